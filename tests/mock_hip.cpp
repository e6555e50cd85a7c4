// The HIP runtime functions that libpbatch.so calls, for tests of its host side on a machine without a GPU: a device of 256
// compute units on which nothing runs; every launch is written down.  Loaded with RTLD_GLOBAL before the library, so that the
// library finds these first.  hipLaunchKernel waits `mock_pause` ms after it has written a launch down: another thread's
// launches come in between if nothing keeps them out.
#include <stdint.h>

#include <chrono>
#include <iterator>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

namespace {

struct Dim { uint32_t x, y, z; };
struct Launch { std::string kernel; Dim grid, block; size_t lds; int caller; };
struct Config { Dim grid, block; size_t lds; void *stream; };

std::mutex g_mutex;
std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;   // (registrations come from the constructors of the library)
    return m;
}
std::vector<Launch> g_launches;
int g_pause = 0;
int g_places = 0;      // waves that fit a SIMD; 0: one workgroup a compute unit
thread_local int t_caller = 0;
thread_local std::vector<Config> t_configs;

}  // namespace

extern "C" {

void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, Dim *, Dim *, int *)
{
    names()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *stream)
{
    t_configs.push_back({grid, block, lds, stream});
    return 0;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, void **stream)
{
    *grid = t_configs.back().grid; *block = t_configs.back().block; *lds = t_configs.back().lds; *stream = t_configs.back().stream;
    t_configs.pop_back();
    return 0;
}
int hipLaunchKernel(const void *fn, Dim grid, Dim block, void **, size_t lds, void *)
{
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        g_launches.push_back({names()[fn], grid, block, lds, t_caller});
    }
    if (g_pause) std::this_thread::sleep_for(std::chrono::milliseconds(g_pause));
    return 0;
}
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }   // (only the number of compute units is asked for)
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = reinterpret_cast<void *>(0x100000); return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int threads, size_t)
{
    *n = g_places ? g_places * 4 / ((threads + 63) / 64) : 1;
    return 0;
}

void mock_pause(int ms) { g_pause = ms; }
void mock_caller(int id) { t_caller = id; }
void mock_places(int n) { g_places = n; }
int mock_launches() { std::lock_guard<std::mutex> lock(g_mutex); return (int)g_launches.size(); }
const char *mock_launch(int i, int *out)   // out: grid x, y, block, LDS, caller
{
    std::lock_guard<std::mutex> lock(g_mutex);
    const Launch &l = g_launches[i];
    out[0] = (int)l.grid.x; out[1] = (int)l.grid.y; out[2] = (int)l.block.x; out[3] = (int)l.lds; out[4] = l.caller;
    return l.kernel.c_str();
}
int mock_kernels() { return (int)names().size(); }
const char *mock_kernel(int i) { return std::next(names().begin(), i)->second.c_str(); }
void mock_clear() { std::lock_guard<std::mutex> lock(g_mutex); g_launches.clear(); }

}  // extern "C"
