"""Which kernels the host side launches, and in which order, worked out without a GPU: libpbatch.so on a HIP runtime that
writes launches down (mock_hip.cpp), in a process of its own."""
import json
import os
import re
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, json, sys, threading
mock = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # before the library, which then finds these functions first
mock.mock_launch.restype = mock.mock_kernel.restype = ctypes.c_char_p
L = ctypes.CDLL(sys.argv[2])
ROWS, BITS, GATES, PAIRS = 0x50420001, 0x50420002, 0x50420003, 0x50420004
F = ctypes.c_void_p(0x10000000)                               # an aligned address that nothing reads
WORK = ctypes.c_void_p(0x20000000)

class Desc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("rows", "cols", "bits", "frac_bits", "act_bits")] + [("layout", ctypes.c_uint32)]

def desc(rows, cols, bits, layout, act_bits=32):
    d = Desc()
    assert L.pb_desc_init_layout(ctypes.byref(d), rows, cols, bits, ctypes.c_uint32(layout)) == 0
    d.act_bits = act_bits
    return d

def launches():
    out, all_ = (ctypes.c_int * 5)(), []
    for i in range(mock.mock_launches()):
        name = mock.mock_launch(i, out).decode()
        all_.append((name, out[4]))
    mock.mock_clear()
    return all_
"""


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    from paper_2003_00822_amd import build
    build.ensure(verbose=False)
    mock = tmp_path_factory.mktemp("mock") / "libmock_hip.so"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", "-o", str(mock),
                           os.path.join(ROOT, "tests", "mock_hip.cpp")])

    def run(code, *args):
        r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(code), str(mock), build.LIB, *args],
                           stdout=subprocess.PIPE, check=True, timeout=300)
        return json.loads(r.stdout)
    return run


def test_calls_on_one_workspace_do_not_mix_their_launches(probe):
    """A call of several launches hands data on through its workspace.  Two host threads that use one workspace on one stream
    must each get their launches in one piece (the stream then keeps them apart)."""
    got = probe("""
        N = 64
        d, p = desc(2000, 3000, 8, BITS), desc(2000, 3000, 8, PAIRS)
        r, lb, lg, s = desc(300, 700, 4, ROWS), desc(400, 300, 4, BITS), desc(6000, 3000, 8, GATES), desc(4096, 4096, 8, BITS)
        ref = ctypes.byref
        cell = lambda l, i: lambda: L.pb_lstm_cell(F, F, ref(l), 4, F, i, ctypes.c_void_p(0x50000000), F, None,
                                                   ctypes.c_void_p(0x60000000), F, N, WORK, None)
        calls = {
            "matmul": lambda: L.pb_matmul(F, F, ref(d), 8, F, N, F, WORK, None),
            "matmul pairs": lambda: L.pb_matmul(F, F, ref(p), 8, F, N, F, WORK, None),
            "matmul rows": lambda: L.pb_matmul(F, F, ref(r), 4, F, 2, F, WORK, None),
            "bias": lambda: L.pb_matmul_bias_act(F, F, ref(d), 8, F, N, F, 1, F, WORK, None),
            "bias rows": lambda: L.pb_matmul_bias_act(F, F, ref(r), 4, F, 2, F, 1, F, WORK, None),
            "static": lambda: L.pb_matmul_static(F, F, ref(s), 8, F, 60, F, None),
            "sums": lambda: L.pb_matmul_acc(F, ref(d), 8, F, N, F, WORK, None),
            "sums of pairs": lambda: L.pb_matmul_acc_pairs(F, ref(d), 8, F, N, F, WORK, None),
            "cell": cell(lb, 200), "cell one launch": cell(lg, 1500),
            "prep": lambda: L.pb_act_prep(ref(d), F, N, WORK, None),
            "fixed point": lambda: L.pb_fixed_point(ref(d), F, N, F, WORK, None),
        }
        single = {}
        for name, f in calls.items():
            assert f() == 0, name
            single[name] = [k for k, _ in launches()]
        mock.mock_pause(3)
        mixed = []
        for a, b in [(n, n) for n in calls] + [("matmul", "prep"), ("matmul", "fixed point"), ("cell", "matmul")]:
            start = threading.Barrier(2)
            def work(me, f):
                mock.mock_caller(me)
                start.wait()
                for _ in range(3):
                    assert f() == 0
            threads = [threading.Thread(target=work, args=(i, calls[n])) for i, n in enumerate((a, b))]
            [t.start() for t in threads]
            [t.join() for t in threads]
            mixed.append((a, b, launches()))
        print(json.dumps([single, mixed]))
    """)
    single, mixed = got
    assert len(single["matmul"]) == len(single["static"]) == len(single["sums"]) == len(single["cell one launch"]) == 2
    assert len(single["bias rows"]) == 3 and len(single["cell"]) >= 2 and len(single["prep"]) == 1
    for a, b, seen in mixed:
        order = []
        while seen:
            me = seen[0][1]
            want = single[(a, b)[me]]
            assert [k for k, who in seen[:len(want)]] == want and {who for _, who in seen[:len(want)]} == {me}, (a, b, seen)
            order.append(me)
            seen = seen[len(want):]
        assert sorted(order) == [0, 0, 0, 1, 1, 1]


def test_the_gpu_tests_reach_every_kernel_for_batches(probe):
    """Every compiled kernel for batches is taken by a case that the GPU tests compare with the oracle: the choice of the kernel
    is fitted, and a change to it must not leave one untested (or unreachable) unnoticed."""
    from tests.test_gpu_imma import CASES, CELLS, DIGITS, KERNELS, PREPARED, with_sums
    products = [c[:6] + (with_sums(c[0], c[2]),) for c in CASES + KERNELS]
    digits = [c + (32, with_sums(c[0], c[2])) for c in DIGITS]
    wide_cells = [c for c in CELLS if c[3] == 32]
    code = """
        products, cells, prepared = json.loads(sys.argv[3])
        reached, ref = set(), ctypes.byref
        def took():
            got = {k for k, _ in launches()}
            reached.update(got)
            return got
        for R, C, N, bits, m, act, sums in products:
            for layout in (BITS, PAIRS):
                d = desc(R, C, bits, layout, act)
                assert L.pb_matmul(F, F, ref(d), m, F, N, F, WORK, None) == 0
                if sums:
                    assert L.pb_matmul_acc(F, ref(d), m, F, N, F, WORK, None) == 0
                    assert L.pb_matmul_acc_pairs(F, ref(d), m, F, N, F, WORK, None) == 0
                took()
        for H, I, N, act, bits, m in cells:
            d = desc(4 * H, I + H, bits, GATES, act)
            assert L.pb_lstm_cell(F, F, ref(d), m, F, I, ctypes.c_void_p(0x50000000), F, None, ctypes.c_void_p(0x60000000), F, N,
                                  WORK, None) == 0
            took()
        for R, C, N, bits, m, act in prepared:
            for layout in (BITS, PAIRS):
                assert L.pb_matmul_prepared(F, F, ref(desc(R, C, bits, layout, act)), m, N, F, WORK, None) == 0
                took()
        compiled = [mock.mock_kernel(i).decode() for i in range(mock.mock_kernels())]
        print(json.dumps([sorted(reached), [k for k in compiled if "k_i8" in k or "k_digits" in k]]))
    """
    reached, compiled = probe(code, json.dumps([products, CELLS, PREPARED]))
    assert len(compiled) > 100
    assert not sorted(set(compiled) - set(reached))
    # 32-bit digits from memory: calls with values beyond three digits reach all; where the top digit may be left out (not in one tile with
    # all four) calls of more than one group of sixteen vectors do, which compare both
    memory = [k for k in compiled if re.search(r"k_i8_tileILi4E|k_i8ILi4ELi\dELb\dELi\dELb0E", k)]
    four = [k for k in memory if re.search(r"k_i8ILi4ELi\dELb\dELi1ELb0E.*Lb0EEE", k)]
    assert len(memory) > 30 and len(four) == 8
    reached, _ = probe(code, json.dumps([digits, wide_cells, PREPARED]))
    assert not sorted(set(memory) - set(reached))
    reached, _ = probe(code, json.dumps([[c for c in digits if c[2] > 16], [c for c in wide_cells if c[2] > 16], [c for c in PREPARED if c[2] > 16]]))
    assert not sorted(set(memory) - set(four) - set(reached))


def test_non_temporal_loads_only_where_they_pay(probe):
    """Weights that fit the L2 caches or nearly so are read with plain loads, which keep them there for the next call."""
    took = probe("""
        took = []
        for rows in (2048, 4016, 4880, 5856, 7808, 10976, 16384):          # 17, 33, 40, 48, 64, 90, 134 MB
            assert L.pb_matmul(F, F, ctypes.byref(desc(rows, 8192, 8, BITS)), 8, F, 2, F, WORK, None) == 0
            took.append([k for k, _ in launches()])
        print(json.dumps(took))
    """)
    assert all(len(t) == 1 and "k_i8I" in t[0] for t in took)
    assert [t[0].split("Li")[-1].startswith("2") for t in took] == [False, False, False, True, True, False, False]


@pytest.mark.parametrize("places,rows,cols,batch,act_bits,bits,layout,want", [
    (3, 12135, 2547, 13, 32, 8, "BITS", 253),      # five waves, two on one SIMD: one workgroup a unit, three row tiles each (380 of two)
    (4, 9551, 2050, 13, 16, 2, "BITS", 199),       # ... two a unit, three row tiles each (299 of two)
    (3, 9000, 9000, 12, 32, 5, "BITS", 188),       # six waves: one
    (3, 1731, 276, 887, 16, 6, "PAIRS", 55),       # one wave, 13120 bytes of LDS in pieces of 1280: eleven a unit
    (4, 9619, 11869, 16, 32, 1, "PAIRS", 201),     # eight waves, two a unit: one with three row tiles is done sooner than two with two
    (4, 14587, 2129, 51, 8, 3, "PAIRS", 456),      # five waves, two a unit with two row tiles each: as many as one with four
])
def test_a_grid_that_runs_at_once(probe, places, rows, cols, batch, act_bits, bits, layout, want):
    """The workgroups along the rows are no more than the compute units run at once: a rest would run by itself."""
    got = probe("""
        places, rows, cols, batch, act, bits, layout = json.loads(sys.argv[3])
        mock.mock_places(places)
        assert L.pb_matmul(F, F, ctypes.byref(desc(rows, cols, bits, globals()[layout], act)), bits, F, batch, F, WORK, None) == 0
        out = (ctypes.c_int * 5)()
        name = mock.mock_launch(mock.mock_launches() - 1, out).decode()
        print(json.dumps([name, out[0]]))
    """, json.dumps([places, rows, cols, batch, act_bits, bits, layout]))
    assert re.search(r"k_i8ILi\dELi\dELb\dELi\dELb0E", got[0]), got     # digits from memory
    assert got[1] == want, got
