"""Registers that the compiler could not keep: scratch memory of the kernels in the built library, from the metadata of its code objects.  A
kernel with scratch takes longer to launch, and a loop that reloads registers longer to run, which no test of results sees."""
import os
import re
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """{kernel (its mangled name): bytes of scratch memory per lane}"""
    if not all(os.path.exists(os.path.join(LLVM, t)) for t in ("llvm-objcopy", "llvm-readelf")):
        pytest.skip("no LLVM tools")
    from paper_2003_00822_amd import build
    build.ensure(verbose=False)
    tmp = tmp_path_factory.mktemp("code")
    fat = str(tmp / "fatbin")
    subprocess.check_call([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, build.LIB, str(tmp / "copy")])
    data, magic, found = open(fat, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", {}
    for start in (m.start() for m in re.finditer(magic, data)):        # one bundle per source file
        entries, at = struct.unpack_from("<Q", data, start + len(magic))[0], start + len(magic) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" not in target:
                continue
            code = str(tmp / "code")
            with open(code, "wb") as f:
                f.write(data[start + offset:start + offset + size])
            notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", code], stdout=subprocess.PIPE, check=True, text=True).stdout
            names = re.findall(r"^\s+\.name:\s+(_Z\S+)$", notes, re.M)
            sizes = re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)
            assert len(names) == len(sizes)
            found.update(zip(names, map(int, sizes)))
    return found


def test_scratch_memory_only_where_four_tiles_fill_the_registers(scratch):
    assert sum("k_i8" in k for k in scratch) > 100 and any("k_mfma" in k for k in scratch)
    spilled = {k: v for k, v in scratch.items() if v}
    # k_i8_tile<digits, slots, layout, eight waves along the digit rows, four tiles each, ...>
    assert all(re.match(r"_ZN2pb9k_i8_tileILi\dELi\dELb\dELi8ELi4E", k) for k in spilled), spilled
    assert max(spilled.values()) <= 200, spilled
