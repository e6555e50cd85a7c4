"""Worst-case sizes of the partial sums of the matrix-core kernels, worked out on the host.

The kernel for one vector (csrc/pb_mfma.hip) keeps the exact integer A_i[r] = sum_c bit_i[r, c] * x_q[c] of Algorithm 2 in
narrower pieces: fp32 accumulators of digit products per slice of columns, one 32-bit integer per lane, four 32-bit "quarter"
sums per (row, bitlayer) in LDS.  The kernels for batches (csrc/pb_imma.h) multiply groups of bitlayers as signed bytes with the
bytes of the activations in 32-bit integers and put those together in fp64.  These tests rebuild the pieces in exact Python
integers for the inputs that make them largest (extreme weights, every activation saturated) at the widest matrix the layout
allows, and check that each fits the type the kernel gives it and that they recombine to the exact sum.
The limits come from csrc/pb_layout.h (compiled for the host); the digit arithmetic is restated here from
Sections 3.1-3.2 of the paper (plane weights 2^j, the sign plane -2^31; two planes = one base-4 digit).
"""
import ctypes
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def limits(tmp_path_factory):
    out = tmp_path_factory.mktemp("limits") / "liblayout_probe.so"
    cmd = ["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__host__=", "-D__device__=",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2003_00822_amd", "csrc"),
           "-o", str(out), os.path.join(ROOT, "tests", "layout_probe.cpp")]
    subprocess.check_call(cmd)
    L = ctypes.CDLL(str(out))
    v = (ctypes.c_int * 2)()
    L.probe_limits(v)
    return {"cols": v[0], "slices": v[1]}


def digits_of(xq):
    """The sixteen base-4 digits of a 32-bit two's-complement value, the top one signed (-2 b31 + b30)."""
    u = xq & 0xFFFFFFFF
    d = [(u >> (2 * i)) & 3 for i in range(16)]
    d[15] = -2 * (d[15] >> 1) + (d[15] & 1)
    assert sum(4 ** i * d[i] for i in range(16)) == (u - (1 << 32) if u >> 31 else u)
    return d


# the four registers of a lane of the result hold the digits b, b + 2, b + 4, b + 6: the quarters
QUARTER_FIRST_DIGIT = [0, 8, 1, 9]
INT32_MAX, INT32_MIN = 2 ** 31 - 1, -2 ** 31
SATURATED = [INT32_MAX, INT32_MIN, 0xFFFF, -1, 0x55555555, -0x55555556, 0x7FFF0000, 1]


def fits_fp32_exactly(v):
    return abs(v) < 2 ** 24


def fits_int32(v):
    return INT32_MIN <= v <= INT32_MAX


def test_partial_sums_fit_at_the_widest_matrix(limits):
    """The kernel for one vector: digit products of a slice, lane integers and quarter sums of (row, bitlayer)."""
    cols = limits["cols"]
    slice_cols = cols // limits["slices"]        # columns of one wave's slice at the widest matrix
    assert slice_cols == 2048
    for xq in SATURATED:
        d = digits_of(xq)
        quarters = []
        for b in QUARTER_FIRST_DIGIT:
            # one lane, one slice: fp32 accumulators of digit products (every weight bit set)
            acc = [d[b + 2 * c] * slice_cols for c in range(4)]
            assert all(fits_fp32_exactly(a) for a in acc)
            t0, t1 = acc[0] + 16 * acc[1], acc[2] + 16 * acc[3]
            assert fits_fp32_exactly(t0) and fits_fp32_exactly(t1)
            lane = t0 + 256 * t1
            assert fits_int32(lane)
            # the LDS word: all slices (and the four lanes that share a slice's columns) add up to all columns
            q = lane * cols // slice_cols
            assert fits_int32(q), (hex(xq & 0xFFFFFFFF), b, q)
            quarters.append(q)
        total = quarters[0] + 4 * quarters[2] + ((quarters[1] + 4 * quarters[3]) << 16)
        signed = xq if xq < 2 ** 31 else xq - 2 ** 32
        assert total == signed * cols
        assert abs(total) < 2 ** 63


K = {1: 0, 2: 0x80, 4: 0x808080}
# the recombination of scaled_sum(), in its order: (digit or the sum of the codes, factor)
CHAIN = {1: [(0, 1)], 2: [(0, 1), ("codes", 0x80), (1, 256)],
         4: [(0, 1), (1, 256), (2, 65536), ("codes", 0x808080), (3, 16777216)]}


def bytes_of(xq, nd):
    """The byte digits of a value of nd bytes: the top one signed, a lower one u as u - 128; x = sum_d 256^d s_d + K."""
    u = [(xq >> (8 * d)) & 0xFF for d in range(nd)]
    s = [v - 128 for v in u[:-1]] + [u[-1] - 256 if u[-1] >= 128 else u[-1]]
    assert sum(256 ** d * s[d] for d in range(nd)) + K[nd] == xq and all(-128 <= v <= 127 for v in s)
    return s


@pytest.mark.parametrize("nd", [1, 2, 4])
@pytest.mark.parametrize("first,size", [(0, 8), (0, 4), (0, 2), (2, 6), (2, 2), (0, 1), (1, 1), (2, 1), (3, 1)])
def test_integer_form_fits_at_the_widest_matrix(limits, nd, first, size):
    """The kernels for batches: a group of bitlayers is a signed byte, its bitlayers at the slots first, first + 1, ... (slot k =
    bit 7 - k; the sign bitlayer stands at slot 0, groups behind the first one at slot 2), times the bytes of the activations.  For
    every code and saturated activations in every column: 32-bit integers hold the sums of a digit's products and of the
    codes, whatever part of the columns they cover and in whatever order they are added; no step of the fp64
    recombination rounds; the bits below the group's last slot are clear."""
    cols, top = limits["cols"], 1 << (8 * nd - 1)
    last = first + size - 1
    for bits in itertools.product([0, 1], repeat=size):
        byte = sum(b << (7 - first - k) for k, b in enumerate(bits))
        code = byte - 256 if byte >= 128 else byte
        # what the group stands for, in units of its last bitlayer
        value = sum((-1 if first + k == 0 else 1) * b << (size - 1 - k) for k, b in enumerate(bits))
        for xq in {top - 1, -top, top - 128, 127 - top, 127, -128, -1, 0}:
            s = bytes_of(xq, nd)
            # partial sums of either sign are no larger than these; FP64 is exact up to 2^53
            assert all(abs(v * code) * cols <= 2 ** 29 for v in s) and abs(code) * cols <= 2 ** 22
            exact, v = 0, 0.0
            for part, factor in CHAIN[nd]:
                term = (code if part == "codes" else s[part] * code) * cols
                exact += factor * term
                v += float(factor) * float(term)
                assert abs(exact) <= 2 ** 53 and int(v) == exact
            assert exact == xq * code * cols
            assert exact % 2 ** (7 - last) == 0 and exact >> (7 - last) == value * xq * cols


def test_popcount_kernel_halves_fit(limits):
    """The AND + popcount kernel keeps sum_j 2^j P_j of the planes 0-15 and 16-31 apart as two 32-bit integers:
    at 32768 columns the low half reaches 32768 * 65535 < 2^31 and the high half -32768 * 32768 = -2^30."""
    cols = 32768
    lo_max = cols * 0xFFFF
    hi_min, hi_max = cols * -(1 << 15), cols * 0x7FFF
    assert fits_int32(lo_max) and fits_int32(hi_min) and fits_int32(hi_max)
    assert lo_max + (hi_min << 16) == cols * ((INT32_MIN) + 0xFFFF)
