"""Packing and unpacking at the edges of their tiles (16 rows x 512 columns), and the clipping search around the sizes from
which a histogram rules thresholds out and the thresholds are no longer shared out, against the oracle's codes and scales."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pb_oracle as po
from tests.test_layout_host import layout_of, probe  # noqa: F401 (the host build of the layout's arithmetic)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pb():
    assert torch.cuda.is_available(), "gpu tests need a GPU"
    from paper_2003_00822_amd import pb as _pb
    _pb.lib()
    return _pb


def check(pb, W, bits, layout, quantizer=0):
    prep = po.prepare(W, bits, quantizer)
    lin = pb.PackedLinear(torch.from_numpy(W).cuda(), bits, layout=layout, quantizer=quantizer)
    assert (lin.unpack().cpu().numpy() == prep["q"]).all()
    assert (lin.scales[:bits].cpu().numpy().view(np.int32) == prep["scales"].view(np.int32)).all()


@pytest.mark.parametrize("layout", [0x50420001, 0x50420002, 0x50420003, 0x50420004])
@pytest.mark.parametrize("bits", [1, 5, 8, 9, 16])
def test_tile_edges(pb, layout, bits):
    g = np.random.default_rng(bits)
    for rows, cols in ((4, 1), (16, 512), (20, 513), (12, 511), (36, 1027), (64, 2046)):
        print("pack", hex(layout), bits, rows, cols, flush=True)
        W = g.normal(0, 0.05, size=(rows, cols)).astype(np.float32)
        # quotients at and next to half-integers, where the code follows the rounding of the division
        qmax = max(1, 2 ** (bits - 1) - 1)
        W[0, 0] = qmax * 0.125
        W[1, :] = (g.integers(-qmax, qmax + 1, size=cols) + 0.5) * np.float32(0.125)
        W[2, :] = np.nextafter(W[1, :], np.float32(0))
        W = np.clip(W, -qmax * 0.125, qmax * 0.125).astype(np.float32)
        check(pb, W, bits, layout)


@pytest.mark.parametrize("layout", [0x50420001, 0x50420002, 0x50420003, 0x50420004])
@pytest.mark.parametrize("bits", [1, 8, 9, 16])
def test_whole_tiles_and_quarters(pb, layout, bits):
    """256 tiles, of which workgroups take quarters, and 257 or more, of which they take the whole."""
    g = np.random.default_rng(bits + 30)
    for rows, cols in ((4092, 3), (4096, 512), (4100, 511), (2064, 513)):
        print("pack", hex(layout), bits, rows, cols, flush=True)
        check(pb, g.normal(0, 0.05, size=(rows, cols)).astype(np.float32), bits, layout)


@pytest.mark.parametrize("layout", [0x50420001, 0x50420002, 0x50420003, 0x50420004])
@pytest.mark.parametrize("bits", [5, 9])
def test_packed_words(pb, probe, layout, bits):  # noqa: F811
    """Every byte of `packed`, padding included, from the oracle's codes and the positions that pb_layout.h gives: quarters of
    tiles and, in the last shape, whole ones."""
    g = np.random.default_rng(bits + 10)
    for rows, cols in ((4, 1), (20, 513), (36, 1027), (52, 31), (4100, 40)):
        print("words", hex(layout), bits, rows, cols, flush=True)
        W = g.normal(0, 0.05, size=(rows, cols)).astype(np.float32)
        q = po.prepare(W, bits)["q"].reshape(rows, cols)
        L = layout_of(probe, layout, rows, cols, bits)
        stored = bits + bits % 2 if layout == pb.PB_LAYOUT_TILE16_PAIRS_V1 else bits
        H = rows // 4
        packed_row = [probe.probe_gates_packed_row(r, H) if L["gate_h"] else r for r in range(rows)]
        codes = np.zeros((L["rows_p"], L["cwp"] * 32), dtype=np.int64)     # (padding has the code 0)
        codes[packed_row, :cols] = q
        layers = [(codes >> (bits - 1 - i)) & 1 if i < bits else codes * 0 for i in range(stored)]   # sign bitlayer first
        words = [np.packbits(b.astype(np.uint8), axis=1, bitorder="little").view("<u4") for b in layers]
        if layout == pb.PB_LAYOUT_TILE16_PAIRS_V1:
            for i in range(0, stored, 2):   # digits 2 upper + lower, of the even and of the odd columns
                up, lo = (1 - layers[i] if i == 0 else layers[i]), layers[i + 1]
                for k in range(2):
                    pair = np.zeros_like(codes, dtype=np.uint8)
                    pair[:, 0::2], pair[:, 1::2] = lo[:, k::2], up[:, k::2]
                    words[i + k] = np.packbits(pair, axis=1, bitorder="little").view("<u4")
        want = np.zeros(L["layer_words"] * stored, dtype=np.uint32)
        at = np.array([[probe.probe_word_index(layout, L["cwp"], L["layer_words"], 0, r, w) for w in range(L["cwp"])]
                       for r in range(L["rows_p"])])
        for i in range(stored):
            want[at + i * L["layer_words"]] = words[i]   # (bitlayer after bitlayer)
        lin = pb.PackedLinear(torch.from_numpy(W).cuda(), bits, layout=layout)
        got = lin.packed.cpu().numpy().view("<u4")
        assert got.size == want.size and (got == want).all()


def test_all_weights_count_in_large_matrices(pb):
    """More weights than one round of the grids takes (2^22 in k_clip_hist, 2^24 elsewhere), an odd number, and all but a few
    of them in one bin of the histogram; with the ragged matrix of 3001 x 5003."""
    g = np.random.default_rng(3)
    ragged = g.normal(0, 0.05, size=(3001, 5003)).astype(np.float32)
    large = g.normal(0, 0.05, size=(4097, 4097)).astype(np.float32)
    onebin = np.full((4097, 4097), 0.3, dtype=np.float32)
    onebin[:, -1], onebin[-1, -1] = -0.31, 0.47
    large[-1, -1], large[0, 0] = 0.9, -1.1
    cases = [(ragged, 4, 0x50420004, 3), (large, 2, 0x50420002, 3), (onebin, 4, 0x50420002, 3), (large, 2, 0x50420002, 2),
             (large, 3, 0x50420002, 1)]
    with ThreadPoolExecutor(3) as pool:   # (the oracle takes 15 seconds for each search)
        expected = list(pool.map(lambda c: po.quantize_mode(c[0], c[1], c[3]), cases))
    for (W, bits, layout, quantizer), (q, d) in zip(cases, expected):
        print("large", W.shape, bits, quantizer, flush=True)
        lin = pb.PackedLinear(torch.from_numpy(W).cuda(), bits, layout=layout, quantizer=quantizer)
        assert (lin.scales[:bits].cpu().numpy().view(np.int32) == po.scales(d, bits).view(np.int32)).all()
        assert (lin.unpack().cpu().numpy() == q).all()


@pytest.mark.parametrize("bits", [1, 4, 8, 12])
def test_clipping_search_with_and_without_histogram(pb, bits):
    g = np.random.default_rng(bits + 50)
    for rows, cols, outlier in ((512, 256, 0.9), (363, 363, 0.9), (400, 701, 30.0), (420, 1000, 0.0)):
        print("clip search", bits, rows, cols, outlier, flush=True)
        W = g.normal(0, 0.05, size=(rows, cols)).astype(np.float32)
        if outlier:
            W[7, 11] = -outlier
        check(pb, W, bits, 0x50420002, quantizer=3)


@pytest.mark.parametrize("bits", [1, 4, 10, 12, 16])
def test_clipping_search_with_thresholds_shared_out(pb, bits):
    """Grids with 32, 16, 4 and 1 workgroups per block of weights, one weight and a single one past a block among them."""
    g = np.random.default_rng(bits + 80)
    for rows, cols in ((1, 1), (91, 90), (8193, 1), (360, 364), (400, 701), (1025, 1024), (2051, 2049)):
        if rows * cols > 1 << 21 and bits not in (4, 16):
            continue
        print("clip search", bits, rows, cols, flush=True)
        W = g.normal(0, 0.05, size=(rows, cols)).astype(np.float32)
        W[0, 0] = 0.3
        check(pb, W, bits, 0x50420002, quantizer=3)


@pytest.mark.parametrize("bits", [1, 3, 4, 8])
def test_clipping_search_between_equal_errors(pb, bits):
    """A few weights, for which several thresholds have the same summed error, or one that differs by the rounding of d q
    alone: -9 with 4 bits is met exactly by the thresholds 32 / 32 (7 steps of RN(9 / 7)) and 28 / 32 (8 steps of 1.125)."""
    for values in ([-9.0], [9.0, -9.0], [1.0, 3.0], [-0.7, 0.1], [5.0, -5.0, 2.5], [0.3], [1e-30, -3e-31]):
        print("clip search", bits, values, flush=True)
        check(pb, np.array([values], dtype=np.float32), bits, 0x50420002, quantizer=3)


@pytest.mark.parametrize("bits", [1, 4, 8, 10, 16])
def test_clipping_search_next_to_the_largest_float(pb, bits):
    """Weights up to the largest float, where d q, rounded, can be beyond it: below and above the size for the histogram."""
    top = np.finfo(np.float32).max
    for rows, cols, std in ((1, 1, 0.0), (20, 513, 2.0 ** 125), (20, 513, 0.05), (512, 600, 2.0 ** 125)):
        print("clip search", bits, rows, cols, std, flush=True)
        W = np.clip(np.random.default_rng(bits).normal(0, 1, size=(rows, cols)) * std, -top, top).astype(np.float32)
        W[-1, -1], W[0, 0] = -top, top
        check(pb, W, bits, 0x50420002, quantizer=3)


@pytest.mark.parametrize("bits,quantizer", [(8, 0), (5, 1), (2, 2), (4, 3)])
def test_statistics_at_the_end_of_the_weights(pb, bits, quantizer):
    """Last blocks of 1 to 8192 weights: all of one sign, so that a weight past the end would change the range or the mean,
    and the largest or smallest one last."""
    g = np.random.default_rng(bits + 20)
    for rows, cols in ((1, 1), (1, 3), (3, 341), (1, 1025), (1, 8191), (1, 8192), (1, 8193), (5, 3277), (3, 8193)):
        for sign, last in ((1, 9.0), (1, 0.25), (-1, 9.0), (-1, 0.25)):
            print("statistics", quantizer, rows, cols, sign, last, flush=True)
            W = (sign * g.uniform(0.5, 1.0, size=(rows, cols))).astype(np.float32)
            W[-1, -1] = sign * last
            check(pb, W, bits, 0x50420002, quantizer)


@pytest.mark.parametrize("nan", [0x7FC00000, 0x7FA00000, 0xFFA00000], ids=["quiet", "signalling", "negative signalling"])
@pytest.mark.parametrize("bits,quantizer", [(8, 0), (16, 0), (5, 1), (2, 2), (4, 3)])
def test_nan_weights_count_as_zero(pb, bits, quantizer, nan):
    """NaN has the code of 0 wherever it stands among the four columns that a lane quantizes together, and does not
    touch the step, also where it follows the largest weight."""
    W = np.random.default_rng(bits).normal(0, 0.05, size=(530, 531)).astype(np.float32)
    W[0, 0], W[0, 5] = -0.9, 0.8
    where = np.zeros(W.shape, dtype=bool)
    for j in range(16):   # every subset of a group of four columns
        for e in range(4):
            where[j + 1, 4 * j + e] = j >> e & 1
            where[j + 514, 512 + e] = j >> e & 1
    where[1:16, 5] = True
    prep = po.prepare(np.where(where, np.float32(0), W), bits, quantizer)
    bitsW = np.where(where, np.uint32(nan), W.view(np.uint32)).view(np.int32)
    lin = pb.PackedLinear(torch.from_numpy(bitsW).cuda().view(torch.float32), bits, quantizer=quantizer)
    assert (lin.unpack().cpu().numpy() == prep["q"]).all()
    assert (lin.scales[:bits].cpu().numpy().view(np.int32) == prep["scales"].view(np.int32)).all()


@pytest.mark.parametrize("bits,quantizer", [(1, 0), (8, 0), (16, 0), (5, 1), (2, 2), (4, 3), (8, 3), (16, 3)])
def test_infinite_missing_and_extreme_weights(pb, bits, quantizer):
    """No weight but NaN: step 1 (the mean is 0); the smallest and the largest floats, whose steps or their inverses are
    beyond the normal range; an infinite weight: an infinite step, in which all codes are 0 (the +-1 code keeps the signs)."""
    g = np.random.default_rng(bits)
    for rows, cols in ((20, 513), (512, 600)):
        normal = g.normal(0, 1, size=(rows, cols)).astype(np.float32)
        for name, W in (("nan", np.full_like(normal, np.nan)), ("zero", np.zeros_like(normal)),
                        ("2^-126", normal * np.float32(2.0 ** -126)), ("2^-145", normal * np.float32(2.0 ** -145)),
                        ("2^-120", normal * np.float32(2.0 ** -120)), ("2^120", normal * np.float32(2.0 ** 120)),
                        ("2^124", normal * np.float32(2.0 ** 124))):
            print("extreme", quantizer, bits, rows, cols, name, flush=True)
            check(pb, W, bits, 0x50420002, quantizer)
        for inf in (np.inf, -np.inf):
            print("extreme", quantizer, bits, rows, cols, inf, flush=True)
            W = normal.copy()
            W[3, 7], W[4, 9] = inf, np.nan
            lin = pb.PackedLinear(torch.from_numpy(W).cuda(), bits, quantizer=quantizer)
            scales = lin.scales[:bits].cpu().numpy()
            assert np.isinf(scales).all() and scales[0] < 0 and (scales[1:] > 0).all()
            q = lin.unpack().cpu().numpy()
            assert (q == (np.where(W < 0, -1, 1) if quantizer == 2 else 0)).all()
