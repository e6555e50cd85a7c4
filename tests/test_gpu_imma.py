"""The kernels on the 8-bit integer matrix cores (csrc/pb_imma.hip, csrc/pb_imma_tile.hip) at the edges of their tiles: every kernel
that is compiled (test_launches.py works out on the host that the cases reach them all), rows and columns that do not fill the
last tile, batches that leave digit rows empty, groups of bitlayers that share a code and groups of one, activations saturated
at both ends.  Oracle: the definition of the per-bitlayer sums on sampled rows (exact integers), then the scales in fp64."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pb_oracle as po
from paper_2003_00822_amd import synth
from tests.helpers import assert_y_close, pair_sums

pytestmark = pytest.mark.gpu

BITS, PAIRS, GATES = 0x50420002, 0x50420004, 0x50420003


@pytest.fixture(scope="module")
def pb():
    assert torch.cuda.is_available(), "gpu tests need a GPU"
    from paper_2003_00822_amd import pb as pbmod
    pbmod.lib()
    return pbmod


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(pb, R, C, N, bits, m, act_bits, frac_bits, layout, sums):
    W, X = synth.ragged(R, C, batch=N, case=700 + R + C + N, xdist="wide")
    X = X.copy()
    X[0, ::2], X[0, 1::2] = 3e38, -3e38                 # both ends of the fixed-point range
    X[N - 1, C - 1] = np.inf
    X[N // 2, :5] = np.nan
    rows = sorted({0, 1, R // 2, (R - 1) // 16 * 16, R - 1} | set(range(min(R, 20))))
    # the codes of the sampled rows: the quantizer's step comes from the largest weight of all
    prep = po.prepare(W[rows + [int(np.abs(W).max(axis=1).argmax())]], bits)
    lin = pb.PackedLinear(dev(W), bits, max_batch=N, frac_bits=frac_bits, act_bits=act_bits, layout=layout)
    Xd = dev(X)
    Y = lin(Xd, m).cpu().numpy()
    Y_again = lin(Xd, m).cpu().numpy()
    assert (Y.view(np.int32) == Y_again.view(np.int32)).all()
    uneven = prep["scales"].copy()
    uneven[0] = np.nextafter(uneven[0], np.float32(0.0))     # one ulp: every bitlayer by itself
    lin.scales[:bits] = dev(uneven)
    Y_uneven = lin(Xd, m).cpu().numpy()
    A = lin.acc(Xd, m).cpu().numpy() if sums else None
    P = lin.acc_pairs(Xd, m).cpu().numpy() if sums else None
    xq = po.fixed_point(X, frac_bits=frac_bits, act_bits=act_bits)
    for k, r in enumerate(rows):
        sub = po.layer_products_direct(prep["layers"][:, k:k + 1, :], m, xq)[:, :, 0]      # [m, N]
        assert_y_close(Y[:, r], po.dequant(sub, prep["scales"], m, frac_bits=frac_bits), sub, prep["scales"], frac_bits=frac_bits)
        want = sum(float(uneven[i]) * sub[i].astype(np.float64) for i in range(m)) * 2.0 ** -frac_bits
        assert_y_close(Y_uneven[:, r], want.astype(np.float32), sub, uneven, frac_bits=frac_bits)
        if sums:
            assert (A[:, :, r] == sub).all(), (r, "sums")
            assert (P[:, :, r] == pair_sums(sub[:, :, None], m)[:, :, 0]).all(), (r, "sums of pairs")


CASES = [
    # rows, columns, vectors, bits, used, activation bits, position of the fixed point
    (17, 511, 2, 4, 4, 32, 16),          # one tile of digit rows, half of it empty; four slots
    (33, 513, 4, 8, 8, 32, 16),          # one full tile, one column in a chunk of its own
    (50, 1100, 5, 7, 5, 32, 16),         # a second tile with one vector
    (16, 300, 9, 5, 1, 16, 10),          # the sign bitlayer by itself
    (95, 2049, 17, 8, 7, 8, 4),          # 8-bit activations, the second tile nearly empty
    (40, 700, 3, 16, 16, 32, 16),        # three groups of bitlayers
    (40, 700, 3, 12, 9, 24, 12),         # two groups, the second of one bitlayer; 24-bit activations
    (100, 9000, 12, 3, 3, 32, 16),       # rows too wide to stage
    (31, 16500, 2, 8, 8, 16, 8),         # two chunks per wave
    (4200, 8192, 2, 8, 8, 32, 16),       # too many weights for the L2 caches
    (4400, 3664, 13, 6, 6, 8, 4),        # digits from memory
    (4022, 2521, 61, 3, 2, 8, 4),        # ... four tiles per wave
    (2100, 5000, 18, 7, 7, 32, 16),      # converted in the launch, two chunks per wave
    (6000, 7871, 18, 7, 7, 16, 8),       # four tiles per wave, several row tiles
    (2000, 3000, 64, 8, 8, 32, 16),
    (4778, 6480, 13, 8, 5, 32, 16),
    (9000, 9000, 16, 6, 6, 32, 16),
    (2620, 2697, 713, 8, 8, 32, 16),     # many digit rows, two tiles per wave
    (9347, 975, 686, 2, 1, 32, 16),
    (1500, 1600, 70, 12, 11, 32, 16),    # two groups per row tile there
    (1128, 1711, 71, 16, 16, 32, 16),    # three
]

# One call for each compiled kernel that the calls above do not take.
# rows, columns, vectors, bits, used, activation bits, position of the fixed point
KERNELS = [
    # many digit rows: four waves along them, eight, eight with four tiles each
    (2669, 520, 187, 2, 1, 32, 16), (2207, 515, 67, 10, 8, 32, 16), (6326, 1189, 388, 8, 8, 32, 16), (4643, 3250, 491, 1, 1, 32, 16),
    (8119, 28, 59, 13, 10, 32, 16), (10964, 23, 101, 5, 3, 32, 16),
    (5782, 1101, 117, 1, 1, 16, 12), (11973, 42, 179, 9, 4, 16, 12), (7339, 1071, 599, 1, 1, 16, 12), (3612, 781, 76, 15, 11, 16, 12),
    (3533, 65, 169, 16, 15, 16, 12), (11768, 1521, 142, 15, 10, 16, 12), (7936, 523, 239, 7, 3, 8, 4), (7100, 18, 600, 14, 3, 8, 4),
    (8782, 1652, 964, 9, 4, 8, 4), (7045, 1197, 70, 14, 11, 8, 4), (9408, 100, 195, 9, 9, 8, 4), (4681, 689, 436, 15, 15, 8, 4),
    # ... the sums themselves
    (1649, 23, 51, 12, 8, 16, 12), (1043, 2813, 438, 7, 5, 16, 12), (1947, 628, 82, 5, 4, 8, 4), (2857, 27, 35, 16, 8, 8, 4),
    (2310, 25, 276, 16, 8, 8, 4),
    # four tiles per wave
    (4379, 18, 105, 13, 1, 32, 16), (8300, 16, 57, 2, 1, 16, 12), (11051, 19, 81, 13, 5, 8, 4), (752, 2612, 168, 1, 1, 8, 4),
    # one tile, digits from memory
    (5782, 16, 34, 11, 9, 32, 16), (4130, 16, 49, 13, 6, 16, 12), (17, 4122, 7, 2, 1, 16, 12), (16, 2134, 13, 1, 1, 8, 4),
    # two tiles, converted in the launch
    (10319, 16, 5, 15, 2, 32, 16), (6172, 16, 9, 13, 7, 16, 12), (6202, 16, 9, 2, 1, 16, 12), (2352, 19, 17, 6, 5, 8, 4),
    (2091, 16, 17, 9, 1, 8, 4), (430, 68, 443, 8, 8, 32, 16),
    # one tile, converted in the launch
    (16, 16, 2, 1, 1, 8, 4), (18, 16, 2, 8, 5, 8, 4),
    # ... non-temporal loads of the weights
    (10700, 8200, 2, 4, 4, 32, 16), (10700, 8200, 2, 4, 4, 16, 12), (10700, 8200, 2, 4, 4, 8, 4), (14713, 1035, 3, 16, 16, 32, 16),
    (14694, 1040, 2, 16, 16, 16, 12), (14745, 1035, 6, 16, 16, 8, 4),
]


def with_sums(R, N):
    return R * N < 700000


@pytest.mark.parametrize("layout", [BITS, PAIRS])
@pytest.mark.parametrize("case", CASES + KERNELS, ids=lambda c: "x".join(map(str, c[:3])) + "-%d/%d-a%d" % (c[4], c[3], c[5]))
def test_every_way(pb, case, layout):
    R, C, N, bits, m, act_bits, frac_bits = case
    print("way", case, hex(layout), flush=True)
    check(pb, R, C, N, bits, m, act_bits, frac_bits, layout, sums=with_sums(R, N))


# Rows, columns, vectors, bits, used: between them these calls take every kernel that reads 32-bit digits from memory and stores Y or the sums, those
# of more than 16 vectors every one that may leave out a digit (test_launches.py works that out)
DIGITS = [(2669, 520, 187, 2, 1), (2207, 515, 67, 10, 8), (2207, 515, 70, 8, 8), (2620, 2697, 113, 8, 8), (6326, 1189, 388, 8, 8),
          (4643, 3250, 491, 1, 1), (4379, 18, 105, 13, 1), (752, 2612, 35, 3, 3), (5782, 16, 34, 11, 9), (100, 9000, 12, 3, 3),
          # one tile; four; many digit rows; the sums
          (1496, 10977, 5, 4, 4), (16337, 1799, 3, 4, 4), (1177, 1605, 50, 4, 2), (1684, 1581, 33, 8, 5), (2213, 1171, 96, 8, 1), (3595, 1146, 40, 7, 7), (4964, 1119, 161, 1, 1),
          (8087, 1125, 120, 7, 5), (964, 1573, 36, 5, 2), (1070, 1620, 62, 5, 2), (1720, 1128, 48, 8, 3), (2722, 1163, 51, 10, 4),
          (2071, 1147, 83, 13, 8)]


def widen(X, columns):
    """Every vector at both ends of three byte digits; of the groups of sixteen vectors the first (and every fourth) keeps to them, where
    there are several; the others have one value beyond, in the first, the middle and the last of `columns` in turn."""
    N = len(X)
    first, middle, last = columns
    for group in range((N + 15) // 16):
        rows = range(16 * group, min(N, 16 * group + 16))
        X[rows[0], first], X[rows[-1], last] = (2 ** 23 - 1) / 65536, -128.0
        kind = 0 if group % 4 == 0 and N > 16 else 1 + (group + N) % 3
        if kind == 1: X[rows[-1], first] = 128.0
        if kind == 2: X[rows[0], middle] = -(2 ** 23 + 1) / 65536
        if kind == 3: X[rows[len(rows) // 2], last] = 3e38


@pytest.mark.parametrize("layout", [BITS, PAIRS])
@pytest.mark.parametrize("case", DIGITS, ids=lambda c: "x".join(map(str, c[:3])) + "-%d/%d" % (c[4], c[3]))
def test_three_digits_or_four(pb, case, layout):
    """Each group of sixteen vectors is multiplied with the digits that it needs; the sums of bitlayers and of pairs beside Y."""
    R, C, N, bits, m = case
    print("digits", case, hex(layout), flush=True)
    g = np.random.default_rng(200300822 + 67)
    W = g.normal(0, 0.02, size=(R, C)).astype(np.float32)
    X = g.normal(size=(N, C)).astype(np.float32)
    widen(X, (0, C // 2, C - 1))
    sample = sorted({0, 1, R // 2, (R - 1) // 16 * 16, R - 1})
    prep = po.prepare(W[sample + [int(np.abs(W).max(axis=1).argmax())]], bits)
    lin = pb.PackedLinear(dev(W), bits, max_batch=N, layout=layout)
    Y = lin(dev(X), m).cpu().numpy()
    A = lin.acc(dev(X), m).cpu().numpy() if with_sums(R, N) else None
    P = lin.acc_pairs(dev(X), m).cpu().numpy() if with_sums(R, N) else None
    xq = po.fixed_point(X, frac_bits=16, act_bits=32)
    for k, r in enumerate(sample):
        sub = po.layer_products_direct(prep["layers"][:, k:k + 1, :], m, xq)[:, :, 0]
        assert_y_close(Y[:, r], po.dequant(sub, prep["scales"], m, frac_bits=16), sub, prep["scales"], frac_bits=16)
        if A is not None:
            assert (A[:, :, r] == sub).all(), r
            assert (P[:, :, r] == pair_sums(sub[:, :, None], m)[:, :, 0]).all(), r


# Rows, columns, vectors, bits, used, activation bits of the two-part calls.  The kernels with one tile of 32-bit digits are compiled for the
# digits that pb_act_prep leaves: these take each of them.
PREPARED = [(30, 21, 19, 8, 1, 32), (19, 17, 24, 6, 5, 32), (114, 1387, 37, 2, 1, 32), (666, 1345, 33, 10, 5, 32), (151, 9063, 13, 8, 8, 32),
            (1231, 1155, 66, 5, 1, 32), (2437, 1135, 393, 1, 1, 32), (700, 1500, 21, 6, 6, 16), (700, 1500, 21, 6, 6, 8)]


@pytest.mark.parametrize("layout", [BITS, PAIRS])
@pytest.mark.parametrize("case", PREPARED, ids=lambda c: "x".join(map(str, c[:3])) + "-%d/%d-a%d" % (c[4], c[3], c[5]))
def test_prepared_digits(pb, case, layout):
    """pb_act_prep and pb_matmul_prepared give what pb_matmul gives, whichever kernel reads the digits, and leave them as they are: two
    matrices on the activations of one preparation."""
    R, C, N, bits, m, act_bits = case
    print("prepared", case, hex(layout), flush=True)
    g = np.random.default_rng(200300822 + 71)
    X = g.normal(size=(N, C)).astype(np.float32)
    if act_bits == 32: widen(X, (0, C // 2, C - 1))
    frac_bits = {32: 16, 16: 12, 8: 4}[act_bits]
    xq = po.fixed_point(X, frac_bits=frac_bits, act_bits=act_bits)
    Xd, first = dev(X), None
    for rows in (R, 2 * R + 5):
        W = g.normal(0, 0.02, size=(rows, C)).astype(np.float32)
        lin = pb.PackedLinear(dev(W), bits, max_batch=N, act_bits=act_bits, frac_bits=frac_bits, layout=layout)
        if first is None:
            first = lin
            pb.pb_act_prep(lin.desc, Xd, N, lin.workspace)
        Y = torch.empty((N, rows), device="cuda")
        pb.pb_matmul_prepared(lin.packed, lin.scales, lin.desc, m, N, Y, first.workspace)
        own = torch.empty_like(lin.workspace)
        want = torch.empty_like(Y)
        pb.pb_matmul(lin.packed, lin.scales, lin.desc, m, Xd, N, want, own)
        assert torch.equal(Y, want)
        sample = sorted({0, 1, rows // 2, rows - 1})
        prep = po.prepare(W[sample + [int(np.abs(W).max(axis=1).argmax())]], bits)
        for k, r in enumerate(sample):
            sub = po.layer_products_direct(prep["layers"][:, k:k + 1, :], m, xq)[:, :, 0]
            assert_y_close(Y.cpu().numpy()[:, r], po.dequant(sub, prep["scales"], m, frac_bits=frac_bits), sub, prep["scales"], frac_bits=frac_bits)


# hidden units, inputs, vectors, activation bits, bits, used; from the second line on: each compiled kernel with the cell update
CELLS = [
    (37, 100, 2, 32, 5, 5), (300, 701, 40, 32, 5, 5), (500, 1500, 100, 16, 5, 5), (600, 79, 11, 8, 5, 5), (40, 1301, 5, 8, 5, 5),
    (200, 601, 1, 32, 5, 5), (1500, 1500, 64, 8, 5, 5), (1500, 1500, 64, 32, 5, 5),
    # many digit rows
    (575, 39, 219, 32, 2, 1), (487, 31, 514, 32, 3, 1), (92, 18, 695, 32, 15, 15), (1036, 46, 449, 32, 12, 1), (485, 41, 272, 32, 15, 15),
    (492, 40, 375, 16, 14, 4), (313, 283, 202, 16, 11, 9), (516, 19, 993, 16, 5, 1), (212, 34, 981, 16, 9, 9), (1034, 89, 935, 16, 10, 1),
    (460, 55, 634, 16, 15, 15), (560, 18, 659, 8, 7, 3), (308, 286, 362, 8, 13, 12), (956, 98, 833, 8, 16, 1), (254, 318, 651, 8, 15, 15),
    (2087, 57, 863, 8, 1, 1), (608, 20, 837, 8, 16, 15),
    # four tiles per wave
    (1365, 177, 9, 32, 5, 5), (1027, 23, 29, 32, 2, 1), (465, 49, 155, 16, 7, 1), (293, 230, 433, 8, 10, 1),
    # one tile, digits from memory
    (1030, 25, 13, 32, 11, 5), (715, 335, 21, 32, 1, 1), (1029, 35, 9, 16, 5, 5), (516, 18, 41, 16, 1, 1), (17, 1528, 17, 8, 14, 5),
    (16, 2153, 13, 8, 4, 1),
    # two tiles, converted in the launch
    (34, 17, 948, 32, 7, 5), (41, 17, 856, 32, 1, 1), (599, 16, 9, 16, 7, 5), (513, 16, 9, 16, 14, 1), (517, 19, 17, 8, 5, 5),
    (518, 20, 17, 8, 4, 1),
    # one tile, converted in the launch
    (16, 16, 2, 32, 8, 1), (16, 17, 2, 16, 15, 5), (16, 16, 2, 16, 13, 1), (16, 17, 2, 8, 9, 1),
    # 32-bit digits from memory, several groups of vectors and chunks of columns: one tile, four, many digit rows
    (342, 1593, 41, 32, 4, 1), (546, 635, 33, 32, 6, 5), (525, 1329, 47, 32, 13, 1), (458, 708, 69, 32, 11, 5), (531, 1008, 113, 32, 4, 1),
    (784, 338, 253, 32, 4, 1), (191, 1553, 53, 32, 15, 15), (140, 1016, 295, 32, 15, 15),
]


@pytest.mark.parametrize("H,I,N,act_bits,bits,m", CELLS)
def test_lstm_cell_of_a_batch(pb, H, I, N, act_bits, bits, m):
    """The cell update at the end of every kernel, the second part of the input also at odd columns, in the chunk where it
    begins and in the chunks behind (2e-6: the bound of the other cell tests).  With 32 bits most groups of sixteen vectors have a value
    beyond three byte digits, in a column of x or of h whose weights are small, so that few gates saturate."""
    g = np.random.default_rng(200300822 + 61)
    frac_bits = {32: 16, 16: 12, 8: 4}[act_bits]
    W = g.uniform(-0.04, 0.04, size=(4 * H, I + H)).astype(np.float32)
    x, h, c = (g.normal(size=(N, n)).astype(np.float32) for n in (I, H, H))
    if act_bits == 32:
        wide = (0, I + H // 2, I + H - 1)
        W[:, wide] *= 0.1
        xh = np.concatenate([x, h], axis=1)
        widen(xh, wide)
        x, h = np.ascontiguousarray(xh[:, :I]), np.ascontiguousarray(xh[:, I:])
    bias = g.normal(0, 0.1, size=4 * H).astype(np.float32)
    prep = po.prepare(W, bits)
    _, Y = po.matmul_words(po.pack_words(prep["layers"]), prep["scales"], m, I + H, np.concatenate([x, h], axis=1),
                           frac_bits=frac_bits, act_bits=act_bits)
    h_ref, c_ref = po.lstm_pointwise(Y, bias, c)
    for lay in (GATES, BITS):
        lin = pb.PackedLinear(dev(W), bits, max_batch=N, act_bits=act_bits, frac_bits=frac_bits, layout=lay)
        ho, co = (torch.empty((N, H), dtype=torch.float32, device="cuda") for _ in range(2))
        pb.pb_lstm_cell(lin.packed, lin.scales, lin.desc, m, dev(x), I, dev(h), dev(c), dev(bias), ho, co, N, lin.workspace)
        assert np.abs(ho.cpu().numpy() - h_ref).max() <= 2e-6
        assert np.abs(co.cpu().numpy() - c_ref).max() <= 2e-6


def test_calls_of_one_layer_on_two_streams(pb):
    """The digits of a batch travel through a workspace: calls of one layer on two streams must not share it."""
    R, C, N = 4000, 3000, 128
    W, X = synth.ragged(R, C, batch=N, case=790, xdist="normal")
    lin = pb.PackedLinear(dev(W), 8, max_batch=N)
    Xs = [dev(X), dev(X[::-1].copy())]
    want = [lin(x).clone() for x in Xs]
    torch.cuda.synchronize()
    streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
    got = [[], []]
    for _ in range(20):
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                got[i].append(lin(Xs[i]))
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(y, want[i]) for y in got[i])


def test_two_threads_on_one_stream_and_workspace(pb):
    """The launches of a call stay together: no thread's product reads the digits of the other's."""
    R, C, N = 2000, 3000, 64
    W, X = synth.ragged(R, C, batch=N, case=793, xdist="normal")
    lin = pb.PackedLinear(dev(W), 8, max_batch=N)
    Xs = [dev(X), dev(X[::-1].copy())]
    want = [lin(x).clone() for x in Xs]
    got = [[torch.empty_like(w) for _ in range(30)] for w in want]
    start = threading.Barrier(2)

    def work(i):
        start.wait()
        for k, y in enumerate(got[i]):
            if k % 2:
                lin(Xs[i], out=y)
            else:
                pb.pb_matmul(lin.packed, lin.scales, lin.desc, 8, Xs[i], N, y, lin.workspace)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(y, want[i]) for y in got[i])


def test_a_captured_call_has_a_workspace_of_its_own(pb):
    """A graph may be replayed on any stream, beside other calls of the layer: also a call that is captured on the layer's
    own stream must not write the workspace that eager calls use."""
    R, C, N = 2000, 3000, 64                            # the digits travel through memory
    W, X = synth.ragged(R, C, batch=N, case=791, xdist="normal")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        lin = pb.PackedLinear(dev(W), 8, max_batch=N)
        Xd = dev(X)
        want = lin(Xd).clone()
        Y = torch.zeros_like(want)
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            lin(Xd, out=Y)
        lin.workspace.fill_(0xA5)
    side.synchronize()
    for _ in range(3):
        Y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want)
    assert (lin.workspace == 0xA5).all()


@pytest.mark.parametrize("R,C,N", [(40, 700, 3), (2000, 3000, 64)])
def test_zero_sums_keep_their_sign(pb, R, C, N):
    """A sum of zeros is +0 whatever the signs of the scales: the fp64 sum starts at +0."""
    W, _ = synth.ragged(R, C, batch=N, case=792, xdist="normal")
    for bits in (1, 5, 12):
        for layout in (BITS, PAIRS):
            lin = pb.PackedLinear(dev(W), bits, max_batch=N, layout=layout)
            halving = lin.scales.clone()
            uneven = halving.clone()
            uneven[0] *= 1.5
            for scales in (halving, uneven):
                lin.scales.copy_(-scales)
                assert (lin(torch.zeros((N, C), device="cuda")).view(torch.int32) == 0).all(), (bits, hex(layout))
