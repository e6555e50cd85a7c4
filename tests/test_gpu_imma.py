"""The kernels on the 8-bit integer matrix cores (csrc/pb_imma.hip, csrc/pb_imma_tile.hip) at the edges of their tiles: every way
the launcher can choose, rows and columns that do not fill the last tile, batches that leave digit rows empty, groups of
bitlayers that share a code and groups of one, activations saturated at both ends.  Oracle: the definition of the
per-bitlayer sums on sampled rows (exact integers), then the scales in fp64."""
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
    prep = po.prepare(W, bits)
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
    rows = sorted({0, 1, R // 2, (R - 1) // 16 * 16, R - 1} | set(range(min(R, 20))))
    for r in rows:
        sub = po.layer_products_direct(prep["layers"][:, r:r + 1, :], m, xq)[:, :, 0]      # [m, N]
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
    (2100, 5000, 18, 7, 7, 32, 16),      # many digit rows, each shape of the kernel for them
    (6000, 7871, 18, 7, 7, 16, 8),
    (2000, 3000, 64, 8, 8, 32, 16),
    (4778, 6480, 13, 8, 5, 32, 16),
    (9000, 9000, 16, 6, 6, 32, 16),
    (2620, 2697, 713, 8, 8, 32, 16),
    (9347, 975, 686, 2, 1, 32, 16),
    (1500, 1600, 70, 12, 11, 32, 16),    # two groups per row tile there
    (1128, 1711, 71, 16, 16, 32, 16),    # three
]


@pytest.mark.parametrize("layout", [BITS, PAIRS])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:3])) + "-%d/%d-a%d" % (c[4], c[3], c[5]))
def test_every_way(pb, case, layout):
    R, C, N, bits, m, act_bits, frac_bits = case
    print("way", case, hex(layout), flush=True)
    check(pb, R, C, N, bits, m, act_bits, frac_bits, layout, sums=R * N < 200000)


@pytest.mark.parametrize("H,I,N,act_bits", [(37, 100, 2, 32), (300, 701, 40, 32), (500, 1500, 100, 16), (600, 79, 11, 8),
                                            (40, 1301, 5, 8), (200, 601, 1, 32), (1500, 1500, 64, 8), (1500, 1500, 64, 32)])
def test_lstm_cell_of_a_batch(pb, H, I, N, act_bits):
    """The cell update at the end of every kernel, the second part of the input also at odd columns, in the chunk where it
    begins and in the chunks behind (2e-6: the bound of the other cell tests)."""
    g = np.random.default_rng(200300822 + 61)
    frac_bits = {32: 16, 16: 12, 8: 4}[act_bits]
    W = g.uniform(-0.04, 0.04, size=(4 * H, I + H)).astype(np.float32)
    x, h, c = (g.normal(size=(N, n)).astype(np.float32) for n in (I, H, H))
    bias = g.normal(0, 0.1, size=4 * H).astype(np.float32)
    prep = po.prepare(W, 5)
    _, Y = po.matmul_words(po.pack_words(prep["layers"]), prep["scales"], 5, I + H, np.concatenate([x, h], axis=1),
                           frac_bits=frac_bits, act_bits=act_bits)
    h_ref, c_ref = po.lstm_pointwise(Y, bias, c)
    for lay in (GATES, BITS):
        lin = pb.PackedLinear(dev(W), 5, max_batch=N, act_bits=act_bits, frac_bits=frac_bits, layout=lay)
        ho, co = (torch.empty((N, H), dtype=torch.float32, device="cuda") for _ in range(2))
        pb.pb_lstm_cell(lin.packed, lin.scales, lin.desc, 5, dev(x), I, dev(h), dev(c), dev(bias), ho, co, N, lin.workspace)
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
