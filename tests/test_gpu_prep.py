"""The plane statistics of the AND + popcount path (largest and smallest activation decide which planes are multiplied)
against the oracle: widths around the rounds of loads, the extreme value at either end, NaN after it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pb_oracle as po

pytestmark = pytest.mark.gpu

ROWMAJOR = 0x50420001


@pytest.mark.parametrize("cols", [1, 3, 255, 257, 1023, 1025, 4099, 8191, 8193, 9000])
def test_extreme_values_decide_the_planes(cols):
    from paper_2003_00822_amd import pb
    assert pb.PB_LAYOUT_ROWMAJOR_V1 == ROWMAJOR
    g = np.random.default_rng(cols)
    W = g.normal(0, 0.05, size=(20, cols)).astype(np.float32)
    X = (g.normal(0, 0.01, size=(8, cols))).astype(np.float32)
    X[0, 0] = 1000.0
    X[1, 0] = -1000.0
    X[2, -1] = 30000.0
    X[3, -1] = -3.0e38
    X[4, -1] = np.inf
    X[5] = -np.abs(X[5]) * np.float32(1e-4)   # (some below one step of the fixed-point grid)
    X[6] = 0.0
    X[7, 0] = -70.0
    bits = X.view(np.int32)
    for n, c in ((0, 1), (1, 2), (7, cols // 2), (7, cols - 1)):   # NaN, quiet and signalling, behind the extreme value
        if 0 < c < cols:
            bits[n, c] = 0x7FA00000 if n else 0x7FC00000
    lin = pb.PackedLinear(torch.from_numpy(W).cuda(), 4, max_batch=8, layout=ROWMAJOR)
    prep = po.prepare(W, 4)
    Xref = np.where(np.isnan(X), np.float32(0), X)
    A_ref, _ = po.matmul_words(po.pack_words(prep["layers"]), prep["scales"], 4, cols, Xref)
    A = lin.acc(torch.from_numpy(bits).cuda().view(torch.float32)).cpu().numpy()
    assert (A == A_ref).all()
