"""The block kernels of the automatic rank (products, FP64 Gram, Cholesky and inverse, each over
chunks and tiles) at the edges of their block widths b = K + 8, against the exact SVD: a matrix
with a geometric spectrum, sigma_i = 0.8^i, so the values converge by a factor of at least
0.8^(2 * 8) per step behind the extra columns; with 30 steps they are exact to the FP32 products,
(n / 16 + q / 16 + 40) 2^-24 of sigma_1.  And a block of rank 3, whose zero pivots must leave it finite.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return _t


# b = 9, 14, 14, 16, 17, 20, 32, 33, 88 (K = min(n, q, m) / 10); contractions of one to many 64-row stages with remainders
@pytest.mark.parametrize("n,q,K", [(10, 10, 1), (65, 127, 8), (129, 63, 9), (80, 127, 8), (129, 90, 9), (300, 200, 12), (257, 640, 24),
                                   (1001, 250, 25), (900, 810, 80)])
@pytest.mark.parametrize("full", [True, False])
def test_values_match_svd(lib, torch, n, q, K, full):
    if not full and K < 8:
        pytest.skip("a rank of 3 needs a wider block")
    m, K = 10 * K, max(1, min(n, q, 10 * K) // 10)
    rng = np.random.default_rng(n + q)
    p = min(n, q)
    sv = 0.8 ** np.arange(p)
    if not full:
        sv[3:] = 0.0
    L0 = (np.linalg.qr(rng.standard_normal((n, p)))[0] * sv) @ np.linalg.qr(rng.standard_normal((q, p)))[0].T
    L0t = np.ascontiguousarray(L0.T, dtype=np.float32)
    ref = np.linalg.svd(L0t.astype(np.float64), compute_uv=False)[:K]
    r = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.zeros(K, dtype=torch.float64, device="cuda")
    lib.altgdmin_op_rank(torch.from_numpy(L0t).cuda(), m, 0.65, 30, r, out)
    got = out.cpu().numpy()
    assert np.isfinite(got).all()
    tol = (n / 16 + q / 16 + 40) * U32
    # a pivot of Z^T Z at or below 1e-13 of the largest, (sigma_i / sigma_1)^4, is a zero direction: such values
    # may be lost, but are never overstated
    seen = ref > 1.1 * 1e-13 ** 0.25 * ref[0]
    assert np.abs(got - ref)[seen].max() <= tol
    assert (got <= ref + tol).all() and (got >= 0).all()
    cum = np.cumsum(ref ** 2) / np.sum(ref ** 2)
    assert int(r.item()) == int(np.argmax(cum >= 0.65)) + 1
