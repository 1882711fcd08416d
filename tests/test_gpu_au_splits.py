"""A_k U with a column's rows split over several workgroups: P_k, and G_k^{-1} from the splits'
Grams, at the edges of the splits, against FP64.

Each entry of P_k is a sum of n products in FP32: within n 2^-24 of the sum of their magnitudes.
G_k is summed in FP64 from P_k as written, so G_k^{-1} G_k is the identity to r m 2^-53 times
the condition number (at most 1e4 here), 1e-8.
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


# one row over a chunk, ragged chunks, the last row count of two, three and four splits; q at the
# most columns that are split and one above; n below the waves that share it
@pytest.mark.parametrize("n,q,m,r", [(40, 3, 257, 1), (301, 128, 258, 4), (301, 129, 400, 10), (1000, 9, 512, 16),
                                     (5, 64, 513, 3), (130, 85, 768, 7), (130, 86, 769, 8), (700, 20, 1000, 10),
                                     (64, 2, 1024, 16)])
def test_rows_and_gram_match_fp64(lib, torch, n, q, m, r):
    g = torch.Generator("cuda").manual_seed(n + m)
    ld = (m + 3) // 4 * 4
    A = torch.randn(q, n, ld, generator=g, device="cuda")
    A[:, :, m:] = 0.0
    U = torch.linalg.qr(torch.randn(n, r, generator=g, device="cuda"))[0].contiguous() if n >= r else None
    prob = lib.make_problem(A, torch.randn(q, m, generator=g, device="cuda"), r, 1, m=m)
    P = torch.full((q, m, r), float("nan"), device="cuda")
    Gi = torch.full((q, r, r), float("nan"), dtype=torch.float64, device="cuda")
    flags = torch.zeros(q, dtype=torch.int32, device="cuda")
    lib.altgdmin_op_au(prob, U, P, Gi, flags)
    A64, U64 = A[:, :, :m].double().cpu().numpy(), U.double().cpu().numpy()
    got, ginv = P.double().cpu().numpy(), Gi.cpu().numpy()
    assert not flags.any().item()
    for k in range(q):
        want = A64[k].T @ U64
        assert (np.abs(got[k] - want) <= n * U32 * (np.abs(A64[k]).T @ np.abs(U64)) + 1e-30).all()
        assert np.abs(ginv[k] @ (got[k].T @ got[k]) - np.eye(r)).max() <= 1e-8
