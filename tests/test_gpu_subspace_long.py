"""The subspace iteration's L_0^T U over long columns against FP64: its FP32 sums stay short."""
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


# One step at r = 1, q = 16, so that the sums over rows are what rounds.  A sum of K rounded terms of random sign
# is off by about sqrt(K / 2) / sqrt(3) units of 2^-24 of its size: 16 products in L_0^T U (1.6 units), 16 columns in
# Z (1.6), and the stores of U_0, T, Z and U (0.6 each, 1.2 together): 2.6 units, allowed 5.  Sums of n / 32 =
# 625 products in a row would be 10 units.
@pytest.mark.parametrize("n", [19999, 20000])
def test_long_columns_round_like_short_ones(lib, torch, n):
    q, err = 16, []
    for seed in range(8):
        rng = np.random.default_rng(seed)
        L0t = rng.standard_normal((q, n)).astype(np.float32)
        start = rng.standard_normal((n, 1)).astype(np.float32)
        U = torch.empty(n, 1, device="cuda")
        lib.altgdmin_op_subspace(torch.from_numpy(L0t).cuda(), 1, torch.from_numpy(start).cuda(), 1, 0.0, U)
        L0 = L0t.T.astype(np.float64)
        z = L0 @ (L0.T @ start.astype(np.float64))
        z /= np.linalg.norm(z)
        err.append(np.linalg.norm(U.cpu().numpy().astype(np.float64) - z))
    assert np.sqrt(np.mean(np.square(err))) <= 5.0 * U32, err
