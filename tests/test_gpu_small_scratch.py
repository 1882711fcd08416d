"""The U-side entry points with the least scratch they take (control block, column splits, one n x r
and one q x r block): the forms that need no room for Gram parts, against FP64."""
import numpy as np
import pytest

from oracle import altgdmin_oracle as O

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return _t


def least_scratch(n, q, r):
    up = lambda b: (b + 255) // 256 * 256
    splits = 4 if q >= 512 else 2 if q >= 64 else 1
    return 256 + up(4 * splits * n * r) + up(4 * n * r) + 4 * q * r


@pytest.mark.parametrize("n,q,r", [(1, 1, 1), (16, 3, 16), (63, 64, 3), (65, 600, 5), (300, 4500, 16), (2100, 40, 8)])
def test_subspace(lib, torch, n, q, r):
    rng = np.random.default_rng(n + q)
    L0 = rng.standard_normal((n, r)) @ rng.standard_normal((r, q)) + 0.1 * rng.standard_normal((n, q))
    L0t, start = np.ascontiguousarray(L0.T, dtype=np.float32), rng.standard_normal((n, r)).astype(np.float32)
    start[:, r - 1] = start[:, 0] + (1e-4 * start[:, r - 1] if r > 1 else 0)   # a second pass for the start block
    if r > min(n, q):
        L0t += 1.0 * np.eye(q, n, dtype=np.float32)
    nb = least_scratch(n, q, r)
    assert nb <= lib.altgdmin_op_scratch_bytes(n, q, r)
    sc = torch.zeros(nb + 4096, dtype=torch.uint8, device="cuda")
    U = torch.empty(n, r, device="cuda")
    its = torch.empty(1, dtype=torch.int32, device="cuda")
    steps = 2 if r <= min(n, q) else 0
    lib.altgdmin_op_subspace(torch.from_numpy(L0t).cuda(), r, torch.from_numpy(start).cuda(), steps, 0.0, U, its,
                             scratch=sc[:nb])
    assert not sc[nb:].any().item()
    Q, _ = O.qr_pos(start.astype(np.float64))
    L0 = L0t.T.astype(np.float64)
    # two CholeskyQR passes with FP64 Grams of rows given exactly, rounded after each
    amp = 4.0 * U32 * np.sqrt(r)
    for _ in range(steps):
        Z = L0 @ (L0.T @ Q)
        amp = amp * np.linalg.cond(Z) + (n / 16 + q / 16 + 40) * U32 * \
            np.linalg.norm(np.abs(L0) @ (np.abs(L0.T) @ np.abs(Q))) / np.linalg.svd(Z, compute_uv=False)[-1]
        Q, _ = O.qr_pos(Z)
    got = U.cpu().numpy().astype(np.float64)
    assert int(its.item()) <= steps
    assert np.abs(got.T @ got - np.eye(r)).max() <= 1e-6
    assert np.linalg.norm(got - Q) <= 4.0 * amp + 1e-6
    # less scratch than that is refused
    with pytest.raises(lib.AltGDminError):
        lib.altgdmin_op_subspace(torch.from_numpy(L0t).cuda(), r, torch.from_numpy(start).cuda(), steps, 0.0, U, its,
                                 scratch=sc[:nb - 1])


@pytest.mark.parametrize("n,r", [(1, 1), (16, 16), (255, 3), (257, 12), (3000, 8)])
@pytest.mark.parametrize("small,first", [(0.0, False), (0.0, True), (1e-4, False)])
def test_qr_step(lib, torch, n, r, small, first):
    rng = np.random.default_rng(n * 3 + r)
    U = O.qr_pos(rng.standard_normal((n, r)))[0].astype(np.float32)
    grad = 0.3 * rng.standard_normal((n, r)) / np.sqrt(n)
    if small > 0 and r > 1:   # U - grad with one direction of size 1e-4
        V = O.qr_pos(rng.standard_normal((n, r)))[0] @ np.diag(np.r_[np.ones(r - 1), small])
        grad = U - V
    grad = grad.astype(np.float32)
    nb = least_scratch(n, 1, r)
    sc = torch.zeros(nb + 4096, dtype=torch.uint8, device="cuda")
    eta = torch.full((1,), 0.0 if first else 1.0, dtype=torch.float64, device="cuda")
    Uo = torch.empty(n, r, device="cuda")
    lib.altgdmin_op_qr_step(torch.from_numpy(U).cuda(), torch.from_numpy(grad).cuda(), 0.14, eta, Uo, scratch=sc[:nb])
    assert not sc[nb:].any().item()
    e = 0.14 / np.linalg.norm(grad.astype(np.float64), 2) if first else 1.0
    assert abs(eta.item() - e) <= 1e-12 * e
    X = U.astype(np.float64) - e * grad.astype(np.float64)
    Q, _ = O.qr_pos(X)
    got = Uo.cpu().numpy().astype(np.float64)
    # X is rounded to FP32 before its first pass: 2^-24 sqrt(r) over its smallest singular value
    assert np.abs(got.T @ got - np.eye(r)).max() <= 1e-6
    assert np.linalg.norm(got - Q) <= 4.0 * U32 * np.sqrt(r) * (1.0 + 1.0 / np.linalg.svd(X, compute_uv=False)[-1])
    with pytest.raises(lib.AltGDminError):
        lib.altgdmin_op_qr_step(torch.from_numpy(U).cuda(), torch.from_numpy(grad).cuda(), 0.14, eta, Uo,
                                scratch=sc[:nb - 1])
