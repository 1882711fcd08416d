"""The U update over many workgroups (gradient rows, Gram parts, one factorisation,
U = X R^{-1}) at the edges of its row blocks, rank groups and column splits, and its
second pass on an ill-conditioned step, against FP64 references."""
import numpy as np
import pytest

from oracle import altgdmin_oracle as O
from paper_2311_03824_amd import instances as I

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return _t


# rows: below, at and above a 64-row block and a 256-row workgroup; ranks at the edges of
# the groups of four; columns: one split (at most 256), and several
@pytest.mark.parametrize("n,q,r", [(16, 3, 1), (63, 5, 4), (64, 65, 5), (65, 20, 8), (255, 256, 9), (256, 257, 12),
                                   (257, 400, 13), (130, 1100, 16), (1025, 17, 3)])
def test_iteration_updates_u_as_in_fp64(lib, torch, n, q, r):
    m = max(12, 2 * r)
    inst = I.make_instance(n=n, q=q, m=m, r=r, rho=1, seed=n * 7 + q)
    A, Y = torch.from_numpy(inst.At).cuda(), torch.from_numpy(inst.Y32).cuda()
    start = torch.from_numpy(inst.U_start).cuda()
    prob = lib.make_problem(A, Y, r, 1, m=m, U_start=start)
    par = lib.default_params(t_max=8, power_iters=0)
    ws = torch.empty(lib.altgdmin_workspace_bytes(prob, par), dtype=torch.uint8, device="cuda")
    h = lib.altgdmin_init(prob, par, ws)
    try:
        for _ in range(2):   # t = 1 sets eta, t = 2 uses it
            lib.altgdmin_step(h, 1)
            U, Un = torch.empty(n, r, device="cuda"), torch.empty(n, r, device="cuda")
            Bt, Si, Sv = (torch.empty(q, r, device="cuda"), torch.empty(q, 1, dtype=torch.int32, device="cuda"),
                          torch.empty(q, 1, device="cuda"))
            lib.altgdmin_get(h, U, Bt, Si, Sv, Un)
            P = torch.empty(q, m, r, device="cuda")
            Gi = torch.empty(q, r, r, dtype=torch.float64, device="cuda")
            B2, H = torch.empty(q, r, device="cuda"), torch.empty(q, n, device="cuda")
            lib.altgdmin_op_au(prob, U, P, Gi)
            lib.altgdmin_op_lsgrad(prob, P, Gi, Si, Sv, B2, H)
            assert torch.equal(B2, Bt)
            eta = lib.altgdmin_status(h)["eta"]
            H64, B64, U64 = (x.cpu().numpy().astype(np.float64) for x in (H, Bt, U))
            G = H64.T @ B64
            X = U64 - eta * G
            Q, _ = O.qr_pos(X)
            # the FP32 sum of grad (q / 64 serial terms per lane and the tree), then one rounding of U
            err_g = eta * (q / 64 + 32) * U32 * np.linalg.norm(np.abs(H64).T @ np.abs(B64))
            smin = np.linalg.svd(X, compute_uv=False)[-1]
            assert np.linalg.norm(Un.cpu().numpy() - Q) <= 4.0 * (err_g / smin + U32 * np.sqrt(r))
    finally:
        lib.altgdmin_destroy(h)


@pytest.mark.parametrize("n,r", [(40, 3), (300, 8), (1000, 16)])
def test_ill_conditioned_step_takes_a_second_pass(lib, torch, n, r):
    rng = np.random.default_rng(n + r)
    U = O.qr_pos(rng.standard_normal((n, r)))[0].astype(np.float32)
    # U - grad has singular values from 1 to 1e-4: pivots spanning 1e-8
    V = O.qr_pos(rng.standard_normal((n, r)))[0] @ np.diag(np.geomspace(1.0, 1e-4, r)) @ O.qr_pos(rng.standard_normal((r, r)))[0]
    grad = (U.astype(np.float64) - V).astype(np.float32)
    eta = torch.ones(1, dtype=torch.float64, device="cuda")
    Uo = torch.empty(n, r, device="cuda")
    lib.altgdmin_op_qr_step(torch.from_numpy(U).cuda(), torch.from_numpy(grad).cuda(), 0.14, eta, Uo)
    got = Uo.cpu().numpy().astype(np.float64)
    Q, _ = O.qr_pos(U.astype(np.float64) - grad.astype(np.float64))
    # cond^2 2^-53 r is 1e-8 * 1.8e-8 at most after the first pass; FP32 rounding afterwards
    assert np.abs(got.T @ got - np.eye(r)).max() <= 1e-6
    assert np.abs(got - Q).max() <= 1e-5


def test_singular_step_leaves_u(lib, torch):
    n, r = 100, 4
    U = O.qr_pos(np.random.default_rng(3).standard_normal((n, r)))[0].astype(np.float32)
    eta = torch.ones(1, dtype=torch.float64, device="cuda")
    Uo = torch.empty(n, r, device="cuda")
    lib.altgdmin_op_qr_step(torch.from_numpy(U).cuda(), torch.from_numpy(U).cuda(), 0.14, eta, Uo)   # U - U = 0
    assert np.array_equal(Uo.cpu().numpy(), U)
