"""IHT steps that provably keep their support read the support columns alone: the
iteration of a solver (whose A_k U kernel hands the column kernel a column norm
bound) against the step-level entry points (which have no bound and take the full
pass in every step) from the same U and S.  The two must agree bit for bit, on
iterations where no step qualifies, where some do and where all do."""
import numpy as np
import pytest

from paper_2311_03824_amd import instances as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return _t


def build(lib, torch, form, cfg, wide_column):
    kw = {"bf16_planes": True} if form == "bf16x2" else {"a_form": "philox"} if form == "philox" else {}
    inst = I.make_instance(**cfg, **kw)
    n, q, m, r, rho = inst.n, inst.q, inst.m, inst.r, inst.rho
    Y = torch.from_numpy(inst.Y32).cuda()
    if form == "philox":
        table = torch.from_numpy(inst.table).cuda()
        return inst, lib.make_problem(None, Y, r, rho, m=m, philox_seed=inst.a_seed, normal_table=table, n=n), (Y, table)
    if form == "bf16x2":
        hi = torch.from_numpy(inst.A_hi.view(np.int16)).cuda()
        lo = torch.from_numpy(inst.A_lo.view(np.int16)).cuda()
        return inst, lib.make_problem(hi, Y, r, rho, A_lo=lo, m=m), (Y, hi, lo)
    At = inst.At.copy()
    if wide_column:   # one column outside every support (its S* and U* rows are zeroed) with a huge norm
        At[:, n - 1, :m] *= 50.0
        X = inst.X_star.copy()
        X[n - 1] = 0.0
        Y = torch.from_numpy(np.einsum("kji,jk->ki", At[:, :, :m].astype(np.float64), X).astype(np.float32)).cuda()
    A = torch.from_numpy(At).cuda()
    return inst, lib.make_problem(A, Y, r, rho, m=m), (Y, A)


# one to four row chunks, ragged m and n, rho = 1, rho at and above the n / 4 limit of the short steps,
# P_k in LDS and in global memory
CASES = [
    ("f32", dict(n=100, q=12, m=40, r=2, rho=2, seed=11), False),
    ("f32", dict(n=131, q=9, m=63, r=1, rho=1, seed=12), False),
    ("f32", dict(n=90, q=8, m=81, r=2, rho=22, seed=13), False),
    ("f32", dict(n=90, q=8, m=81, r=2, rho=23, seed=14), False),
    ("f32", dict(n=310, q=10, m=301, r=7, rho=19, seed=15), False),
    ("f32", dict(n=601, q=6, m=518, r=10, rho=70, seed=16), False),
    ("f32", dict(n=1100, q=5, m=1020, r=16, rho=90, seed=17), False),
    ("f32", dict(n=200, q=12, m=100, r=3, rho=5, seed=18), True),
    ("bf16x2", dict(n=310, q=10, m=301, r=7, rho=19, seed=19), False),
    ("philox", dict(n=150, q=8, m=101, r=3, rho=6, seed=20), False),
]


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("form,cfg,wide_column", CASES)
def test_iteration_equals_full_passes(lib, torch, monkeypatch, form, cfg, wide_column, waves):
    monkeypatch.setenv("ALTGDMIN_COL_WAVES", str(waves))
    inst, prob, keep = build(lib, torch, form, cfg, wide_column)
    n, q, m, r, rho = inst.n, inst.q, inst.m, inst.r, inst.rho
    # a subspace close to U* with a short step: S settles within a few iterations
    start = torch.from_numpy((inst.U_star + 1e-4 / np.sqrt(n) * inst.U_start).astype(np.float32)).cuda()
    prob.U_start = lib.ptr(start)
    par = lib.default_params(t_max=64, power_iters=0, eta_c=5e-5)
    ws = torch.empty(lib.altgdmin_workspace_bytes(prob, par), dtype=torch.uint8, device="cuda")
    h = lib.altgdmin_init(prob, par, ws)
    try:
        def state():
            o = dict(U=torch.empty(n, r, device="cuda"), Bt=torch.empty(q, r, device="cuda"),
                     S_idx=torch.empty(q, rho, dtype=torch.int32, device="cuda"),
                     S_val=torch.empty(q, rho, device="cuda"), U_next=torch.empty(n, r, device="cuda"))
            lib.altgdmin_get(h, o["U"], o["Bt"], o["S_idx"], o["S_val"], o["U_next"])
            return o

        for ahead in (0, 1, 1, 2, 4, 12, 20):   # iterations 1, 2, 3, 5, 9, 21, 41 are compared
            if ahead > 1:
                lib.altgdmin_step(h, ahead - 1)
            s = state()
            P = torch.empty(q, m, r, device="cuda")
            Gi = torch.empty(q, r, r, dtype=torch.float64, device="cuda")
            lib.altgdmin_op_au(prob, s["U_next"], P, Gi)
            lib.altgdmin_op_iht(prob, True, P, Gi, par.tau, True, s["S_idx"], s["S_val"])
            Bt, H = torch.empty(q, r, device="cuda"), torch.empty(q, n, device="cuda")
            lib.altgdmin_op_lsgrad(prob, P, Gi, s["S_idx"], s["S_val"], Bt, H)
            lib.altgdmin_step(h, 1)
            got = state()
            assert torch.equal(got["U"], s["U_next"])
            assert torch.equal(got["S_idx"], s["S_idx"])
            assert torch.equal(got["S_val"], s["S_val"])
            assert torch.equal(got["Bt"], Bt)
        if not wide_column:   # IHT does not settle with a column 50 times longer; there only the equality counts
            assert lib.altgdmin_status(h)["resid"] < 1e-3   # S has settled: the last iterations take the short steps
    finally:
        lib.altgdmin_destroy(h)
