"""Solves with and without short IHT steps (ALTGDMIN_FULL_STEPS at init withholds the norm bound)
agree bit for bit in every real form, and the short steps do run."""
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


def build(lib, torch, form, cfg):
    kw = {"a_form": "philox"} if form == "philox" else {} if form == "f32" else {"bf16_planes": True}
    inst = I.make_instance(**cfg, **kw)
    Y = torch.from_numpy(inst.Y32).cuda()
    start = torch.from_numpy((inst.U_star + 1e-4 / np.sqrt(inst.n) * inst.U_start).astype(np.float32)).cuda()
    if form == "philox":
        table = torch.from_numpy(inst.table).cuda()
        prob = lib.make_problem(None, Y, inst.r, inst.rho, m=inst.m, philox_seed=inst.a_seed, normal_table=table,
                                n=inst.n, U_start=start)
        keep = (Y, table, start)
    elif form == "f32":
        A = torch.from_numpy(inst.At).cuda()
        prob, keep = lib.make_problem(A, Y, inst.r, inst.rho, m=inst.m, U_start=start), (Y, A, start)
    else:
        hi, lo = (torch.from_numpy(x.view(np.int16)).cuda() for x in (inst.A_hi, inst.A_lo))
        prob, keep = lib.make_problem(hi, Y, inst.r, inst.rho, A_lo=lo, m=inst.m, U_start=start), (Y, hi, lo, start)
    par = lib.default_params(t_max=64, power_iters=0, eta_c=5e-5)
    if form == "mixed":
        par.flags = lib.FLAG_BF16_MIXED
    if form == "hi_phase":
        par.bf16_hi_max = 6
    return inst, prob, par, keep


def handle(lib, torch, prob, par, monkeypatch, full):
    if full:
        monkeypatch.setenv("ALTGDMIN_FULL_STEPS", "1")
    else:
        monkeypatch.delenv("ALTGDMIN_FULL_STEPS", raising=False)
    ws = torch.empty(lib.altgdmin_workspace_bytes(prob, par), dtype=torch.uint8, device="cuda")
    return lib.altgdmin_init(prob, par, ws), ws


CASES = [dict(n=100, q=12, m=40, r=2, rho=2, seed=1), dict(n=310, q=10, m=301, r=7, rho=19, seed=2),
         dict(n=90, q=40, m=81, r=2, rho=22, seed=3), dict(n=601, q=6, m=518, r=10, rho=70, seed=4),
         dict(n=1100, q=5, m=1020, r=16, rho=90, seed=5)]


@pytest.mark.parametrize("form", ["f32", "bf16x2", "mixed", "hi_phase", "philox"])
@pytest.mark.parametrize("cfg", CASES)
def test_short_steps_change_no_bit(lib, torch, monkeypatch, form, cfg):
    inst, prob, par, keep = build(lib, torch, form, cfg)
    out = []
    for full in (False, True):
        h, ws = handle(lib, torch, prob, par, monkeypatch, full)
        try:
            res = []
            for _ in range(4):
                lib.altgdmin_step(h, 6)
                U, Bt = torch.empty(inst.n, inst.r, device="cuda"), torch.empty(inst.q, inst.r, device="cuda")
                Si = torch.empty(inst.q, inst.rho, dtype=torch.int32, device="cuda")
                Sv = torch.empty(inst.q, inst.rho, device="cuda")
                lib.altgdmin_get(h, U, Bt, Si, Sv)
                res += [U, Bt, Si, Sv]
            out.append([x.cpu().numpy() for x in res] + [lib.altgdmin_residual_log(h, 64)])
        finally:
            lib.altgdmin_destroy(h)
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_batched_short_steps_change_no_bit(lib, torch, monkeypatch):
    out = []
    probs = [build(lib, torch, f, c) for f, c in (("f32", CASES[1]), ("mixed", CASES[3]), ("philox", CASES[0]))]
    for full in (False, True):
        hs, wss = zip(*(handle(lib, torch, p[1], p[2], monkeypatch, full) for p in probs))
        try:
            grp = torch.empty(lib.altgdmin_group_bytes(list(hs)), dtype=torch.uint8, device="cuda")
            lib.altgdmin_step_many(list(hs), 20, grp)
            res = []
            for h, (inst, *_rest) in zip(hs, probs):
                U, Sv = torch.empty(inst.n, inst.r, device="cuda"), torch.empty(inst.q, inst.rho, device="cuda")
                lib.altgdmin_get(h, U, None, None, Sv)
                res += [U.cpu().numpy(), Sv.cpu().numpy()]
            out.append(res)
        finally:
            for h in hs:
                lib.altgdmin_destroy(h)
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("form", ["f32", "mixed", "philox"])
def test_short_steps_run(lib, torch, monkeypatch, form):
    """Settled iterations at n = 1000, q = 125, m = 400: the column kernel takes at most three quarters of its
    time with full passes (about half in FP32)."""
    inst, prob, par, keep = build(lib, torch, form, dict(n=1000, q=125, m=400, r=10, rho=50, seed=6))
    ms = []
    for full in (False, True):
        h, ws = handle(lib, torch, prob, par, monkeypatch, full)
        try:
            lib.altgdmin_step(h, 30)
            ms.append(min(lib.altgdmin_profile_iteration(h, 8)["k_col"] for _ in range(5)))
        finally:
            lib.altgdmin_destroy(h)
    print(form, ms)
    assert ms[0] <= 0.75 * ms[1], ms
