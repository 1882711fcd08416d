"""A_k U in 8-wave workgroups on both sides of 256 workgroups, where the loads in flight change:
the same bits, and no step in time beyond the second workgroup of a CU."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return _t


def _problem(lib, torch, form, n, q, m, r):
    g = torch.Generator("cuda").manual_seed(n + m)
    A = torch.zeros(q, n, (m + 7) // 8 * 8, device="cuda")
    A[:, :, :m] = torch.randn(q, n, m, generator=g, device="cuda")
    Y = torch.randn(q, m, generator=g, device="cuda")
    if form == "f32":
        return lib.make_problem(A, Y, r, 2, m=m), (A, Y)
    hi = A.bfloat16()
    lo = (A - hi.float()).bfloat16()
    hi, lo = hi.view(torch.int16), lo.view(torch.int16)
    return lib.make_problem(hi, Y, r, 2, A_lo=lo, m=m), (hi, lo, Y)


@pytest.mark.parametrize("form", ["f32", "bf16x2"])
@pytest.mark.parametrize("n,m,r", [(7, 16, 1), (130, 65, 4), (301, 100, 7), (90, 256, 10), (75, 120, 16)])
def test_depths_give_the_same_bits(lib, torch, form, n, m, r):
    out = []
    for q in (257, 20):   # a column's P_k and Gram depend on its own A_k alone
        prob, keep = _problem(lib, torch, form, n, 257, m, r)
        prob.q = q
        U = torch.randn(n, r, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
        P, Gi = torch.empty(q, m, r, device="cuda"), torch.empty(q, r, r, dtype=torch.float64, device="cuda")
        lib.altgdmin_op_au(prob, U, P, Gi)
        out.append((P[:20].clone(), Gi[:20].clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_no_step_in_time_above_one_workgroup_per_cu(lib, torch):
    """n = 300, m = 100, r = 7: 23 us at 256 columns, 26 at 300 (39 with the depth of one workgroup per CU)."""
    ms = {}
    for q in (256, 300):
        prob, keep = _problem(lib, torch, "f32", 300, q, 100, 7)
        par = lib.default_params(t_max=200, power_iters=2)
        ws = torch.empty(lib.altgdmin_workspace_bytes(prob, par), dtype=torch.uint8, device="cuda")
        h = lib.altgdmin_init(prob, par, ws)
        try:
            lib.altgdmin_profile_iteration(h, 3)
            ms[q] = min(lib.altgdmin_profile_iteration(h, 8)["k_au"] for _ in range(6))
        finally:
            lib.altgdmin_destroy(h)
    assert ms[300] <= 1.45 * ms[256], ms
