"""The spectral starts with a part of their workgroups: the roll is closed after a wait forced
from the host (at once, or soon), so the work is done by whichever workgroups have come.  The
result does not depend on how many those are."""
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


@pytest.mark.parametrize("n,q,r", [(40, 17, 2), (65, 130, 5), (1000, 1000, 10), (6500, 40, 8), (333, 1700, 16)])
def test_real_start_with_few_workgroups(lib, torch, monkeypatch, n, q, r):
    g = torch.Generator("cuda").manual_seed(n + q)
    L0t = torch.randn(q, n, generator=g, device="cuda")
    start = torch.randn(n, r, generator=g, device="cuda")
    its = torch.empty(1, dtype=torch.int32, device="cuda")

    def run():
        U = torch.full((n, r), float("nan"), device="cuda")
        lib.altgdmin_op_subspace(L0t, r, start, 5, 0.0, U, its)
        return U, int(its.item())

    ref, steps = run()
    for us in ("0", "0", "1", "2", "5", "1000"):
        monkeypatch.setenv("ALTGDMIN_START_GRACE_US", us)
        U, k = run()
        assert torch.equal(U, ref) and k == steps


@pytest.mark.parametrize("n1,n2,q,r", [(4, 15, 30, 2), (20, 20, 300, 4), (48, 64, 40, 8)])
def test_fourier_start_with_few_workgroups(lib, torch, monkeypatch, n1, n2, q, r):
    n, m = n1 * n2, n1 * n2 // 2
    g = torch.Generator("cuda").manual_seed(n)
    mask = torch.sort(torch.topk(torch.rand(q, n, generator=g, device="cuda"), m, 1).indices, 1).values.int().contiguous()
    Y = torch.randn(q, m, generator=g, device="cuda", dtype=torch.complex64)
    prob = lib.make_fourier_problem(mask, Y, n1, n2, r, 2)
    par = lib.default_params(t_max=4, power_iters=5, power_tol=0.0)
    ws = torch.empty(lib.altgdmin_workspace_bytes(prob, par), dtype=torch.uint8, device="cuda")
    out = []
    for us in (None, "0", "0", "1", "3", "1000"):
        if us is not None:
            monkeypatch.setenv("ALTGDMIN_START_GRACE_US", us)
        h = lib.altgdmin_init(prob, par, ws)
        U = torch.empty(n, r, dtype=torch.complex64, device="cuda")
        lib.altgdmin_get(h, None, None, None, None, U)
        rep = lib.altgdmin_status(h)
        lib.altgdmin_destroy(h)
        out.append((U, rep["power_iterations"], rep["error_flags"]))
    for U, k, err in out[1:]:
        assert torch.equal(U, out[0][0]) and k == out[0][1] and err == out[0][2] == 0


def test_many_starts_at_once(lib, torch, monkeypatch):
    """Twelve streams of 96-workgroup starts, mostly with a short wait, beside each other."""
    n, q, r = 3000, 1500, 8
    g = torch.Generator("cuda").manual_seed(3)
    L0t, start = torch.randn(q, n, generator=g, device="cuda"), torch.randn(n, r, generator=g, device="cuda")
    sc = [torch.empty(lib.altgdmin_op_scratch_bytes(n, q, r) + 256, dtype=torch.uint8, device="cuda") for _ in range(12)]
    ref = torch.empty(n, r, device="cuda")
    lib.altgdmin_op_subspace(L0t, r, start, 6, 0.0, ref, scratch=sc[0])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in sc]
    got = [torch.empty(n, r, device="cuda") for _ in sc]
    for i, st in enumerate(streams):
        monkeypatch.setenv("ALTGDMIN_START_GRACE_US", str((0, 10, 2000)[i % 3]))
        lib.altgdmin_op_subspace(L0t, r, start, 6, 0.0, got[i], scratch=sc[i], stream=st)
    torch.cuda.synchronize()
    for x in got:
        assert torch.equal(x, ref)


def test_solve_with_a_partial_roll(lib, torch, monkeypatch):
    inst = I.make_instance(n=100, q=100, m=40, r=2, rho=2, seed=1)
    res = []
    for us in (None, "0"):
        if us is not None:
            monkeypatch.setenv("ALTGDMIN_START_GRACE_US", us)
        s = lib.Solver(inst.At, inst.Y32, 40, 2, 2, lib.default_params(t_max=20), U_start=inst.U_start)
        s.init().step(20)
        res.append(s.get())
        s.close()
    for k in res[0]:
        assert np.array_equal(res[0][k], res[1][k])
