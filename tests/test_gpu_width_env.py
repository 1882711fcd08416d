"""A handle keeps the A_k U width and row splits of its initialisation: a change of
ALTGDMIN_AU_WAVES between init and the iterations changes neither what they compute nor where
they write."""
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


@pytest.mark.parametrize("how", ["step", "step_many", "profile"])
@pytest.mark.parametrize("first,then", [("4", None), ("8", "4")])
def test_width_is_taken_at_init(lib, torch, monkeypatch, how, first, then):
    n, q, m, r, rho = 120, 9, 301, 3, 4
    inst = I.make_instance(n=n, q=q, m=m, r=r, rho=rho, seed=31)
    A, Y = torch.from_numpy(inst.At).cuda(), torch.from_numpy(inst.Y32).cuda()
    prob = lib.make_problem(A, Y, r, rho, m=m)
    par = lib.default_params(t_max=8, power_iters=20)
    got = []
    for change in (False, True):
        monkeypatch.setenv("ALTGDMIN_AU_WAVES", first)
        nb = lib.altgdmin_workspace_bytes(prob, par)
        ws = torch.zeros(nb + (1 << 20), dtype=torch.uint8, device="cuda")
        h = lib.altgdmin_init(prob, par, ws)
        if change and then is None:
            monkeypatch.delenv("ALTGDMIN_AU_WAVES")
        elif change:
            monkeypatch.setenv("ALTGDMIN_AU_WAVES", then)
        try:
            if how == "step":
                lib.altgdmin_step(h, 4)
            elif how == "profile":
                lib.altgdmin_profile_iteration(h, 4)
            else:
                grp = torch.empty(lib.altgdmin_group_bytes([h]), dtype=torch.uint8, device="cuda")
                lib.altgdmin_step_many([h], 4, grp)
            U, Bt = torch.empty(n, r, device="cuda"), torch.empty(q, r, device="cuda")
            Si, Sv = torch.empty(q, rho, dtype=torch.int32, device="cuda"), torch.empty(q, rho, device="cuda")
            lib.altgdmin_get(h, U, Bt, Si, Sv)
            assert lib.altgdmin_status(h)["error_flags"] == 0
            got.append([x.cpu().numpy() for x in (U, Bt, Si, Sv)])
            assert not ws[nb:].any().item()   # nothing beyond the workspace
        finally:
            lib.altgdmin_destroy(h)
    for a, b in zip(*got):
        assert np.array_equal(a, b)
