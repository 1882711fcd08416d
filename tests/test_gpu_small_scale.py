"""A of a magnitude whose squares underflow in FP32: the column norm bound of the short IHT
steps must not fall below the norms.  Scaling A and x by powers of two must not change the
supports (their values it may, in the last bits: A_k g_T comes near the end of the range in a
few columns, in the full pass too).
The problem is one where a bound that lost its small terms keeps a wrong support:

U is close to the unit vector of the only support entry w, so the projected column
Pi A_w is short and the step length large; the step then replaces w by j, although ||u|| is
small against s_w.  All entries of A are +-1, but one is 4: of their squares at 2^-76 it alone
is not rounded to zero, 4 where the norms are 20.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return _t


@pytest.mark.parametrize("q", [8, 130])   # with row splits of A_k U, and without
def test_bound_holds_where_squares_underflow(lib, torch, q):
    n, m, w, j = 64, 400, 20, 41
    rng = np.random.default_rng(q)
    At = rng.choice([-1.0, 1.0], size=(q, n, m)).astype(np.float32)
    At[:, 3, 7] *= 4.0
    v = rng.standard_normal(n)
    v[[w, j]] = 0.0
    U = 0.1 * v / np.linalg.norm(v)
    U[w] = 1.0
    U = (U / np.linalg.norm(U)).astype(np.float32).reshape(n, 1)
    Y = (At[:, w] + 0.02 * At[:, j]).astype(np.float32)
    res = []
    for a, x in ((0, 0), (-76, 110)):
        A = torch.from_numpy(np.ldexp(At, a)).cuda()
        Yd = torch.from_numpy(np.ldexp(Y, a + x)).cuda()
        Ud = torch.from_numpy(U).cuda()
        prob = lib.make_problem(A, Yd, 1, 1, m=m, U_start=Ud)
        par = lib.default_params(t_max=4, power_iters=0, tau=1)
        ws = torch.empty(lib.altgdmin_workspace_bytes(prob, par), dtype=torch.uint8, device="cuda")
        h = lib.altgdmin_init(prob, par, ws)
        idx, val = torch.empty(q, 1, dtype=torch.int32, device="cuda"), torch.empty(q, 1, device="cuda")
        try:
            lib.altgdmin_step(h, 1)
            lib.altgdmin_get(h, None, None, idx, val)
        finally:
            lib.altgdmin_destroy(h)
        res.append(idx.cpu().numpy())
    assert (res[0] == j).all()   # the step does replace the support
    assert np.array_equal(res[1], res[0])
