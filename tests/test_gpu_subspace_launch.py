"""The subspace iteration in one launch (workgroups that meet at a counter): the edges of its
row units, column groups and splits against FP64, and several launches at once."""
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


def _l0(n, q, r, seed):
    rng = np.random.default_rng(seed)
    L0 = rng.standard_normal((n, r)) @ rng.standard_normal((r, q)) + 0.1 * rng.standard_normal((n, q))
    return np.ascontiguousarray(L0.T, dtype=np.float32), rng.standard_normal((n, r)).astype(np.float32)


# one and several workgroups, 16-column groups and 64-row units with remainders, column splits
# (q >= 64 with more workgroups than row units), more units than workgroups, r at its ends
@pytest.mark.parametrize("n,q,r", [(1, 1, 1), (5, 3, 2), (63, 16, 3), (64, 17, 4), (65, 130, 5), (200, 1000, 16),
                                   (1000, 1000, 10), (6500, 40, 8), (333, 1700, 12)])
def test_fixed_steps_match_fp64(lib, torch, n, q, r):
    L0t, start = _l0(n, q, r, n + q + r)
    U = torch.empty(n, r, device="cuda")
    its = torch.empty(1, dtype=torch.int32, device="cuda")
    steps = 2
    lib.altgdmin_op_subspace(torch.from_numpy(L0t).cuda(), r, torch.from_numpy(start).cuda(), steps, 0.0, U, its)
    Q, _ = O.qr_pos(start.astype(np.float64))
    L0 = L0t.T.astype(np.float64)
    amp = 0.0
    for _ in range(steps):
        Z = L0 @ (L0.T @ Q)
        # FP32 sums of n then q terms, at worst 2^-24 per term, against the smallest direction of Z
        amp += (n / 16 + q / 16 + 40) * U32 * np.linalg.norm(np.abs(L0) @ (np.abs(L0.T) @ np.abs(Q))) / \
            np.linalg.svd(Z, compute_uv=False)[-1]
        Q, _ = O.qr_pos(Z)
    got = U.cpu().numpy().astype(np.float64)
    assert 1 <= int(its.item()) <= steps
    assert np.linalg.norm(got - Q) <= 4.0 * amp + 1e-6
    assert np.abs(got.T @ got - np.eye(r)).max() <= 1e-6


def test_launches_on_several_streams_at_once(lib, torch):
    """Four streams, each with its own buffers, against the same calls one after the other."""
    n, q, r = 3000, 1500, 8
    data = [tuple(torch.from_numpy(x).cuda() for x in _l0(n, q, r, 50 + i)) for i in range(4)]
    sc = [torch.empty(lib.altgdmin_op_scratch_bytes(n, q, r) + 256, dtype=torch.uint8, device="cuda") for _ in data]

    def call(i, out, stream=None):
        lib.altgdmin_op_subspace(data[i][0], r, data[i][1], 12, 1e-6, out, scratch=sc[i], stream=stream)

    ref = [torch.empty(n, r, device="cuda") for _ in data]
    for i in range(4):
        call(i, ref[i])
    torch.cuda.synchronize()
    got = [torch.empty(n, r, device="cuda") for _ in data]
    streams = [torch.cuda.Stream() for _ in data]
    for _ in range(3):
        for i in range(4):
            call(i, got[i], streams[i])
    torch.cuda.synchronize()
    for i in range(4):
        assert torch.equal(got[i], ref[i])


def test_rank_deficient_start_is_reported(lib, torch):
    """A start block without full rank: error bit 1, as before, and no wait left open."""
    from paper_2311_03824_amd import instances as I
    inst = I.make_instance(n=90, q=40, m=30, r=3, rho=2, seed=9)
    start = np.ones((90, 3), np.float32)
    s = lib.Solver(inst.At, inst.Y32, 30, 3, 2, lib.default_params(t_max=2), U_start=start)
    assert s.init().status()["error_flags"] & 2
    s.close()
