"""The subspace iteration with many more columns than rows: column blocks that go through LDS
together, and many column splits of L_0 T, against FP64; and its time."""
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


# 256 workgroups of 16 columns hold 4096: at and above that, two to four blocks at once with ragged last
# ones, and several rounds of four; 1 to 32 splits
@pytest.mark.parametrize("n,q,r", [(63, 4096, 2), (64, 4097, 16), (100, 9000, 5), (40, 16385, 3), (65, 20011, 4),
                                   (700, 5000, 10)])
def test_many_columns_match_fp64(lib, torch, n, q, r):
    rng = np.random.default_rng(n + q)
    L0 = rng.standard_normal((n, r)) @ rng.standard_normal((r, q)) + 0.1 * rng.standard_normal((n, q))
    L0t = np.ascontiguousarray(L0.T, dtype=np.float32)
    start = rng.standard_normal((n, r)).astype(np.float32)
    U = torch.empty(n, r, device="cuda")
    steps = 2
    lib.altgdmin_op_subspace(torch.from_numpy(L0t).cuda(), r, torch.from_numpy(start).cuda(), steps, 0.0, U)
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
    assert np.linalg.norm(got - Q) <= 4.0 * amp + 1e-6
    assert np.abs(got.T @ got - np.eye(r)).max() <= 1e-6


def test_a_step_over_many_columns_fills_the_gpu(lib, torch):
    """n = 100, q = 50,000: 0.13 ms a step (0.53 with 96 workgroups, of which 8 formed L_0 T)."""
    n, q, r, steps = 100, 50000, 5, 10
    g = torch.Generator("cuda").manual_seed(1)
    L0t, start = torch.randn(q, n, generator=g, device="cuda"), torch.randn(n, r, generator=g, device="cuda")
    U = torch.empty(n, r, device="cuda")
    sc = torch.empty(lib.altgdmin_op_scratch_bytes(n, q, r) + 256, dtype=torch.uint8, device="cuda")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    t = []
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(st)
        lib.altgdmin_op_subspace(L0t, r, start, steps, 0.0, U, scratch=sc, stream=st)
        e1.record(st)
        torch.cuda.synchronize()
        t.append(e0.elapsed_time(e1) / steps)
    assert min(t) <= 0.25, t
