"""The gradient's entry point in 16-wave workgroups (at most 128 of them) and in 4-wave ones, against
FP64; and its time where there are few."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return _t


# 128 and 132 workgroups, one, and columns fewer than the waves take at once; ragged rows and ranks
@pytest.mark.parametrize("n,q,r", [(2048, 512, 8), (2049, 600, 3), (64, 63, 16), (1, 1, 1), (65, 5, 5), (257, 70, 12),
                                   (100, 5000, 4)])
def test_grad_matches_fp64(lib, torch, n, q, r):
    g = torch.Generator("cuda").manual_seed(n + q)
    H, B = torch.randn(q, n, generator=g, device="cuda"), torch.randn(q, r, generator=g, device="cuda")
    G = torch.empty(n, r, device="cuda")
    lib.altgdmin_op_grad(H, B, G)
    H64, B64 = H.double().cpu().numpy(), B.double().cpu().numpy()
    # FP32 sums: at most q / 16 serial terms per lane, then a tree
    tol = (q / 16 + 32) * U32 * (np.abs(H64).T @ np.abs(B64))
    assert (np.abs(G.cpu().numpy() - H64.T @ B64) <= tol).all()


def test_few_row_blocks_with_many_columns(lib, torch):
    """n = 100, q = 20,000, r = 4: 53 us (104 in 4-wave workgroups)."""
    n, q, r = 100, 20000, 4
    H, B, G = torch.randn(q, n, device="cuda"), torch.randn(q, r, device="cuda"), torch.empty(n, r, device="cuda")
    sc = torch.empty(lib.altgdmin_op_scratch_bytes(n, q, r) + 256, dtype=torch.uint8, device="cuda")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    t = []
    for _ in range(6):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(st)
        for _ in range(4):
            lib.altgdmin_op_grad(H, B, G, scratch=sc, stream=st)
        e1.record(st)
        torch.cuda.synchronize()
        t.append(e0.elapsed_time(e1) / 4)
    assert min(t) <= 0.08, t
