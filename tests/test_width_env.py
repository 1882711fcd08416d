"""The workspace of a problem has one size: ALTGDMIN_AU_WAVES (which forces the width of the
A_k U workgroups, and with it their row splits) may change between the calls of a program."""
import pytest


def _problem(lib, n, q, m, r):
    p = lib.Problem()   # placeholder pointers: validated, never dereferenced
    p.n, p.q, p.m, p.r, p.rho = n, q, m, r, 3
    p.a_format = lib.ALTGDMIN_A_F32
    p.A, p.Y = 1 << 20, 1 << 24
    p.lda = p.ldy = (m + 3) // 4 * 4
    p.a_stride_k = p.lda * n
    return p


@pytest.mark.parametrize("n,q,m,r", [(300, 20, 257, 3), (1000, 125, 400, 10), (700, 1, 1024, 16), (90, 64, 256, 4),
                                     (90, 600, 400, 4)])
def test_workspace_size_does_not_follow_the_environment(lib, monkeypatch, n, q, m, r):
    sizes = set()
    for width in (None, "4", "8"):
        if width is None:
            monkeypatch.delenv("ALTGDMIN_AU_WAVES", raising=False)
        else:
            monkeypatch.setenv("ALTGDMIN_AU_WAVES", width)
        sizes.add(lib.altgdmin_workspace_bytes(_problem(lib, n, q, m, r), lib.default_params()))
    assert len(sizes) == 1
