"""The orthonormalisation's controller at the block sizes where its factor
changes: up to 8 and up to 16 columns in one wave's registers, wider ones
column by column, with and without a basis to stay orthogonal to; and with a
nearly dependent pair of columns, whose last pivot is rounding, of either sign
(the plain factorisation fails for about half of them).

Bounds: the algorithm stops at 1e-14 in the overlaps it forms itself (or at a
bound of them); another summation of the same unit vectors is off by no more
than 8 epsilon.  The span is kept to 1e-12, or to epsilon times the condition
number (1e10, with a factor 100 for its constant)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BAR = 1e-14 + 8 * np.finfo(float).eps


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_06668_amd as P

    return P


@pytest.mark.parametrize("near", [False, True])
@pytest.mark.parametrize(
    "ny,nw", [(0, 1), (3, 1), (0, 2), (5, 7), (0, 8), (16, 8), (0, 9), (18, 9), (30, 15), (0, 16), (32, 16),
              (0, 17), (34, 17), (62, 31), (64, 32)]
)
def test_ortho_block_sizes(P, ny, nw, near):
    if near and nw == 1:
        pytest.skip("one column has no pair")
    print("ortho edges", ny, nw, near, flush=True)
    g = synth.rng(100 * ny + nw)
    n = 5000
    Y = np.linalg.qr(g.standard_normal((n, ny)))[0] if ny else np.zeros((n, 0))
    X = g.standard_normal((n, nw))
    if near:
        X[:, -1] = X[:, 0] + 1e-10 * X[:, -1]
    buf = torch.from_numpy(np.hstack([Y, X])).cuda()
    s = P.Solver(n)
    s.ensure_workspace(max(8, nw))
    if ny:
        info = P.lobpcg_ortho_against(s.h, buf[:, ny:], buf[:, :ny])
    else:
        info = P.lobpcg_ortho(s.h, buf)
    out = buf.cpu().numpy()
    Q = out[:, ny:]
    assert np.array_equal(out[:, :ny], Y)
    assert info["stalled"] == 0 and info["svqb"] == 0
    assert near or (info["failed"] == 0 and info["shifted"] == 0)
    assert np.abs(Q.T @ Q - np.eye(nw)).max() <= BAR
    if ny:
        assert np.abs(Y.T @ Q).max() <= BAR
    Z = X - Y @ (Y.T @ X)
    Z /= np.linalg.norm(Z, axis=0)
    if near:
        Z = Z[:, :-1]  # (the pair's difference is left to rounding)
    assert np.linalg.norm(Z - Q @ (Q.T @ Z)) <= (1e-12 if not near else 100 * 2.3e-6)
