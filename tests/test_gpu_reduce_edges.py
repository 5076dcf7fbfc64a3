"""Second stage of the reductions (partial sums of the workgroups, added in a
fixed order) at the workgroup counts where its batches change: one, 128, 129,
512 and, in the orthonormalisation, more; and the sign rule of the returned
vectors, whose largest entry is found over every workgroup.

Bounds: an overlap within 1e-13 of sum_k |a_ik| |b_kj|, the bound of the other
overlap tests; orthonormal to the 1e-14 that the algorithm stops at, plus 8
epsilon for the other summation order; signs exactly."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_06668_amd as P

    return P


@pytest.mark.parametrize("n", [24, 64 * 8, 64 * 8 + 1, 64 * 128, 64 * 128 + 1, 64 * 129, 64 * 512, 64 * 512 + 1])
@pytest.mark.parametrize("p,q", [(1, 1), (17, 3)])
def test_gram_workgroups(P, n, p, q):
    print("reduce edges", n, p, q, flush=True)
    g = synth.rng(n + p)
    A, B = g.standard_normal((n, p)), g.standard_normal((n, q))
    s = P.Solver(n)
    s.ensure_workspace(8)
    Cd = torch.zeros((p, q), dtype=torch.float64, device="cuda")
    P.lobpcg_gram(s.h, torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), Cd)
    C = Cd.cpu().numpy()
    assert np.all(np.abs(C - A.T @ B) <= 1e-13 * (np.abs(A).T @ np.abs(B)))


@pytest.mark.parametrize("n", [64 * 600, 64 * 1024 + 64])
def test_ortho_workgroups(P, n):
    print("reduce edges ortho", n, flush=True)
    X = synth.rng(n).standard_normal((n, 5))
    s = P.Solver(n)
    s.ensure_workspace(8)
    Xd = torch.from_numpy(X).cuda()
    P.lobpcg_ortho(s.h, Xd)
    Q = Xd.cpu().numpy()
    assert np.abs(Q.T @ Q - np.eye(5)).max() <= 1e-14 + 8 * np.finfo(float).eps


@pytest.mark.parametrize("n,m", [(9, 3), (65, 16), (700, 17), (3000, 2)])
def test_returned_signs(P, n, m):
    print("reduce edges signs", n, m, flush=True)
    lam = np.arange(1.0, n + 1)
    A, _ = synth.prescribed_spectrum(lam, n)
    s = P.Solver(n)
    s.set_operator_dense(torch.from_numpy(A).cuda())
    s.set_option(P.OPT_MAX_ITER, 5)
    s.set_initial_guess(torch.from_numpy(synth.start_block(n, m, 7)).cuda())
    V = s.solve(m, 1e-12).evecs.cpu().numpy()
    assert V.shape == (n, m)
    assert np.all(V[np.abs(V).argmax(axis=0), np.arange(m)] > 0.0)
