"""The Rayleigh-Ritz kernel at the block sizes where its layout changes: the
basis of 3 m vectors below and above 33, 49 and 64 (row strides of the
reduction, registers of the Sturm counts, one or two rows per lane), factors
of 8 and of 16 columns and the general ones, odd sizes; on a spectrum with
repeated eigenvalues, which the inverse iteration returns as mixtures.

Bounds: each pair's residual is at most the solve's own tolerance, an
eigenvalue is within its residual of the spectrum (Weyl), and the vectors are
orthonormal to 1e-12, as in the other solves' tests."""
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


@pytest.mark.parametrize("m", [1, 2, 3, 5, 8, 9, 11, 12, 16, 17, 21, 22, 31, 32])
def test_solve_block_sizes(P, m):
    print("rr edges", m, flush=True)
    n = 320
    lam = np.sort(np.concatenate([np.repeat(np.arange(1.0, 13.0), 3), np.linspace(20.0, 40.0, n - 36)]))
    A, _ = synth.prescribed_spectrum(lam, 50 + m)
    tol = 1e-9
    s = P.Solver(n)
    s.set_operator_dense(torch.from_numpy(A).cuda())
    s.set_option(P.OPT_MAX_ITER, 3000)
    s.set_initial_guess(torch.from_numpy(synth.start_block(n, m, 7)).cuda())
    r = s.solve(m, tol)
    assert r.status == 0 and r.stats["rr_eig_fallbacks"] == 0
    X, ev = r.evecs.cpu().numpy(), np.asarray(r.evals)
    res = np.linalg.norm(A @ X - X * ev, axis=0)
    assert np.all(res <= tol * 40.0 * (1 + 1e-6))
    assert np.abs(X.T @ X - np.eye(m)).max() <= 1e-12
    assert np.all(np.abs(ev - lam[:m]) <= tol * 40.0 * (1 + 1e-6))
    s.close()
