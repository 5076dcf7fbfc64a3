"""The register/LDS eigensolver of small matrices at the sizes where
its layout changes (one and two rows per lane, panels of 16 columns, rows of
the inverse iteration by eights, the packed reflector store) and on matrices
that its shortcuts could trip over: decoupled blocks (zero reflectors, zero
couplings), clusters, entries near the ends of the exponent range.

Tolerance: the eigensolver is backward stable, |lambda - lambda'| and the
residual within p eps ||A|| times a constant; the bound of the other small
eigensolver tests, 1e-13 ||A||, is 4.7 p eps at p = 96, and orthogonality
within the same 1e-13."""
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


def matrix(kind, p):
    g = synth.rng(1000 + p)
    if kind == "random":
        return synth.random_symmetric(p, p)
    if kind == "clusters":  # repeated and 1e-14-separated eigenvalues
        lam = np.sort(np.repeat(np.arange(1.0, 2.0 + p // 4), 4)[:p] + 1e-14 * np.arange(p))
        return synth.prescribed_spectrum(lam, p)[0]
    if kind == "blocks":  # decoupled 3 x 3 blocks in scattered order
        a = np.zeros((p, p))
        perm = g.permutation(p)
        for i in range(0, p, 3):
            b = perm[i : i + 3]
            a[np.ix_(b, b)] = synth.random_symmetric(b.size, i + 1)
        return a
    if kind == "diagonal":
        return np.diag(g.permutation(np.arange(p, dtype=float)))
    if kind == "tiny":
        return 1e-140 * synth.random_symmetric(p, p)
    if kind == "huge":
        return 1e140 * synth.random_symmetric(p, p)
    if kind == "zero":
        return np.zeros((p, p))
    raise ValueError(kind)


@pytest.mark.parametrize("kind", ["random", "clusters", "blocks", "diagonal", "tiny", "huge", "zero"])
@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 8, 15, 16, 17, 32, 33, 47, 49, 63, 64, 65, 79, 81, 95, 96])
def test_small_eigh_edges(P, p, kind):
    print("small_eigh edges", p, kind, flush=True)
    a = matrix(kind, p)
    s = P.Solver(300)
    ev = torch.zeros(p, dtype=torch.float64, device="cuda")
    U = torch.zeros((p, p), dtype=torch.float64, device="cuda")
    P.lobpcg_small_eigh(s.h, torch.from_numpy(a).cuda(), ev, U)
    lam, Uh = ev.cpu().numpy(), U.cpu().numpy()
    nrm = np.linalg.norm(a, 2)
    assert np.all(np.abs(lam - np.linalg.eigvalsh(a)) <= 1e-13 * nrm)
    assert np.all(np.diff(lam) >= 0)
    assert np.abs(Uh.T @ Uh - np.eye(p)).max() <= 1e-13
    assert np.abs(a @ Uh - Uh * lam).max() <= 1e-13 * nrm
    assert np.all(np.diag(Uh) >= 0)
    s.close()


@pytest.mark.parametrize("p", [3, 33, 64, 65, 96])
def test_small_eigh_fallback(P, p):
    """Entries whose squares are near the end of the exponent range: the reflectors'
    scale overflows, and the matrix is read again and goes through the Jacobi
    sweeps, as when a Cholesky factorisation breaks down.  The same bounds."""
    print("small_eigh fallback", p, flush=True)
    a = 1e-158 * synth.random_symmetric(p, p)
    s = P.Solver(300)
    ev = torch.zeros(p, dtype=torch.float64, device="cuda")
    U = torch.zeros((p, p), dtype=torch.float64, device="cuda")
    P.lobpcg_small_eigh(s.h, torch.from_numpy(a).cuda(), ev, U)
    lam, Uh = ev.cpu().numpy() * 2.0**500, U.cpu().numpy()
    a = a * 2.0**500  # (the checks' own squares)
    nrm = np.linalg.norm(a, 2)
    assert np.all(np.abs(lam - np.linalg.eigvalsh(a)) <= 1e-13 * nrm)
    assert np.all(np.diff(lam) >= 0)
    assert np.abs(Uh.T @ Uh - np.eye(p)).max() <= 1e-13
    assert np.abs(a @ Uh - Uh * lam).max() <= 1e-13 * nrm
    assert np.all(np.diag(Uh) >= 0)
    s.close()


@pytest.mark.parametrize("off", [0.0, 1e-17, 1e-9, 1e-5, 1e-3, 0.02, 0.5])
@pytest.mark.parametrize("p", [1, 2, 76, 77, 83, 84, 90, 96])
def test_small_eigh_nearly_diagonal(P, p, off):
    """Off-diagonal entries small against the distances on the diagonal, which
    large matrices solve by rotations, on both sides of the choice; also in
    place, where they do not.  The same bounds."""
    print("small_eigh nearly diagonal", p, off, flush=True)
    g = synth.rng(p)
    a = np.diag(g.permutation(np.arange(p, dtype=float))) + off * synth.random_symmetric(p, p)
    s = P.Solver(300)
    for inplace in (False, True):
        A = torch.from_numpy(a).cuda()
        ev = torch.zeros(p, dtype=torch.float64, device="cuda")
        U = A if inplace else torch.zeros((p, p), dtype=torch.float64, device="cuda")
        P.lobpcg_small_eigh(s.h, A, ev, U)
        lam, Uh = ev.cpu().numpy(), U.cpu().numpy()
        nrm = np.linalg.norm(a, 2)
        assert np.all(np.abs(lam - np.linalg.eigvalsh(a)) <= 1e-13 * nrm)
        assert np.all(np.diff(lam) >= 0)
        assert np.abs(Uh.T @ Uh - np.eye(p)).max() <= 1e-13
        assert np.abs(a @ Uh - Uh * lam).max() <= 1e-13 * nrm
        assert np.all(np.diag(Uh) >= 0)
    s.close()
