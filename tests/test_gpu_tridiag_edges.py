"""The partition method of the tridiagonal preconditioner at the sizes where
its split changes: chunks of 16 and 32 rows, groups of 256 / CW chunks, column
blocks of 4, 8 and 16, more groups than the fixed buffers hold, and as many
that a thread of the top level takes several; strided blocks, weak dominance
over long runs.

Tolerance: the bound of the other tests of this solve, 1e-13 times the
Gershgorin condition bound of T_j (at least 10), relative to the largest
entry of the column."""
import numpy as np
import pytest

import synth
from oracle import lobpcg_oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_06668_amd as P

    return P


def tridiag_csr(d, e):
    """CSR of tridiag(e, d, e), built row by row (diagonal always stored)."""
    n = d.size
    i = np.arange(n)
    rows = np.concatenate([i, i[:-1], i[1:]])
    cols = np.concatenate([i, i[1:], i[:-1]])
    vals = np.concatenate([d, e, e])
    o = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, dtype=np.int64)
    rp[1:] = np.cumsum(np.bincount(rows, minlength=n))
    return rp.astype(np.int32), cols[o].astype(np.int32), vals[o]


@pytest.mark.parametrize(
    "n,m,ld",
    [
        (3, 1, 1), (15, 4, 4), (16, 5, 5), (17, 1, 3), (97, 32, 32), (255, 9, 12), (256, 16, 16), (257, 17, 20),
        (511, 8, 8), (513, 3, 3), (1024, 8, 8), (1025, 4, 4), (2049, 13, 40),
        (262144, 4, 4),  # the fixed buffers are full
        (262145, 16, 48),  # ... and passed
        (600011, 16, 16),  # chunks of 32 rows, several groups per thread at the top
        (600011, 6, 7),
    ],
)
def test_tridiag_apply_edges(P, n, m, ld):
    print("tridiag edges", n, m, ld, flush=True)
    g = synth.rng(n + m)
    e = g.uniform(-0.5, 0.5, n - 1)
    e[g.integers(0, n - 1, max(1, n // 50))] = 0.0  # runs that do not couple
    d = 1.0 + g.uniform(0.0, 2.0, n)
    theta = np.sort(g.uniform(0.5, 1.5, m))  # t_i at its floor |e| + |e| + delta in places
    rp, ci, val = tridiag_csr(d, e)
    s = P.Solver(n)
    s.set_operator_csr(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), torch.from_numpy(val).cuda())
    s.ensure_workspace(min(m, n // 3))
    s.set_preconditioner(P.PRECOND_TRIDIAG)
    R = g.standard_normal((n, ld))
    mm = min(m, n // 3)
    Rd = torch.from_numpy(R).cuda()
    P.lobpcg_tridiag_apply(s.h, Rd[:, :mm], torch.from_numpy(theta[:mm].copy()).cuda())
    W = Rd.cpu().numpy()
    assert np.array_equal(W[:, mm:], R[:, mm:])  # other columns untouched
    Wo = O.precondition_tridiag(np.ascontiguousarray(R[:, :mm]), d, e, theta[:mm])
    off = np.zeros(n)
    off[:-1] += np.abs(e)
    off[1:] += np.abs(e)
    for j in range(mm):
        t = np.maximum(np.abs(d - theta[j]), off + O.PRECOND_GUARD * max(1.0, abs(theta[j])))
        kap = float((t + off).max() / (t - off).min())
        err = np.abs(W[:, j] - Wo[:, j]).max() / np.abs(Wo[:, j]).max()
        assert err <= 1e-13 * max(kap, 10.0), (j, err, kap)
    s.close()


@pytest.mark.parametrize("where", ["inside", "ends", "seams", "alternate", "run"])
@pytest.mark.parametrize("n,m", [(40, 3), (1025, 4), (5003, 16), (262145, 8)])
def test_tridiag_apply_frozen_rows(P, n, m, where):
    """Infinite entries of a diagonal that the caller gives, and an infinite
    theta: w is 0 in these rows (in the whole column), and the rows beside
    them are solved without the coupling.  Tolerance as above."""
    from scipy.linalg import solve_banded

    print("tridiag frozen rows", n, m, where, flush=True)
    g = synth.rng(3 * n + m)
    e = g.uniform(-0.5, 0.5, n - 1)
    d = 1.0 + g.uniform(0.0, 2.0, n)
    frozen = {
        "inside": np.array([n // 3]),
        "ends": np.array([0, n - 1]),
        "seams": np.arange(15, n, 16),  # last rows of chunks, of groups
        "alternate": np.arange(1, n, 2),
        "run": np.arange(n // 4, n // 2),
    }[where]
    theta = np.sort(g.uniform(0.5, 1.5, m))
    theta[-1] = np.inf
    rp, ci, val = tridiag_csr(d, e)
    du = d.copy()
    du[frozen] = np.where(np.arange(frozen.size) % 2 == 0, np.inf, -np.inf)
    dd = torch.from_numpy(du).cuda()
    s = P.Solver(n)
    s.set_operator_csr(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), torch.from_numpy(val).cuda())
    s.set_preconditioner(P.PRECOND_TRIDIAG, dd)
    s.ensure_workspace(m)
    R = g.standard_normal((n, m))
    Rd = torch.from_numpy(R).cuda()
    P.lobpcg_tridiag_apply(s.h, Rd, torch.from_numpy(theta).cuda())
    W = Rd.cpu().numpy()
    off = np.zeros(n)
    off[:-1] += np.abs(e)
    off[1:] += np.abs(e)
    for j in range(m - 1):
        t = np.maximum(np.abs(d - theta[j]), off + O.PRECOND_GUARD * max(1.0, abs(theta[j])))
        kap = float((t + off).max() / (t - off).min())
        band = np.zeros((3, n))
        band[0, 1:], band[1], band[2, :-1], r = e, t, e, R[:, j].copy()
        band[1, frozen], r[frozen] = 1.0, 0.0
        for b, k in ((0, 0), (0, 1), (2, 0), (2, -1)):  # the couplings of row i: band[0, i], [0, i + 1], [2, i], [2, i - 1]
            at = frozen + k
            band[b, at[(at >= 0) & (at < n)]] = 0.0
        ref = solve_banded((1, 1), band, r)
        assert np.all(W[frozen, j] == 0.0), (j, W[frozen, j])
        err = np.abs(W[:, j] - ref).max() / np.abs(ref).max()
        assert err <= 1e-13 * max(kap, 10.0), (j, err, kap)
    assert np.all(W[:, -1] == 0.0)
    s.close()
