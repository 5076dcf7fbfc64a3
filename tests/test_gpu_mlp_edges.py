"""The fp32 learned preconditioner at the sizes where its screening changes: one
entry of a tile, a full tile and one entry more, a group of tiles and one
more, a ragged one, and more groups than a workgroup screens at once; with
entries inside the window at both ends of the block and between.

Bounds, those of the other sizes' test: 1e-4 relative to the fp64 oracle inside
the window (an fp32 net), 1e-14 outside (the Jacobi step, fp64 on both sides)."""
import numpy as np
import pytest

import synth
from oracle import lobpcg_oracle as O
from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_06668_amd as P

    return P


@pytest.mark.parametrize("n,m", [(3, 1), (64, 1), (65, 1), (512, 1), (513, 1), (700, 3), (300_007, 8)])
def test_learned_apply_sizes(P, n, m):
    import scipy.sparse as sp

    print("mlp edges", n, m, flush=True)
    d = np.arange(n, dtype=np.float64) + 1.0
    off = np.full(n - 1, 0.5)
    As = sp.diags([off, d, off], [-1, 0, 1], format="csr")
    rho = np.asarray(abs(As).sum(1)).ravel() - np.abs(d)
    theta = np.linspace(1.3, n - 0.4, m) if m > 1 else np.array([n - 0.4])
    p = M.init_params(5, out_bias=-1.0)
    p.W3 *= 10.0
    w32 = p.flat().astype(np.float32)
    p = M.Params.from_flat(w32.astype(np.float64))
    s = P.Solver(n)
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    s.set_operator_csr(cu(As.indptr.astype(np.int32)), cu(As.indices.astype(np.int32)), cu(As.data.astype(np.float64)))
    s.ensure_workspace(m)
    s.set_learned_weights(w32)
    s.set_option(P.OPT_LEARNED_BF16, 0)
    R = synth.rng(n).standard_normal((n, m))
    Rd = cu(R)
    P.lobpcg_learned_apply(s.h, Rd, cu(theta), cu(np.zeros(m, dtype=np.int32)))
    W = Rd.cpu().numpy()
    s_ = M.scale_of(d)
    for j in range(m):
        near = np.abs(d - theta[j]) <= 16 * rho
        assert near.any()
        ref = O.precondition_diag(R[:, [j]], d, theta[[j]])[:, 0]
        assert np.all(np.abs(W[~near, j] - ref[~near]) <= 1e-14 * np.abs(ref[~near])), j
        ref, _ = M.precondition(p, R[near, j], d[near], theta[j], rho[near], s_)
        assert np.all(np.abs(W[near, j] - ref) <= 1e-4 * np.abs(ref)), j


@pytest.mark.parametrize("n,m", [(512 * 256, 1), (512 * 256 + 1, 1), (512 * 256 * 4, 1), (512 * 256 * 4 + 1, 1), (512 * 256 * 16 + 700, 1)])
def test_learned_apply_group_counts(P, n, m):
    """One group for every workgroup and one more, four and one more (the groups of
    a pass), sixteen (all that are screened at once) and two more."""
    test_learned_apply_sizes(P, n, m)
