"""The CSR product at the sizes where its row kernel changes: rows of 0, of a
few entries around a batch of gathers, around what the LDS of a wave holds per
row, and much longer; a group of rows that fits and its neighbour that does
not; matrices of few rows, less than a wave's and a workgroup's rows; the last
lane of a row whole, shifted, and at any alignment of W.

Entry by entry against the definition within the summation bound
(row length + 2) u sum_j |a_ij| |w_j|."""
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


def matrix(n, seed):
    import scipy.sparse as sp

    g = np.random.default_rng(seed)
    lens = g.choice([0, 1, 2, 3, 4, 5, 7, 8, 9, 47, 48, 49, 95, 97, 300], size=n)
    lens[: n // 3] = g.choice([39, 41, 43, 47, 48, 49], size=n // 3)  # groups that just fit, or not
    lens = np.minimum(lens, n)
    rows = np.repeat(np.arange(n), lens)
    cols = np.concatenate([np.sort(g.choice(n, size=k, replace=False)) for k in lens] + [np.zeros(0, int)])
    return sp.csr_matrix((g.uniform(-1, 1, rows.size), (rows, cols.astype(int))), shape=(n, n))


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [3, 7, 9, 33, 1000, 5003])
@pytest.mark.parametrize("m,ldw,q", [(5, 5, 0), (8, 9, 1), (9, 9, 0), (16, 16, 0), (13, 31, 7), (17, 33, 3), (31, 32, 1), (32, 32, 0), (33, 33, 0), (64, 64, 0)])
def test_csr_row_edges(P, n, m, ldw, q, prec):
    print("csr row edges", n, m, ldw, q, prec, flush=True)
    S = matrix(n, 100 + n)
    s = P.Solver(n)
    s.set_operator_csr(
        torch.from_numpy(S.indptr.astype(np.int32)).cuda(),
        torch.from_numpy(S.indices.astype(np.int32)).cuda(),
        torch.from_numpy(S.data.astype(np.float64)).cuda(),
    )
    f32 = prec == "f32"
    if f32:
        s.set_option(P.OPT_PRECISION, P.PREC_FP32)
    s.ensure_workspace(1)
    dt, u = (torch.float32, 2.0**-24) if f32 else (torch.float64, 2.0**-53)
    Wd = torch.from_numpy(synth.rng(n + m).standard_normal((n, ldw))).to(dt).cuda()
    Y = torch.full((n, ldw + 2), 5.0, dtype=dt, device="cuda")
    (P.lobpcg_apply_operator_f32 if f32 else P.lobpcg_apply_operator)(s.h, Wd[:, q : q + m], Y[:, q : q + m])
    out = Y.cpu().numpy().astype(np.float64)
    W = Wd.cpu().numpy().astype(np.float64)[:, q : q + m]
    A = S.copy()
    if f32:
        A.data = S.data.astype(np.float32).astype(np.float64)
    bound = (np.diff(S.indptr)[:, None] + 2) * u * (abs(A) @ np.abs(W))
    assert np.all(np.abs(out[:, q : q + m] - A @ W) <= bound)
    assert np.all(out[:, :q] == 5.0) and np.all(out[:, q + m :] == 5.0)  # other columns untouched
    s.close()
