"""The Kronecker-sum operator where its loads and its order of tiles change:
sizes around a tile (32), a chunk of k (16) and a strip of 8 rows of tiles, odd
ones, blocks of less and more than 8 columns, columns of a wider basis.

Entry by entry against the definition within the summation bound
(2 na + 3) u (|A| |W_b| + |W_b| |A| + |V| |W_b|)."""
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


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("m,ldw,q", [(8, 8, 0), (3, 3, 0), (9, 11, 1), (16, 16, 0)])
@pytest.mark.parametrize("na", [2, 3, 15, 16, 17, 31, 32, 33, 34, 47, 64, 65, 97, 255, 257, 289])
def test_kron_edges(P, na, m, ldw, q, prec):
    print("kron edges", na, m, ldw, q, prec, flush=True)
    g = synth.rng(7 * na + m)
    n = na * na
    B = g.standard_normal((na, na))
    A, V = 0.5 * (B + B.T), g.standard_normal((na, na))
    s = P.Solver(n)
    s.set_operator_kronsum(torch.from_numpy(A).cuda(), torch.from_numpy(V).cuda())
    f32 = prec == "f32"
    if f32:
        s.set_option(P.OPT_PRECISION, P.PREC_FP32)
    s.ensure_workspace(1)
    dt, u = (torch.float32, 2.0**-24) if f32 else (torch.float64, 2.0**-53)
    Wd = torch.from_numpy(g.standard_normal((n, ldw))).to(dt).cuda()
    Y = torch.full((n, ldw), 5.0, dtype=dt, device="cuda")
    (P.lobpcg_apply_operator_f32 if f32 else P.lobpcg_apply_operator)(s.h, Wd[:, q : q + m], Y[:, q : q + m])
    out = Y.cpu().numpy().astype(np.float64)
    W = Wd.cpu().numpy().astype(np.float64)
    if f32:
        A, V = A.astype(np.float32).astype(np.float64), V.astype(np.float32).astype(np.float64)
    for b in range(q, q + m):
        Wb = W[:, b].reshape(na, na)
        ref = A @ Wb + Wb @ A + V * Wb
        bound = (2 * na + 3) * u * (abs(A) @ abs(Wb) + abs(Wb) @ abs(A) + abs(V) * abs(Wb))
        assert np.all(np.abs(out[:, b].reshape(na, na) - ref) <= bound)
    assert np.all(out[:, :q] == 5.0) and np.all(out[:, q + m :] == 5.0)  # other columns untouched
    s.close()


@pytest.mark.parametrize("m,ldw,q", [(8, 8, 0), (8, 11, 3), (16, 18, 2), (16, 19, 1), (24, 24, 0), (3, 3, 0), (9, 11, 1)])
@pytest.mark.parametrize("na", [1, 2, 16, 17, 33, 65, 257, 289])
def test_kron_no_workspace(P, na, m, ldw, q):
    """Without a workspace there is no packed copy: the kernel reads the caller's
    block itself, at its leading dimension, alignment and number of columns, eight
    columns to a row of the grid."""
    print("kron no workspace", na, m, ldw, q, flush=True)
    g = synth.rng(11 * na + m)
    n = na * na
    B = g.standard_normal((na, na))
    A, V = 0.5 * (B + B.T), g.standard_normal((na, na))
    s = P.Solver(n)
    s.set_operator_kronsum(torch.from_numpy(A).cuda(), torch.from_numpy(V).cuda())
    W = g.standard_normal((n, ldw))
    Y = torch.full((n, ldw), 5.0, dtype=torch.float64, device="cuda")
    P.lobpcg_apply_operator(s.h, torch.from_numpy(W).cuda()[:, q : q + m], Y[:, q : q + m])
    out = Y.cpu().numpy()
    for b in range(q, q + m):
        Wb = W[:, b].reshape(na, na)
        ref = A @ Wb + Wb @ A + V * Wb
        bound = (2 * na + 3) * 2.0**-53 * (abs(A) @ abs(Wb) + abs(Wb) @ abs(A) + abs(V) * abs(Wb))
        assert np.all(np.abs(out[:, b].reshape(na, na) - ref) <= bound)
    assert np.all(out[:, :q] == 5.0) and np.all(out[:, q + m :] == 5.0)  # other columns untouched
    s.close()
