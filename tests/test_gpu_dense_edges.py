"""The dense operator where its kernel changes: sizes around a tile of rows
(16), a chunk of columns (32) and the chunks of a workgroup, below and above the
switches between its shapes, rows of any alignment, 1 to 33 columns of a
wider basis.

Entry by entry against the definition within the summation bound
(n + 1) u sum_j |a_ij| |w_j|."""
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
@pytest.mark.parametrize("n,pad", [(3, 0), (15, 1), (16, 0), (17, 0), (31, 2), (32, 0), (33, 0), (255, 0), (257, 0), (300, 3), (4095, 0), (4096, 1), (4097, 0), (5999, 0), (6000, 0), (6031, 1)])
@pytest.mark.parametrize("m,ldw,q", [(1, 1, 0), (4, 7, 2), (5, 5, 0), (16, 16, 0), (17, 20, 3), (33, 33, 0)])
def test_dense_edges(P, n, pad, m, ldw, q, prec):
    print("dense edges", n, pad, m, ldw, q, prec, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + m)
    A = torch.randn((n, n + pad), generator=g, device="cuda", dtype=torch.float64)
    A[:, :n] = 0.5 * (A[:, :n] + A[:, :n].T.clone())
    s = P.Solver(n)
    s.set_operator_dense(A[:, :n])
    f32 = prec == "f32"
    if f32:
        s.set_option(P.OPT_PRECISION, P.PREC_FP32)
    s.ensure_workspace(1)
    dt, u = (torch.float32, 2.0**-24) if f32 else (torch.float64, 2.0**-53)
    W = torch.randn((n, ldw), generator=g, device="cuda", dtype=torch.float64).to(dt)
    Y = torch.full((n, ldw + 1), 5.0, dtype=dt, device="cuda")
    (P.lobpcg_apply_operator_f32 if f32 else P.lobpcg_apply_operator)(s.h, W[:, q : q + m], Y[:, q : q + m])
    Ad = A[:, :n].to(dt).double().contiguous()
    Wd = W[:, q : q + m].double().contiguous()
    bound = (n + 1) * u * (Ad.abs() @ Wd.abs())
    assert bool(((Y[:, q : q + m].double() - Ad @ Wd).abs() <= bound).all())
    assert bool((Y[:, :q] == 5.0).all()) and bool((Y[:, q + m :] == 5.0).all())  # other columns untouched
    s.close()


@pytest.mark.parametrize("n,pad", [(1, 0), (2, 1), (7, 0), (127, 1), (128, 0), (1799, 0), (1800, 0), (4095, 1), (4096, 0), (4099, 1), (5799, 0), (8193, 1), (8194, 0), (12499, 1), (12502, 0), (16386, 0)])
def test_dense_few_columns(P, n, pad):
    """Up to four columns of a block whose rows lie close together: the sizes,
    row alignments, widths and offsets between which the kernel changes."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    A = torch.randn((n, n + pad), generator=g, device="cuda", dtype=torch.float64)
    Ad = A[:, :n].contiguous()
    Aa = Ad.abs()
    s = P.Solver(n)
    s.set_operator_dense(A[:, :n])
    for m, ldw, q in [(1, 1, 0), (1, 4, 3), (2, 2, 0), (2, 3, 1), (2, 4, 1), (2, 4, 2), (3, 3, 0), (3, 4, 1), (4, 4, 0), (4, 5, 1)]:
        print("dense few", n, pad, m, ldw, q, flush=True)
        W = torch.randn((n, ldw), generator=g, device="cuda", dtype=torch.float64)
        Y = torch.full((n, ldw + 1), 5.0, dtype=torch.float64, device="cuda")
        P.lobpcg_apply_operator(s.h, W[:, q : q + m], Y[:, q : q + m])
        Wd = W[:, q : q + m].contiguous()
        bound = (n + 1) * 2.0**-53 * (Aa @ Wd.abs())
        # (the oracle's own products round too: as much again)
        assert bool(((Y[:, q : q + m] - Ad @ Wd).abs() <= 2 * bound).all())
        assert bool((Y[:, :q] == 5.0).all()) and bool((Y[:, q + m :] == 5.0).all())  # other columns untouched
    s.close()


@pytest.mark.parametrize("prec,n,pad", [("f64", 6001, 0), ("f64", 6047, 1), ("f64", 8192, 0), ("f64", 16999, 0), ("f64", 17000, 0), ("f32", 12999, 0), ("f32", 13000, 0), ("f32", 13023, 1), ("f32", 16999, 0)])
def test_dense_workgroups_apart(P, prec, n, pad):
    """Sizes at which the workgroups begin at different columns of their rows."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    f32 = prec == "f32"
    dt, u = (torch.float32, 2.0**-24) if f32 else (torch.float64, 2.0**-53)
    A = torch.randn((n, n + pad), generator=g, device="cuda", dtype=torch.float64)
    s = P.Solver(n)
    s.set_operator_dense(A[:, :n])
    if f32:
        s.set_option(P.OPT_PRECISION, P.PREC_FP32)
        s.ensure_workspace(1)
    Ad = A[:, :n].to(dt).double().contiguous()
    Aa = Ad.abs()
    for m, ldw, q in [(5, 5, 0), (8, 24, 16), (17, 17, 0)]:
        print("dense apart", prec, n, pad, m, ldw, q, flush=True)
        W = torch.randn((n, ldw), generator=g, device="cuda", dtype=torch.float64).to(dt)
        Y = torch.full((n, ldw + 1), 5.0, dtype=dt, device="cuda")
        (P.lobpcg_apply_operator_f32 if f32 else P.lobpcg_apply_operator)(s.h, W[:, q : q + m], Y[:, q : q + m])
        Wd = W[:, q : q + m].double().contiguous()
        bound = (n + 1) * u * (Aa @ Wd.abs())
        assert bool(((Y[:, q : q + m].double() - Ad @ Wd).abs() <= 2 * bound).all())
        assert bool((Y[:, :q] == 5.0).all()) and bool((Y[:, q + m :] == 5.0).all())  # other columns untouched
    s.close()
