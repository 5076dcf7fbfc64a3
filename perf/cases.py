"""Performance cases: the work that programs have this library do.

A case is a dict of plain values.  ``prepare(case, seed)`` makes what a program
holds before the call (matrices, blocks, a solver handle with its workspace),
``run(state)`` is one pass through the public entry points and returns its
outputs, ``work(case)`` the bytes and operations that the pass cannot do
without, and ``exact(case, seed)`` the same outputs in plain 64-bit torch.

The kinds are the whole solves and the steps that a solve is made of (each is
an entry point of its own, for callers with their own iteration):

  solve_dense  lowest pairs of a dense, diagonally dominant matrix
  solve_csr    lowest eigenvalues of a sparse banded matrix, mixed precision
  csr          sparse operator on a block (fp64, or the fp32 phase's product)
  dense        dense operator on a block (fp64 or fp32)
  kron         matrix-free Kronecker-sum operator on a block
  gram         overlap of two blocks
  ortho        block made orthonormal to itself and to the basis left of it
  rotate       basis rotation with residual and Jacobi step
  eigh         small symmetric eigensolve
  tridiag      tridiagonal preconditioner on a block
  train        steps of the learned preconditioner's training (forward,
               backward and Adam)
"""
from __future__ import annotations

import math

import torch

import paper_2305_06668_amd as P

DEV = "cuda:0"
SOLVE_TOL = 1e-8  # residual tolerance of the eigenvalue solves
# Vectors are returned by the dense solve: its lowest eigenvalues lie 0.05
# apart, so this residual tolerance fixes them to about ten digits.
VECTOR_TOL = 1e-11


def listed():
    return [
        # A small whole problem (SCF-Hessian-like, n = 2000, 8 pairs, a block
        # wider than k by 5): launches, host read-backs and the small dense
        # kernels count.
        dict(name="solve_dense_2000", kind="solve_dense", n=2000, k=8, block=13),
        # A whole sparse solve, learned preconditioner with mixed precision.
        dict(name="solve_csr_200k", kind="solve_csr", n=200_000, k=8, block=12, learned=True, mixed=True),
        # The operator of the quoted benchmark: n = 1e6, 16 columns, compact.
        dict(name="csr_1m_f64", kind="csr", n=1_000_000, m=16, ldw=16, col=0, f32=False),
        # The fp32 phase's product: the W columns of an [X P W] basis, odd n.
        dict(name="csr_300k_f32", kind="csr", n=300_007, m=16, ldw=48, col=32, f32=True),
        # The dense operator at its full size.
        dict(name="dense_20k", kind="dense", n=20_000, m=8, f32=False),
        # The matrix-free operator at its full size, n = 16.8 million.
        dict(name="kron_4096", kind="kron", na=4096, m=8),
        # The Rayleigh-Ritz Gram of a 48-column basis.
        dict(name="gram_1m_48", kind="gram", n=1_000_000, p=48, q=48),
        # W made orthonormal to [X P] (32 columns) at n = 1e6.
        dict(name="ortho_1m_32_16", kind="ortho", n=1_000_000, ny=32, nw=16),
        # The rotation of the whole basis at n = 1e6, every column active.
        dict(name="rotate_1m_16", kind="rotate", n=1_000_000, m=16, nact=16),
        # The Rayleigh-Ritz eigensolve of a 48-column basis: the smallest call.
        dict(name="eigh_48", kind="eigh", p=48),
        # The tridiagonal preconditioner on 16 columns at n = 1e6.
        dict(name="tridiag_1m_16", kind="tridiag", n=1_000_000, m=16),
        # Training: 4 Adam steps on 8 of a snapshot's 16 columns, n = 2e5.
        dict(name="train_200k", kind="train", n=200_000, m=16, cols=8, steps=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(
        ["solve_dense", "solve_csr", "csr", "csr", "dense", "kron", "gram", "ortho", "rotate", "eigh", "tridiag", "train"]
    )
    if kind == "solve_dense":
        k = rng.randint(2, 8)
        return dict(kind=kind, n=_log_int(rng, 300, 2000), k=k, block=k + rng.randint(2, 5))
    if kind == "solve_csr":
        k = rng.randint(3, 8)
        return dict(
            kind=kind, n=_log_int(rng, 20_000, 100_000), k=k, block=k + 4,
            learned=rng.random() < 0.5, mixed=rng.random() < 0.7,
        )
    if kind == "csr":
        # a compact block, or columns of a wider basis as the solver holds them
        m = rng.randint(1, 32)
        n = _log_int(rng, 5_000, 1_000_000)
        f32 = rng.random() < 0.4
        if rng.random() < 0.5:
            return dict(kind=kind, n=n, m=m, ldw=m, col=0, f32=f32)
        col = rng.randint(m, 2 * m)
        return dict(kind=kind, n=n, m=m, ldw=col + m, col=col, f32=f32)
    if kind == "dense":
        return dict(kind=kind, n=_log_int(rng, 300, 16_000), m=rng.randint(1, 16), f32=rng.random() < 0.4)
    if kind == "kron":
        return dict(kind=kind, na=_log_int(rng, 64, 2048), m=rng.randint(1, 16))
    if kind == "gram":
        return dict(kind=kind, n=_log_int(rng, 1_000, 1_000_000), p=rng.randint(1, 96), q=rng.randint(1, 48))
    if kind == "ortho":
        nw = rng.randint(1, 32)
        return dict(kind=kind, n=_log_int(rng, 2_000, 1_000_000), ny=rng.randint(0, 2 * nw), nw=nw)
    if kind == "rotate":
        m = rng.randint(2, 24)
        return dict(kind=kind, n=_log_int(rng, 2_000, 1_000_000), m=m, nact=rng.randint(1, m))
    if kind == "eigh":
        return dict(kind=kind, p=rng.randint(6, 96))
    if kind == "tridiag":
        return dict(kind=kind, n=_log_int(rng, 2_000, 1_000_000), m=rng.randint(1, 32))
    m = rng.randint(6, 16)
    return dict(kind="train", n=_log_int(rng, 20_000, 200_000), m=m, cols=rng.randint(2, 6), steps=rng.randint(2, 4))


# ---- inputs -----------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device=DEV, dtype=torch.float64) * (hi - lo) + lo


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float64)


def _banded_csr(g, n, diag, per_row=20, value=1e-3, chain=False):
    """Symmetric CSR: per_row offsets in 1 .. band above the diagonal of each
    row (repeats dropped), values U(-value, value), mirrored; `chain` also
    stores every entry next to the diagonal."""
    band = min(5000, n // 4)
    off = torch.randint(1, band + 1, (n, per_row), generator=g, device=DEV)
    if chain:
        off[:, 0] = 1
    off = off.sort(1).values
    keep = torch.ones_like(off, dtype=torch.bool)
    keep[:, 1:] = off[:, 1:] != off[:, :-1]
    i = torch.arange(n, device=DEV)[:, None].expand_as(off)
    j = i + off
    keep &= j < n
    v = _uniform(g, off.shape, -value, value)[keep]
    i, j = i[keep], j[keep]
    d = torch.arange(n, device=DEV)
    key, order = torch.cat([i * n + j, j * n + i, d * n + d]).sort()
    val = torch.cat([v, v, diag])[order].contiguous()
    rows = torch.div(key, n, rounding_mode="floor")
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.bincount(rows, minlength=n).cumsum(0)
    return rp.to(torch.int32), (key - rows * n).to(torch.int32), val


def _dominant_diag(g, n):
    """1 + a slope that reaches 11 at the last row + U(0, 0.1)."""
    return 1.0 + torch.arange(n, device=DEV, dtype=torch.float64) * (10.0 / n) + _uniform(g, (n,), 0.0, 0.1)


def _orthonormal(X):
    for _ in range(2):
        X = torch.linalg.solve_triangular(torch.linalg.cholesky(X.T @ X), X.T, upper=False).T.contiguous()
    return X


def _inputs(case, seed):
    """The case's arrays on the GPU, from the seed alone."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "solve_dense":
        n = case["n"]
        A = torch.triu(_normal(g, n, n) * 1e-3, 1)
        A = A + A.T
        A.diagonal().copy_(1.0 + 0.05 * torch.arange(n, device=DEV, dtype=torch.float64) + _uniform(g, (n,), 0.0, 0.01))
        return dict(A=A, X0=_normal(g, n, case["block"]))
    if kind == "solve_csr":
        n = case["n"]
        rp, ci, val = _banded_csr(g, n, _dominant_diag(g, n))
        return dict(rp=rp, ci=ci, val=val, X0=_normal(g, n, case["block"]))
    if kind == "csr":
        n = case["n"]
        rp, ci, val = _banded_csr(g, n, _dominant_diag(g, n))
        W = _normal(g, n, case["ldw"])
        return dict(rp=rp, ci=ci, val=val, W=W.float() if case["f32"] else W)
    if kind == "dense":
        n = case["n"]
        A = _normal(g, n, n).mul_(0.05)
        A = A + A.T
        W = _normal(g, n, case["m"])
        return dict(A=A, W=W.float() if case["f32"] else W)
    if kind == "kron":
        na = case["na"]
        A = torch.triu(_normal(g, na, na) * 1e-2, 1)
        A = A + A.T
        A.diagonal().copy_(_uniform(g, (na,), 0.0, 20.0).sort().values)
        i = torch.arange(na, device=DEV)
        V = 0.1 * torch.cos(((i[:, None] * i[None, :]) % 97).double())
        return dict(A=A, V=V, W=_normal(g, na * na, case["m"]))
    if kind == "gram":
        return dict(A=_normal(g, case["n"], case["p"]), B=_normal(g, case["n"], case["q"]))
    if kind == "ortho":
        n, ny, nw = case["n"], case["ny"], case["nw"]
        V = torch.empty((n, ny + nw), dtype=torch.float64, device=DEV)
        # columns of very different sizes that overlap with the basis and,
        # moderately, with each other
        W = _normal(g, n, nw) + 0.5 * _normal(g, n, 1)
        if ny:
            Y = _orthonormal(_normal(g, n, ny))
            V[:, :ny] = Y
            W += Y @ (_normal(g, ny, nw) * math.sqrt(n) * 0.3)
        W *= 10.0 ** _uniform(g, (nw,), -6.0, 0.0)
        return dict(V=V, W=W)
    if kind == "rotate":
        n, m, nact = case["n"], case["m"], case["nact"]
        p, q = m + 2 * nact, m + nact
        return dict(
            V=_normal(g, n, p), AV=_normal(g, n, p), U=_orthonormal(_normal(g, p, q)),
            theta=_uniform(g, (m,), 1.0, 2.0).sort().values, diag=_dominant_diag(g, n),
        )
    if kind == "eigh":
        p = case["p"]
        a = _normal(g, p, p)
        return dict(a=(a + a.T) * 0.5 + torch.diag(torch.arange(p, device=DEV, dtype=torch.float64)))
    if kind == "tridiag":
        n = case["n"]
        diag = _dominant_diag(g, n)
        rp, ci, val = _banded_csr(g, n, diag, per_row=3, value=0.3, chain=True)
        return dict(
            rp=rp, ci=ci, val=val, diag=diag, R=_normal(g, n, case["m"]),
            theta=_uniform(g, (case["m"],), 0.8, 1.2).sort().values,
        )
    if kind == "train":
        n = case["n"]
        rp, ci, val = _banded_csr(g, n, _dominant_diag(g, n))
        return dict(rp=rp, ci=ci, val=val, X0=_normal(g, n, case["m"]))
    raise ValueError(kind)


class _Learner:
    """A learner handle that goes with its owner."""

    def __init__(self, seed):
        self.h = P.lobpcg_learner_create(0, seed)

    def __del__(self):
        try:
            P.lobpcg_learner_destroy(self.h)
        except Exception:
            pass


def prepare(case, seed):
    kind = case["kind"]
    t = _inputs(case, seed)
    st = dict(case=case, t=t)
    if kind in ("solve_dense", "solve_csr"):
        s = P.Solver(case["n"])
        if kind == "solve_dense":
            s.set_operator_dense(t["A"])
            s.set_preconditioner(P.PRECOND_DIAG)
        else:
            s.set_operator_csr(t["rp"], t["ci"], t["val"])
            s.set_preconditioner(P.PRECOND_LEARNED if case["learned"] else P.PRECOND_DIAG)
            if case["learned"]:
                net = _Learner(1)  # the initial weights
                s.set_learned_weights(P.lobpcg_learner_get_weights(net.h))
            if case["mixed"]:
                s.set_option(P.OPT_PRECISION, P.PREC_FP32)
        s.set_initial_guess(t["X0"])
    elif kind in ("csr", "dense"):
        s = P.Solver(case["n"])
        if kind == "csr":
            s.set_operator_csr(t["rp"], t["ci"], t["val"])
        else:
            s.set_operator_dense(t["A"])
        if case["f32"]:
            s.set_option(P.OPT_PRECISION, P.PREC_FP32)
        s.ensure_workspace(1)
        t["Y"] = torch.zeros_like(t["W"])
    elif kind == "kron":
        s = P.Solver(case["na"] ** 2)
        s.set_operator_kronsum(t["A"], t["V"])
        s.ensure_workspace(1)
        t["Y"] = torch.zeros_like(t["W"])
    elif kind == "gram":
        s = P.Solver(case["n"])
        s.ensure_workspace(32)
        t["C"] = torch.zeros((case["p"], case["q"]), dtype=torch.float64, device=DEV)
    elif kind == "ortho":
        s = P.Solver(case["n"])
        s.ensure_workspace(32)
    elif kind == "rotate":
        m, nact = case["m"], case["nact"]
        s = P.Solver(case["n"])
        s.set_preconditioner(P.PRECOND_DIAG, t["diag"])
        s.ensure_workspace(m)
        p = m + 2 * nact
        t["Vout"] = torch.zeros((case["n"], p), dtype=torch.float64, device=DEV)
        t["AVout"] = torch.zeros((case["n"], p), dtype=torch.float64, device=DEV)
        t["r2"] = torch.zeros(m, dtype=torch.float64, device=DEV)
    elif kind == "eigh":
        p = case["p"]
        s = P.Solver(3 * p)
        s.ensure_workspace(1)
        t["ev"] = torch.zeros(p, dtype=torch.float64, device=DEV)
        t["U"] = torch.zeros((p, p), dtype=torch.float64, device=DEV)
    elif kind == "tridiag":
        s = P.Solver(case["n"])
        s.set_operator_csr(t["rp"], t["ci"], t["val"])
        s.set_preconditioner(P.PRECOND_TRIDIAG)
        s.ensure_workspace(case["m"])
        t["X"] = torch.empty_like(t["R"])
    else:
        s = P.Solver(case["n"])
        s.set_operator_csr(t["rp"], t["ci"], t["val"])
        s.set_preconditioner(P.PRECOND_DIAG)
        s.set_initial_guess(t["X0"])
        s.set_option(P.OPT_MAX_ITER, 5)
        X = s.solve(case["m"], 1e-300).evecs
        L = _Learner(1)
        P.lobpcg_learner_set_supervision(L.h, 1.0)
        P.lobpcg_learner_add_snapshot(L.h, s.h, X, 20, 1e-6)
        st["learner"] = L
        st["w0"] = P.lobpcg_learner_get_weights(L.h)
    st["solver"] = s
    return st


def run(st):
    case, t, s = st["case"], st["t"], st["solver"]
    kind = case["kind"]
    if kind == "solve_dense":
        r = s.solve(case["k"], VECTOR_TOL)
        return dict(evals=r.evals, evecs=r.evecs, status=r.status)
    if kind == "solve_csr":
        # the lowest eigenvalues of this matrix lie 1e-3 apart: a residual of
        # 1e-8 fixes them to rounding, the vectors only to five digits
        r = s.solve(case["k"], SOLVE_TOL, want_vectors=False)
        return dict(evals=r.evals, status=r.status)
    if kind == "csr":
        a, b = case["col"], case["col"] + case["m"]
        apply = P.lobpcg_apply_operator_f32 if case["f32"] else P.lobpcg_apply_operator
        apply(s.h, t["W"][:, a:b], t["Y"][:, a:b])
        return t["Y"][:, a:b]
    if kind == "dense":
        (P.lobpcg_apply_operator_f32 if case["f32"] else P.lobpcg_apply_operator)(s.h, t["W"], t["Y"])
        return t["Y"]
    if kind == "kron":
        P.lobpcg_apply_operator(s.h, t["W"], t["Y"])
        return t["Y"]
    if kind == "gram":
        P.lobpcg_gram(s.h, t["A"], t["B"], t["C"])
        return t["C"]
    if kind == "ortho":
        ny = case["ny"]
        X = t["V"][:, ny:]
        X.copy_(t["W"])  # the call works in place: a new block each time
        if ny:
            P.lobpcg_ortho_against(s.h, X, t["V"][:, :ny])
        else:
            P.lobpcg_ortho(s.h, X)
        return X
    if kind == "rotate":
        m, nact = case["m"], case["nact"]
        p, q = m + 2 * nact, m + nact
        P.lobpcg_rotate(s.h, t["V"], t["AV"], p, t["U"], m, q, t["theta"], m - nact, t["Vout"], t["AVout"], t["r2"])
        return dict(V=t["Vout"], AV=t["AVout"][:, :q], r2=t["r2"])
    if kind == "eigh":
        P.lobpcg_small_eigh(s.h, t["a"], t["ev"], t["U"])
        return dict(evals=t["ev"], evecs=t["U"])
    if kind == "tridiag":
        t["X"].copy_(t["R"])  # the call works in place: a new block each time
        P.lobpcg_tridiag_apply(s.h, t["X"], t["theta"])
        return t["X"]
    L = st["learner"].h
    P.lobpcg_learner_set_weights(L, st["w0"])
    P.lobpcg_learner_train(L, case["steps"], case["cols"], 1e-3, 7)
    return dict(weights=P.lobpcg_learner_get_weights(L))


# ---- what a pass cannot do without -------------------------------------------

_ITERS = 20  # iterations that a whole solve is charged with


def _csr_work(n, m, val, vec):
    nnz = n * 41
    return nnz * (val + 4) + 4 * (n + 1) + 2 * n * m * vec, 2 * nnz * m


def work(case):
    kind = case["kind"]
    if kind in ("solve_dense", "solve_csr"):
        # an iteration: the operator read once, the basis [X P W] and its
        # product read once and written once
        n, m = case["n"], case["block"]
        if kind == "solve_dense":
            op, fl = 8 * n * n, 2 * n * n * m
        else:
            op, fl = _csr_work(n, m, 8, 8)
        return dict(bytes=_ITERS * (op + 2 * 2 * 3 * n * m * 8), flops=_ITERS * (fl + 2 * n * (9 + 2 * 6) * m * m))
    if kind == "csr":
        b, f = _csr_work(case["n"], case["m"], *((4, 4) if case["f32"] else (8, 8)))
        return dict(bytes=b, flops=f)
    if kind == "dense":
        n, m, s = case["n"], case["m"], 4 if case["f32"] else 8
        return dict(bytes=s * (n * n + 2 * n * m), flops=2 * n * n * m)
    if kind == "kron":
        na, m = case["na"], case["m"]
        return dict(bytes=8 * (2 * na * na * m + 2 * na * na), flops=4 * na**3 * m)
    if kind == "gram":
        n, p, q = case["n"], case["p"], case["q"]
        return dict(bytes=8 * (n * (p + q) + p * q), flops=2 * n * p * q)
    if kind == "ortho":
        n, ny, nw = case["n"], case["ny"], case["nw"]
        return dict(bytes=8 * n * (ny + 2 * nw), flops=2 * n * nw * (2 * ny + 2 * nw))
    if kind == "rotate":
        n, m, a = case["n"], case["m"], case["nact"]
        p, q = m + 2 * a, m + a
        return dict(bytes=8 * n * (2 * p + 2 * q + a + 1), flops=4 * n * p * q)
    if kind == "eigh":
        p = case["p"]
        return dict(bytes=8 * (2 * p * p + p), flops=9 * p**3)
    if kind == "tridiag":
        n, m = case["n"], case["m"]
        return dict(bytes=8 * n * (2 * m + 2), flops=8 * n * m)
    # train: per step the gathered columns R and T, the operator once, the
    # gradient block once; forward and backward through the 3-128-128-1 net
    n, c = case["n"], case["cols"]
    b, f = _csr_work(n, c, 8, 8)
    return dict(bytes=case["steps"] * (b + 8 * n * (4 * c + 16)), flops=case["steps"] * (f + 8 * n * c * 8))


# ---- the same outputs in plain 64-bit torch ----------------------------------


def _orient(U, by):
    pick = U.gather(0, by[None, :])[0]
    return U * torch.where(pick < 0, -1.0, 1.0)


def _csr_product(rp, ci, val, W):
    """A W, a few million stored entries at a time."""
    n = rp.numel() - 1
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), (rp[1:] - rp[:-1]).long())
    Y = torch.zeros((n, W.shape[1]), dtype=torch.float64, device=DEV)
    step = 4_000_000
    for a in range(0, ci.numel(), step):
        z = min(a + step, ci.numel())
        Y.index_add_(0, rows[a:z], val[a:z, None] * W[ci[a:z].long()])
    return Y


def _cyclic_reduction(t, e, R):
    """Solves tridiag(e, t, e) x = r for each column of t and R (n x m) by
    parallel cyclic reduction (the rows' off-diagonal e: n, last one 0)."""
    n = t.shape[0]
    hi = e[:, None].expand_as(t).clone()  # coupling of row i to row i + s
    lo = torch.zeros_like(hi)  # coupling of row i to row i - s
    lo[1:] = hi[:-1]
    b, d, s = t.clone(), R.clone(), 1
    while s < n:
        def up(x, fill):  # row i - s
            return torch.cat([torch.full_like(x[:s], fill), x[:-s]])

        def down(x, fill):  # row i + s
            return torch.cat([x[s:], torch.full_like(x[:s], fill)])

        al, ah = -lo / up(b, 1.0), -hi / down(b, 1.0)
        b, d, lo, hi = (
            b + al * up(hi, 0.0) + ah * down(lo, 0.0),
            d + al * up(d, 0.0) + ah * down(d, 0.0),
            al * up(lo, 0.0),
            ah * down(hi, 0.0),
        )
        s *= 2
    return d / b


def exact(case, seed):
    kind = case["kind"]
    if kind in ("train", "solve_csr"):  # a long iteration, and no closed form
        return None
    t = _inputs(case, seed)
    if kind == "solve_dense":
        lam, U = torch.linalg.eigh(t["A"].cpu())
        U = U[:, : case["k"]]
        return dict(evals=lam[: case["k"]], evecs=_orient(U, U.abs().argmax(0)), status=None)
    if kind == "csr":
        val = t["val"].float().double() if case["f32"] else t["val"]
        W = t["W"][:, case["col"] : case["col"] + case["m"]].double().contiguous()
        return _csr_product(t["rp"], t["ci"], val, W)
    if kind == "dense":
        A = t["A"].float().double() if case["f32"] else t["A"]
        return A @ t["W"].double()
    if kind == "kron":
        na, m = case["na"], case["m"]
        Y = torch.empty((na * na, m), dtype=torch.float64, device=DEV)
        for j in range(m):
            Wj = t["W"][:, j].reshape(na, na).contiguous()
            Y[:, j] = (t["A"] @ Wj + Wj @ t["A"] + t["V"] * Wj).reshape(-1)
        return Y
    if kind == "gram":
        return t["A"].T @ t["B"]
    if kind == "ortho":
        W = t["W"] / t["W"].norm(dim=0)
        Y = t["V"][:, : case["ny"]]
        for _ in range(2):
            W = _orthonormal(W - Y @ (Y.T @ W))
        return W
    if kind == "rotate":
        m, nact = case["m"], case["nact"]
        q = m + nact
        VU, AVU = t["V"] @ t["U"], t["AV"] @ t["U"]
        R = AVU[:, :m] - VU[:, :m] * t["theta"]
        T = (t["diag"][:, None] - t["theta"][None, m - nact :]).abs()
        T = torch.maximum(T, 1e-8 * t["theta"][m - nact :].abs().clamp(min=1.0))
        return dict(V=torch.cat([VU, R[:, m - nact :] / T], 1), AV=AVU, r2=(R * R).sum(0))
    if kind == "eigh":
        lam, U = torch.linalg.eigh(t["a"].cpu())
        return dict(evals=lam, evecs=_orient(U, torch.arange(case["p"])))
    if kind == "tridiag":
        n = case["n"]
        rp, ci = t["rp"].long(), t["ci"].long()
        rows = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
        at = ci == rows + 1
        e = torch.zeros(n, dtype=torch.float64, device=DEV)
        e[rows[at]] = t["val"][at]
        off = e.abs()
        off[1:] += e[:-1].abs()
        delta = 1e-8 * t["theta"].abs().clamp(min=1.0)
        T = torch.maximum((t["diag"][:, None] - t["theta"]).abs(), off[:, None] + delta)
        return _cyclic_reduction(T, e, t["R"])
    raise ValueError(kind)
