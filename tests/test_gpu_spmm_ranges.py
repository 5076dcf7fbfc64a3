"""The CSR product over the row lengths and sizes by which it picks a kernel:
means from a few entries to several hundred, even and very uneven lengths, below
and above what the waves on the chip take in one step, more steps than a wave
counts its leftover groups for, and W on both sides of 4 GB (32-bit offsets
below, 64-bit addresses above).

Entry by entry against the definition in fp64 by plain torch, within the
summation bound (row length + 2) u sum_j |a_ij| |w_j|."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2305_06668_amd as P

    return P


def gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def matrix(n, mean, kind, seed, tail=False):
    """row_ptr, col, val on the GPU; `tail`: a third of the columns are the last 100."""
    g = gen(seed)
    if kind == "even":
        lens = (mean * (1.0 + 0.11 * torch.randn(n, generator=g, device="cuda"))).round()
    elif kind == "uneven":  # geometric
        lens = (-mean * torch.log(torch.rand(n, generator=g, device="cuda").clamp(min=1e-4))).floor()
    else:  # "few": most rows short, some very long, some empty
        lens = (mean * 0.5 * torch.rand(n, generator=g, device="cuda")).floor()
        lens[::997] = min(250.0 * mean, 4000.0)
    lens = lens.clamp(min=0).long()
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = lens.cumsum(0)
    nnz = int(rp[-1])
    ci = torch.randint(0, n, (nnz,), generator=g, device="cuda")
    if tail:
        last = torch.rand(nnz, generator=g, device="cuda") < 0.3
        ci = torch.where(last, n - 1 - ci % 100, ci)
    val = torch.rand(nnz, generator=g, device="cuda", dtype=torch.float64) * 2 - 1
    return rp.int(), ci.int(), val


def check(rp, ci, val, W, Y, u):
    """Y against A W, a few million entries at a time."""
    n, m = Y.shape
    lens = (rp[1:] - rp[:-1]).long()
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), lens)
    ref = torch.zeros((n, m), dtype=torch.float64, device="cuda")
    mag = torch.zeros_like(ref)
    for a in range(0, ci.numel(), 2_000_000):
        z = min(a + 2_000_000, ci.numel())
        p = val[a:z, None] * W[ci[a:z].long()].double()
        ref.index_add_(0, rows[a:z], p)
        mag.index_add_(0, rows[a:z], p.abs())
    # (the reference's own sums are in 64 bits, in some order: the same bound)
    bound = (lens[:, None] + 2) * (u + 2.0**-53) * mag
    assert bool(((Y.double() - ref).abs() <= bound).all())


def product(P, rp, ci, val, W, a, m, f32):
    n = rp.numel() - 1
    s = P.Solver(n)
    s.set_operator_csr(rp, ci, val)
    if f32:
        s.set_option(P.OPT_PRECISION, P.PREC_FP32)
    s.ensure_workspace(1)
    Y = torch.full((n, m), 5.0, dtype=W.dtype, device="cuda")
    (P.lobpcg_apply_operator_f32 if f32 else P.lobpcg_apply_operator)(s.h, W[:, a : a + m], Y)
    torch.cuda.synchronize()
    s.close()
    return Y


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("m", [8, 16, 32, 64])
@pytest.mark.parametrize(
    "n,mean,kind",
    [
        (70001, 3, "even"), (70001, 22, "even"), (70001, 38, "even"), (70001, 50, "even"), (70001, 100, "even"),
        (70001, 300, "even"), (70001, 38, "uneven"), (70001, 100, "uneven"), (70001, 24, "few"), (2003, 38, "uneven"),
        (2003, 100, "even"), (2003, 300, "few"),
    ],
)
def test_csr_row_lengths(P, n, mean, kind, m, prec):
    print("csr row lengths", n, mean, kind, m, prec, flush=True)
    rp, ci, val = matrix(n, mean, kind, n + mean)
    f32 = prec == "f32"
    W = torch.randn(n, m, generator=gen(m), device="cuda", dtype=torch.float64)
    if f32:
        W, val32 = W.float(), val.float().double()
    Y = product(P, rp, ci, val, W, 0, m, f32)
    check(rp, ci, val32 if f32 else val, W, Y, 2.0**-24 if f32 else 2.0**-53)


@pytest.mark.parametrize("kind", ["even", "few"])
def test_csr_many_steps(P, kind):
    """n = 2.3 million: a wave takes 70 groups of 8 rows."""
    n, m = 2_300_003, 16
    print("csr many steps", kind, flush=True)
    rp, ci, val = matrix(n, 31, kind, 5) if kind == "even" else matrix(n, 62, kind, 5)
    W = torch.randn(n, m, generator=gen(6), device="cuda", dtype=torch.float64)
    check(rp, ci, val, W, product(P, rp, ci, val, W, 0, m, False), 2.0**-53)


@pytest.mark.parametrize("mean,kind", [(4, "even"), (33, "even"), (34, "few")])
@pytest.mark.parametrize("n", [1_048_575, 1_048_576])
def test_csr_large_w(P, n, mean, kind):
    """A W of 512 fp64 columns spans 4 GB from n = 1048576 on; its last rows are
    referenced, and the last columns of each."""
    ldw, m = 512, 16
    print("csr large W", n, mean, kind, flush=True)
    rp, ci, val = matrix(n, mean, kind, 7, tail=True)
    W = torch.randn(n, ldw, generator=gen(8), device="cuda", dtype=torch.float64)
    a = ldw - m
    Y = product(P, rp, ci, val, W, a, m, False)
    check(rp, ci, val, W[:, a:], Y, 2.0**-53)


@pytest.mark.parametrize("m", [33, 34, 36, 40, 41, 64])
def test_csr_misaligned_tail_bits(P, m):
    """More than 32 fp64 columns at an odd leading dimension add a row's entries
    in order, as a block aligned to 16 bytes does, also the last one to eight: the
    same bits."""
    n = 5003
    print("csr misaligned tail", m, flush=True)
    rp, ci, val = matrix(n, 41, "even", 3)
    W = torch.randn(n, m | 1, generator=gen(m), device="cuda", dtype=torch.float64)
    Y = torch.full_like(W, 5.0)
    s = P.Solver(n)
    s.set_operator_csr(rp, ci, val)
    P.lobpcg_apply_operator(s.h, W[:, :m], Y[:, :m])
    torch.cuda.synchronize()
    s.close()
    for a in list(range(0, m - 15, 16)) + [m - 16]:
        Z = product(P, rp, ci, val, W[:, a : a + 16].contiguous(), 0, 16, False)
        assert torch.equal(Y[:, a : a + 16], Z), (m, a)
    check(rp, ci, val, W[:, :m], Y[:, :m], 2.0**-53)
    assert bool((Y[:, m:] == 5.0).all())


@pytest.mark.parametrize("n,mean,kind", [(12_000, 80, "even"), (5_003, 60, "uneven"), (9_001, 400, "few"), (15_001, 80, "even"), (30_001, 48, "uneven"), (44_003, 25, "even"), (65_537, 48, "even"), (109_999, 25, "uneven"), (75_001, 30, "even")])
def test_csr_misaligned_f32(P, n, mean, kind):
    """Nine to sixteen fp32 columns whose rows are not aligned to 16 bytes, and more
    of them around them."""
    rp, ci, val = matrix(n, mean, kind, n)
    for m, ldw, a in [(8, 9, 1), (9, 27, 9), (12, 12 * 3 + 1, 3), (13, 13, 0), (16, 48, 33), (16, 17, 1), (17, 17, 0), (31, 31, 0)]:
        print("csr misaligned f32", n, mean, kind, m, ldw, a, flush=True)
        ldw = max(ldw, a + m)
        W = torch.randn((n, ldw), generator=gen(m), device="cuda", dtype=torch.float64).float()
        Y = torch.full((n, ldw), 5.0, dtype=torch.float32, device="cuda")
        s = P.Solver(n)
        s.set_operator_csr(rp, ci, val)
        s.set_option(P.OPT_PRECISION, P.PREC_FP32)
        s.ensure_workspace(1)
        P.lobpcg_apply_operator_f32(s.h, W[:, a : a + m], Y[:, a : a + m])
        check(rp, ci, val, W[:, a : a + m], Y[:, a : a + m], 2.0**-24)
        assert bool((Y[:, :a] == 5.0).all()) and bool((Y[:, a + m :] == 5.0).all())  # other columns untouched
        s.close()


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("n,mean,kind", [(60_000, 3, "even"), (50_000, 50, "even"), (200_003, 52, "uneven"), (30_001, 80, "even"), (100_003, 64, "even"), (100_003, 100, "few"), (30_001, 300, "even")])
def test_csr_passes(P, n, mean, kind, f32):
    """Each size of the workgroups' LDS, one pass and several, and longer rows of
    products that the cache holds."""
    rp, ci, val = matrix(n, mean, kind, n)
    for m in (6, 12, 16, 32, 64):
        print("csr passes", n, mean, kind, f32, m, flush=True)
        W = torch.randn((n, m), generator=gen(m), device="cuda", dtype=torch.float64)
        W = W.float() if f32 else W
        Y = torch.full((n, m), 5.0, dtype=W.dtype, device="cuda")
        s = P.Solver(n)
        s.set_operator_csr(rp, ci, val)
        if f32:
            s.set_option(P.OPT_PRECISION, P.PREC_FP32)
        s.ensure_workspace(1)
        (P.lobpcg_apply_operator_f32 if f32 else P.lobpcg_apply_operator)(s.h, W, Y)
        check(rp, ci, val, W, Y, 2.0**-24 if f32 else 2.0**-53)
        s.close()
