"""GPU parity of fmt_gemm_fmac8 (Sec. IV-A, Algorithm 1) against the CPU oracle: the order of the
roundings is fixed by the algorithm, so the results must be identical bit for bit."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VARIANTS = [(5, 10, True), (5, 10, False), (6, 9, True), (6, 9, False), (8, 7, True), (8, 7, False)]
LAYOUTS = [(False, False), (False, True), (True, False), (True, True)]


@pytest.fixture(scope="module")
def fmt():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2103_15940_amd as lib
    return lib


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def run(fmt, A, B, f, tA=False, tB=False):
    Ain = np.ascontiguousarray(A.T) if tA else A
    Bin = np.ascontiguousarray(B.T) if tB else B
    C = fmt.fmt_gemm_fmac8(dev(Ain), dev(Bin), f, transA=tA, transB=tB)
    torch.cuda.synchronize()
    ref = oracle.gemm_fmac8(Ain, Bin, f[0], f[1], f[2], transA=tA, transB=tB)
    return C.cpu().numpy(), ref


def assert_bits(got, ref, what):
    g, r = got.view(np.uint32), ref.view(np.uint32)
    if not np.array_equal(g, r):
        bad = np.argwhere(g != r)
        i, j = bad[0]
        raise AssertionError("%s: %d outputs differ; first at (%d,%d): got %r want %r" %
                             (what, len(bad), i, j, got[i, j], ref[i, j]))


@pytest.mark.parametrize("tA,tB", LAYOUTS)
@pytest.mark.parametrize("e,m,d", VARIANTS)
def test_bit_exact_random(fmt, e, m, d, tA, tB):
    rng = np.random.default_rng(100 * e + m)
    M, N, K = 150, 70, 203                # ragged tiles; K not a multiple of 8 or of the stage
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = (rng.standard_normal((K, N)) * 2.0 ** -3).astype(np.float32)
    got, ref = run(fmt, A, B, (e, m, d), tA, tB)
    assert_bits(got, ref, "1/%d/%d/%s" % (e, m, d))
    # results are values of the format
    assert np.array_equal(oracle.quantize(got, e, m, d).view(np.uint32), got.view(np.uint32))


@pytest.mark.parametrize("e,m,d", VARIANTS + [(4, 3, True), (7, 14, False), (3, 5, True), (6, 11, True), (6, 11, False),
                                             (2, 11, True), (6, 12, True), (7, 9, True)])
def test_bit_exact_wide_range(fmt, e, m, d):
    """Operands spread over the whole range of the format: accumulator and product exponents far
    apart (the sticky-bit cases), denormal and flushed accumulators, overflowing accumulators."""
    rng = np.random.default_rng(7 * e + m)
    c = oracle.format_constants(e, m)
    span = c["Emax"] - c["Emin"]
    A = workloads.log2_normal((90, 130), (c["Emin"] + c["Emax"]) / 4, span / 6, 0.05, rng)
    B = workloads.log2_normal((130, 75), (c["Emin"] + c["Emax"]) / 4, span / 6, 0.05, rng)
    got, ref = run(fmt, A, B, (e, m, d), False, True)
    nan = np.isnan(ref)
    assert np.array_equal(np.isnan(got), nan)
    assert_bits(np.where(nan, 0, got).astype(np.float32), np.where(nan, 0, ref).astype(np.float32), "wide range")


@pytest.mark.parametrize("e,m,d", [(5, 10, True), (6, 9, True), (6, 9, False), (6, 11, True)])
def test_single_and_double_precision_steps_agree(fmt, e, m, d, monkeypatch):
    """Formats with e <= 6 and m <= 11 run the fused step in single precision; forced onto the
    double-precision step they must give the same bits (and both equal the oracle)."""
    rng = np.random.default_rng(e + m)
    c = oracle.format_constants(e, m)
    span = c["Emax"] - c["Emin"]
    A = workloads.log2_normal((70, 96), (c["Emin"] + c["Emax"]) / 4, span / 5, 0.05, rng)
    B = workloads.log2_normal((96, 66), (c["Emin"] + c["Emax"]) / 4, span / 5, 0.05, rng)
    fast, ref = run(fmt, A, B, (e, m, d))
    monkeypatch.setenv("FMT_FMAC8_F64", "1")
    slow, _ = run(fmt, A, B, (e, m, d))
    nan = np.isnan(ref)
    assert np.array_equal(np.isnan(fast), nan) and np.array_equal(np.isnan(slow), nan)
    assert np.array_equal(fast[~nan].view(np.uint32), slow[~nan].view(np.uint32))
    assert np.array_equal(fast[~nan].view(np.uint32), ref[~nan].view(np.uint32))


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 7), (64, 64, 8), (65, 63, 9), (10, 300, 40), (200, 17, 1000)])
def test_shapes(fmt, shape):
    M, N, K = shape
    rng = np.random.default_rng(M + 3 * N + 5 * K)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((K, N)).astype(np.float32)
    got, ref = run(fmt, A, B, (6, 9, True))
    assert_bits(got, ref, str(shape))


def test_k_zero_and_nonfinite(fmt):
    C = fmt.fmt_gemm_fmac8(torch.empty((4, 0), device="cuda"), torch.empty((0, 6), device="cuda"), (6, 9, True))
    torch.cuda.synchronize()
    assert float(C.abs().sum()) == 0.0
    rng = np.random.default_rng(3)
    A = rng.standard_normal((20, 24)).astype(np.float32)
    B = rng.standard_normal((24, 20)).astype(np.float32)
    A[2, 3] = np.inf
    A[5, 7] = np.nan
    B[1, 4] = 1e30                     # overflows binary16
    got, ref = run(fmt, A, B, (5, 10, True))
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    fin = ~np.isnan(ref)
    assert np.array_equal(got[fin].view(np.uint32), ref[fin].view(np.uint32))


def test_mlp_layer_shapes(fmt):
    """Configuration 2's first layer (256 x 784 -> 1024) forward with FMAC-8 in 1/6/9 and binary16."""
    cfg = workloads.config2()
    for f in [(6, 9, True), (5, 10, True)]:
        got, ref = run(fmt, cfg["X"], cfg["W"][0].T.copy(), f)
        assert_bits(got, ref, "mlp layer 1 %s" % (f,))


@pytest.mark.parametrize("f", [(6, 9, True), (5, 10, False)])
def test_bench_size_sampled(fmt, f):
    """The size the bench times (2048 x 2048 x 1024): every output is its own chain of K fused steps,
    so the oracle run on 48 sampled rows of A and 48 sampled columns of B gives those 48 x 48 outputs."""
    M, N, K = 2048, 2048, 1024
    rng = np.random.default_rng(17)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = (rng.standard_normal((K, N)) * 0.02).astype(np.float32)
    C = fmt.fmt_gemm_fmac8(dev(A), dev(B), f)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([rng.integers(0, M, 44), [0, 1, M - 2, M - 1]]))
    cols = np.unique(np.concatenate([rng.integers(0, N, 44), [0, 1, N - 2, N - 1]]))
    ref = oracle.gemm_fmac8(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), f[0], f[1], f[2])
    got = C.cpu().numpy()[np.ix_(rows, cols)]
    assert_bits(np.ascontiguousarray(got), ref, "sampled %s" % (f,))


def test_operand_of_more_than_2_to_the_32_elements(fmt):
    """A is (2^22 + 70) x 1024 (16 GiB), B 1024 x 8: sampled rows bit for bit against the oracle."""
    M, K, N = (1 << 22) + 70, 1024, 8
    f = (6, 9, True)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    A = torch.randn((M, K), device="cuda", generator=g)
    B = torch.randn((K, N), device="cuda", generator=g) * 0.05
    C = fmt.fmt_gemm_fmac8(A, B, f)
    torch.cuda.synchronize()
    rng = np.random.default_rng(4)
    edge = [(1 << 31) // K, (1 << 32) // K]
    rows = np.unique(np.concatenate([np.arange(8), np.arange(M - 72, M), rng.integers(0, M, 60)] +
                                    [np.arange(r - 4, r + 4) for r in edge]))
    rows_d = torch.from_numpy(rows).cuda()
    ref = oracle.gemm_fmac8(A[rows_d].cpu().numpy(), B.cpu().numpy(), *f)
    assert_bits(C[rows_d].cpu().numpy(), ref, "sampled rows, M*K > 2^32")


@pytest.mark.parametrize("e,m,d", VARIANTS + [(7, 8, True), (7, 8, False), (4, 3, True)])
def test_against_the_plain_definition(fmt, e, m, d):
    """fmt_gemm_fmac8 compared directly with Algorithm 1 run in exact rational arithmetic
    (oracle/fmac_exact.py: the sum a + w*x as a Fraction, rounded once by a search over the enumerated
    value set) -- no fp64 construction in between.  Operands span the whole exponent range of the
    format, so accumulator and product are often far apart; 1/8/7 and 1/7/8 take the kernel's
    double-precision step, the others its single-precision one.  Small: the definition is slow."""
    from oracle import fmac_exact
    rng = np.random.default_rng(1000 + 10 * e + m + int(d))
    c = oracle.format_constants(e, m)
    span = c["Emax"] - c["Emin"]
    M, N, K = 16, 16, 40
    # two recipes: products mostly inside the range (accumulators wander through the denormal range and
    # far-apart exponents), and products that often overflow the accumulator or the final rounding
    for centre, sigma, min_finite in [(-span / 8, span / 6, M * N * 3 // 4), ((c["Emin"] + c["Emax"]) / 4, span / 5, 8)]:
        A = workloads.log2_normal((M, K), centre, sigma, 0.05, rng)
        B = workloads.log2_normal((K, N), centre, sigma, 0.05, rng)
        want = fmac_exact.gemm_fmac8(A, B, e, m, d)
        assert np.isfinite(want).sum() >= min_finite        # the case is not degenerate
        for tA, tB in LAYOUTS if (e, m, d) == (6, 9, True) else [(False, False)]:
            Ain = np.ascontiguousarray(A.T) if tA else A
            Bin = np.ascontiguousarray(B.T) if tB else B
            got = fmt.fmt_gemm_fmac8(dev(Ain), dev(Bin), (e, m, d), transA=tA, transB=tB)
            torch.cuda.synchronize()
            got = got.cpu().numpy()
            nan = np.isnan(want)
            assert np.array_equal(np.isnan(got), nan)
            assert_bits(np.where(nan, 0, got).astype(np.float32), np.where(nan, 0, want).astype(np.float32),
                        "definition, 1/%d/%d/%s layout %s" % (e, m, d, (tA, tB)))


@pytest.mark.parametrize("M,N", [(17, 33), (16, 16), (700, 800), (2000, 2010)])
@pytest.mark.parametrize("e,m,d", [(6, 9, True), (6, 9, False), (5, 10, True), (6, 11, False), (2, 11, True), (3, 1, True)])
def test_forms_of_the_step_by_stage(fmt, e, m, d, M, N):
    """Every tile size of the kernel (1, 4 and 16 outputs per thread), with stages of 32 k on both sides of the bound
    that decides which form of the fused step a stage takes: products far below it, the largest operands the last values of
    the format whose product is below 2^(Emin-m+52) (or 2^Emax) over the growth of a group and the first above it, a stage with an overflow, one with an infinity, one of
    values around the smallest denormal, and large products that meet a tiny accumulator.  Bit for bit on sampled rows and columns."""
    rng = np.random.default_rng(10 * e + m + M)
    c = oracle.format_constants(e, m)
    limit = min(c["Emin"] - m + 52, c["Emax"])
    K = 32 * 7 + 5
    A = workloads.log2_normal((M, K), -2.0, 3.0, 0.02, rng)
    B = workloads.log2_normal((K, N), -2.0, 3.0, 0.02, rng)
    top = 2.0 ** (limit / 2)

    def clip(X, hi):
        return np.clip(X, -hi, hi).astype(np.float32)
    A, B = clip(A, top / 16), clip(B, top / 16)
    growth = sum((1.0 + 2.0 ** -(m + 1)) ** i for i in range(9))  # of |a + w x| over a group, each step rounded up by half a unit
    edge = np.sqrt(0.99 * 2.0 ** limit / growth)
    step = 2.0 ** (max(np.floor(np.log2(edge)), c["Emin"]) - m)   # of the format at the edge
    below = np.floor(edge / step) * step
    assert below ** 2 < 0.99 * 2.0 ** limit / growth < (below + step) ** 2
    for stage, largest in ((1, below), (2, below + step), (3, 1.5 * top)):
        s = slice(32 * stage, 32 * stage + 32)
        A[:, s] = clip(workloads.log2_normal((M, 32), limit / 2 - 4, 4.0, 0.0, rng), largest)
        B[s, :] = clip(workloads.log2_normal((32, N), limit / 2 - 4, 4.0, 0.0, rng), largest)
    A[M // 2, 32 * 4 + 3] = np.inf
    s = slice(32 * 5, 32 * 6)
    A[:, s] = workloads.log2_normal((M, 32), (c["Emin"] - m) / 2.0, 1.0, 0.0, rng)
    B[s, :] = workloads.log2_normal((32, N), (c["Emin"] - m) / 2.0, 1.0, 0.0, rng)
    s = slice(32 * 6, 32 * 7)                                     # tiny accumulator, then a product with its last bit set
    A[:, s] = clip(workloads.log2_normal((M, 32), limit / 2 - 3, 0.5, 0.0, rng), 0.25 * top)
    B[s, :] = clip(workloads.log2_normal((32, N), limit / 2 - 3, 0.5, 0.0, rng), 0.25 * top)
    A[:, 32 * 6:32 * 7:2] = np.float32(c["minD"] if e > 2 else 1.0)
    B[32 * 6:32 * 7:2, :] = np.float32(1.0)
    C = fmt.fmt_gemm_fmac8(dev(A), dev(B), (e, m, d))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([rng.integers(0, M, 30), [0, M // 2, M - 1]]))
    cols = np.unique(np.concatenate([rng.integers(0, N, 30), [0, N - 1]]))
    ref = oracle.gemm_fmac8(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), e, m, d)
    got = np.ascontiguousarray(C.cpu().numpy()[np.ix_(rows, cols)])
    nan = np.isnan(ref)
    assert np.array_equal(np.isnan(got), nan)
    assert_bits(np.where(nan, 0, got).astype(np.float32), np.where(nan, 0, ref).astype(np.float32), "stages")


@pytest.mark.parametrize("M,N,K", [(31, 33, 63), (32, 32, 64), (33, 65, 65), (1, 2, 9), (2000, 2010, 45), (2048, 1999, 33)])
@pytest.mark.parametrize("d", [True, False])
def test_binary16_tiles(fmt, d, M, N, K):
    """1/5/10 at the edges of the 32 x 32 and 64 x 64 tiles and of their stages of 64 and 32 k, with accumulators that wander
    through the denormals and that overflow.  Bit for bit on sampled rows and columns, all layouts."""
    rng = np.random.default_rng(M + N + K)
    A = workloads.log2_normal((M, K), -6.0, 4.0, 0.05, rng)
    B = workloads.log2_normal((K, N), -6.0, 4.0, 0.05, rng)
    A[M // 2] = workloads.log2_normal((K,), 8.0, 2.0, 0.0, rng)
    rows = np.unique(np.concatenate([rng.integers(0, M, 24), [0, M // 2, M - 1]]))
    cols = np.unique(np.concatenate([rng.integers(0, N, 24), [0, N - 1]]))
    ref = oracle.gemm_fmac8(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), 5, 10, d)
    for tA, tB in LAYOUTS:
        C = fmt.fmt_gemm_fmac8(dev(A.T if tA else A), dev(B.T if tB else B), (5, 10, d), transA=tA, transB=tB)
        torch.cuda.synchronize()
        got = np.ascontiguousarray(C.cpu().numpy()[np.ix_(rows, cols)])
        nan = np.isnan(ref)
        assert np.array_equal(np.isnan(got), nan)
        assert_bits(np.where(nan, 0, got).astype(np.float32), np.where(nan, 0, ref).astype(np.float32), "layout %s" % ((tA, tB),))


@pytest.mark.parametrize("e,m,d", [(6, 9, True), (6, 9, False), (6, 11, True), (6, 3, True)])
def test_sums_next_to_a_power_of_two(fmt, e, m, d):
    """A power of two plus a product far below it that fills the last places of the 53-bit sum, on either side: the sum lies next to
    the end of a binade with its last bit set."""
    rng = np.random.default_rng(e + m)
    n = 96
    A, B = np.zeros((n, 16), np.float32), np.zeros((16, n), np.float32)
    A[:, 0] = 2.0 ** rng.integers(-6, 7, n)
    B[0] = rng.choice([-1.0, 1.0], n) * 2.0 ** rng.integers(-6, 7, n)
    frac = lambda k: 1.0 + (2 * rng.integers(0, 1 << (m - 1), k) + 1) * 2.0 ** -m      # noqa: E731  (last bit set)
    A[:, 1] = rng.choice([-1.0, 1.0], n) * frac(n) * 2.0 ** rng.integers(-22, -12, n)
    B[1] = frac(n) * 2.0 ** rng.integers(-22, -12, n)
    got, ref = run(fmt, A, B, (e, m, d))
    assert_bits(got, ref, "1/%d/%d" % (e, m))


FLUSHING = [(6, 9), (6, 11), (6, 3), (4, 3), (5, 2), (3, 1), (5, 10)]


@pytest.mark.parametrize("M,N", [(40, 70), (700, 800), (2000, 2010)])
@pytest.mark.parametrize("e,m", FLUSHING)
def test_flush_next_to_the_smallest_normal(fmt, e, m, M, N):
    """Sums that round to minN or just miss it, at every tile size: products and accumulator-plus-product sums half a step below minN
    (a tie, which goes to minN), one bit of the product on either side of it, and between there and minN.  Both signs.  A second
    product that adds nothing but its own bits follows, so that a sum wrongly flushed shows in every later step as well."""
    rng = np.random.default_rng(10 * e + m)
    c = oracle.format_constants(e, m)
    lo = c["Emin"]
    h = 2.0 ** (lo // 2)                                          # B's values; h * g = 2^Emin
    g = 2.0 ** (lo - lo // 2)
    last = 2.0 ** -m
    # in units of 2^Emin; values of the format times a power of two that the operands' exponents absorb
    heads = np.array([0.0, 1.0 - last, 1.0 - last / 2, 0.5 * (2.0 - last), 0.5 * (2.0 - 2 * last), 1.0, 1.0 + last, 0.75, 2.0])
    tails = np.array([0.0, last / 2, last / 4, last / 8, last, -last / 2, -last / 4, -last / 8, -last])
    A, B = np.zeros((M, 16), np.float32), np.zeros((16, N), np.float32)
    head, tail = rng.choice(heads, M), rng.choice(tails, M)
    head[:9], tail[:9] = heads, 0.0
    A[:, 0], A[:, 1] = head * g, tail * g
    A[:, 2] = rng.choice([0.0, last / 2, -last / 2], M) * g
    B[:3] = rng.choice([-h, h], N)
    B[1:3] *= rng.choice([1.0, 1.0, -1.0], N)
    A[:, 8:11], B[8:11] = A[:, :3], B[:3]                         # and in a second group
    C = fmt.fmt_gemm_fmac8(dev(A), dev(B), (e, m, False))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(36), rng.integers(0, M, 120)]))
    cols = np.unique(np.concatenate([rng.integers(0, N, 24), [0, N - 1]]))
    ref = oracle.gemm_fmac8(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), e, m, False)
    assert_bits(np.ascontiguousarray(C.cpu().numpy()[np.ix_(rows, cols)]), ref, "next to minN")


@pytest.mark.parametrize("M,N", [(200, 200), (700, 800), (2000, 2010)])
@pytest.mark.parametrize("e,m", FLUSHING)
def test_flush_of_random_sums_around_the_smallest_normal(fmt, e, m, M, N):
    """Flushing formats with operands around 2^(Emin/2), so that sums wander about minN."""
    rng = np.random.default_rng(100 * e + m)
    c = oracle.format_constants(e, m)
    A = workloads.log2_normal((M, 64), c["Emin"] / 2, 1.0, 0.02, rng)
    B = workloads.log2_normal((64, N), c["Emin"] / 2, 1.0, 0.02, rng)
    C = fmt.fmt_gemm_fmac8(dev(A), dev(B), (e, m, False))
    torch.cuda.synchronize()
    rows, cols = np.unique(rng.integers(0, M, 150)), np.unique(rng.integers(0, N, 150))
    ref = oracle.gemm_fmac8(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), e, m, False)
    assert (ref == 0.0).any() and (ref != 0.0).any()
    assert_bits(np.ascontiguousarray(C.cpu().numpy()[np.ix_(rows, cols)]), ref, "around minN")


@pytest.mark.parametrize("M,N", [(16, 48), (70, 133), (700, 800), (2000, 2050)])
@pytest.mark.parametrize("e,m,d", [(6, 9, True), (6, 9, False), (6, 11, True), (8, 7, True), (7, 14, False)])
def test_rare_elements_limits_and_strides(fmt, e, m, d, M, N):
    """What the loads, the roundings and the choice of the form of a stage of 32 k look at, at every tile size, in all layouts and with
    leading dimensions of their own: rows and columns of which all, or a few at an edge, lie inside a tile (their elements come without
    tests of their own); elements around the overflow threshold, infinities and NaN in one row, so that one wave of a stage rounds in
    the general form and the others in the short one; and stages whose largest magnitudes, which are taken before the rounding, have a
    product at the limit of the wide form, or beyond it before or after the rounding only."""
    K = 11 * 32 + 5
    rng = np.random.default_rng(100 * e + m + M)
    c = oracle.format_constants(e, m)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = (rng.standard_normal((K, N)) * 2.0 ** -3).astype(np.float32)
    growth = sum((1.0 + 2.0 ** -(m + 1)) ** i for i in range(9))
    limit = 0.99 * 2.0 ** min(c["Emin"] - m + 52, c["Emax"]) / growth
    for s, by in enumerate((0.0, 2.0 ** -(m + 2), -2.0 ** -(m + 2), 2.0 ** -(m + 4), -2.0 ** -(m + 4), 2.0 ** -m, -2.0 ** -m)):
        w = 12.0 * (1.0 + rng.random() / 4)
        A[rng.integers(0, M), 32 * s + 3], B[32 * s + 3, rng.integers(0, N)] = w, min(limit / w * (1.0 + by), 2.0 ** 60)
    top, ulp = float(c["maxN"]), 2.0 ** (c["Emax"] - m)
    over = np.array([top, min(top + ulp / 2, 3.4e38), np.nextafter(np.float32(min(top + ulp / 2, 3.4e38)), np.float32(0)), np.inf, np.nan], np.float32)
    A[M // 2, 32 * 7 + 1: 32 * 7 + 6], B[32 * 9 + 7, N // 2] = over, over[1]
    A[M - 1, 32 * 8], B[32 * 10, N - 1] = -top, np.inf
    rows = np.unique(np.concatenate([[0, M - 1, M // 2, M - 2], rng.integers(0, M, 40)])) if M > 100 else np.arange(M)
    cols = np.unique(np.concatenate([[0, N - 1, N // 2, N - 2], rng.integers(0, N, 40)])) if M > 100 else np.arange(N)
    ref = oracle.gemm_fmac8(np.ascontiguousarray(A[rows]), np.ascontiguousarray(B[:, cols]), e, m, d)
    nan = np.isnan(ref)
    assert nan.any() and np.isfinite(ref).sum() > ref.size / 2
    for tA, tB in LAYOUTS:
        a, b = (dev(x.T if t else x) for x, t in ((A, tA), (B, tB)))
        wide = [torch.full((x.shape[0], x.shape[1] + 5), float("nan"), device="cuda") for x in (a, b)]
        for w, x in zip(wide, (a, b)):
            w[:, :x.shape[1]] = x
        C = fmt.fmt_gemm_fmac8(wide[0][:, :a.shape[1]], wide[1][:, :b.shape[1]], (e, m, d), transA=tA, transB=tB)
        torch.cuda.synchronize()
        got = np.ascontiguousarray(C.cpu().numpy()[np.ix_(rows, cols)])
        assert np.array_equal(np.isnan(got), nan), "layout %s" % ((tA, tB),)
        assert_bits(np.where(nan, 0, got).astype(np.float32), np.where(nan, 0, ref).astype(np.float32), "layout %s" % ((tA, tB),))
