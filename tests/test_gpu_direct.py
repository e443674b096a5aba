"""Small products of fp32 matrices: fmt_gemm in one launch, operands rounded on the way into the matrix cores, against the CPU
oracle, against the general route (forced through FMT_GEMM_PLAN=general) and against the prepared calls."""
import ctypes

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# every pair of rounding and pieces that takes the route: one fp16 piece, one bf16 piece (e < 8 and e == 8), two bf16 pieces
FORMATS = [(5, 10, True), (5, 10, False), (4, 3, True), (8, 7, True), (8, 7, False), (8, 3, True), (6, 9, True), (6, 9, False),
           (7, 8, True), (2, 15, False)]
LAYOUTS = [(False, False), (False, True), (True, False), (True, True)]
SHAPES = [(1, 1, 1), (2, 3, 7), (5, 4, 8), (31, 33, 31), (32, 32, 32), (33, 65, 33), (64, 40, 64), (9, 20, 86), (7, 100, 129),
          (256, 10, 1024), (130, 70, 257), (512, 200, 100)]


@pytest.fixture(scope="module")
def fmt():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2103_15940_amd as lib
    return lib


@pytest.fixture(autouse=True)
def plain_environment(monkeypatch):
    for name in ("FMT_GEMM_PLAN", "FMT_GEMM_WINDOW"):
        monkeypatch.delenv(name, raising=False)


def stored(X, transposed, pad, offset):
    """X (or its transpose) on the GPU with `pad` extra columns, the first element `offset` floats past a 16-byte boundary."""
    S = np.ascontiguousarray(X.T if transposed else X)
    ld = S.shape[1] + pad
    buf = torch.full((S.shape[0] * ld + offset,), float("nan"), device="cuda")
    view = buf[offset:].view(S.shape[0], ld)[:, :S.shape[1]]
    view.copy_(torch.from_numpy(S))
    return view


def product(fmt, A, B, f, tA, tB, pad=0, offset=0):
    C = torch.full((A.shape[0], B.shape[1] + pad), 7.0, device="cuda")
    out = C[:, :B.shape[1]]
    fmt.fmt_gemm(stored(A, tA, pad, offset), stored(B, tB, pad, offset), f, transA=tA, transB=tB, out=out)
    torch.cuda.synchronize()
    assert bool((C[:, B.shape[1]:] == 7.0).all())                    # nothing beyond the result is written
    return out.cpu().numpy()


def launches(fmt, call):
    """Kernels that a call launches: the nodes of a graph recorded from it."""
    lib = fmt.raw_library()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        call()                                                       # grows the stream's scratch
        stream.synchronize()
        graph, count = ctypes.c_void_p(), ctypes.c_size_t()
        assert lib.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), 1) == 0
        call()
        assert lib.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    assert lib.hipGraphDestroy(graph) == 0
    return count.value


def bits(t):
    return t.view(torch.int32)


@pytest.mark.parametrize("e,m,d", FORMATS)
@pytest.mark.parametrize("shape", SHAPES)
def test_every_layout_and_alignment(fmt, e, m, d, shape, monkeypatch):
    """Integers small enough for every partial sum to be exact: the oracle's bits whatever the order of the sums.  All layouts,
    leading dimensions and base alignments (k-contiguous rows of any alignment, k that ends inside a block of 32 or of 8)."""
    monkeypatch.setenv("FMT_GEMM_PLAN", "direct")
    M, N, K = shape
    rng = np.random.default_rng(M + 10 * N + 100 * K + e)
    top = 3 if m >= 3 else 1
    A = rng.integers(-top, top + 1, (M, K)).astype(np.float32) * np.float32(0.25)
    B = rng.integers(-top, top + 1, (K, N)).astype(np.float32) * np.float32(0.25)
    want = oracle.gemm(A, B, e, m, d)
    for i, (tA, tB) in enumerate(LAYOUTS):
        for pad, offset in ((0, 0), (4, 0), (1, 0), (3, 1)):
            got = product(fmt, A, B, (e, m, d), tA, tB, pad, offset)
            assert np.array_equal(got, want), (tA, tB, pad, offset)


@pytest.mark.parametrize("M,N,K,parts", [(60, 50, 200, 1), (40, 70, 512, 2), (40, 70, 523, 2), (33, 31, 800, 3), (100, 64, 1030, 4),
                                         (64, 64, 2048, 8), (70, 130, 2075, 8), (250, 300, 777, 3)])
@pytest.mark.parametrize("e,m,d", [(5, 10, True), (8, 7, True), (8, 7, False), (7, 8, True), (6, 9, True), (6, 9, False)])
def test_bits_of_the_general_route_with_k_in_parts(fmt, e, m, d, M, N, K, parts, monkeypatch):
    """Sums that round at every step, k in 1 to 8 parts (as the plan of the general route has it), K ragged or not: one launch
    gives the bits of the general route's two or three, and of the prepared calls.  The formats whose prepared operands are planes
    choose their parts themselves, and take the plan's where FMT_GEMM_WINDOW=0 turns the planes off."""
    if e == 6:
        monkeypatch.setenv("FMT_GEMM_WINDOW", "0")
    g = torch.Generator(device="cuda").manual_seed(K + M)
    f = (e, m, d)
    for tA, tB in LAYOUTS:
        A = torch.randn((K, M) if tA else (M, K), device="cuda", generator=g)
        B = torch.randn((N, K) if tB else (K, N), device="cuda", generator=g)
        C = [torch.full((M, N), float("nan"), device="cuda") for _ in range(3)]
        monkeypatch.setenv("FMT_GEMM_PLAN", "direct")
        assert launches(fmt, lambda: fmt.fmt_gemm(A, B, f, transA=tA, transB=tB, out=C[0])) == 1
        monkeypatch.setenv("FMT_GEMM_PLAN", "general")
        assert launches(fmt, lambda: fmt.fmt_gemm(A, B, f, transA=tA, transB=tB, out=C[1])) == (2 if parts == 1 else 3)
        fmt.fmt_gemm_prepared(fmt.fmt_prepare(A, f, trans=tA), fmt.fmt_prepare(B, f, trans=not tB), out=C[2])
        torch.cuda.synchronize()
        assert torch.equal(bits(C[0]), bits(C[1])), (tA, tB)
        assert torch.equal(bits(C[0]), bits(C[2])), (tA, tB)


def test_which_route_a_product_takes(fmt):
    """One launch where the rule's estimate is on its side, two or three where it is not: far on either side of the line."""
    for f, shape, want in [((6, 9, True), (64, 64, 32), 1), ((8, 7, True), (64, 64, 32), 1), ((6, 9, True), (256, 256, 512), 1),
                           ((6, 9, True), (1000, 1000, 256), 2), ((8, 7, True), (256, 1024, 512), 2), ((6, 9, True), (64, 64, 2400), 3),
                           ((7, 18, True), (64, 64, 32), 2), ((7, 23, True), (64, 64, 32), 2)]:
        M, N, K = shape
        A, B, C = torch.ones(M, K, device="cuda"), torch.ones(N, K, device="cuda"), torch.empty(M, N, device="cuda")
        assert launches(fmt, lambda: fmt.fmt_gemm(A, B, f, transB=True, out=C)) == want, (f, shape)


@pytest.mark.parametrize("e,m,d", FORMATS)
def test_values_over_the_whole_range(fmt, e, m, d, monkeypatch):
    """Random operands (normal, denormal and flushed values, zeros): within the accumulation bound of the oracle; the bits
    of the prepared calls where they share the representation; and next to the general route."""
    monkeypatch.setenv("FMT_GEMM_PLAN", "direct")
    rng = np.random.default_rng(50 + e + m)
    c = oracle.format_constants(e, m)
    M, N, K = 96, 70, 128
    A = workloads.log2_normal((M, K), max(c["Emin"] / 2.0, -20.0), 3.0, 0.05, rng)
    A[5, :] = workloads.log2_normal(K, c["Emin"] - m / 2.0, 2.0, 0.0, rng) if e < 8 else 0.0
    B = (rng.standard_normal((K, N)) * 0.5).astype(np.float32)
    top = np.float32(min(c["maxN"], 1e30) / 2)                       # overflow is another test's: stay below it in the narrow formats
    A, B = np.clip(A, -top, top), np.clip(B, -top, top)
    got = product(fmt, A, B, (e, m, d), False, False)
    ref = oracle.gemm(A, B, e, m, d).astype(np.float64)
    assert np.linalg.norm(got - ref) <= 1e-6 * np.linalg.norm(ref)   # K = 128: sqrt(K) 2^-24 = 7e-7 at most
    if not (e == 6 and m in (8, 9)):
        pa = fmt.fmt_prepare(torch.from_numpy(A).cuda(), (e, m, d))
        pb = fmt.fmt_prepare(torch.from_numpy(B).cuda(), (e, m, d), trans=True)
        assert np.array_equal(fmt.fmt_gemm_prepared(pa, pb).cpu().numpy().view(np.uint32), got.view(np.uint32))
    monkeypatch.setenv("FMT_GEMM_PLAN", "general")
    general = product(fmt, A, B, (e, m, d), False, False)
    assert np.linalg.norm(got - general) <= 1e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("e,m,d", [(5, 10, True), (6, 9, False), (8, 7, True), (4, 3, True)])
def test_overflow_infinity_nan(fmt, e, m, d, monkeypatch):
    """Elements that overflow the format, infinities and NaN: non-finite results exactly where the oracle has them, NaN where it
    has NaN, and the other outputs untouched by them."""
    monkeypatch.setenv("FMT_GEMM_PLAN", "direct")
    rng = np.random.default_rng(9)
    M, N, K = 70, 66, 100
    A = rng.integers(-2, 3, (M, K)).astype(np.float32)
    B = rng.integers(-2, 3, (K, N)).astype(np.float32)
    A[3, 97], A[40, 0], A[69, 50], B[99, 65], B[10, 2], B[31, 33] = np.inf, np.nan, -3e38, -np.inf, np.nan, 3e38
    A[12, 20], A[12, 21] = np.array([0x7F800001], dtype=np.uint32).view(np.float32)[0], np.inf
    for tA, tB in LAYOUTS:
        got, want = product(fmt, A, B, (e, m, d), tA, tB), oracle.gemm(A, B, e, m, d)
        assert np.array_equal(np.isfinite(got), np.isfinite(want))
        assert np.isnan(got[np.isnan(want)]).all()
        inf = np.isinf(want)
        assert ((got[inf] == want[inf]) | np.isnan(got[inf])).all()
        fin = np.isfinite(want)
        assert np.array_equal(got[fin], want[fin])


@pytest.mark.parametrize("e,m,d", [(5, 10, True), (5, 10, False), (8, 7, True), (8, 7, False)])
@pytest.mark.parametrize("K", [1, 5])
def test_conversion_of_binary16_and_bfloat16(fmt, e, m, d, K, monkeypatch):
    """The vector units' own conversions: every exponent with ties, their neighbours and random mantissas, both signs, and the
    patterns around the thresholds of overflow and flush, times 1 and 2^20 (K = 1: loaded singly, K = 5: in vectors), in one launch
    and as prepared operands: the oracle's roundings, exactly (both factors are powers of two)."""
    rng = np.random.default_rng(e + K)
    half = 1 << (22 - m)
    mant = np.concatenate([[0, 1, half - 1, half, half + 1, 3 * half - 1, 3 * half, 3 * half + 1, 0x7FFFFF], rng.integers(0, 1 << 23, 7)])
    u = (np.arange(255, dtype=np.uint32)[:, None] << 23 | mant.astype(np.uint32)[None, :]).ravel()
    c = oracle.format_constants(e, m)
    edges = np.array([c["minN"], c["minD"], c["minD"] / 2, c["minN"] - c["minD"] / 2, c["maxN"]], dtype=np.float64).astype(np.float32).view(np.uint32)
    u = np.concatenate([u] + [edges + np.uint32(j) for j in (0, 1)] + [edges - np.uint32(1)])
    x = np.concatenate([u, u | np.uint32(0x80000000)]).view(np.float32)
    q = oracle.quantize(x, e, m, d).astype(np.float64)
    A = np.zeros((x.size, K), dtype=np.float32)
    A[:, K - 1] = x
    B = np.zeros((K, 2), dtype=np.float32)
    B[K - 1] = 1.0, 2.0 ** (10 if e == 5 else 20)
    want = q[:, None] * B[K - 1].astype(np.float64)[None, :]
    monkeypatch.setenv("FMT_GEMM_PLAN", "direct")
    got = [product(fmt, A, B, (e, m, d), False, False)]
    monkeypatch.delenv("FMT_GEMM_PLAN")
    pa, pb = fmt.fmt_prepare(torch.from_numpy(A).cuda(), (e, m, d)), fmt.fmt_prepare(torch.from_numpy(B).cuda(), (e, m, d), trans=True)
    got.append(fmt.fmt_gemm_prepared(pa, pb).cpu().numpy())
    plain = np.isfinite(want) & ((want == 0) | (np.abs(want) >= 2.0 ** -126)) & (np.abs(want) < 2.0 ** 127)
    inf = np.isinf(want[:, 0])
    assert plain.sum() > 6000 and (inf.any() or e == 8)
    for g in got:
        assert np.array_equal(g[plain], want[plain].astype(np.float32))
        assert np.array_equal(g[inf, 0], want[inf, 0].astype(np.float32)) or K > 1        # K > 1: infinity times a zero of the padding
