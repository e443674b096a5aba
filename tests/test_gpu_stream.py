"""GPU parity of fmt_quantize / fmt_histogram (through the C ABI) against the CPU oracle:
bit-exact values, bit-exact integer counts."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VARIANTS = [(5, 10, True), (5, 10, False), (6, 9, True), (6, 9, False), (8, 7, True), (8, 7, False)]
OTHER = [(2, 1, True), (3, 2, False), (4, 3, True), (7, 16, False), (8, 23, True), (7, 23, True), (5, 23, False),
         (8, 1, False), (2, 22, True)]


@pytest.fixture(scope="module")
def fmt():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2103_15940_amd as lib
    return lib


def bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def assert_same_values(got, want, what):
    g, w = bits(got), bits(want)
    if not np.array_equal(g, w):
        bad = np.flatnonzero(g != w)
        i = bad[0]
        raise AssertionError("%s: %d of %d elements differ; first at %d: got %08x want %08x" %
                             (what, bad.size, g.size, i, g[i], w[i]))


def assert_same_hist(fmtlib, hist, want, what):
    h = fmtlib.hist_to_dict(hist)
    for k in fmtlib.CLASS_NAMES:
        assert h[k] == want[k], "%s: class %s got %d want %d" % (what, k, h[k], want[k])
    assert np.array_equal(h["bins"], want["bins"]), "%s: bins differ\n%s\n%s" % (what, h["bins"], want["bins"])


def mixed(n, seed):
    rng = np.random.default_rng(seed)
    parts = [workloads.random_bits(n // 3, seed), workloads.log2_normal(n // 3, -14, 6, 0.01, rng)]
    rest = n - sum(p.size for p in parts)
    sp = workloads.special_values()
    parts.append(np.resize(sp, rest))
    x = np.concatenate(parts)
    rng.shuffle(x)
    return x


@pytest.mark.parametrize("e,m,d", VARIANTS + OTHER)
def test_quantize_and_fused_hist_bit_exact(fmt, e, m, d):
    n = (1 << 18) + 37                      # several workgroups' worth of tiles and a ragged tail
    x = mixed(n, 17 * e + m)
    xd = dev(x)
    hist = fmt.new_hist()
    y = fmt.fmt_quantize(xd, (e, m, d), hist=hist)
    y2 = fmt.fmt_quantize(xd, (e, m, d))   # store-only kernel
    torch.cuda.synchronize()
    want = oracle.quantize(x, e, m, d)
    assert_same_values(y.cpu().numpy(), want, "fused 1/%d/%d/%s" % (e, m, d))
    assert_same_values(y2.cpu().numpy(), want, "plain 1/%d/%d/%s" % (e, m, d))
    assert_same_hist(fmt, hist, oracle.histogram(x, e, m), "fused hist 1/%d/%d" % (e, m))
    h2 = fmt.fmt_histogram(xd, (e, m, d))
    torch.cuda.synchronize()
    assert_same_hist(fmt, h2, oracle.histogram(x, e, m), "hist-only 1/%d/%d" % (e, m))


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 63, 64, 65, 511, 2048, 2049, 8191, 8192 * 4 + 1, 70001])
def test_ragged_sizes(fmt, n):
    x = mixed(max(n, 8), n)[:n]
    xd = dev(x)
    for (e, m, d) in [(6, 9, True), (5, 10, False), (8, 7, True)]:
        hist = fmt.new_hist()
        y = fmt.fmt_quantize(xd, (e, m, d), hist=hist)
        torch.cuda.synchronize()
        assert_same_values(y.cpu().numpy(), oracle.quantize(x, e, m, d), "n=%d" % n)
        assert_same_hist(fmt, hist, oracle.histogram(x, e, m), "n=%d" % n)


def test_empty_input(fmt):
    xd = torch.empty(0, dtype=torch.float32, device="cuda")
    hist = torch.full((72,), 7, dtype=torch.int64, device="cuda")
    y = fmt.fmt_quantize(xd, (6, 9, True), hist=hist)
    torch.cuda.synchronize()
    assert y.numel() == 0 and int(hist.abs().sum()) == 0
    hist.fill_(5)
    fmt.fmt_histogram(xd, (6, 9, True), hist=hist)
    torch.cuda.synchronize()
    assert int(hist.abs().sum()) == 0


@pytest.mark.parametrize("ox,oy", [(0, 0), (1, 1), (3, 3), (1, 0), (0, 2), (2, 3)])
def test_misaligned_pointers(fmt, ox, oy):
    """Offsets in elements from a 256-byte aligned base: equal offsets take the vector path with a
    scalar head, unequal ones the dword fallback."""
    n = 50003
    x = mixed(n + 8, 5 + ox * 4 + oy)
    xb = dev(x)
    yb = torch.zeros(n + 8, dtype=torch.float32, device="cuda")
    xs, ys = xb[ox:ox + n], yb[oy:oy + n]
    hist = fmt.new_hist()
    fmt.fmt_quantize(xs, (6, 9, False), out=ys, hist=hist)
    h2 = fmt.fmt_histogram(xs, (6, 9, False))
    torch.cuda.synchronize()
    assert_same_values(ys.cpu().numpy(), oracle.quantize(x[ox:ox + n], 6, 9, False), "offsets %d,%d" % (ox, oy))
    want = oracle.histogram(x[ox:ox + n], 6, 9)
    assert_same_hist(fmt, hist, want, "fused")
    assert_same_hist(fmt, h2, want, "hist-only")
    # nothing outside [oy, oy+n) was written
    full = yb.cpu().numpy()
    assert np.all(full[:oy] == 0) and np.all(full[oy + n:] == 0)


def test_in_place(fmt):
    x = mixed(100000, 3)
    xd = dev(x)
    out = fmt.fmt_quantize(xd, (5, 10, True), out=xd)
    torch.cuda.synchronize()
    assert out.data_ptr() == xd.data_ptr()
    assert_same_values(xd.cpu().numpy(), oracle.quantize(x, 5, 10, True), "in place")


@pytest.mark.parametrize("exp_lo", [-192, -160, -149, -127, -126, -48, -24, 0, 64, 128])
def test_histogram_windows(fmt, exp_lo):
    """Windows that reach into the fp32-denormal binades use the per-binade rows."""
    den = (workloads.random_bits(60000, 9).view(np.uint32) & np.uint32(0x807FFFFF)).view(np.float32)   # fp32 denormals
    x = np.concatenate([mixed(60000, exp_lo + 500), den])
    xd = dev(x)
    hist = fmt.fmt_histogram(xd, (8, 7, True), exp_lo=exp_lo)
    h2 = fmt.new_hist()
    y = fmt.fmt_quantize(xd, (8, 7, True), hist=h2, exp_lo=exp_lo)
    torch.cuda.synchronize()
    want = oracle.histogram(x, 8, 7, exp_lo=exp_lo)
    assert_same_hist(fmt, hist, want, "exp_lo=%d" % exp_lo)
    assert_same_hist(fmt, h2, want, "fused exp_lo=%d" % exp_lo)
    assert_same_values(y.cpu().numpy(), oracle.quantize(x, 8, 7, True), "values")


@pytest.mark.parametrize("e,m", [(5, 10), (6, 9), (8, 7)])
def test_exhaustive_codes_and_boundaries(fmt, e, m):
    """Every code of the format, every midpoint between adjacent codes and the fp32 neighbours of
    each midpoint, both signs -- the same probes that pin the oracle, now through the GPU."""
    from fmtdef import decode_codes
    v = decode_codes(e, m)
    pos = v[: 1 << 15].astype(np.float64)
    last = ((1 << e) - 1) << m
    lo, hi = pos[:last].copy(), pos[1:last + 1].copy()
    hi[-1] = 2.0 ** (2 ** (e - 1))
    mid = ((lo + hi) / 2).astype(np.float32)
    probes = np.concatenate([v, mid, np.nextafter(mid, np.float32(0)), np.nextafter(mid, np.float32(np.inf))])
    probes = np.concatenate([probes, -probes])
    xd = dev(probes)
    for d in (True, False):
        hist = fmt.new_hist()
        y = fmt.fmt_quantize(xd, (e, m, d), hist=hist)
        torch.cuda.synchronize()
        got, want = y.cpu().numpy(), oracle.quantize(probes, e, m, d)
        nan = np.isnan(want)
        assert_same_values(got, want, "codes 1/%d/%d/%s" % (e, m, d))
        assert np.all(bits(got[nan]) == 0x7FC00000)
        assert_same_hist(fmt, hist, oracle.histogram(probes, e, m), "codes hist")


def test_config1_full(fmt):
    """Configuration 1: 2^20 values, log2|x| ~ N(-14, 6^2), 1 % zeros, 1/6/9 with denormals and flushed."""
    x = workloads.config1()["x"]
    xd = dev(x)
    ho = oracle.histogram(x, 6, 9)
    for d in (True, False):
        hist = fmt.new_hist()
        y = fmt.fmt_quantize(xd, (6, 9, d), hist=hist)
        torch.cuda.synchronize()
        assert_same_values(y.cpu().numpy(), oracle.quantize(x, 6, 9, d), "config1 d=%s" % d)
        assert_same_hist(fmt, hist, ho, "config1")


def test_config5_reduced_all_variants(fmt):
    """Configuration 5's heavy-tailed tensor at 2^23 elements: all six variants element by element."""
    x = workloads.config5(n=1 << 23)
    xd = dev(x)
    for (e, m, d) in VARIANTS:
        hist = fmt.new_hist()
        y = fmt.fmt_quantize(xd, (e, m, d), hist=hist)
        torch.cuda.synchronize()
        assert_same_values(y.cpu().numpy(), oracle.quantize(x, e, m, d), "config5 1/%d/%d/%s" % (e, m, d))
        assert_same_hist(fmt, hist, oracle.histogram(x, e, m), "config5 hist")


def test_repeated_calls_are_deterministic(fmt):
    x = workloads.config5(n=1 << 22)
    xd = dev(x)
    ref = None
    for _ in range(5):
        hist = fmt.fmt_histogram(xd, (5, 10, True))
        torch.cuda.synchronize()
        h = hist.cpu().numpy()
        if ref is None:
            ref = h
        assert np.array_equal(h, ref)


def test_non_default_stream(fmt):
    x = mixed(300000, 77)
    s = torch.cuda.Stream()
    xd = dev(x)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        hist = fmt.new_hist()
        y = fmt.fmt_quantize(xd, (6, 9, True), hist=hist, stream=s)
    s.synchronize()
    assert_same_values(y.cpu().numpy(), oracle.quantize(x, 6, 9, True), "side stream")
    assert_same_hist(fmt, hist, oracle.histogram(x, 6, 9), "side stream")


def test_config5_full_size(fmt):
    """Configuration 5 at its full size (2^28 elements, the launch shape bench.py times): the
    integer statistics must equal the oracle's over the whole tensor, and the values are checked
    element by element on a 2^22-element sample made of 64 slices spread over the tensor
    (including its first and last elements)."""
    n = 1 << 28
    x = workloads.config5(n=n)
    xd = dev(x)
    y = torch.empty_like(xd)
    want_hist = oracle.histogram(x, 6, 9)                     # one pass of the oracle over 2^28 elements
    rng = np.random.default_rng(55)
    starts = np.concatenate([[0, n - (1 << 16)], rng.integers(0, n - (1 << 16), 62)])
    for (e, m, d) in [(6, 9, True), (6, 9, False)]:
        hist = fmt.new_hist()
        fmt.fmt_quantize(xd, (e, m, d), out=y, hist=hist)
        torch.cuda.synchronize()
        assert_same_hist(fmt, hist, want_hist, "config5 full 1/%d/%d" % (e, m))
        for s in starts:
            s = int(s)
            got = y[s:s + (1 << 16)].cpu().numpy()
            assert_same_values(got, oracle.quantize(x[s:s + (1 << 16)], e, m, d), "slice at %d" % s)
    # the other formats: statistics must satisfy the format-independent invariants at full size
    for (e, m) in [(5, 10), (8, 7)]:
        h = fmt.hist_to_dict(fmt.fmt_histogram(xd, (e, m, True)))
        assert h["total"] == n == sum(h[k] for k in fmt.CLASS_NAMES[1:])
        assert np.array_equal(h["bins"], want_hist["bins"])
        assert int(h["bins"].sum()) == n - h["zero"] - h["nan"]
        assert h["zero"] == want_hist["zero"] and h["nan"] == want_hist["nan"] and h["inf"] == want_hist["inf"]


def test_more_than_2_to_the_32_elements(fmt):
    """A tensor whose element indices do not fit 32 bits (2^32 + 12293 elements, 16 GiB): the tensor is
    a 2^24-element chunk repeated, so the statistics are 256 times the chunk's plus those of the ragged
    rest, and the values are checked on samples around every power-of-two index boundary and at the
    end.  Fused fp32 pass, statistics-only pass and the 16-bit code pass."""
    chunk_n = 1 << 24
    tail = 3 * 4096 + 5
    n = (1 << 32) + tail
    chunk = mixed(chunk_n, 1234)
    xd = dev(chunk).repeat(257)[:n]
    assert xd.numel() == n
    hc, ht = oracle.histogram(chunk, 6, 9), oracle.histogram(chunk[:tail], 6, 9)
    want = {k: 256 * hc[k] + ht[k] for k in fmt.CLASS_NAMES}
    want["bins"] = 256 * np.asarray(hc["bins"]) + np.asarray(ht["bins"])
    # sample positions: both ends, around 2^31 and 2^32, and random ones
    rng = np.random.default_rng(9)
    near = np.concatenate([np.arange(-2048, 2048) + b for b in (1 << 31, 1 << 32, (1 << 32) - (1 << 24))])
    idx = np.unique(np.concatenate([np.arange(4096), np.arange(n - 4096, n), near, rng.integers(0, n, 1 << 16)]))
    idx_d = torch.from_numpy(idx).cuda()
    src = chunk[idx % chunk_n]
    f = (6, 9, True)

    hist = fmt.new_hist()
    y = torch.empty_like(xd)
    fmt.fmt_quantize(xd, f, out=y, hist=hist)
    torch.cuda.synchronize()
    assert_same_hist(fmt, hist, want, "fused, n > 2^32")
    assert_same_values(y[idx_d].cpu().numpy(), oracle.quantize(src, *f), "sampled values, n > 2^32")
    del y

    assert_same_hist(fmt, fmt.fmt_histogram(xd, f), want, "statistics only, n > 2^32")

    hist = fmt.new_hist()
    c = fmt.fmt_pack16(xd, f, hist=hist)
    torch.cuda.synchronize()
    assert_same_hist(fmt, hist, want, "pack16, n > 2^32")
    got = c[idx_d].cpu().numpy().view(np.uint16)
    assert np.array_equal(got, oracle.pack16(src, *f)), "sampled codes, n > 2^32"
    back = fmt.fmt_unpack16(c, f)
    torch.cuda.synchronize()
    assert_same_values(back[idx_d].cpu().numpy(), oracle.quantize(src, *f), "unpacked values, n > 2^32")


@pytest.mark.parametrize("seed", range(40))
def test_seeded_random_cases(fmt, seed):
    """Format (any 2 <= e <= 8, 1 <= m <= 23, d or n), length, pointer offsets of input and output,
    histogram window and call (fused, values only, statistics only, 16-bit codes, in place) drawn from a
    seeded generator; everything bit for bit against the oracle, and nothing written outside the output."""
    rng = np.random.default_rng(5000 + seed)
    e, m, d = int(rng.integers(2, 9)), int(rng.integers(1, 24)), bool(rng.integers(0, 2))
    n = int(rng.choice([int(rng.integers(0, 64)), int(rng.integers(64, 20000)), int(rng.integers(20000, 400000))]))
    ox, oy = int(rng.integers(0, 4)), int(rng.integers(0, 4))
    exp_lo = int(rng.integers(-192, 129))
    x = mixed(n + 8, seed)[:n] if n else np.zeros(0, np.float32)
    xb = torch.zeros(n + 8, device="cuda")
    xb[ox:ox + n] = dev(x)
    xin = xb[ox:ox + n]
    want_h = oracle.histogram(x, e, m, exp_lo=exp_lo)
    want_y = oracle.quantize(x, e, m, d)
    what = "seed %d: 1/%d/%d/%s n=%d ox=%d oy=%d exp_lo=%d" % (seed, e, m, "d" if d else "n", n, ox, oy, exp_lo)
    kind = seed % 5
    if kind == 0:                                   # fused
        yb = torch.full((n + 8,), 7.0, device="cuda")
        hist = fmt.new_hist()
        fmt.fmt_quantize(xin, (e, m, d), out=yb[oy:oy + n], hist=hist, exp_lo=exp_lo)
        torch.cuda.synchronize()
        got = yb.cpu().numpy()
        assert_same_values(got[oy:oy + n], want_y, what)
        assert np.all(got[:oy] == 7.0) and np.all(got[oy + n:] == 7.0), what
        assert_same_hist(fmt, hist, want_h, what)
    elif kind == 1:                                 # values only
        yb = torch.full((n + 8,), 7.0, device="cuda")
        fmt.fmt_quantize(xin, (e, m, d), out=yb[oy:oy + n])
        torch.cuda.synchronize()
        got = yb.cpu().numpy()
        assert_same_values(got[oy:oy + n], want_y, what)
        assert np.all(got[:oy] == 7.0) and np.all(got[oy + n:] == 7.0), what
    elif kind == 2:                                 # statistics only
        hist = fmt.new_hist()
        fmt.fmt_histogram(xin, (e, m, d), hist=hist, exp_lo=exp_lo)
        torch.cuda.synchronize()
        assert_same_hist(fmt, hist, want_h, what)
        assert_same_values(xb.cpu().numpy()[ox:ox + n], x, what + ": input changed")
    elif kind == 3:                                 # in place, with statistics
        hist = fmt.new_hist()
        fmt.fmt_quantize(xin, (e, m, d), out=xin, hist=hist, exp_lo=exp_lo)
        torch.cuda.synchronize()
        assert_same_values(xb.cpu().numpy()[ox:ox + n], want_y, what)
        assert_same_hist(fmt, hist, want_h, what)
    else:                                           # 16-bit codes where the format has them
        if 1 + e + m > 16:
            e, m = 6, 9
            want_h = oracle.histogram(x, e, m, exp_lo=exp_lo)
        cb = torch.full((n + 8,), 0x5555, dtype=torch.int16, device="cuda")
        hist = fmt.new_hist()
        fmt.fmt_pack16(xin, (e, m, d), out=cb[oy:oy + n], hist=hist, exp_lo=exp_lo)
        torch.cuda.synchronize()
        got = cb.cpu().numpy().view(np.uint16)
        assert np.array_equal(got[oy:oy + n], oracle.pack16(x, e, m, d)), what
        assert np.all(got[:oy] == 0x5555) and np.all(got[oy + n:] == 0x5555), what
        assert_same_hist(fmt, hist, want_h, what)


def test_config2_every_tensor_of_a_step(fmt):
    """Config 2 call by call: one forward + backward step of the 784-1024-1024-10 MLP at batch 256 with
    loss scale 1024; fmt_quantize + statistics of EVERY tensor the step rounds -- the input, the three
    weight matrices, the three layer outputs, the loss-scaled gradient of the logits and the two
    back-propagated gradients (256 x 784 ... 256 x 10) -- against the oracle, bit for bit, in the three
    formats.  The step itself (products, ReLU, softmax) is harness glue in float64 on the host: parity is
    per call on identical inputs."""
    import oracle
    cfg = workloads.config2()
    X, W = cfg["X"], cfg["W"]
    tensors = [("X", X)] + [("W%d" % l, W[l]) for l in range(3)]
    acts = [X.astype(np.float64)]
    for l in range(3):
        z = acts[-1] @ W[l].astype(np.float64).T
        tensors.append(("Y%d" % l, z.astype(np.float32)))
        acts.append(np.maximum(z, 0) if l < 2 else z)
    z = acts[-1]
    p = np.exp(z - z.max(1, keepdims=True))
    p /= p.sum(1, keepdims=True)
    p[np.arange(z.shape[0]), cfg["labels"]] -= 1.0
    g = p / z.shape[0] * cfg["loss_scale"]
    tensors.append(("dY2", g.astype(np.float32)))
    for l in (2, 1):
        g = (g @ W[l].astype(np.float64)) * (acts[l] > 0)
        tensors.append(("dY%d" % (l - 1), g.astype(np.float32)))
    assert {t.shape for _, t in tensors} >= {(256, 784), (1024, 784), (256, 1024), (10, 1024), (256, 10)}
    for e, m, d in [(6, 9, True), (5, 10, True), (8, 7, False)]:
        for name, t in tensors:
            flat = np.ascontiguousarray(t).ravel()
            xd = torch.from_numpy(flat).cuda()
            hist = fmt.new_hist(xd.device)
            y = fmt.fmt_quantize(xd, (e, m, d), hist=hist)
            torch.cuda.synchronize()
            want = oracle.quantize(flat, e, m, d)
            assert np.array_equal(y.cpu().numpy().view(np.uint32), want.view(np.uint32)), (name, e, m, d)
            got, ho = fmt.hist_to_dict(hist), oracle.histogram(flat, e, m)
            assert all(got[k] == ho[k] for k in fmt.CLASS_NAMES), (name, e, m, d, got, ho)
            assert np.array_equal(got["bins"], ho["bins"]), (name, e, m, d)


@pytest.mark.parametrize("tiles,rest", [(0, 9), (1, 0), (2, 3), (64, 0), (64, 1), (65, 4095), (1024, 1), (4 * 1024 + 1, 17)])
@pytest.mark.parametrize("offset", [0, 1])
def test_statistics_in_one_launch(fmt, tiles, rest, offset):
    """The statistics are summed by the pass itself: one workgroup (up to a tile of 4096 elements), one record (64 workgroups),
    records summed by a second addition (more), several tiles per workgroup -- aligned and not, twice in a row with the
    sizes and kinds of pass mixed, so that whatever a launch leaves in the records shows in the next one."""
    n = 4096 * tiles + rest
    x = mixed(n + offset, 40 + tiles + offset)[offset:]
    buf = torch.empty(n + offset, device="cuda")
    buf[offset:] = dev(x)
    xd = buf[offset:]
    want = oracle.histogram(x, 6, 9)
    small = mixed(70001, 5)
    small_d, want_small = dev(small), oracle.histogram(small, 5, 10)
    for _ in range(2):
        hist = [fmt.new_hist().fill_(-1) for _ in range(4)]
        y = fmt.fmt_quantize(xd, (6, 9, True), hist=hist[0])
        fmt.fmt_histogram(xd, (6, 9, True), hist=hist[1])
        fmt.fmt_quantize(small_d, (5, 10, False), hist=hist[2])
        fmt.fmt_pack16(xd, (6, 9, True), hist=hist[3])
        torch.cuda.synchronize()
        assert_same_values(y.cpu().numpy(), oracle.quantize(x, 6, 9, True), "n = %d" % n)
        for i, w in ((0, want), (1, want), (2, want_small), (3, want)):
            assert_same_hist(fmt, hist[i], w, "n = %d, pass %d" % (n, i))


@pytest.mark.parametrize("n", [(1 << 26) - 1, 1 << 26, (1 << 27) - 4095, (1 << 27) + 4097])
def test_statistics_of_large_tensors(fmt, n):
    """Sizes around the lines where a pass takes more replicas of its table: the three passes agree with a count of the classes and of
    the binades by torch (exponents and thresholds of the patterns), and with one another."""
    f = (6, 9, True)
    x = torch.randn(n, device="cuda").mul_(12.0).exp2_()
    x[::1001] = 0.0
    x[5::100003] = float("inf")
    x[7::100003] = float("nan")
    hist = [fmt.new_hist().fill_(-1) for _ in range(3)]
    y = fmt.fmt_quantize(x, f, hist=hist[0])
    fmt.fmt_histogram(x, f, hist=hist[1])
    fmt.fmt_pack16(x, f, hist=hist[2])
    torch.cuda.synchronize()
    assert torch.equal(hist[0], hist[1]) and torch.equal(hist[0], hist[2])
    h = fmt.hist_to_dict(hist[0])
    minn = 2.0 ** -30
    inf, nan, zero = int(torch.isinf(x).sum()), int(torch.isnan(x).sum()), int((x == 0).sum())
    want = {"total": n, "zero": zero, "inf": inf, "nan": nan, "underflow": int((y == 0).sum()) - zero,
            "denormal": int(((y > 0) & (y < minn)).sum()), "overflow": int(torch.isinf(y).sum()) - inf,
            "normal": int(((y >= minn) & torch.isfinite(y)).sum())}
    assert {k: h[k] for k in want} == want
    e = ((x.view(torch.int32) >> 23) & 255)[(x != 0) & ~torch.isnan(x)]          # no fp32 denormals among them
    bins = torch.bincount((e.to(torch.int64) - 127 + 48).clamp_(0, 63), minlength=64)
    assert np.array_equal(h["bins"], bins.cpu().numpy())


def test_statistics_after_records_left_over(fmt):
    """Passes that overlap on one stream's scratch leave counts and arrivals in its partial records.  Here the test leaves them
    there itself (every word of the buffer: seven arrivals and a count), so that nothing races: the first pass of few
    workgroups and the first of many may be wrong, the next ones are right, whatever their sizes, and so are replays of a recorded pass."""
    import ctypes
    lib = fmt.raw_library()
    stream = torch.cuda.Stream()
    xs = [mixed(n, 3 + n) for n in (70001, 9000, 6 * 4096 * 1024 + 5, 4097, 300)]
    xd = [dev(x) for x in xs]
    want = [oracle.histogram(x, 6, 9) for x in xs]
    A, W = torch.randint(-3, 4, (300, 64), device="cuda").float(), torch.randint(-3, 4, (2100, 64), device="cuda").float()
    mats = [torch.randn(64 + 32 * i, 100, device="cuda") for i in range(3)]
    bufs = [[torch.empty(fmt.fmt_operand_bytes(*m.shape[::o], (6, 9, True)), dtype=torch.uint8, device="cuda") for m in mats]
            for o in (1, -1)]

    def passes():
        h = [fmt.new_hist().fill_(-1) for _ in range(2 * len(xs) + 1 + len(mats))]
        for i, x in enumerate(xd):
            fmt.fmt_quantize(x, (6, 9, True), hist=h[2 * i])
            fmt.fmt_histogram(x, (6, 9, True), hist=h[2 * i + 1])
        fmt.fmt_linear(A, W, None, (6, 9, True), hist=h[2 * len(xs)])
        fmt.fmt_quantize_prepare_pair_batch(mats, (6, 9, True), [torch.empty_like(m) for m in mats], h[2 * len(xs) + 1:],
                                            outs=bufs[0], outs_t=bufs[1])
        return h

    def leave():
        scratch = (ctypes.c_uint64 * 8)()            # the library's record of the stream's buffers: address, bytes, ...
        get = getattr(lib, "_ZN3fmt11get_scratchEP12ihipStream_tmmPNS_7ScratchE")
        assert get(ctypes.c_void_p(stream.cuda_stream), ctypes.c_size_t(0), ctypes.c_size_t(0), scratch) == 0
        left = np.full(scratch[1] // 8, (7 << 48) | 5, dtype=np.uint64)
        lib.hipDeviceSynchronize()
        assert lib.hipMemcpy(ctypes.c_void_p(scratch[0]), ctypes.c_void_p(left.ctypes.data), ctypes.c_size_t(left.nbytes), 1) == 0

    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        right = passes()
        graph = torch.cuda.CUDAGraph()
        rec = [fmt.new_hist() for _ in xs]
        y = [torch.empty_like(x) for x in xd]
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            for x, q, h in zip(xd, y, rec):
                fmt.fmt_quantize(x, (6, 9, True), out=q, hist=h)
        leave()
        for first in ((0, 2), (2, 1), (1, 2)):       # one pass of 18 or 3 workgroups, one of 1024
            for i in first:
                fmt.fmt_histogram(xd[i], (6, 9, True))
            after = passes()
            stream.synchronize()
            for a, r in zip(after, right):
                assert torch.equal(a, r)
            leave()
        for replay in range(3):
            for h in rec:
                h.fill_(-1)
            graph.replay()
            stream.synchronize()
            for i, h in enumerate(rec):
                if replay > 0:
                    assert_same_hist(fmt, h, want[i], "replay %d of n = %d" % (replay, xs[i].size))
    for i in range(len(xs)):
        assert_same_hist(fmt, right[2 * i], want[i], "n = %d" % xs[i].size)
