"""GPU parity of fmt_conv2d_fwd / _dgrad / _wgrad (convolutions of Sec. IV-A on rounded operands,
patches gathered on the fly) against the CPU oracle's plain definitions: bit for bit where every
partial sum is exact in fp32, within the GEMM tolerance (1e-5 relative Frobenius) otherwise."""
import numpy as np
import pytest

import oracle
import workloads
from graph_kernels import kernels_of

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 1e-5
VARIANTS = [(5, 10, True), (5, 10, False), (6, 9, True), (6, 9, False), (8, 7, True), (8, 7, False)]
GEOMS = [  # N, C, H, W, K, R, S, pad, stride
    (2, 3, 7, 6, 4, 3, 3, (1, 1), (1, 1)),
    (1, 2, 9, 8, 3, 3, 3, (1, 1), (2, 2)),
    (2, 4, 6, 6, 5, 1, 1, (0, 0), (1, 1)),
    (1, 3, 8, 9, 2, 5, 3, (2, 1), (1, 2)),
    (3, 2, 5, 5, 3, 2, 2, (0, 0), (1, 1)),
    (1, 1, 10, 7, 2, 3, 3, (0, 2), (3, 1)),
    (2, 40, 14, 14, 70, 3, 3, (1, 1), (1, 1)),       # several tiles and k-blocks, ragged everywhere
    (3, 33, 15, 13, 65, 3, 3, (1, 1), (2, 2)),
    # channel counts that are multiples of 32: forward and (stride 1) dgrad gather inside the product kernel
    (2, 32, 9, 8, 64, 3, 3, (1, 1), (1, 1)),
    (1, 64, 7, 7, 32, 3, 3, (1, 1), (2, 2)),          # forward in-kernel, dgrad through the gathered operand
    (2, 96, 6, 5, 32, 1, 1, (0, 0), (1, 1)),
    (1, 32, 8, 9, 96, 5, 3, (2, 1), (1, 1)),
    (3, 64, 5, 11, 160, 2, 4, (0, 3), (1, 1)),        # even taps, pad wider than the filter reaches on one side
    (5, 32, 12, 12, 40, 3, 3, (2, 2), (1, 2)),        # only forward qualifies (40 filters)
]


@pytest.fixture(scope="module")
def fmt():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2103_15940_amd as lib
    return lib


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def rel_err(got, ref):
    return float(np.linalg.norm(got.astype(np.float64) - ref.astype(np.float64)) /
                 max(np.linalg.norm(ref.astype(np.float64)), 1e-300))


def run_all(fmt, X, W, dY, f, pad, stride):
    Y = fmt.fmt_conv2d_fwd(dev(X), dev(W), f, pad=pad, stride=stride)
    dX = fmt.fmt_conv2d_dgrad(dev(dY), dev(W), X.shape, f, pad=pad, stride=stride)
    dW = fmt.fmt_conv2d_wgrad(dev(dY), dev(X), W.shape, f, pad=pad, stride=stride)
    torch.cuda.synchronize()
    return Y.cpu().numpy(), dX.cpu().numpy(), dW.cpu().numpy()


def oracle_all(X, W, dY, f, pad, stride):
    e, m, d = f
    return (oracle.conv2d_fwd(X, W, e, m, d, pad, stride), oracle.conv2d_dgrad(dY, W, X.shape, e, m, d, pad, stride),
            oracle.conv2d_wgrad(dY, X, W.shape, e, m, d, pad, stride))


@pytest.mark.parametrize("parts", [2, 3, 9])
def test_parts_of_k_into_images(fmt, parts, monkeypatch):
    """Forward and dgrad with k in parts: the sums go to NCHW, whose images (35 positions) end inside groups of four elements."""
    monkeypatch.setenv("FMT_GEMM_PLAN", "1,1,%d" % parts)
    rng = np.random.default_rng(parts)
    X = rng.integers(-4, 5, (2, 96, 7, 5)).astype(np.float32)
    W = rng.integers(-4, 5, (32, 96, 3, 3)).astype(np.float32)
    dY = rng.integers(-4, 5, (2, 32, 7, 5)).astype(np.float32)
    f, pad, stride = (6, 9, True), (1, 1), (1, 1)
    Y, dX = fmt.fmt_conv2d_fwd(dev(X), dev(W), f, pad=pad, stride=stride), fmt.fmt_conv2d_dgrad(dev(dY), dev(W), X.shape, f, pad=pad, stride=stride)
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy(), oracle.conv2d_fwd(X, W, 6, 9, True, pad, stride))
    assert np.array_equal(dX.cpu().numpy(), oracle.conv2d_dgrad(dY, W, X.shape, 6, 9, True, pad, stride))


@pytest.mark.parametrize("geom", GEOMS)
@pytest.mark.parametrize("f", [(6, 9, True), (5, 10, False), (8, 7, True)])
def test_bit_exact_integer_data(fmt, geom, f):
    """Small integers times powers of two: every partial sum is exact in fp32 in any order."""
    n, c, h, w, k, r, s, pad, stride = geom
    rng = np.random.default_rng(n + 10 * c + 100 * h)
    X = (rng.integers(-4, 5, (n, c, h, w)) * 0.5).astype(np.float32)
    W = (rng.integers(-4, 5, (k, c, r, s)) * 0.25).astype(np.float32)
    P, Q = oracle.conv_out_size(h, w, r, s, pad, stride)
    dY = (rng.integers(-4, 5, (n, k, P, Q)) * 2.0 ** -6).astype(np.float32)
    got = run_all(fmt, X, W, dY, f, pad, stride)
    want = oracle_all(X, W, dY, f, pad, stride)
    for name, g_, w_ in zip(("Y", "dX", "dW"), got, want):
        assert g_.shape == w_.shape
        assert np.array_equal(g_.view(np.uint32), w_.view(np.uint32)), "%s differs for %r" % (name, geom)


@pytest.mark.parametrize("geom", GEOMS)
@pytest.mark.parametrize("f", VARIANTS)
def test_real_data_within_tolerance(fmt, geom, f):
    n, c, h, w, k, r, s, pad, stride = geom
    rng = np.random.default_rng(7 * n + c + f[0])
    X = np.maximum(rng.standard_normal((n, c, h, w)), 0).astype(np.float32)         # ReLU activations
    W = (rng.standard_normal((k, c, r, s)) * np.sqrt(2.0 / (c * r * s))).astype(np.float32)
    P, Q = oracle.conv_out_size(h, w, r, s, pad, stride)
    dY = workloads.log2_normal((n, k, P, Q), -12.0, 3.0, 0.0, rng)
    got = run_all(fmt, X, W, dY, f, pad, stride)
    want = oracle_all(X, W, dY, f, pad, stride)
    for name, g_, w_ in zip(("Y", "dX", "dW"), got, want):
        assert rel_err(g_, w_) <= TOL, "%s: %.3g for %r" % (name, rel_err(g_, w_), geom)


def test_operands_are_rounded(fmt):
    """The convolution of unrounded operands differs; the convolution of pre-rounded operands agrees."""
    rng = np.random.default_rng(8)
    X = rng.standard_normal((2, 8, 10, 10)).astype(np.float32)
    W = rng.standard_normal((6, 8, 3, 3)).astype(np.float32)
    f = (5, 10, True)
    Y = fmt.fmt_conv2d_fwd(dev(X), dev(W), f).cpu().numpy()
    Yq = fmt.fmt_conv2d_fwd(dev(oracle.quantize(X, *f)), dev(oracle.quantize(W, *f)), f).cpu().numpy()
    Y32 = torch.nn.functional.conv2d(torch.from_numpy(X).double(), torch.from_numpy(W).double(), padding=1).numpy()
    assert np.array_equal(Y, Yq)
    assert rel_err(Y, Y32) > 1e-4


def test_empty_and_degenerate(fmt):
    f = (6, 9, True)
    cuda = torch.device("cuda")
    # no images / no filters: empty outputs
    Y = fmt.fmt_conv2d_fwd(torch.empty((0, 3, 5, 5), device=cuda), torch.empty((4, 3, 3, 3), device=cuda), f)
    assert tuple(Y.shape) == (0, 4, 5, 5)
    Y = fmt.fmt_conv2d_fwd(torch.empty((2, 3, 5, 5), device=cuda), torch.empty((0, 3, 3, 3), device=cuda), f)
    assert tuple(Y.shape) == (2, 0, 5, 5)
    # no input channels: an empty sum, zeros
    Y = fmt.fmt_conv2d_fwd(torch.empty((2, 0, 5, 5), device=cuda), torch.empty((4, 0, 3, 3), device=cuda), f,
                           out=torch.full((2, 4, 5, 5), 7.0, device=cuda))
    torch.cuda.synchronize()
    assert float(Y.abs().sum()) == 0.0
    # wgrad over an empty batch: zeros
    dW = fmt.fmt_conv2d_wgrad(torch.empty((0, 4, 5, 5), device=cuda), torch.empty((0, 3, 5, 5), device=cuda), (4, 3, 3, 3), f,
                              out=torch.full((4, 3, 3, 3), 7.0, device=cuda))
    torch.cuda.synchronize()
    assert float(dW.abs().sum()) == 0.0
    # a filter as large as the padded image: one output position
    rng = np.random.default_rng(0)
    X = rng.integers(-3, 4, (1, 2, 3, 3)).astype(np.float32)
    W = rng.integers(-3, 4, (2, 2, 5, 5)).astype(np.float32)
    Y = fmt.fmt_conv2d_fwd(dev(X), dev(W), f, pad=1).cpu().numpy()
    assert Y.shape == (1, 2, 1, 1)
    assert np.array_equal(Y, oracle.conv2d_fwd(X, W, 6, 9, True, (1, 1), (1, 1)))


@pytest.mark.parametrize("f", [(6, 9, True), (5, 10, True), (8, 7, False)])
def test_config3_full_size_sampled(fmt, f):
    """ResNet-style 3x3 convolution of config 3 (batch 64, 256 -> 256 channels, 14 x 14), forward,
    dgrad and wgrad at full size: sampled outputs against the oracle -- one in every 64 x 64 block of
    the underlying product (rows: filters or channels; columns: positions or taps), the smallest tile
    the product kernel has, so that no tile and no k part can be skipped, plus 2000 random ones --
    error measured against the norm of the sampled reference values."""
    cfg = workloads.config3()
    X, W2, dY2 = cfg["X"], cfg["W"], cfg["dY"]
    n, c, h, w = X.shape
    k = W2.shape[0]
    W = W2.reshape(k, c, 3, 3)
    dY = np.ascontiguousarray(dY2.reshape(n, h, w, k).transpose(0, 3, 1, 2))        # the same values as NCHW
    Y, dX, dW = run_all(fmt, X, W, dY, f, (1, 1), (1, 1))
    e, m, d = f
    rng = np.random.default_rng(33)
    def blocks(rows, cols, to_flat):
        bi, bj = np.meshgrid(np.arange(0, rows, 64), np.arange(0, cols, 64), indexing="ij")
        r = np.minimum(bi + rng.integers(0, 64, bi.shape), rows - 1).ravel()
        q = np.minimum(bj + rng.integers(0, 64, bj.shape), cols - 1).ravel()
        return to_flat(r, q)
    hw = h * w
    nchw = lambda chans: (lambda r, q: ((q // hw) * chans + r) * hw + q % hw)       # row = channel, column = (image, position)
    for name, got, ref_fn, pinned in (
            ("Y", Y, lambda s: oracle.conv2d_fwd(X, W, e, m, d, sample=s), blocks(k, n * hw, nchw(k))),
            ("dX", dX, lambda s: oracle.conv2d_dgrad(dY, W, X.shape, e, m, d, sample=s), blocks(c, n * hw, nchw(c))),
            ("dW", dW, lambda s: oracle.conv2d_wgrad(dY, X, W.shape, e, m, d, sample=s), blocks(k, c * 9, lambda r, q: r * c * 9 + q))):
        idx = np.concatenate([pinned, rng.integers(0, got.size, 2000)])
        ref = ref_fn(idx)
        assert np.all(np.isfinite(got))
        assert rel_err(got.ravel()[idx], ref) <= TOL, "%s: %.3g" % (name, rel_err(got.ravel()[idx], ref))


def test_equals_im2col_product_config3_shape(fmt):
    """Forward (patches gathered inside the product kernel, k running tap-major) against fmt_gemm on the
    materialised patch matrix (k running channel-major): the same rounded operands and exact products,
    summed in fp32 in two different orders of the K = 576 terms.  Each order is within about
    sqrt(K) * 2^-24 = 1.4e-6 of the exact sum relative to the Frobenius norm, typically a tenth of that."""
    rng = np.random.default_rng(12)
    X = np.maximum(rng.standard_normal((4, 64, 14, 14)), 0).astype(np.float32)
    W = (rng.standard_normal((96, 64, 3, 3)) * 0.05).astype(np.float32)
    f = (6, 9, True)
    Y = fmt.fmt_conv2d_fwd(dev(X), dev(W), f).cpu().numpy()
    Xcol = workloads.im2col_3x3(X)
    Y2 = fmt.fmt_gemm(dev(Xcol), dev(W.reshape(96, -1)), f, transB=True).cpu().numpy()    # [n*h*w, k]
    Y2 = Y2.reshape(4, 14, 14, 96).transpose(0, 3, 1, 2)
    assert rel_err(Y, Y2) <= 1e-6


@pytest.mark.parametrize("seed", range(36))
def test_seeded_random_geometries(fmt, seed):
    """Batch, channels, image and filter size (filters up to 7 x 6: more than 32 taps included), padding
    (also wider than the filter), stride and format drawn from a seeded generator; exact data, so
    forward, dgrad and wgrad must match the oracle bit for bit."""
    rng = np.random.default_rng(9000 + seed)
    n, c, k = int(rng.integers(1, 4)), int(rng.integers(1, 41)), int(rng.integers(1, 41))
    h, w = int(rng.integers(1, 18)), int(rng.integers(1, 18))
    pad = (int(rng.integers(0, 4)), int(rng.integers(0, 4)))
    r = int(rng.integers(1, min(7, h + 2 * pad[0]) + 1))
    s = int(rng.integers(1, min(6, w + 2 * pad[1]) + 1))
    stride = (int(rng.integers(1, 4)), int(rng.integers(1, 4)))
    f = [(6, 9, True), (5, 10, False), (8, 7, True), (6, 9, False), (7, 12, True), (4, 3, True)][seed % 6]
    X = (rng.integers(-3, 4, (n, c, h, w)) * 0.5).astype(np.float32)
    W = (rng.integers(-3, 4, (k, c, r, s)) * 0.25).astype(np.float32)
    P, Q = oracle.conv_out_size(h, w, r, s, pad, stride)
    dY = (rng.integers(-3, 4, (n, k, P, Q)) * 2.0 ** -3).astype(np.float32)
    got = run_all(fmt, X, W, dY, f, pad, stride)
    want = oracle_all(X, W, dY, f, pad, stride)
    what = "seed %d: n=%d c=%d k=%d %dx%d filter %dx%d pad %r stride %r 1/%d/%d" % (seed, n, c, k, h, w, r, s, pad, stride, f[0], f[1])
    for name, g_, w_ in zip(("Y", "dX", "dW"), got, want):
        assert g_.shape == w_.shape, what
        assert np.all(np.isfinite(w_)), what
        assert np.array_equal(g_.view(np.uint32), w_.view(np.uint32)), "%s differs, %s" % (name, what)


@pytest.mark.parametrize("seed", range(30))
def test_seeded_random_geometries_with_channel_multiples_of_32(fmt, seed):
    """The same draw with channel and filter counts from {32, 64, 96, 128} and at most 32 taps, so that forward
    (any stride) and dgrad (stride 1, every third seed at least) gather their patches inside the product kernel:
    images of several sizes incl. one pixel, padding wider than the filter, strides, six formats (one, two and
    three 16-bit pieces); exact data, bit for bit against the oracle."""
    rng = np.random.default_rng(9500 + seed)
    n = int(rng.integers(1, 4))
    c, k = int(rng.choice([32, 64, 96, 128])), int(rng.choice([32, 64, 96, 128]))
    h, w = int(rng.integers(1, 16)), int(rng.integers(1, 16))
    pad = (int(rng.integers(0, 4)), int(rng.integers(0, 4)))
    r = int(rng.integers(1, min(5, h + 2 * pad[0]) + 1))
    s = int(rng.integers(1, min(6, w + 2 * pad[1]) + 1))
    stride = (1, 1) if seed % 3 == 0 else (int(rng.integers(1, 4)), int(rng.integers(1, 4)))
    f = [(6, 9, True), (5, 10, False), (8, 7, True), (6, 9, False), (7, 20, True), (4, 3, True)][seed % 6]
    X = (rng.integers(-3, 4, (n, c, h, w)) * 0.5).astype(np.float32)
    W = (rng.integers(-3, 4, (k, c, r, s)) * 0.25).astype(np.float32)
    P, Q = oracle.conv_out_size(h, w, r, s, pad, stride)
    dY = (rng.integers(-3, 4, (n, k, P, Q)) * 2.0 ** -3).astype(np.float32)
    got = run_all(fmt, X, W, dY, f, pad, stride)
    want = oracle_all(X, W, dY, f, pad, stride)
    what = "seed %d: n=%d c=%d k=%d %dx%d filter %dx%d pad %r stride %r 1/%d/%d" % (seed, n, c, k, h, w, r, s, pad, stride, f[0], f[1])
    for name, g_, w_ in zip(("Y", "dX", "dW"), got, want):
        assert g_.shape == w_.shape, what
        assert np.all(np.isfinite(w_)), what
        assert np.array_equal(g_.view(np.uint32), w_.view(np.uint32)), "%s differs, %s" % (name, what)


def test_in_kernel_gather_equals_gathered_operand(fmt, monkeypatch):
    """Forward and dgrad with the patches gathered inside the product kernel give, on data whose partial sums
    are exact, the same bits as the route through a gathered operand (FMT_CONV_IMPLICIT=0), and within the
    tolerance on real data; both routes are held to the oracle by the tests above."""
    n, c, h, w, k, r, s, pad, stride = 2, 64, 10, 9, 96, 3, 3, (1, 1), (1, 1)
    rng = np.random.default_rng(11)
    f = (6, 9, True)
    for exact in (True, False):
        if exact:
            X = (rng.integers(-4, 5, (n, c, h, w)) * 0.5).astype(np.float32)
            W = (rng.integers(-4, 5, (k, c, r, s)) * 0.25).astype(np.float32)
            dY = (rng.integers(-4, 5, (n, k, h, w)) * 2.0 ** -6).astype(np.float32)
        else:
            X = rng.standard_normal((n, c, h, w)).astype(np.float32)
            W = (rng.standard_normal((k, c, r, s)) * 0.05).astype(np.float32)
            dY = (rng.standard_normal((n, k, h, w)) * 1e-3).astype(np.float32)
        monkeypatch.delenv("FMT_CONV_IMPLICIT", raising=False)
        a = run_all(fmt, X, W, dY, f, pad, stride)
        monkeypatch.setenv("FMT_CONV_IMPLICIT", "0")
        b = run_all(fmt, X, W, dY, f, pad, stride)
        monkeypatch.delenv("FMT_CONV_IMPLICIT", raising=False)
        for name, g_, w_ in zip(("Y", "dX", "dW"), a, b):
            if exact:
                assert np.array_equal(g_.view(np.uint32), w_.view(np.uint32)), name
            else:
                assert rel_err(g_, w_) <= TOL, name


def test_scratch_of_forward_and_dgrad_is_of_the_size_of_the_tensor(fmt):
    """With the patches gathered inside the product kernel, forward and dgrad hold the rounded tensor (two
    bytes per element and 16-bit piece: 4 B for 1/6/9), the prepared filter and, when k is split, partial sums
    in scratch -- nothing of the size of the patch matrix (R*S times the tensor).  wgrad still prepares a
    patch-sized operand, which the last assertion records."""
    n, c, h, w, k, r, s = 8, 64, 28, 28, 64, 3, 3
    rng = np.random.default_rng(5)
    X = dev(rng.standard_normal((n, c, h, w)).astype(np.float32))
    W = dev((rng.standard_normal((k, c, r, s)) * 0.05).astype(np.float32))
    dY = dev((rng.standard_normal((n, k, h, w)) * 1e-3).astype(np.float32))
    f = (6, 9, True)
    tensor = n * c * h * w
    patch_operand = tensor * r * s * 4                      # what a gathered operand of two 16-bit pieces takes
    filt = 256 * c * r * s * 4                              # the filter operand, rows padded to 256
    slabs = 8 * k * n * h * w * 4                           # generous room for split-k partial sums
    torch.cuda.synchronize()
    fmt.fmt_release_scratch()
    fmt.fmt_conv2d_fwd(X, W, f, pad=(1, 1))
    torch.cuda.synchronize()
    fwd = fmt.fmt_scratch_bytes()["products"]
    assert 4 * tensor <= fwd <= 4 * tensor + filt + slabs + 65536
    assert fwd < patch_operand / 2
    fmt.fmt_release_scratch()
    fmt.fmt_conv2d_dgrad(dY, W, (n, c, h, w), f, pad=(1, 1))
    torch.cuda.synchronize()
    dgrad = fmt.fmt_scratch_bytes()["products"]
    assert 4 * tensor <= dgrad <= 4 * tensor + filt + slabs + 65536
    assert dgrad < patch_operand / 2
    fmt.fmt_release_scratch()
    fmt.fmt_conv2d_wgrad(dY, X, (k, c, r, s), f, pad=(1, 1))
    torch.cuda.synchronize()
    assert fmt.fmt_scratch_bytes()["products"] >= patch_operand
    fmt.fmt_release_scratch()


def test_config3_full_size_every_element(fmt):
    """Config 3 at full size, 1/6/9/d: every element of forward, dgrad and wgrad against the oracle's full
    convolutions (3 x 14.8 GFLOP on the host's cores), within the 1e-5 relative Frobenius bound."""
    f = (6, 9, True)
    cfg = workloads.config3()
    X, W2, dY2 = cfg["X"], cfg["W"], cfg["dY"]
    n, c, h, w = X.shape
    k = W2.shape[0]
    W = W2.reshape(k, c, 3, 3)
    dY = np.ascontiguousarray(dY2.reshape(n, h, w, k).transpose(0, 3, 1, 2))
    Y, dX, dW = run_all(fmt, X, W, dY, f, (1, 1), (1, 1))
    e, m, d = f
    for name, got, ref in (("Y", Y, oracle.conv2d_fwd(X, W, e, m, d)),
                           ("dX", dX, oracle.conv2d_dgrad(dY, W, X.shape, e, m, d)),
                           ("dW", dW, oracle.conv2d_wgrad(dY, X, W.shape, e, m, d))):
        assert got.shape == ref.shape and np.all(np.isfinite(got)), name
        assert rel_err(got, ref) <= TOL, "%s: %.3g" % (name, rel_err(got, ref))


def in_64_bits(X, W, dY, pad, stride):
    """The three products in 64 bits, of values and of magnitudes: (Y, dX, dW), (|Y|, |dX|, |dW|)."""
    def three(x, w, dy):
        x, w = torch.from_numpy(x).double().requires_grad_(), torch.from_numpy(w).double().requires_grad_()
        y = torch.nn.functional.conv2d(x, w, padding=pad, stride=stride)
        y.backward(torch.from_numpy(dy).double())
        return y.detach().numpy(), x.grad.numpy(), w.grad.numpy()
    return three(X, W, dY), three(np.abs(X), np.abs(W), np.abs(dY))


@pytest.mark.parametrize("plan", [None, "1,1,1", "2,2,2", "4,2,1", "2,4,1", "4,4,1"])
@pytest.mark.parametrize("spread", ["images", "elements", "single", "gradient"])
def test_elements_outside_plane_0(fmt, spread, plan, monkeypatch):
    """1/6/8 and 1/6/9 on exponent planes with one scale per tensor: operands of which much lies in a second plane, images and channels of their
    own magnitudes (where whole outputs live outside plane 0), and a few elements outside plane 0 (operands with elements both above and
    below: test_all_pairs_of_planes_meet).  |sum in fp32 - sum in 64 bits| <= (K + 2) 2^-24 sum|a b| for products that are exact, in any order."""
    if plan is not None:
        monkeypatch.setenv("FMT_GEMM_PLAN", plan)
    monkeypatch.setenv("FMT_GEMM_WINDOW", "1")           # by size these take two bf16 pieces
    rng = np.random.default_rng(len(spread))
    for e, m, d, (n, c, h, w, k, r, s, pad, stride) in (
            (6, 9, True, (5, 64, 9, 8, 96, 3, 3, (1, 1), (1, 1))), (6, 9, False, (3, 32, 13, 11, 40, 2, 4, (0, 3), (1, 2))),
            (6, 8, True, (2, 96, 17, 5, 32, 5, 3, (2, 1), (1, 1))), (6, 9, True, (4, 33, 8, 7, 65, 3, 3, (1, 1), (2, 2)))):
        P, Q = oracle.conv_out_size(h, w, r, s, pad, stride)
        X, W, dY = (rng.standard_normal(shape) for shape in ((n, c, h, w), (k, c, r, s), (n, k, P, Q)))
        if spread == "images":          # 2^-36 .. 2^26
            X *= 2.0 ** (rng.integers(-30, 21, (n, 1, 1, 1)) + rng.integers(-6, 6, (1, c, 1, 1)))
            W *= 2.0 ** rng.integers(-20, 11, (k, c, 1, 1))
            dY *= 2.0 ** (rng.integers(-30, 21, (n, 1, 1, 1)) + rng.integers(-6, 6, (1, k, 1, 1)))
        elif spread == "elements":
            X, W, dY = (t * 2.0 ** np.clip(rng.normal(-4, 12, t.shape), -36, 26) for t in (X, W, dY))
        elif spread == "single":
            for t in (X, W, dY):
                flat = t.reshape(-1)
                at = np.concatenate([[0, flat.size - 1], rng.integers(0, flat.size, 6)])
                flat[at] = np.where(rng.random(at.size) < 0.5, 2.0 ** 24, 2.0 ** -33) * 1.5
        else:
            dY = workloads.log2_normal(dY.shape, -20.0, 5.0, 0.0, rng)
            dY.reshape(-1)[rng.integers(0, dY.size, 5)] = 6.0
        X, W, dY = (oracle.quantize(np.ascontiguousarray(t.astype(np.float32)), e, m, d) for t in (X, W, dY))
        got = run_all(fmt, X, W, dY, (e, m, d), pad, stride)
        want, size = in_64_bits(X, W, dY, pad, stride)
        for name, g_, w_, z_, K in zip(("Y", "dX", "dW"), got, want, size, (c * r * s, k * r * s, n * P * Q)):
            bad = np.abs(g_ - w_) > (K + 2) * 2.0 ** -24 * z_ + 2.0 ** -149
            assert not bad.any(), "%s 1/%d/%d: %d of %d" % (name, e, m, bad.sum(), bad.size)


def sampled(n, runs=64):
    """The elements that a tensor's scale is chosen from: 32 or 64 runs of 32, an odd number of runs apart."""
    if n < 32 * runs + 32:
        return np.arange(min(n, 32 * runs))
    step = (((n - 32) // (runs - 1) // 32 - 1) | 1) * 32
    return (np.arange(runs)[:, None] * step + np.arange(32)).ravel()


def planes_of(x, m):
    """The plane of every element of a tensor in 1/6/m: 0, 1 above, 2 below (zeros: 0)."""
    emin, wid = -30, 39 - m
    flat = x.ravel()
    a = np.abs(flat[sampled(flat.size)].astype(np.float64))
    E = np.frexp(a[a > 0])[1] - 1
    hi, lo = int(E.max()), int(max(E.min(), emin - 1))
    top, room = hi + 1, lo + wid
    T = 9 - m if lo < emin else room if top >= room else top + min(4, (room - top) // 2)
    sc = x.astype(np.float64) * 2.0 ** (15 - min(max(T, 0), 31))
    above = np.abs(sc) >= 65536.0
    return np.where(above, 1, np.where(np.where(above, 0, sc).astype(np.float16) != sc, 2, 0) * ~above)


def place(x, at, value):
    """x[at] = value, or in the first element after it that the scale does not look at."""
    i, seen = int(np.ravel_multi_index(at, x.shape)), set(sampled(x.size).tolist()) | set(sampled(x.size, 32).tolist())
    while i % x.size in seen:
        i += 1
    x.ravel()[i % x.size] = value


def check_three(fmt, X, W, dY, f, pad, stride):
    """|sum in fp32 - sum in 64 bits| <= (K + 2) 2^-24 sum|a b| for products that are exact, in any order; nothing overflows."""
    for t in (X, W, dY):
        assert np.array_equal(t, oracle.quantize(t, *f))
    got = run_all(fmt, X, W, dY, f, pad, stride)
    want, size = in_64_bits(X, W, dY, pad, stride)
    n, _, P, Q = dY.shape
    k, c, r, s = W.shape
    for name, g_, w_, z_, K in zip(("Y", "dX", "dW"), got, want, size, (c * r * s, k * r * s, n * P * Q)):
        assert np.isfinite(g_).all(), "%s 1/%d/%d: %d not finite" % (name, f[0], f[1], (~np.isfinite(g_)).sum())
        bad = np.abs(g_ - w_) > (K + 2) * 2.0 ** -24 * z_ + 2.0 ** -149
        assert not bad.any(), "%s 1/%d/%d: %d of %d" % (name, f[0], f[1], bad.sum(), bad.size)


def normal_clipped(rng, shape, f):
    """N(0, 1) of which nothing is below 2^-8: a scale in the middle of its range, with planes above and below."""
    x = rng.standard_normal(shape)
    return oracle.quantize(np.ascontiguousarray((np.sign(x) * np.maximum(np.abs(x), 2.0 ** -8)).astype(np.float32)), *f)


@pytest.mark.parametrize("m", [8, 9])
@pytest.mark.parametrize("plan", [None, "1,1,1", "2,2,1", "4,2,1", "2,4,1", "4,4,1", "1,1,3", "2,2,2"])
def test_all_pairs_of_planes_meet(fmt, m, plan, monkeypatch):
    """Elements above and below plane 0 in both operands of all three products, large ones that meet large ones in the outputs of
    waves where small ones meet small ones: the sums reach 2^(2 (26 + S)) in plane 0's units, and the pair of the planes below has a
    scale of 2^62 (2^64 with m = 8) in them."""
    if plan is not None:
        monkeypatch.setenv("FMT_GEMM_PLAN", plan)
    monkeypatch.setenv("FMT_GEMM_WINDOW", "1")
    f, rng = (6, m, True), np.random.default_rng(m)
    for n, c, h, w, k, pad in ((4, 64, 12, 10, 96, (1, 1)), (3, 96, 14, 14, 64, (1, 1))):
        X, W, dY = (normal_clipped(rng, shape, f) for shape in ((n, c, h, w), (k, c, 3, 3), (n, k, h, w)))
        big, small = 2.0 ** 26, 1.5 * 2.0 ** -33
        # the large ones meet in Y[., 5], dX[., 3] and dW[5, 3], the small ones in the channels beside them
        for t, at in ((X, (0, 3, 4, 4)), (X, (1, 3, 0, 1)), (X, (n - 1, c - 1, h - 1, w - 2)), (W, (5, 3, 1, 1)), (W, (5, 7, 0, 2)), (W, (k - 1, c - 1, 2, 1)),
                      (dY, (0, 5, 4, 4)), (dY, (1, 5, 0, 2)), (dY, (n - 1, k - 1, h - 1, w - 2))):
            place(t, at, big)
        for t, at in ((X, (0, 4, 4, 6)), (X, (1, 9, 2, 2)), (X, (n - 1, c - 2, h - 2, 1)), (W, (6, 4, 1, 1)), (W, (9, 3, 0, 0)), (W, (k - 2, c - 2, 1, 2)),
                      (dY, (0, 6, 4, 6)), (dY, (1, 9, 3, 2)), (dY, (n - 1, k - 2, 1, 1))):
            place(t, at, small)
        for t in (X, W, dY):
            assert np.array_equal(np.bincount(planes_of(t, m).ravel(), minlength=3)[1:], [3, 3])
        check_three(fmt, X, W, dY, f, pad, (1, 1))


@pytest.mark.parametrize("plan", ["1,1,1", "2,2,1", "4,4,1", "2,2,2", "1,1,3"])
def test_elements_outside_plane_0_in_long_sums(fmt, plan, monkeypatch):
    """Sums of more than 128 blocks of 32 k, whose masks are looked at in several steps of 64 blocks (in one part, and in parts that are
    no multiple of 64 blocks long), with elements above and below plane 0 in the first, the last, and the blocks on both sides of a step."""
    monkeypatch.setenv("FMT_GEMM_PLAN", plan)
    monkeypatch.setenv("FMT_GEMM_WINDOW", "1")
    f, rng = (6, 9, True), np.random.default_rng(7)
    big, small = 2.0 ** 26, 1.5 * 2.0 ** -33
    blocks = (0, 63, 64, 127, 128, 143)
    # 512 channels, 3 x 3 taps: block b is tap b / 16, channels 32 (b % 16) on, for the forward product of X and the input gradient of dY
    n, c, h, w, k = 1, 512, 6, 5, 40
    for which in ("fwd", "dgrad"):
        T, O = normal_clipped(rng, (n, c, h, w), f), normal_clipped(rng, (n, k, h, w), f)
        F = normal_clipped(rng, (k, c, 3, 3) if which == "fwd" else (c, k, 3, 3), f)
        for i, b in enumerate(blocks):
            ch, tap = 32 * (b % 16), (b // 16 // 3, b // 16 % 3)
            for j, v in enumerate((big, small)):
                place(T, (0, ch + 5 + 9 * j, i % h, (i + j) % w), v)
                place(F, ((3 + i + 17 * j, ch + 5 + 9 * j) if which == "fwd" else (ch + 5 + 9 * j, 3 + i + 17 * j)) + tap, v)
        for t in (T, F):
            assert (np.bincount(planes_of(t, 9).ravel(), minlength=3)[1:] >= 4).all()
        check_three(fmt, *((T, F, O) if which == "fwd" else (O, F, T)), f, (1, 1), (1, 1))
    # 3 images of 40 x 40: block b of the weight gradient is positions 32 b on
    n, c, h, w, k = 3, 24, 40, 40, 40
    X, W, dY = normal_clipped(rng, (n, c, h, w), f), normal_clipped(rng, (k, c, 3, 3), f), normal_clipped(rng, (n, k, h, w), f)
    for i, b in enumerate(blocks + (149,)):
        for j, v in enumerate((big, small)):
            image, at = divmod(32 * b + 3 + 8 * j, h * w)
            place(dY, (image, 3 + i + 20 * j, at // w, at % w), v)
            place(X, (image, 2 + i + 11 * j, at // w, at % w), v)
    for t in (X, dY):
        assert (np.bincount(planes_of(t, 9).ravel(), minlength=3)[1:] >= 4).all()
    check_three(fmt, X, W, dY, f, (1, 1), (1, 1))


def spread_over(rng, shape, mean, sigma, f):
    """log2|x| ~ N(mean, sigma^2), random signs."""
    x = np.where(rng.random(shape) < 0.5, -1.0, 1.0) * 2.0 ** np.clip(rng.normal(mean, sigma, shape), -60, 30)
    return oracle.quantize(np.ascontiguousarray(x.astype(np.float32)), *f)


WIDE = {"high": (-10.0, 7.0), "low": (-5.0, 6.0), "all": (-6.0, 12.0), "top": (28.0, 2.0)}
# with denormals; without; most of the format; not wide, at the format's top


@pytest.mark.parametrize("plan", ["1,1,1", "2,2,1", "4,2,1", "2,4,1", "4,4,1", "1,1,3", "2,2,2"])
@pytest.mark.parametrize("f", [(6, 9, True), (6, 9, False), (6, 8, True)])
def test_tensors_wider_than_a_plane(fmt, f, plan, monkeypatch):
    """Tensors that span more than a plane take two bf16 pieces: the bits of these where either operand is such a tensor, the
    bits of planes where none is."""
    monkeypatch.setenv("FMT_GEMM_PLAN", plan)
    rng = np.random.default_rng(len(plan))
    n, c, h, w, k = 3, 64, 14, 14, 96
    for wide in ("none", "high", "low", "all", "top"):
        for which in ((), ) if wide == "none" else ((0,), (1,), (2,), (0, 1, 2)):
            X, W, dY = (spread_over(rng, shape, *(WIDE[wide] if i in which else (-3.0, 1.5)), f)
                        for i, shape in enumerate(((n, c, h, w), (k, c, 3, 3), (n, k, h, w))))
            got = {}
            for mode in "013":
                monkeypatch.setenv("FMT_GEMM_WINDOW", mode)
                got[mode] = run_all(fmt, X, W, dY, f, (1, 1), (1, 1))
            for i, operands in enumerate(((0, 1), (1, 2), (0, 2))):
                pieces = wide != "top" and bool(set(operands) & set(which))
                assert not np.array_equal(got["0"][i], got["1"][i]), "the test cannot tell"
                assert np.array_equal(got["3"][i], got["0" if pieces else "1"][i]), (wide, which, i)


def test_wide_tensors_by_default(fmt, monkeypatch):
    """The same at sizes that take planes by default."""
    f, rng = (6, 9, True), np.random.default_rng(3)
    n, c, h, w, k = 64, 96, 14, 14, 96
    monkeypatch.setenv("FMT_GEMM_PLAN", "2,2,1")
    X, W = spread_over(rng, (n, c, h, w), -3.0, 1.5, f), spread_over(rng, (k, c, 3, 3), -3.0, 1.5, f)
    for wide in (False, True):
        dY = spread_over(rng, (n, k, h, w), *(WIDE["high"] if wide else (-3.0, 1.5)), f)
        monkeypatch.delenv("FMT_GEMM_WINDOW", raising=False)
        got = run_all(fmt, X, W, dY, f, (1, 1), (1, 1))
        for mode in "01":
            monkeypatch.setenv("FMT_GEMM_WINDOW", mode)
            other = run_all(fmt, X, W, dY, f, (1, 1), (1, 1))
            for i in range(3):
                assert np.array_equal(got[i], other[i]) == ((mode == "0") == (wide and i > 0)), (wide, mode, i)


@pytest.mark.parametrize("shape", [(1, 32, 4, 4, 32, 1), (2, 32, 6, 6, 33, 1), (1, 64, 33, 1, 32, 1), (1, 32, 35, 2, 33, 3), (2, 64, 16, 16, 64, 3)])
def test_samples_of_tensors_that_start_inside_a_line(fmt, shape, monkeypatch):
    """Tensors at any address, of fewer elements than a sample takes, about as many (1024 + 32, 2048 + 32) and more: the samples lie inside
    the tensor, whose neighbours would change the answer, and the bits are those of a tensor that starts at a line, also where a few of the
    samples' elements alone decide (the first of every run)."""
    monkeypatch.setenv("FMT_GEMM_WINDOW", "3")
    n, c, h, w, k, r = shape
    f, rng = (6, 9, True), np.random.default_rng(sum(shape))
    g = {"pad": (r // 2, r // 2), "stride": (1, 1)}

    def at(x, offset):
        buf = torch.full((x.size + 64,), 2.0 ** 30, device="cuda")
        buf[1::2] = 2.0 ** -39
        buf[offset: offset + x.size] = dev(x).flatten()
        return buf[offset: offset + x.size].view(x.shape)
    for values in ("narrow", "wide", "wide in the sample"):
        X, dY = (spread_over(rng, s, *((-6.0, 12.0) if values == "wide" else (-3.0, 1.5)), f) for s in ((n, c, h, w), (n, k, h, w)))
        if values == "wide in the sample":
            for t in (X, dY):
                for runs in (32, 64):
                    firsts = sampled(t.size, runs)[::32]
                    t.ravel()[firsts] = np.where(np.arange(firsts.size) % 2, 2.0 ** 24, 1.5 * 2.0 ** -34)
        W = spread_over(rng, (k, c, r, r), -3.0, 1.5, f)
        got = []
        for offset in (0, 1, 17, 31):
            x, y, v = at(X, offset), at(dY, offset), at(W, offset)
            got.append((fmt.fmt_conv2d_fwd(x, v, f, **g), fmt.fmt_conv2d_dgrad(y, v, x.shape, f, **g), fmt.fmt_conv2d_wgrad(y, x, v.shape, f, **g)))
        torch.cuda.synchronize()
        for other in got[1:]:
            assert all(torch.equal(a, b) for a, b in zip(got[0], other))


@pytest.mark.parametrize("shape", [(36, 288, 27, 480, 1), (73, 64, 41, 160, 3), (13, 96, 50, 512, 1), (8, 64, 14, 96, 3)])
def test_products_of_planes_stay_in_registers(fmt, shape, monkeypatch):
    """Large products, for which 256 x 256 results per workgroup would be the fastest without the code for the elements outside plane 0, and a
    small one: none of the kernels keeps sums or fragments in private memory."""
    monkeypatch.setenv("FMT_GEMM_WINDOW", "1")
    n, c, h, k, r = shape
    X, W = torch.randn(n, c, h, h, device="cuda"), torch.randn(k, c, r, r, device="cuda")
    f, g = (6, 9, True), {"pad": (r // 2, r // 2), "stride": (1, 1)}
    Y = torch.empty(n, k, h, h, device="cuda")
    dX, dW = torch.empty_like(X), torch.empty_like(W)
    for call in (lambda: fmt.fmt_conv2d_fwd(X, W, f, out=Y, **g), lambda: fmt.fmt_conv2d_dgrad(Y, W, X.shape, f, out=dX, **g),
                 lambda: fmt.fmt_conv2d_dgrad(X, W.transpose(0, 1).contiguous(), Y.shape, f, out=Y, **g), lambda: fmt.fmt_conv2d_wgrad(Y, X, W.shape, f, out=dW, **g)):
        kernels = kernels_of(call)
        assert any("window" in name for name, _, _ in kernels) and all(local == 0 for _, local, _ in kernels), kernels


def test_small_input_gradients_take_pieces(fmt, monkeypatch):
    """At 2.6e8 products the forward product takes planes and the input gradient, whose gradients have elements outside plane 0, pieces."""
    f, rng = (6, 9, True), np.random.default_rng(4)
    monkeypatch.setenv("FMT_GEMM_PLAN", "2,2,1")
    X, W = spread_over(rng, (16, 96, 14, 14), -3.0, 1.5, f), spread_over(rng, (96, 96, 3, 3), -3.0, 1.5, f)
    dY = spread_over(rng, (16, 96, 14, 14), -20.0, 5.0, f)
    monkeypatch.delenv("FMT_GEMM_WINDOW", raising=False)
    got = run_all(fmt, X, W, dY, f, (1, 1), (1, 1))
    for mode in "01":
        monkeypatch.setenv("FMT_GEMM_WINDOW", mode)
        other = run_all(fmt, X, W, dY, f, (1, 1), (1, 1))
        assert [np.array_equal(a, b) for a, b in zip(got, other)] == [mode == "1", mode == "0", mode == "0"]


def test_infinities_on_exponent_planes(fmt, monkeypatch):
    """An infinite element makes the outputs that meet it non-finite and leaves the others as they are, also where other elements
    lie outside plane 0."""
    monkeypatch.setenv("FMT_GEMM_WINDOW", "1")
    n, c, h, w, k = 2, 32, 9, 8, 40
    rng = np.random.default_rng(2)
    X = rng.integers(-4, 5, (n, c, h, w)).astype(np.float32)
    W = (rng.integers(1, 5, (k, c, 3, 3)) * 0.25).astype(np.float32)
    X[1, 3, 0, 0] = 2.0 ** -37
    clean = fmt.fmt_conv2d_fwd(dev(X), dev(W), (6, 9, True)).cpu().numpy()
    X[0, 5, 4, 4] = np.inf
    Y = fmt.fmt_conv2d_fwd(dev(X), dev(W), (6, 9, True)).cpu().numpy()
    met = np.zeros(Y.shape, bool)
    met[0, :, 3:6, 3:6] = True
    assert not np.isfinite(Y[met]).any()
    assert np.array_equal(Y[~met].view(np.uint32), clean[~met].view(np.uint32))


@pytest.mark.parametrize("seed", [s for s in range(36) if s % 6 in (0, 3)])
def test_seeded_random_geometries_on_exponent_planes(fmt, seed, monkeypatch):
    """The drawn geometries in 1/6/9, which by size take two bf16 pieces, on exponent planes."""
    monkeypatch.setenv("FMT_GEMM_WINDOW", "1")
    test_seeded_random_geometries(fmt, seed)
    if seed < 30:
        test_seeded_random_geometries_with_channel_multiples_of_32(fmt, seed)


def test_exponent_planes_under_capture(fmt, monkeypatch):
    """The three calls recorded into a graph on exponent planes: every replay, on inputs that change in between (with and without elements
    outside plane 0, and so wide that they take two bf16 pieces), gives the bits of the eager calls."""
    monkeypatch.setenv("FMT_GEMM_WINDOW", "3")
    f, g = (6, 9, True), {"pad": (1, 1), "stride": (1, 1)}
    gen = torch.Generator(device="cuda").manual_seed(1)
    draw = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731
    X, W, dY = draw(16, 96, 14, 14), draw(96, 96, 3, 3) * 0.05, draw(16, 96, 14, 14) * 1e-3
    Y, dX, dW = torch.empty_like(dY), torch.empty_like(X), torch.empty_like(W)

    def three(y, dx, dw):
        fmt.fmt_conv2d_fwd(X, W, f, out=y, **g)
        fmt.fmt_conv2d_dgrad(dY, W, X.shape, f, out=dx, **g)
        fmt.fmt_conv2d_wgrad(dY, X, W.shape, f, out=dw, **g)

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        three(Y, dX, dW)                                 # scratch of the stream
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            three(Y, dX, dW)
    torch.cuda.synchronize()
    for turn in range(5):
        if turn == 4:
            turn = 2
            W *= torch.exp2(6.0 * draw(*W.shape))
        X.copy_(draw(*X.shape) * 2.0 ** (8 * turn))
        dY.copy_(draw(*dY.shape) * 2.0 ** (-12 * turn))
        if turn % 2:
            X[3, 5, 0, :] = 2.0 ** -36
            dY[1, 7, 3, 3] = 2.0 ** 25
        eager = [torch.empty_like(t) for t in (Y, dX, dW)]
        three(*eager)
        torch.cuda.synchronize()
        for t in (Y, dX, dW):
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        for a, b in zip((Y, dX, dW), eager):
            assert torch.equal(a, b)


def test_capture_in_the_scratch_of_two_pieces(fmt, monkeypatch):
    """Exponent planes take half as much scratch again as two bf16 pieces.  A stream that is being captured, whose scratch cannot grow,
    records the calls on the pieces if there is room for these only: every replay gives their bits."""
    f, g = (6, 9, True), {"pad": (1, 1), "stride": (1, 1)}
    X, W, dY = torch.randn(8, 64, 14, 14, device="cuda"), torch.randn(64, 64, 3, 3, device="cuda") * 0.05, torch.randn(8, 64, 14, 14, device="cuda")
    Y, dX, dW = torch.empty_like(dY), torch.empty_like(X), torch.empty_like(W)
    calls = ((lambda o: fmt.fmt_conv2d_fwd(X, W, f, out=o, **g), Y), (lambda o: fmt.fmt_conv2d_dgrad(dY, W, X.shape, f, out=o, **g), dX),
             (lambda o: fmt.fmt_conv2d_wgrad(dY, X, W.shape, f, out=o, **g), dW))
    for call, out in calls:
        fmt.fmt_release_scratch()
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            monkeypatch.setenv("FMT_GEMM_WINDOW", "0")
            call(out)
            stream.synchronize()
            want, had = out.clone(), fmt.fmt_scratch_bytes()["products"]
            monkeypatch.setenv("FMT_GEMM_WINDOW", "1")
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                call(out)
            assert fmt.fmt_scratch_bytes()["products"] == had
            for _ in range(3):
                out.fill_(float("nan"))
                stream.synchronize()
                graph.replay()
                stream.synchronize()
                assert torch.equal(out, want)
            call(out)                                    # not captured: the scratch grows
            stream.synchronize()
            assert fmt.fmt_scratch_bytes()["products"] > had
    fmt.fmt_release_scratch()
