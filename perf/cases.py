"""The work that a training or serving program has this library do, as cases that can be timed and checked.

A case is a dict of plain values; ``kind`` names the calls that a pass makes:

  round      fmt_quantize with statistics: every tensor of a step is rounded and logged (Sec. IV-A, Sec. V)
  histogram  fmt_histogram: a tensor is logged and left as it is
  pack       fmt_pack16 with statistics, then fmt_unpack16: a tensor is put away as 16-bit codes and read back
  mlp        fmt_gemm: forward, input and weight gradients of a small multilayer perceptron, operands in fp32
  gemm       fmt_gemm: one product of any size and layout, operands in fp32
  linear     fmt_linear / fmt_linear_pack16: forward of a fully connected layer with bias (and statistics)
  serve      fmt_prepare + fmt_linear_prepared: forward with a weight operand that is kept prepared
  step       the rounding pass over X, W and dY of every layer, prepared operands, and the three products per layer
  conv       fmt_conv2d_fwd, _dgrad, _wgrad of one layer
  fmac8      fmt_gemm_fmac8: the product with the 16-bit accumulation of Algorithm 1

Inputs are drawn on the GPU with the distributions of the benchmark's configurations.
"""
from __future__ import annotations

import math

import torch

import paper_2103_15940_amd as fmt

FORMATS = ("1/5/10/d", "1/5/10/n", "1/6/9/d", "1/6/9/n", "1/8/7/d", "1/8/7/n")


def listed():
    return [
        # the last layer's weights and bias of the 784-1024-1024-10 perceptron, 1024 * 10 + 10 values: the smallest
        # tensors of a step, of which a model has many
        {"name": "round_small", "kind": "round", "n": 10250, "format": "1/6/9/d"},
        # one layer's activations or weights (2^20 values)
        {"name": "round_1m", "kind": "round", "n": 1 << 20, "format": "1/5/10/d"},
        # the largest tensor, a heavy-tailed gradient of 2^28 values
        {"name": "round_256m", "kind": "round", "n": 1 << 28, "format": "1/6/9/n"},
        # logging of a tensor of odd size, 3000 rows of 4097
        {"name": "histogram_12m", "kind": "histogram", "n": 3000 * 4097, "format": "1/6/9/d"},
        # an activation kept as 16-bit codes between forward and backward, odd size
        {"name": "pack_30m", "kind": "pack", "n": 30000001, "format": "1/8/7/n"},
        # the 784-1024-1024-10 perceptron at batch 256
        {"name": "mlp_256", "kind": "mlp", "batch": 256, "inputs": 784, "hidden": 1024, "outputs": 10, "format": "1/6/9/d"},
        # an odd product in binary16, weight-gradient layout
        {"name": "gemm_ragged", "kind": "gemm", "M": 1001, "N": 3003, "K": 1530, "transA": True, "transB": False,
         "format": "1/5/10/d"},
        # query, key and value projection of an encoder layer at 4096 tokens, with the statistics of the output
        {"name": "linear_qkv", "kind": "linear", "batch": 4096, "inputs": 1024, "outputs": 3072, "format": "1/6/9/d",
         "packed": False, "stats": True},
        # inference of a short batch through the first feed-forward matrix, bfloat16
        {"name": "serve_ffn1", "kind": "serve", "batch": 333, "inputs": 1024, "outputs": 4096, "format": "1/8/7/n"},
        # one training step's rounding passes and products of an encoder layer at 4096 tokens
        {"name": "step_encoder", "kind": "step", "tokens": 4096, "hidden": 1024, "inner": 4096, "format": "1/6/9/d"},
        # 3x3 convolution, 256 -> 256 channels at 14 x 14, batch 64, all three directions
        {"name": "conv_3x3", "kind": "conv", "batch": 64, "channels": 256, "size": 14, "filters": 256, "window": 3,
         "pad": 1, "stride": 1, "format": "1/6/9/d"},
        # Algorithm 1 on a mid-sized product
        {"name": "fmac8_2048", "kind": "fmac8", "M": 2048, "N": 2048, "K": 1024, "format": "1/6/9/d"},
    ]


def _size(rng, lo, hi, step=8):
    """A size from lo to hi, spread over its logarithm; half of them multiples of `step`."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        v = max(step, v // step * step)
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(("round", "round", "histogram", "pack", "mlp", "gemm", "linear", "serve", "step", "conv", "fmac8"))
    c = {"kind": kind, "format": rng.choice(FORMATS)}
    if kind == "round":
        c["n"] = _size(rng, 1000, 1 << 28, 1024)
    elif kind == "histogram":
        c["n"] = _size(rng, 1 << 16, 1 << 27, 1024)
    elif kind == "pack":
        c["n"] = _size(rng, 1 << 16, 1 << 27, 1024)
    elif kind == "mlp":
        c.update(batch=_size(rng, 32, 512), inputs=_size(rng, 100, 1024), hidden=_size(rng, 128, 1024),
                 outputs=_size(rng, 10, 100))
    elif kind == "gemm":
        c.update(M=_size(rng, 64, 4096), N=_size(rng, 64, 4096), K=_size(rng, 64, 4096), transA=rng.random() < 0.5,
                 transB=rng.random() < 0.5)
    elif kind == "linear":
        c.update(batch=_size(rng, 64, 4096), inputs=_size(rng, 128, 4096), outputs=_size(rng, 128, 4096),
                 packed=rng.random() < 0.5, stats=rng.random() < 0.5)
    elif kind == "serve":
        c.update(batch=_size(rng, 1, 1024), inputs=_size(rng, 256, 4096), outputs=_size(rng, 256, 4096))
    elif kind == "step":
        hidden = _size(rng, 128, 1024)
        c.update(tokens=_size(rng, 128, 4096), hidden=hidden, inner=hidden * rng.randint(2, 4))
    elif kind == "conv":
        window = rng.choice((1, 3, 3, 5))
        c.update(batch=_size(rng, 4, 64), channels=_size(rng, 16, 256, 32), filters=_size(rng, 16, 256, 32), window=window,
                 size=rng.randint(7, 14 if window > 3 else 28), pad=window // 2, stride=rng.choice((1, 1, 2)))
        while _conv_flops(c) > 15e9:        # a third of the listed layer's three products
            c["batch"] = max(4, c["batch"] // 2)
            c["filters"] = max(16, c["filters"] // 2)
    else:
        c.update(M=_size(rng, 64, 2048), N=_size(rng, 64, 2048), K=_size(rng, 64, 1024),
                 format=rng.choice(("1/5/10/d", "1/5/10/n", "1/6/9/d", "1/6/9/n")))
    return c


# ------------------------------------------------------------------------------------------------ helpers

def _format(case):
    _, e, m, d = case["format"].split("/")
    return int(e), int(m), d == "d"


def _layers(case):
    """(inputs, outputs) of an encoder layer's four matrices: query-key-value, attention output, feed-forward 1 and 2."""
    h, i = case["hidden"], case["inner"]
    return ((h, 3 * h), (h, h), (h, i), (i, h))


def _mlp_layers(case):
    return ((case["inputs"], case["hidden"]), (case["hidden"], case["hidden"]), (case["hidden"], case["outputs"]))


def _conv_out(case):
    return (case["size"] + 2 * case["pad"] - case["window"]) // case["stride"] + 1


def _conv_flops(case):
    """One of the three products."""
    return 2.0 * case["batch"] * _conv_out(case) ** 2 * case["filters"] * case["channels"] * case["window"] ** 2


class _Draw:
    """Seeded numbers on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, *shape, scale=1.0):
        return torch.randn(shape, generator=self.g, device="cuda") * scale

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, device="cuda")

    def gradient(self, *shape, mean=-24.0, sigma=6.0):
        """Activation gradients: log2|x| normal, random sign."""
        x = torch.randn(shape, generator=self.g, device="cuda").mul_(sigma).add_(mean).exp2_()
        return x.mul_(torch.randint(0, 2, shape, generator=self.g, device="cuda", dtype=torch.int8).mul_(2).sub_(1))

    def heavy(self, n):
        """log2|x| = -18 + 8 T with T of Student's t(3), 2 % zeros: the heavy-tailed gradient tensor."""
        out = torch.empty(n, device="cuda")
        for a in range(0, n, 1 << 26):
            k = min(1 << 26, n - a)
            s = torch.zeros(k, device="cuda")
            for _ in range(3):
                s += torch.randn(k, generator=self.g, device="cuda").square_()
            t = torch.randn(k, generator=self.g, device="cuda").div_(s.div_(3.0).sqrt_())
            x = t.mul_(8.0).sub_(18.0).exp2_()
            u = torch.rand(k, generator=self.g, device="cuda")
            x[u < 0.02] = 0.0
            out[a:a + k] = torch.where(u < 0.51, x, -x)
        return out

    def values(self, n):
        """Activations and small tensors: log2|x| ~ N(-14, 6^2), 1 % zeros."""
        x = self.gradient(n, mean=-14.0, sigma=6.0)
        x[torch.rand(n, generator=self.g, device="cuda") < 0.01] = 0.0
        return x


# ------------------------------------------------------------------------------------------------ the cases

def _inputs(case, seed):
    """The fp32 tensors of a case."""
    d, kind = _Draw(seed), case["kind"]
    if kind in ("round", "histogram", "pack"):
        return {"x": d.heavy(case["n"]) if case["n"] > 1 << 22 else d.values(case["n"])}
    if kind == "mlp":
        layers = []
        for i, o in _mlp_layers(case):
            layers.append({"X": d.uniform(case["batch"], i), "W": d.normal(o, i, scale=math.sqrt(2.0 / i)),
                           "dY": d.gradient(case["batch"], o, mean=-12.0, sigma=4.0)})
        return {"layers": layers}
    if kind in ("gemm", "fmac8"):
        M, N, K = case["M"], case["N"], case["K"]
        tA, tB = case.get("transA", False), case.get("transB", False)
        A = d.normal(*((K, M) if tA else (M, K)))
        return {"A": A, "B": d.normal(*((N, K) if tB else (K, N)), scale=0.05)}
    if kind in ("linear", "serve"):
        return {"X": d.normal(case["batch"], case["inputs"]), "W": d.normal(case["outputs"], case["inputs"], scale=0.02),
                "b": d.normal(case["outputs"], scale=0.02)}
    if kind == "step":
        return {"layers": [{"X": d.normal(case["tokens"], i), "W": d.normal(o, i, scale=0.02), "dY": d.gradient(case["tokens"], o)}
                           for i, o in _layers(case)]}
    c, k, r, p = case["channels"], case["filters"], case["window"], _conv_out(case)
    return {"X": d.normal(case["batch"], c, case["size"], case["size"]).relu_(),
            "W": d.normal(k, c, r, r, scale=math.sqrt(2.0 / (c * r * r))),
            "dY": d.gradient(case["batch"], k, p, p, mean=-20.0, sigma=5.0)}


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, f = case["kind"], _format(case)
    s.update(kind=kind, f=f)
    if kind in ("round", "histogram", "pack"):
        s["hist"] = fmt.new_hist()
    if kind == "round":
        s["y"] = torch.empty_like(s["x"])
    elif kind == "pack":
        s["codes"], s["y"] = torch.empty(s["x"].shape, dtype=torch.int16, device="cuda"), torch.empty_like(s["x"])
    elif kind in ("gemm", "fmac8"):
        s.update(tA=case.get("transA", False), tB=case.get("transB", False))
        s["C"] = torch.empty((case["M"], case["N"]), device="cuda")
    elif kind == "linear":
        s.update(packed=case["packed"], hist=fmt.new_hist() if case["stats"] else None)
        s["Y"] = torch.empty((case["batch"], case["outputs"]), dtype=torch.int16 if case["packed"] else torch.float32, device="cuda")
    elif kind == "serve":
        s["Wp"] = fmt.fmt_prepare(s["W"], f)
        s["Xbuf"] = torch.empty(fmt.fmt_operand_bytes(case["batch"], case["inputs"], f), dtype=torch.uint8, device="cuda")
        s["Y"] = torch.empty((case["batch"], case["outputs"]), device="cuda")
    elif kind == "step":
        # a step's buffers: rounded copies, statistics, both orientations of every operand, results
        s["src"] = [L[t] for L in s["layers"] for t in ("X", "W", "dY")]
        s["rounded"] = [torch.empty_like(t) for t in s["src"]]
        s["hists"] = [fmt.new_hist() for _ in s["src"]]
        empty = lambda r, c: torch.empty(fmt.fmt_operand_bytes(r, c, f), dtype=torch.uint8, device="cuda")  # noqa: E731
        s["ops"] = [empty(*t.shape) for t in s["src"]]
        s["ops_t"] = [empty(t.shape[1], t.shape[0]) for t in s["src"]]
        s["out"] = []
        for L in s["layers"]:
            s["out"] += [torch.empty_like(L["dY"]), torch.empty_like(L["X"]), torch.empty_like(L["W"])]
    elif kind == "conv":
        s.update(pad=case["pad"], stride=case["stride"], Y=torch.empty_like(s["dY"]), dX=torch.empty_like(s["X"]),
                 dW=torch.empty_like(s["W"]))
    return s


def run(s):
    kind, f = s["kind"], s["f"]
    if kind == "round":
        return {"y": fmt.fmt_quantize(s["x"], f, out=s["y"], hist=s["hist"]), "hist": s["hist"]}
    if kind == "histogram":
        return {"hist": fmt.fmt_histogram(s["x"], f, hist=s["hist"])}
    if kind == "pack":
        fmt.fmt_pack16(s["x"], f, out=s["codes"], hist=s["hist"])
        fmt.fmt_unpack16(s["codes"], f, out=s["y"])
        return {"codes": s["codes"], "hist": s["hist"], "y": s["y"]}
    if kind == "mlp":
        out = []
        for i, L in enumerate(s["layers"]):
            o = {"Y": fmt.fmt_gemm(L["X"], L["W"], f, transB=True)}
            if i:                                            # the network's input needs no gradient
                o["dX"] = fmt.fmt_gemm(L["dY"], L["W"], f)
            o["dW"] = fmt.fmt_gemm(L["dY"], L["X"], f, transA=True)
            out.append(o)
        return out
    if kind == "gemm":
        return fmt.fmt_gemm(s["A"], s["B"], f, transA=s["tA"], transB=s["tB"], out=s["C"])
    if kind == "fmac8":
        return fmt.fmt_gemm_fmac8(s["A"], s["B"], f, out=s["C"])
    if kind == "linear":
        call = fmt.fmt_linear_pack16 if s["packed"] else fmt.fmt_linear
        out = {"Y": call(s["X"], s["W"], s["b"], f, out=s["Y"], hist=s["hist"])}
        if s["hist"] is not None:
            out["counts"] = s["hist"].to(torch.float64)      # as they are logged
        return out
    if kind == "serve":
        return fmt.fmt_linear_prepared(fmt.fmt_prepare(s["X"], f, out=s["Xbuf"]), s["Wp"], s["b"], out=s["Y"])
    if kind == "step":
        if f[0] == 6:
            pairs = fmt.fmt_quantize_prepare_pair_batch(s["src"], f, s["rounded"], s["hists"], outs=s["ops"], outs_t=s["ops_t"])
        else:
            for x, y, h in zip(s["src"], s["rounded"], s["hists"]):
                fmt.fmt_quantize(x, f, out=y, hist=h)
            pairs = fmt.fmt_prepare_pair_batch(s["src"], f, outs=s["ops"], outs_t=s["ops_t"])
        A, B = [], []
        for i in range(0, len(pairs), 3):
            X, W, dY = pairs[i:i + 3]
            A += [X[0], dY[0], dY[1]]                        # Y = X W^T, dX = dY W, dW = dY^T X
            B += [W[0], W[1], X[1]]
        return {"products": fmt.fmt_gemm_prepared_batch(A, B, out=s["out"]), "rounded": s["rounded"], "hists": s["hists"]}
    g = {"pad": s["pad"], "stride": s["stride"]}
    return {"Y": fmt.fmt_conv2d_fwd(s["X"], s["W"], f, out=s["Y"], **g),
            "dX": fmt.fmt_conv2d_dgrad(s["dY"], s["W"], s["X"].shape, f, out=s["dX"], **g),
            "dW": fmt.fmt_conv2d_wgrad(s["dY"], s["X"], s["W"].shape, f, out=s["dW"], **g)}


def work(case):
    kind = case["kind"]
    if kind in ("round", "histogram", "pack"):
        per = {"round": 8, "histogram": 4, "pack": 12}[kind]    # pack: 4 read + 2 written, 2 read + 4 written
        return {"bytes": per * case["n"] + 576, "flops": 0}
    if kind in ("gemm", "fmac8"):
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 4 * (M * K + K * N + M * N), "flops": 2.0 * M * N * K}
    if kind in ("linear", "serve"):
        M, N, K = case["batch"], case["outputs"], case["inputs"]
        return {"bytes": 4 * (M * K + N) + (2 if kind == "serve" else 4) * N * K + (2 if case.get("packed") else 4) * M * N,
                "flops": 2.0 * M * N * K}
    if kind == "mlp":
        b, flops = 0, 0.0
        for n, (i, o) in enumerate(_mlp_layers(case)):
            x, w, y = case["batch"] * i, i * o, case["batch"] * o
            b += 4 * (x + 2 * y + 2 * w + (x if n else 0))
            flops += (6.0 if n else 4.0) * case["batch"] * i * o
        return {"bytes": b, "flops": flops}
    if kind == "step":
        b, flops = 0, 0.0
        for i, o in _layers(case):
            x, w, y = case["tokens"] * i, i * o, case["tokens"] * o
            b += 12 * (x + w + y)                               # read, rounded copy and result
            flops += 6.0 * case["tokens"] * i * o
        return {"bytes": b, "flops": flops}
    x = case["batch"] * case["channels"] * case["size"] ** 2
    w = case["filters"] * case["channels"] * case["window"] ** 2
    y = case["batch"] * case["filters"] * _conv_out(case) ** 2
    return {"bytes": 4 * 3 * (x + w + y), "flops": 3 * _conv_flops(case)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("round", "histogram", "pack", "fmac8"):
        return "exact"                  # one rounding per value, counts, and an order of roundings that the algorithm fixes
    if kind in ("linear", "serve"):
        # the output is rounded to the format: a sum that falls on the other side of a midpoint moves by a unit
        return {"rel": 2e-4, "max": 2e-2, "differ": 5e-3}
    return {"rel": 2e-6, "max": 3e-5}   # exact products, sums in fp32


# ------------------------------------------------------------------------------------------------ in 64 bits

def _q(x, f, chunk=1 << 25):
    """Q(x) by its definition, in 64 bits: to the nearest multiple of the format's step at x, ties to even."""
    e, m, den = f
    emax = (1 << (e - 1)) - 1
    emin = 1 - emax
    flat = x.reshape(-1)
    out = torch.empty(flat.shape, dtype=torch.float64, device=x.device)
    for a in range(0, flat.numel(), chunk):
        v = flat[a:a + chunk].to(torch.float64)
        _, ex = torch.frexp(v)
        step = (((ex - 1).clamp_(min=emin) - m + 1023).to(torch.int64) << 52).view(torch.float64)   # 2^(E - m), exactly
        r = torch.round(v / step) * step
        r = torch.where(r.abs() >= 2.0 ** (emax + 1), torch.copysign(torch.full_like(r, math.inf), v), r)
        if not den:
            r = torch.where(r.abs() < 2.0 ** emin, torch.copysign(torch.zeros_like(r), v), r)
        out[a:a + chunk] = torch.where(torch.isfinite(v), r, v)
    return out.reshape(x.shape)


def _fmac8(A, B, f):
    """Algorithm 1 with every fused step in 64 bits and one rounding to the format."""
    a = torch.zeros(A.shape[0], B.shape[1], dtype=torch.float64, device=A.device)
    total = torch.zeros(a.shape, dtype=torch.float32, device=A.device)
    for k in range(A.shape[1]):
        if k % 8 == 0:
            total += a.to(torch.float32)
            a.zero_()
        a = _q(torch.addcmul(a, A[:, k:k + 1], B[k:k + 1, :]), f)
    return _q(total + a.to(torch.float32), f)


def exact(case, seed):
    s, kind, f = _inputs(case, seed), case["kind"], _format(case)
    if kind == "round":
        return {"y": _q(s["x"], f), "hist": None}
    if kind == "histogram":
        return None
    if kind == "pack":
        return {"codes": None, "hist": None, "y": _q(s["x"], f)}
    if kind == "mlp":
        out = []
        for i, L in enumerate(s["layers"]):
            X, W, dY = (_q(L[t], f) for t in ("X", "W", "dY"))
            o = {"Y": X @ W.t(), "dW": dY.t() @ X}
            if i:
                o["dX"] = dY @ W
            out.append(o)
        return out
    if kind in ("gemm", "fmac8"):
        A, B = _q(s["A"], f), _q(s["B"], f)
        if kind == "fmac8":
            return _fmac8(A, B, f)
        return (A.t() if case["transA"] else A) @ (B.t() if case["transB"] else B)
    if kind in ("linear", "serve"):
        if case.get("packed"):
            return None                                                      # codes
        acc = _q(s["X"], f) @ _q(s["W"], f).t()
        Y = _q(_q(acc, f) + _q(s["b"], f), f)
        return Y if kind == "serve" else {"Y": Y, "counts": None}
    if kind == "step":
        products, rounded = [], []
        for L in s["layers"]:
            X, W, dY = (_q(L[t], f) for t in ("X", "W", "dY"))
            products += [X @ W.t(), dY @ W, dY.t() @ X]
            rounded += [X, W, dY]
        return {"products": products, "rounded": rounded, "hists": None}
    X, W, dY = (_q(s[t], f) for t in ("X", "W", "dY"))
    n, k, r = case["batch"], case["filters"], case["window"]
    g = {"kernel_size": r, "padding": case["pad"], "stride": case["stride"]}
    cols = torch.nn.functional.unfold(X, **g)                                # [n, c r r, p p]
    cols = cols.transpose(0, 1).reshape(cols.shape[1], -1)
    dY2 = dY.reshape(n, k, -1).transpose(0, 1).reshape(k, -1)
    W2 = W.reshape(k, -1)
    Y = (W2 @ cols).reshape(k, n, -1).transpose(0, 1).reshape(dY.shape)
    dcols = (W2.t() @ dY2).reshape(W2.shape[1], n, -1).transpose(0, 1)
    dX = torch.nn.functional.fold(dcols, X.shape[2:], **g)
    return {"Y": Y, "dX": dX, "dW": (dY2 @ cols.t()).reshape(W.shape)}
