"""Performance cases of the approximate-multiplier library: calls that its users make, through the
binding and the autograd layers, with the inputs such a program holds.

A case is one call (a GEMM, the passes of a convolution or dense layer, a LeNet-5 training step) with
its sizes and its multiplier: the table's design (`table`) and mantissa bits (`m`), or the native
multiply, or a (1, e, m) format.  Three designs stand for the tables users bring: Mitchell's
logarithmic multiplier, the exact product of truncated operands (bfloat16 at M = 7), and a
logarithmic multiplier with a per-segment error compensation, which depends on both operands and
stands for a design of a user's own.
"""
import functools
import math

import numpy as np
import torch

from paper_2209_04161_amd import binding, modules

# LeNet-5 on 28 x 28 images: convolutions (c_in, c_out, kernel, pad) and dense layers (in, out).
_LENET_CONV = ((1, 6, 5, 2), (6, 16, 5, 0))
_LENET_FC = ((400, 120), (120, 84), (84, 10))


def listed():
    return [
        # a small dense product, the latency of one call
        dict(name="gemm_64", kind="gemm", m_=64, n=64, k=64, ta=False, tb=False, dist="uniform", table="mitchell", m=7),
        # a large dense product, the benchmark's GEMM
        dict(name="gemm_4096", kind="gemm", m_=4096, n=4096, k=4096, ta=False, tb=False, dist="normal",
             table="mitchell", m=7),
        # the same at the paper's 12-bit significand (M = 11, a 16 MiB table)
        dict(name="gemm_4096_m11", kind="gemm", m_=4096, n=4096, k=4096, ta=False, tb=False, dist="normal",
             table="mitchell", m=11),
        # ragged sizes, a transposed operand and a table of the user's own design
        dict(name="gemm_ragged", kind="gemm", m_=1000, n=777, k=1111, ta=False, tb=True, dist="normal",
             table="compensated", m=7),
        # half-precision arithmetic: the exact product in a (1, 5, 10) format
        dict(name="gemm_1024_e5", kind="gemm", m_=1024, n=1024, k=1024, ta=False, tb=False, dist="normal",
             table="exact_trunc", m=10, e_bits=5),
        # training step of a ResNet 3x3 layer at batch 128, activations after a ReLU
        dict(name="resnet_3x3", kind="conv", n=128, h=32, w=32, ci=64, co=64, kk=3, stride=1, pad=1, x="relu",
             table="mitchell", m=7),
        # training step of the ResNet-50 stem (images: three channels, stride 2)
        dict(name="r50_stem", kind="conv", n=32, h=224, w=224, ci=3, co=64, kk=7, stride=2, pad=3, x="image",
             table="mitchell", m=7),
        # training step of a deep ResNet-50 3x3 layer with a table of the user's own design
        dict(name="r50_3x3", kind="conv", n=32, h=14, w=14, ci=256, co=256, kk=3, stride=1, pad=1, x="relu",
             table="compensated", m=7),
        # training step of a ResNet-50 pointwise layer in bfloat16 arithmetic
        dict(name="r50_1x1", kind="conv", n=32, h=14, w=14, ci=1024, co=256, kk=1, stride=1, pad=0, x="relu",
             table="exact_trunc", m=7),
        # the same layer family with the native multiply in the library's kernels, the paper's baseline
        dict(name="resnet_native", kind="conv", n=128, h=32, w=32, ci=64, co=64, kk=3, stride=1, pad=1, x="relu",
             table="native", m=7),
        # a dense classifier layer at batch 1: forward and both gradients of one sample
        dict(name="dense_b1", kind="dense", b=1, fi=2048, fo=1000, table="mitchell", m=7),
        # a whole LeNet-5 training step at batch 64 (14 small calls and their glue)
        dict(name="lenet5", kind="lenet", b=64, table="exact_trunc", m=7),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _multiplier(rng, kind):
    """The multiplier of a drawn case: mostly M = 7, as most of the paper's designs are 16-bit ones."""
    c = dict(table=rng.choice(["mitchell", "mitchell", "compensated", "exact_trunc"]),
             m=rng.choice([7, 7, 7, 7, 5, 8, 10, 11]))
    if kind != "dense":
        other = rng.random()
        if other < 0.08:
            c.update(table="native", m=7)
        elif other < 0.16 and c["m"] >= 7:
            c.update(e_bits=5)
    return c


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "conv", "conv", "dense"])
    while True:
        mult = _multiplier(rng, kind)
        if kind == "gemm":
            c = dict(kind=kind, m_=_log(rng, 16, 4096), n=_log(rng, 16, 4096), k=_log(rng, 16, 4096),
                     ta=rng.random() < 0.3, tb=rng.random() < 0.3, dist=rng.choice(["normal", "uniform", "relu"]), **mult)
        elif kind == "dense":
            c = dict(kind=kind, b=rng.choice([1, _log(rng, 2, 256), _log(rng, 2, 256)]), fi=_log(rng, 16, 4096),
                     fo=_log(rng, 10, 4096), **mult)
        else:
            kk = rng.choice([1, 3, 3, 5, 7])
            h = _log(rng, 7, 64)
            c = dict(kind=kind, n=_log(rng, 1, 128), h=h, w=max(7, h + rng.choice([0, 0, -1, 3])),
                     ci=rng.choice([1, 3, _log(rng, 4, 256), _log(rng, 4, 256)]), co=_log(rng, 6, 256), kk=kk,
                     stride=rng.choice([1, 1, 2]), pad=rng.choice([0, kk // 2]), x=rng.choice(["relu", "normal"]), **mult)
        # wide tables, formats and the native multiply run slower than M <= 7 tables: smaller limits
        most = 2 ** 33 if c["m"] <= 7 and "e_bits" not in c and c["table"] != "native" else 2 ** 31
        if _macs(c) <= most:
            return c


def _out_hw(c):
    return ((c["h"] + 2 * c["pad"] - c["kk"]) // c["stride"] + 1, (c["w"] + 2 * c["pad"] - c["kk"]) // c["stride"] + 1)


def _lenet_layers(b):
    """(rows, reduction, columns) of the layers' forward products."""
    hw = ((28, 28), (10, 10))
    conv = [(b * oh * ow, kk * kk * ci, co) for (ci, co, kk, _), (oh, ow) in zip(_LENET_CONV, hw)]
    return conv + [(b, fi, fo) for fi, fo in _LENET_FC]


def _macs(c):
    """Approximate multiplies of one pass of the case."""
    if c["kind"] == "gemm":
        return c["m_"] * c["n"] * c["k"]
    if c["kind"] == "dense":
        return 3 * c["b"] * c["fi"] * c["fo"]
    if c["kind"] == "lenet":
        each = [r * k * n for r, k, n in _lenet_layers(c["b"])]
        return 3 * sum(each) - each[0]  # the images need no gradient
    oh, ow = _out_hw(c)
    return 3 * c["n"] * oh * ow * c["co"] * c["kk"] ** 2 * c["ci"]


def work(case):
    c = case
    if c["kind"] == "gemm":
        elems = c["m_"] * c["k"] + c["k"] * c["n"] + c["m_"] * c["n"]
    elif c["kind"] == "dense":  # x, w, dy read; y, dx, dw written
        elems = 2 * (c["b"] * c["fi"] + c["fi"] * c["fo"] + c["b"] * c["fo"])
    elif c["kind"] == "lenet":  # images; activations and weights, and the gradients of both
        layers = _lenet_layers(c["b"])
        elems = c["b"] * 784 + sum(2 * (r * n + k * n) for r, k, n in layers)
    else:
        oh, ow = _out_hw(c)
        elems = 2 * (c["n"] * c["h"] * c["w"] * c["ci"] + c["kk"] ** 2 * c["ci"] * c["co"] + c["n"] * oh * ow * c["co"])
    table = 0 if c["table"] == "native" else 4 << (2 * c["m"])
    return {"bytes": 4 * elems + table, "flops": 2 * _macs(c)}


def tolerance(case):
    if case["kind"] == "lenet":
        # a last-bit difference in one layer's sums moves a few activations across a 7-bit truncation
        # step of the next layer, each by 2^-7 of its value; measured with last-bit noise on every
        # product's sums over 30 seeds: up to 1.8e-2 in a small gradient
        return {"rel": 3e-2, "max": 0.9}
    # FP32 sums of up to 131072 products in another order: up to 4.3e-7 from the 64-bit sums
    return {"rel": 2e-6}


# ------------------------------------------------------------------ tables -----------------


def _factors(design, m):
    """v(ka, kb) = 2^carry * mantissa of a design's product of 1.ka and 1.kb, as float64 [2^M][2^M]."""
    f = np.arange(1 << m, dtype=np.float64) / (1 << m)
    x, y = f[:, None], f[None, :]
    if design == "exact_trunc":
        return (1.0 + x) * (1.0 + y)
    log = np.where(x + y < 1.0, 1.0 + x + y, 2.0 * (x + y))
    if design == "mitchell":
        return log
    # compensated: the mean error of each of 4 x 4 operand segments added, the result cut to M bits
    s = 1 << max(0, m - 2)
    err = ((1.0 + x) * (1.0 + y) - log).reshape((1 << m) // s, s, (1 << m) // s, s).mean(axis=(1, 3))
    v = log + np.repeat(np.repeat(err, s, axis=0), s, axis=1)
    ulp = np.where(v >= 2.0, 2.0, 1.0) / (1 << m)
    return np.floor(v / ulp) * ulp


@functools.lru_cache(maxsize=None)
def _table(design, m):
    """The design's table in the library's interchange format (carry << 23 | mantissa)."""
    if design in ("mitchell", "exact_trunc"):
        return binding.lut_build(m, design)
    bits = _factors(design, m).astype(np.float32).view(np.uint32)
    return np.ascontiguousarray((bits - np.uint32(0x3F800000)) & np.uint32(0x00FFFFFF)).reshape(-1)


# ------------------------------------------------------------------ inputs -----------------


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _values(g, shape, dist):
    if dist in ("uniform", "image"):
        x = torch.rand(shape, generator=g, device="cuda")
        return x if dist == "image" else 2.0 * x - 1.0
    x = torch.randn(shape, generator=g, device="cuda")
    return torch.relu(x) if dist == "relu" else x


def _desc(c):
    return dict(n=c["n"], h=c["h"], w=c["w"], c_in=c["ci"], c_out=c["co"], kh=c["kk"], kw=c["kk"],
                stride_h=c["stride"], stride_w=c["stride"], pad_top=c["pad"], pad_bottom=c["pad"], pad_left=c["pad"],
                pad_right=c["pad"])


def _operands(c, seed):
    """The tensors of a gemm, dense or conv case: (A, B), or (x, w, dy)."""
    g = _gen(seed)
    if c["kind"] == "gemm":
        a = _values(g, (c["k"], c["m_"]) if c["ta"] else (c["m_"], c["k"]), c["dist"])
        b = _values(g, (c["n"], c["k"]) if c["tb"] else (c["k"], c["n"]), "normal" if c["dist"] == "relu" else c["dist"])
        return a, b
    if c["kind"] == "dense":
        x = _values(g, (c["b"], c["fi"]), "relu")
        w = _values(g, (c["fi"], c["fo"]), "uniform") * math.sqrt(6.0 / (c["fi"] + c["fo"]))
        return x, w, _values(g, (c["b"], c["fo"]), "normal") * 0.05
    oh, ow = _out_hw(c)
    x = _values(g, (c["n"], c["h"], c["w"], c["ci"]), c["x"])
    w = _values(g, (c["kk"], c["kk"], c["ci"], c["co"]), "normal") * math.sqrt(2.0 / (c["kk"] ** 2 * c["ci"]))
    return x, w, _values(g, (c["n"], oh, ow, c["co"]), "normal")


def prepare(case, seed):
    c = case
    s = dict(case=c, lut=None if c["table"] == "native" else binding.device_lut(_table(c["table"], c["m"])))
    if c["kind"] == "lenet":
        g = _gen(seed)
        s["x"] = _values(g, (c["b"], 28, 28, 1), "image")
        s["labels"] = torch.randint(0, 10, (c["b"],), generator=g, device="cuda")
        conv = [modules.AMConv2d(ci, co, kk, s["lut"], c["m"], padding=pad) for ci, co, kk, pad in _LENET_CONV]
        fc = [modules.AMLinear(fi, fo, s["lut"], c["m"]) for fi, fo in _LENET_FC]
        for layer in conv + fc:
            with torch.no_grad():
                shape = layer.weight.shape
                taps = shape[0] * shape[1] if len(shape) == 4 else 1
                limit = math.sqrt(6.0 / (taps * (shape[-2] + shape[-1])))
                layer.weight.copy_(_values(g, tuple(shape), "uniform") * limit)
        s["conv"], s["fc"] = conv, fc
        s["params"] = [p for layer in conv + fc for p in layer.parameters()]
        return s
    s["t"] = _operands(c, seed)
    if c["kind"] != "gemm":
        if c["table"] != "native" and "e_bits" not in c:
            s["t"][0].requires_grad_()
            s["t"][1].requires_grad_()
        else:
            s["desc"] = _desc(c)
    return s


# ------------------------------------------------------------------ the calls --------------


def _options(c):
    return dict(multiply="native" if c["table"] == "native" else "table", e_bits=c.get("e_bits", 8))


def run(state):
    c, lut = state["case"], state["lut"]
    if c["kind"] == "gemm":
        a, b = state["t"]
        if c["table"] == "native" or "e_bits" in c:
            return binding.approx_gemm_ex(a, b, lut, c["m"], trans_a=c["ta"], trans_b=c["tb"], **_options(c))
        return binding.approx_gemm(a, b, lut, c["m"], trans_a=c["ta"], trans_b=c["tb"])
    if c["kind"] == "lenet":
        h = state["x"]
        for layer in state["conv"]:
            h = torch.relu(layer(h)).permute(0, 3, 1, 2)
            h = torch.nn.functional.max_pool2d(h, 2).permute(0, 2, 3, 1)
        h = h.reshape(c["b"], -1)
        for i, layer in enumerate(state["fc"]):
            h = layer(h)
            if i + 1 < len(state["fc"]):
                h = torch.relu(h)
        loss = torch.nn.functional.cross_entropy(h, state["labels"])
        return [h.detach()] + list(torch.autograd.grad(loss, state["params"]))
    x, w, dy = state["t"]
    if c["kind"] == "conv" and "desc" in state:  # the layers take no options: the three passes by themselves
        opt = _options(c)
        return (binding.approx_conv2d_fwd_ex(state["desc"], x, w, lut, c["m"], **opt),
                binding.approx_conv2d_bwd_data_ex(state["desc"], dy, w, lut, c["m"], **opt),
                binding.approx_conv2d_bwd_weight_ex(state["desc"], x, dy, lut, c["m"], **opt))
    if c["kind"] == "conv":
        y = modules.am_conv2d(x, w, lut, c["m"], (c["stride"],) * 2, (c["pad"],) * 4)
    else:
        y = modules.am_linear(x, w, lut, c["m"])
    return (y.detach(),) + torch.autograd.grad(y, (x, w), dy)


# ------------------------------------------------------------------ 64-bit results ---------


def _decode(t, c):
    """(mantissa index, +-2^exponent or 0, unbiased exponent) of an operand, cast to the case's format."""
    u = t.detach().contiguous().view(torch.int32)
    e = ((u >> 23) & 0xFF) - 127
    k = (u >> (23 - c["m"])) & ((1 << c["m"]) - 1)
    p = torch.ldexp(torch.where(u < 0, -1.0, 1.0).double(), e)
    beta = (1 << (c.get("e_bits", 8) - 1)) - 1
    if beta < 127:  # beyond the format: Inf above (none in these inputs), a zero below
        assert int(e.max()) <= beta
    return k, torch.where(e < 1 - beta if beta < 127 else e == -127, 0.0, p), e


def _gemm64(a, b, c):
    """sum over k of amul(a[i, k], b[k, j]) in float64; a [r][k] and b [k][j] 2-D."""
    if c["table"] == "native":
        return a.detach().double() @ b.detach().double()
    table = torch.from_numpy(_factors(c["table"], c["m"])).to(a.device).reshape(-1)
    ka, pa, ea = _decode(a, c)
    kb, pb, eb = _decode(b, c)
    if c["table"] == "exact_trunc" and "e_bits" not in c:  # the factors' own product
        return (pa * table[ka << c["m"]]) @ (pb * table[kb << c["m"]])
    beta = (1 << (c.get("e_bits", 8) - 1)) - 1
    out = torch.zeros(a.shape[0], b.shape[1], dtype=torch.float64, device=a.device)
    kstep = max(1, min(a.shape[1], (1 << 26) // b.shape[1]))
    for k0 in range(0, a.shape[1], kstep):
        ks = slice(k0, k0 + kstep)
        rows = max(1, (1 << 26) // (kb[ks].numel()))
        for r0 in range(0, a.shape[0], rows):
            rs = slice(r0, r0 + rows)
            v = table[(ka[rs, ks, None] << c["m"]) + kb[None, ks]]
            v *= pb[None, ks]
            if beta < 127:
                v *= (ea[rs, ks, None] + eb[None, ks]) > -beta  # the format's zero rule
            out[rs] += torch.bmm(pa[rs, None, ks], v)[:, 0]
    return out


def _im2col(x, c):
    """[n * oh * ow][kh * kw * ci] of an NHWC tensor inside its zero border."""
    oh, ow = _out_hw(c)
    p, s = c["pad"], c["stride"]
    xp = torch.nn.functional.pad(x.detach(), (0, 0, p, p, p, p))
    taps = [xp[:, i:i + s * (oh - 1) + 1:s, j:j + s * (ow - 1) + 1:s] for i in range(c["kk"]) for j in range(c["kk"])]
    return torch.stack(taps, dim=3).reshape(c["n"] * oh * ow, -1)


def exact(case, seed):
    c = case
    if c["kind"] == "lenet":  # truncation between the layers makes 64-bit sums another function
        return None
    t = _operands(c, seed)
    if c["kind"] == "gemm":
        a, b = t
        return _gemm64(a.t().contiguous() if c["ta"] else a, b.t().contiguous() if c["tb"] else b, c)
    x, w, dy = t
    if c["kind"] == "dense":
        return (_gemm64(x, w, c), _gemm64(dy, w.t().contiguous(), c), _gemm64(x.t().contiguous(), dy, c))
    if _macs(c) > 2e10:
        return None
    oh, ow = _out_hw(c)
    n, h, wd, ci, co, kk, s, p = (c[i] for i in ("n", "h", "w", "ci", "co", "kk", "stride", "pad"))
    cols, dyr = _im2col(x, c), dy.reshape(-1, co)
    y = _gemm64(cols, w.reshape(-1, co), c).reshape(n, oh, ow, co)
    dw = _gemm64(cols.t().contiguous(), dyr, c).reshape(w.shape)
    # each tap's products, added where the tap reads x
    dcol = _gemm64(dyr, w.reshape(-1, co).t().contiguous(), c).reshape(n, oh, ow, kk, kk, ci)
    dx = torch.zeros(n, h + 2 * p, wd + 2 * p, ci, dtype=torch.float64, device=x.device)
    for i in range(kk):
        for j in range(kk):
            dx[:, i:i + s * (oh - 1) + 1:s, j:j + s * (ow - 1) + 1:s] += dcol[:, :, :, i, j]
    return y, dx[:, p:p + h, p:p + wd], dw
