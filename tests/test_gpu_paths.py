"""Which body a call runs, read from the path flags in its workspace, and its results there.

Additive and exact-product tables and the native multiply run in bodies with tiles of their own
(own_kernel) where the call is large enough (M <= 7, native: 2^27 products), the result is wide enough and
the operands' exponents allow it; every other call runs the gathers.  Each condition is driven on both
sides, with the table of the kind and with the same table one entry away from it: entries of the first
operand's largest mantissa index, which no first operand here has, so that the products are the model's on
either table.  The changed tables keep the gathers' bodies covered where the tables of a kind no longer
reach them: the bf16, hi/lo, exact, sum-indexed and row-staging bodies in large calls.
"""
import numpy as np
import pytest

import oracle
from parity import assert_within_tolerance
from paper_2209_04161_amd import workloads as W
from test_gpu_canary import GUARD, SENTINEL, WS_BYTE, _guarded, _guarded_workspace

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MODELS = {"mitchell": oracle.MITCHELL, "exact_trunc": oracle.EXACT_TRUNC, "native": oracle.MITCHELL}
UNSET = 0x7F7F7F7F  # a flag that no launch has written


@pytest.fixture(scope="module")
def B():
    from paper_2209_04161_amd import binding
    binding.lib()
    return binding


_LUTS = {}


def lut_of(B, model, m, variant):
    """The device table: "kind" as built; "general" with an entry changed that makes it neither of a kind nor
    sum-indexed; "sum" with the last entry changed, the only one of its index sum."""
    if model == "native":
        return None
    key = (model, m, variant)
    if key not in _LUTS:
        t, n = B.lut_build(m, model).copy(), 1 << m
        flip = np.uint32(1 << (23 - m) if model == "mitchell" else 0x100)
        if variant == "general":
            t[(n - 1) * n + 1] ^= flip
        elif variant == "sum":
            t[-1] ^= flip
        _LUTS[key] = B.device_lut(t)
    return _LUTS[key]


def operand(rng, shape, m, lo, hi, first):
    """Exponent fields spanning exactly [lo, hi]; a first operand never has the largest mantissa index.  Only one
    value has hi, the others at most hi - 12: one product at most comes near the largest finite value, so that
    no partial sum overflows in one order of summation and not in another."""
    n = int(np.prod(shape))
    e = rng.integers(lo, max(lo, hi - 12) + 1, n).astype(np.uint32)
    e[0], e[-1] = lo, hi
    u = (e << 23) | rng.integers(0, 1 << 23, n, dtype=np.uint32) | (rng.integers(0, 2, n).astype(np.uint32) << 31)
    top = np.uint32(((1 << m) - 1) << (23 - m))
    if first:
        u = np.where((u & top) == top, u ^ np.uint32(1 << 22), u)
    return np.ascontiguousarray(rng.permutation(u.astype(np.uint32)).view(np.float32).reshape(shape))


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _align(x):
    return -(-x // 256) * 256


def read_flags(ws, m):
    """The four path flags of a call on tables of m bits, from its workspace: they follow the table's rows
    (rows of 128 entries and one of zeros for M <= 7), the bf16 path's rows and, for M <= 7, the hi/lo rows."""
    rl = max(m, 7)
    off = _align((1 << rl) * ((1 << rl) + (rl == 7)) * 4) + _align(129 * 128) + (_align(129 * 512) if rl == 7 else 0)
    torch.cuda.synchronize()
    return ws[off:off + 16].cpu().numpy().view(np.int32).tolist()


def workspace(nbytes):
    return torch.full((max(nbytes, 256),), 0x7F, dtype=torch.uint8, device="cuda")


def options(model, e_bits, exp_cast="inf"):
    return dict(multiply="native" if model == "native" else "table", e_bits=e_bits, exp_cast=exp_cast)


def gemm_flags(B, a, b, model, m, variant, e_bits=8, exp_cast="inf"):
    M, K = a.shape
    N = b.shape[1]
    ws = workspace(B.amsim_gemm_workspace_size(0, 0, M, N, K, m))
    C = B.approx_gemm_ex(cuda(a), cuda(b), lut_of(B, model, m, variant), m, workspace=ws,
                         **options(model, e_bits, exp_cast))
    flags = read_flags(ws, m)
    return C.cpu().numpy().reshape(-1), flags


def check_sampled(got, model, m, a, b, e_bits, what, seed, sat=False):
    idx = np.sort(np.random.default_rng(seed).choice(got.size, min(got.size, 3000), replace=False))
    ref, S = oracle.gemm(MODELS[model], m, a, b, idx=idx, e_bits=e_bits, native=model == "native", sat=sat)
    with np.errstate(invalid="ignore"):
        assert_within_tolerance(got[idx], ref, S, what)


LARGE = (4096, 64, 1024)  # 2^28 products
IN, LO, HI, A_254, B_253, B_254 = (((64, 130), (64, 127)), ((64, 130), (63, 127)), ((120, 254), (100, 127)),
                                   ((120, 254), (100, 126)), ((100, 127), (100, 253)), ((100, 126), (100, 254)))
AT_380 = ((120, 253), (100, 127))
HL_IN, HL_B15, HL_IN2, HL_142 = (((127, 130), (16, 127)), ((128, 130), (15, 127)), ((120, 130), (23, 127)),
                                 ((120, 130), (22, 127)))
MID = ((110, 140), (110, 140))
# model, table, m, e_bits, size, operands' exponents, path
PATHS = (
    # the window of the bodies for M <= 7, each side; the largest first exponent 254 inside it: bf16 path
    [("mitchell", "kind", 7, 8, LARGE, r, p) for r, p in ((IN, 3), (LO, 0), (AT_380, 3), (HI, 0), (A_254, 1), (B_253, 3), (B_254, 0))]
    + [("exact_trunc", "kind", 7, 8, LARGE, r, p) for r, p in ((IN, 4), (LO, 0), (AT_380, 4), (HI, 0), (A_254, 4), (B_253, 4), (B_254, 0))]
    + [("native", "kind", 7, 8, LARGE, r, p) for r, p in ((IN, 3), (LO, 0), (AT_380, 3), (HI, 0), (A_254, 3), (B_253, 3), (B_254, 0))]
    # general tables: the bf16 path's and the hi/lo path's thresholds
    + [("mitchell", "general", 7, 8, LARGE, r, p) for r, p in ((IN, 1), (LO, 0), (AT_380, 1), (HI, 0), (A_254, 1), (B_253, 1), (B_254, 0))]
    + [("exact_trunc", "general", 7, 8, (4096, 1024, 64), r, p) for r, p in ((HL_IN, 2), (HL_B15, 0), (HL_IN2, 2), (HL_142, 0))]
    + [("mitchell", "kind", 6, 8, LARGE, MID, 3), ("exact_trunc", "kind", 4, 8, LARGE, MID, 4),
       ("mitchell", "kind", 2, 8, LARGE, MID, 1), ("mitchell", "kind", 7, 5, LARGE, ((112, 142), (112, 142)), 0)]
    # full-size products on the gathers: the benchmark's GEMM, and wide tables from g and from staged rows
    + [("mitchell", "general", 7, 8, (4096, 4096, 4096), MID, 1), ("exact_trunc", "general", 7, 8, (4096, 4096, 1024), MID, 2),
       ("mitchell", "sum", 11, 8, (4096, 4096, 512), MID, 0), ("exact_trunc", "general", 11, 8, (4096, 4096, 512), MID, 0)]
    # narrow results are the gathers' (the exact product's GEMMs are not)
    + [("mitchell", "kind", 7, 8, (8192, 16, 1024), MID, 1), ("mitchell", "kind", 7, 8, (8192, 17, 1024), MID, 3),
       ("exact_trunc", "kind", 7, 8, (65536, 2, 1024), MID, 4), ("native", "kind", 7, 8, (16384, 8, 1024), MID, UNSET),
       ("native", "kind", 7, 8, (16384, 13, 1024), MID, 3)]
    # small calls decide in the table kernel
    + [("mitchell", "kind", 7, 8, (512, 64, 1024), MID, UNSET), ("native", "kind", 7, 8, (512, 64, 1024), MID, UNSET)]
    # wide tables: any size, rounded products outside the window
    + [("mitchell", "kind", 9, 8, (300, 64, 97), r, p) for r, p in ((IN, 3), (LO, 5), (HI, 5), (A_254, 5), (B_253, 3), (B_254, 5))]
    + [("exact_trunc", "kind", 9, 8, (300, 64, 97), r, p) for r, p in ((IN, 4), (LO, 6), (HI, 6), (A_254, 4), (B_253, 4), (B_254, 6))]
    + [(t, v, m, e, (300, 64, 97), MID, 0) for t, v in (("mitchell", "general"), ("mitchell", "sum"), ("exact_trunc", "general"))
       for m, e in ((8, 8), (11, 8), (10, 5))]
    + [("mitchell", "kind", 8, 8, (300, 12, 97), MID, 0), ("mitchell", "kind", 8, 8, (300, 13, 97), MID, 3),
       ("mitchell", "kind", 8, 8, (300, 13, 97), LO, 0),  # rounded products from 29 columns
       ("mitchell", "kind", 8, 8, (300, 29, 97), LO, 5),
       ("mitchell", "kind", 11, 5, (300, 28, 97), MID, 0), ("mitchell", "kind", 11, 5, (300, 29, 97), MID, 5),
       ("exact_trunc", "kind", 11, 5, (300, 19, 97), MID, 0), ("exact_trunc", "kind", 11, 5, (300, 20, 97), MID, 6),
       ("exact_trunc", "kind", 10, 8, (300, 3, 97), MID, 4), ("exact_trunc", "kind", 10, 8, (300, 3, 97), HI, 0)]
)


@pytest.mark.parametrize("case", range(len(PATHS)))
def test_path_of_gemm(B, case):
    model, variant, m, e_bits, (M, N, K), (ra, rb), path = PATHS[case]
    rng = np.random.default_rng(case)
    a, b = operand(rng, (M, K), m, *ra, True), operand(rng, (K, N), m, *rb, False)
    got, flags = gemm_flags(B, a, b, model, m, variant, e_bits)
    what = "%s %s M=%d e=%d %s" % (model, variant, m, e_bits, (M, N, K))
    assert flags[1] == path, what + ": flags %s" % flags
    if m > 7 and path == 0:  # the gathers' body: one array of factors, or rows
        assert flags[3] == (0 if variant == "general" or model == "exact_trunc" else 1), what + ": flags %s" % flags
    check_sampled(got, model, m, a, b, e_bits, what, case)


@pytest.mark.parametrize("model,m,path", [("mitchell", 7, 0), ("exact_trunc", 7, 0), ("native", 7, 0), ("mitchell", 9, 5),
                                          ("exact_trunc", 11, 6)])
def test_special_operands(B, model, m, path):
    """NaN and Inf operands: the exact path, or the rounded form."""
    rng = np.random.default_rng(900 + m)
    a, b = operand(rng, LARGE[::2], m, 110, 140, True), operand(rng, (LARGE[2], LARGE[1]), m, 110, 140, False)
    a[3, 10], a[70, 20], b[5, 7], b[40, 7], b[20, 9] = np.nan, -np.inf, np.inf, -np.inf, np.inf
    got, flags = gemm_flags(B, a, b, model, m, "kind")
    assert flags[1] == path
    got = got.reshape(LARGE[0], LARGE[1])[:80]
    ref, S = oracle.gemm(MODELS[model], m, a[:80], b, native=model == "native")
    with np.errstate(invalid="ignore"):
        assert_within_tolerance(got, ref, S, "special operands")


@pytest.mark.parametrize("model", ["mitchell", "exact_trunc"])
def test_saturating_cast_on_a_computed_wide_table(B, model):
    rng = np.random.default_rng(950)
    a, b = operand(rng, (200, 65), 9, 100, 160, True), operand(rng, (65, 40), 9, 100, 160, False)
    for variant, path in (("kind", 5 if model == "mitchell" else 6), ("general", 0)):
        got, flags = gemm_flags(B, a, b, model, 9, variant, 5, "saturate")
        assert flags[1] == path
        check_sampled(got, model, 9, a, b, 5, "saturate, " + variant, 951, sat=True)


# n, h, w, ci, co, kernel, stride, pad, m, e_bits and, per pass, whether the additive and the exact kind run in
# a body with tiles of its own
CONVS = [
    (16, 33, 31, 64, 64, 3, 2, 1, 7, 8, ((1, 1), (1, 1), (1, 1))),
    (32, 32, 32, 64, 16, 3, 1, 1, 7, 8, ((0, 1), (1, 1), (1, 1))),
    (24, 40, 40, 16, 17, 5, 1, 2, 7, 8, ((1, 1), (0, 1), (1, 1))),
    (200, 28, 28, 32, 8, 5, 1, 2, 7, 8, ((0, 0), (1, 1), (1, 1))),
    (4, 15, 17, 12, 24, 3, 1, 1, 9, 8, ((1, 1), (0, 1), (1, 1))),
    (4, 15, 17, 20, 30, 3, 2, 1, 10, 5, ((1, 1), (0, 1), (1, 1))),
    (4, 15, 17, 20, 8, 3, 1, 1, 11, 5, ((0, 0), (0, 1), (0, 1))),
    (128, 32, 32, 64, 64, 3, 1, 1, 7, 8, ((1, 1), (1, 1), (1, 1))),  # the benchmark's ResNet 3x3 layer
]


@pytest.mark.parametrize("case", range(len(CONVS)))
def test_path_of_convolution_passes(B, case):
    n, h, w, ci, co, kk, s, pad, m, e_bits, own = CONVS[case]
    d = W.conv_desc(n, h, w, ci, co, kk, kk, s, pad)
    assert m > 7 or W.conv_macs(d) >= 1 << 27
    oh, ow = W.conv_out_hw(d)
    rng = np.random.default_rng(1000 + case)
    x, wt = operand(rng, (n, h, w, ci), m, 113, 141, True), operand(rng, (kk, kk, ci, co), m, 113, 141, False)
    dy = operand(rng, (n, oh, ow, co), m, 113, 141, True)
    # backward weight takes x first: w and dy are second operands or, in backward data, dy the first
    calls = ((B.approx_conv2d_fwd_ex, (x, wt), oracle.conv2d_fwd), (B.approx_conv2d_bwd_data_ex, (dy, wt), oracle.conv2d_bwd_data),
             (B.approx_conv2d_bwd_weight_ex, (x, dy), oracle.conv2d_bwd_weight))
    for pass_id, (fn, ins, ref_fn) in enumerate(calls):
        size = [n * oh * ow * co, n * h * w * ci, kk * kk * ci * co][pass_id]
        idx = np.sort(rng.choice(size, min(size, 1500), replace=False))
        for ki, model in enumerate(("mitchell", "exact_trunc")):
            ref, S = ref_fn(MODELS[model], m, d, *ins, idx=idx, e_bits=e_bits)
            for variant in ("kind", "general"):
                ws = workspace(B.amsim_conv2d_workspace_size(d, pass_id, m))
                got = fn(d, *map(cuda, ins), lut_of(B, model, m, variant), m, workspace=ws, **options(model, e_bits))
                flags = read_flags(ws, m)
                what = "%s %s %s" % (fn.__name__, model, variant)
                assert (flags[1] >= 3) == bool(variant == "kind" and own[pass_id][ki]), what + ": flags %s" % flags
                with np.errstate(invalid="ignore"):
                    assert_within_tolerance(got.cpu().numpy().reshape(-1)[idx], ref, S, what)


GUARDED = [  # (model, table, m), GEMM or convolution at or beyond the sizes of the bodies with tiles of their own
    (t, v, m, shape) for t, v, m in (("mitchell", "kind", 7), ("exact_trunc", "kind", 7), ("native", "kind", 7), ("exact_trunc", "general", 7))
    for shape in ((63, 41, 60007), (1030, 300, 500), W.conv_desc(16, 33, 31, 64, 66, 3, 3, 2, 1), W.conv_desc(30, 57, 53, 3, 34, 7, 7, 1, 3))
] + [
    (t, v, m, shape) for t, v, m in (("mitchell", "kind", 11), ("mitchell", "sum", 11), ("exact_trunc", "general", 9), ("exact_trunc", "kind", 8))
    for shape in ((63, 41, 9007), (300, 130, 257), W.conv_desc(4, 19, 17, 20, 34, 3, 3, 2, 1))
]


@pytest.mark.parametrize("case", range(len(GUARDED)))
def test_writes_stay_in_the_buffers(B, case):
    model, variant, m, shape = GUARDED[case]
    lut = lut_of(B, model, m, variant)
    rng = np.random.default_rng(1100 + case)
    calls = []
    if isinstance(shape, tuple):
        M, N, K = shape
        a, b = cuda(operand(rng, (M, K), m, 110, 140, True)), cuda(operand(rng, (K, N), m, 110, 140, False))
        calls.append(((M, N), B.amsim_gemm_workspace_size(0, 0, M, N, K, m), lambda **kw: B.approx_gemm_ex(a, b, lut, m, **kw)))
    else:
        d, (oh, ow) = shape, W.conv_out_hw(shape)
        xs, wsh, ys = ((d["n"], d["h"], d["w"], d["c_in"]), (d["kh"], d["kw"], d["c_in"], d["c_out"]), (d["n"], oh, ow, d["c_out"]))
        x, w, dy = (cuda(operand(rng, sh, m, 110, 140, True)) for sh in (xs, wsh, ys))
        for pass_id, (fn, i0, i1, out) in enumerate(((B.approx_conv2d_fwd_ex, x, w, ys), (B.approx_conv2d_bwd_data_ex, dy, w, xs),
                                                     (B.approx_conv2d_bwd_weight_ex, x, dy, wsh))):
            calls.append((out, B.amsim_conv2d_workspace_size(d, pass_id, m),
                          lambda fn=fn, i0=i0, i1=i1, **kw: fn(d, i0, i1, lut, m, **kw)))
    sentinel = np.int32(np.uint32(SENTINEL).view(np.int32))
    for out_shape, nbytes, call in calls:
        ref = call(**options(model, 8))
        buf, out = _guarded(out_shape)
        wbuf, ws = _guarded_workspace(nbytes)
        call(out=out, workspace=ws, **options(model, 8))
        torch.cuda.synchronize()
        g = buf.cpu().numpy()
        assert np.all(g[:GUARD] == sentinel) and np.all(g[-GUARD:] == sentinel), "a write outside the result"
        assert np.array_equal(g[GUARD:-GUARD], ref.cpu().numpy().view(np.int32).reshape(-1)), "the result differs"
        assert np.all(wbuf[nbytes:].cpu().numpy() == WS_BYTE), "a write past the workspace (%d bytes)" % nbytes


def test_captured_call_decides_at_each_replay(B):
    """One captured GEMM (split reduction, 2^27 products and more) replayed on operands and tables that take
    different bodies: every replay equals the eager call's bits."""
    M, N, K = 130, 72, 16000
    rng = np.random.default_rng(1200)
    ins = [(cuda(operand(rng, (M, K), 7, *ra, True)), cuda(operand(rng, (K, N), 7, *rb, False))) for ra, rb in (MID, LO, A_254)]
    luts = [lut_of(B, "mitchell", 7, "kind"), lut_of(B, "mitchell", 7, "general"), lut_of(B, "exact_trunc", 7, "kind")]
    a, b, lut = ins[0][0].clone(), ins[0][1].clone(), luts[0].clone()
    ws = workspace(B.amsim_gemm_workspace_size(0, 0, M, N, K, 7))
    out = torch.empty(M, N, device="cuda")
    eager = [[B.approx_gemm(x, y, t, 7).cpu().numpy().view(np.int32).copy() for t in luts] for x, y in ins]
    B.approx_gemm(a, b, lut, 7, out=out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.approx_gemm(a, b, lut, 7, out=out, workspace=ws)
    paths = set()
    for rep in range(2):
        for i, (x, y) in enumerate(ins):
            for k, t in enumerate(luts):
                a.copy_(x), b.copy_(y), lut.copy_(t)
                graph.replay()
                paths.add(read_flags(ws, 7)[1])
                assert np.array_equal(out.cpu().numpy().view(np.int32), eager[i][k]), "replay %d, operands %d, table %d" % (rep, i, k)
    assert paths == {0, 1, 3, 4}


def test_two_streams_on_different_bodies(B):
    """Calls of the bodies with tiles of their own and of the gathers on two streams at once."""
    rng = np.random.default_rng(1300)
    a, b = cuda(operand(rng, (1024, 1024), 7, *MID[0], True)), cuda(operand(rng, (1024, 200), 7, *MID[1], False))
    a2, b2 = cuda(operand(rng, (300, 700), 7, *MID[0], True)), cuda(operand(rng, (700, 64), 7, *MID[1], False))

    def work(variant, model):
        return [B.approx_gemm(a, b, lut_of(B, model, 7, variant), 7),
                B.approx_gemm_ex(a, b, None, 7, multiply="native"),
                B.approx_gemm(a2, b2, lut_of(B, model, 9, variant), 9)]

    jobs = (("kind", "mitchell"), ("general", "exact_trunc"))
    ref = [[t.cpu().numpy().view(np.int32).copy() for t in work(*j)] for j in jobs]
    streams = [torch.cuda.Stream() for _ in jobs]  # default priority
    for _ in range(3):
        torch.cuda.synchronize()
        got = []
        for st, j in zip(streams, jobs):
            with torch.cuda.stream(st):
                got.append(work(*j))
        torch.cuda.synchronize()
        for g, r in zip(got, ref):
            assert all(np.array_equal(t.cpu().numpy().view(np.int32), x) for t, x in zip(g, r))
