"""The bodies that compute additive and exact-product tables (matrix cores at M = 3..7, FP32 at M = 8..11)
and the native multiply's, against the general bodies and the oracle.

A table with one entry changed takes the general path: (2^M - 1, 2^M - 1), which the operands here never
select, so both paths have the same products.  Shapes sit at the edges of the matrix-core tiles (128 or
256 rows, 16, 32 or 64 columns, slabs of 32 steps); operands hold zeros of both signs, and whole rows
and columns of them.  Single products must be equal bit for bit, sums within the parity bar of the
oracle on either path, and exactly-zero sums of zero products have the oracle's sign.
"""
import numpy as np
import pytest

import oracle
from parity import assert_bits_equal, assert_within_tolerance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MODELS = {"mitchell": oracle.MITCHELL, "exact_trunc": oracle.EXACT_TRUNC}


@pytest.fixture(scope="module")
def B():
    from paper_2209_04161_amd import binding
    binding.lib()
    return binding


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _tables(B, model, m):
    """(the table, the same with an entry changed that no operand selects), on the device."""
    lut = B.lut_build(m, model)
    other = lut.copy()
    other[-1] ^= np.uint32(1 << (23 - m) if model == "mitchell" else 0x100)
    return B.device_lut(lut), B.device_lut(other)


def _operand(rng, shape, m, zeros=0.0):
    """Exponents 100..150, never the largest mantissa index; a share of zeros of both signs."""
    u = rng.integers(0, 1 << 23, shape, dtype=np.uint32)
    top = np.uint32(((1 << m) - 1) << (23 - m))
    u = np.where((u & top) == top, u ^ np.uint32(1 << 22), u)
    u |= rng.integers(100, 151, shape).astype(np.uint32) << np.uint32(23)
    u |= rng.integers(0, 2, shape).astype(np.uint32) << np.uint32(31)
    u = np.where(rng.random(shape) < zeros, u & np.uint32(0x80000000), u)
    return np.ascontiguousarray(u.astype(np.uint32).view(np.float32))


# m, n, k, trans_a, trans_b; at least 2^27 products each: smaller calls take the general path
GEMMS = [
    (127, 15, 72001, False, False), (128, 16, 66000, True, False), (129, 17, 62003, False, True),
    (257, 33, 16102, True, True), (255, 65, 8103, False, False), (16, 64, 131080, False, False),
    (300, 32, 14001, False, True), (5, 2100, 12801, True, False), (640, 200, 1111, False, False),
    (3000, 4100, 17, False, False), (1025, 513, 513, False, False),
]


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("case", range(len(GEMMS)))
def test_gemm_matches_general_path(B, model, case):
    m, n, k, ta, tb = GEMMS[case]
    assert m * n * k >= 1 << 27
    mb = (3, 5, 7)[case % 3]
    rng = np.random.default_rng(case)
    a, b = _operand(rng, (m, k), mb, 0.3), _operand(rng, (k, n), mb, 0.2)
    a[m // 2] = -0.0
    b[:, n // 2] = np.where(rng.random(k) < 0.5, 0.0, -0.0)
    da = torch.from_numpy(np.ascontiguousarray(a.T if ta else a)).cuda()
    db = torch.from_numpy(np.ascontiguousarray(b.T if tb else b)).cuda()
    c, g = (host(B.approx_gemm(da, db, lut, mb, trans_a=ta, trans_b=tb)) for lut in _tables(B, model, mb))
    cols = np.unique(np.r_[0, n // 2, n - 1, rng.integers(0, n, 40)])
    idx = (np.arange(m)[:, None] * n + cols).reshape(-1)
    ref, S = oracle.gemm(MODELS[model], mb, a, b, idx=idx)
    for got, what in ((c, "matrix cores"), (g, "general path")):
        assert_within_tolerance(got.reshape(-1)[idx], ref, S, what)
    zero = np.asarray(S).reshape(-1) == 0.0  # sums of zero products
    assert zero.any()
    assert_bits_equal(c.reshape(-1)[idx][zero], np.asarray(ref).reshape(-1)[zero], "zero sums")


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("m", [3, 5, 7])
def test_single_products(B, model, m):
    """K = 2 with a zero second step: every output is one product (k = 1 has kernels of its own)."""
    rng = np.random.default_rng(m)
    rows, cols = 8200, 8200  # 2 * rows * cols >= 2^27
    a, b = _operand(rng, (rows, 2), m, 0.05), _operand(rng, (2, cols), m, 0.05)
    a[:, 1] = 0.0
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    c = host(B.approx_gemm(da, db, _tables(B, model, m)[0], m))
    p = oracle.mul(MODELS[model], m, np.repeat(a[:, 0], cols), np.tile(b[0], rows)).reshape(rows, cols)
    keep = p != 0.0  # a zero product's sign is that of the two-product sum
    assert_bits_equal(c[keep], p[keep], "products")
    assert not c[~keep].any()


# n, h, w, ci, co, kh, kw, stride, pads (top, bottom, left, right); at least 2^27 products a pass
CONVS = [
    (100, 19, 21, 5, 80, 3, 3, 1, (1, 1, 1, 1)), (20, 57, 53, 3, 64, 7, 7, 2, (3, 3, 3, 3)),
    (130, 8, 8, 64, 33, 3, 3, 1, (1, 1, 1, 1)), (150, 31, 31, 16, 17, 5, 3, 2, (2, 1, 0, 1)),
    (250, 14, 14, 40, 72, 1, 1, 1, (0, 0, 0, 0)), (1000, 30, 31, 1, 6, 5, 5, 1, (2, 2, 2, 2)),
]


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("case", range(len(CONVS)))
def test_convolution_passes_match_general_path(B, model, case):
    n, h, w, ci, co, kh, kw, s, (pt, pb, pl, pr) = CONVS[case]
    d = dict(n=n, h=h, w=w, c_in=ci, c_out=co, kh=kh, kw=kw, stride_h=s, stride_w=s, pad_top=pt, pad_bottom=pb,
             pad_left=pl, pad_right=pr)
    oh, ow = B.conv_out_hw(d)
    assert n * oh * ow * co * kh * kw * ci >= 1 << 27
    rng = np.random.default_rng(100 + case)
    m = 7 if case % 2 else 4
    x = _operand(rng, (n, h, w, ci), m, 0.4)
    wt = _operand(rng, (kh, kw, ci, co), m, 0.1)
    dy = _operand(rng, (n, oh, ow, co), m, 0.4)
    dx, dwt, ddy = (torch.from_numpy(t).cuda() for t in (x, wt, dy))
    mid = MODELS[model]
    for fn, ins, ref in ((B.approx_conv2d_fwd, (dx, dwt), oracle.conv2d_fwd(mid, m, d, x, wt)),
                         (B.approx_conv2d_bwd_data, (ddy, dwt), oracle.conv2d_bwd_data(mid, m, d, dy, wt)),
                         (B.approx_conv2d_bwd_weight, (dx, ddy), oracle.conv2d_bwd_weight(mid, m, d, x, dy))):
        for lut, what in zip(_tables(B, model, m), ("matrix cores", "general path")):
            assert_within_tolerance(host(fn(d, *ins, lut, m)), *ref, "%s, %s" % (fn.__name__, what))


WIDE = [  # m, n, k, trans_a, trans_b: the arithmetic bodies' tiles are 128 or 256 rows, 64 or 128 columns
    (2, 2, 2, False, False), (127, 63, 15, False, True), (257, 65, 17, True, False), (130, 129, 33, True, True),
    (300, 7, 1000, False, False), (33, 300, 9, False, False),
]


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("e_bits,exps", [(8, (100, 151)), (8, (1, 255)), (5, (110, 143))])
@pytest.mark.parametrize("case", range(len(WIDE)))
def test_wide_tables_match_general_path(B, model, e_bits, exps, case):
    """M = 8..11: inside the operand window, outside it (products that under- and overflow) and in a
    (1, 5, M) format.  Class and sign of Inf and NaN sums as the oracle's on either path."""
    m, n, k, ta, tb = WIDE[case]
    mb = (8, 11, 9, 10)[(case + len(model)) % 4]
    rng = np.random.default_rng(1000 + case)

    def operand(shape, zeros):
        x = _operand(rng, shape, mb, zeros).view(np.uint32)
        e = rng.integers(exps[0], exps[1], shape).astype(np.uint32) << np.uint32(23)
        return np.where(x << np.uint32(1) == 0, x, (x & np.uint32(0x807FFFFF)) | e).astype(np.uint32).view(np.float32)

    a, b = operand((m, k), 0.2), operand((k, n), 0.1)
    a[m // 2] = -0.0
    da = torch.from_numpy(np.ascontiguousarray(a.T if ta else a)).cuda()
    db = torch.from_numpy(np.ascontiguousarray(b.T if tb else b)).cuda()
    ref, S = oracle.gemm(MODELS[model], mb, a, b, e_bits=e_bits)
    for lut, what in zip(_tables(B, model, mb), ("computed", "general path")):
        got = host(B.approx_gemm_ex(da, db, lut, mb, trans_a=ta, trans_b=tb, e_bits=e_bits))
        with np.errstate(invalid="ignore"):
            assert_within_tolerance(got, ref, S, what)
        zero = np.asarray(S) == 0.0
        assert zero.any()
        assert_bits_equal(got[zero], np.asarray(ref)[zero], "zero sums, " + what)


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("case", range(len(CONVS)))
def test_wide_convolution_passes(B, model, case):
    n, h, w, ci, co, kh, kw, s, (pt, pb, pl, pr) = CONVS[case]
    n = max(1, n // 10)
    d = dict(n=n, h=h, w=w, c_in=ci, c_out=co, kh=kh, kw=kw, stride_h=s, stride_w=s, pad_top=pt, pad_bottom=pb,
             pad_left=pl, pad_right=pr)
    oh, ow = B.conv_out_hw(d)
    rng = np.random.default_rng(200 + case)
    m = (8, 9, 10, 11)[case % 4]
    x, wt = _operand(rng, (n, h, w, ci), m, 0.4), _operand(rng, (kh, kw, ci, co), m, 0.1)
    dy = _operand(rng, (n, oh, ow, co), m, 0.4)
    dx, dwt, ddy = (torch.from_numpy(t).cuda() for t in (x, wt, dy))
    mid = MODELS[model]
    for fn, ins, ref in ((B.approx_conv2d_fwd, (dx, dwt), oracle.conv2d_fwd(mid, m, d, x, wt)),
                         (B.approx_conv2d_bwd_data, (ddy, dwt), oracle.conv2d_bwd_data(mid, m, d, dy, wt)),
                         (B.approx_conv2d_bwd_weight, (dx, ddy), oracle.conv2d_bwd_weight(mid, m, d, x, dy))):
        for lut, what in zip(_tables(B, model, m), ("computed", "general path")):
            assert_within_tolerance(host(fn(d, *ins, lut, m)), *ref, "%s, %s" % (fn.__name__, what))


@pytest.mark.parametrize("inside", [True, False])
@pytest.mark.parametrize("case", range(len(GEMMS)))
def test_native_multiply_gemm(B, case, inside):
    """Large calls with the native multiply: the matrix cores inside the operand window, the fma kernels
    with an operand so large that some product could overflow (none does); denormal operands, read as
    zero, on either."""
    m, n, k, ta, tb = GEMMS[case]
    rng = np.random.default_rng(300 + case)
    a, b = _operand(rng, (m, k), 7, 0.3), _operand(rng, (k, n), 7, 0.2)
    a[m // 2] = -0.0
    b[:, n // 2] = np.where(rng.random(k) < 0.5, 0.0, -0.0)
    a[0] = (a[0].view(np.uint32) & np.uint32(0x807FFFFF)).view(np.float32)
    if not inside:
        a[m - 1, 0] = np.float32(2.0) ** 120
        b[0] = np.float32(2.0) ** -27
    da = torch.from_numpy(np.ascontiguousarray(a.T if ta else a)).cuda()
    db = torch.from_numpy(np.ascontiguousarray(b.T if tb else b)).cuda()
    got = host(B.approx_gemm_ex(da, db, None, 7, trans_a=ta, trans_b=tb, multiply="native"))
    cols = np.unique(np.r_[0, n // 2, n - 1, rng.integers(0, n, 40)])
    idx = (np.arange(m)[:, None] * n + cols).reshape(-1)
    ref, S = oracle.gemm(MODELS["mitchell"], 7, a, b, idx=idx, native=True)
    got = got.reshape(-1)[idx]
    with np.errstate(invalid="ignore"):
        assert_within_tolerance(got, ref, S, "native GEMM")
    zero = np.asarray(S) == 0.0
    assert zero.any()
    assert_bits_equal(got[zero], np.asarray(ref)[zero], "zero sums")


@pytest.mark.parametrize("case", range(len(CONVS)))
def test_native_multiply_convolutions(B, case):
    n, h, w, ci, co, kh, kw, s, (pt, pb, pl, pr) = CONVS[case]
    d = dict(n=n, h=h, w=w, c_in=ci, c_out=co, kh=kh, kw=kw, stride_h=s, stride_w=s, pad_top=pt, pad_bottom=pb,
             pad_left=pl, pad_right=pr)
    oh, ow = B.conv_out_hw(d)
    rng = np.random.default_rng(400 + case)
    x, wt = _operand(rng, (n, h, w, ci), 7, 0.4), _operand(rng, (kh, kw, ci, co), 7, 0.1)
    dy = _operand(rng, (n, oh, ow, co), 7, 0.4)
    dx, dwt, ddy = (torch.from_numpy(t).cuda() for t in (x, wt, dy))
    mid = MODELS["mitchell"]
    for fn, ins, ref in (
            (B.approx_conv2d_fwd_ex, (dx, dwt), oracle.conv2d_fwd(mid, 7, d, x, wt, native=True)),
            (B.approx_conv2d_bwd_data_ex, (ddy, dwt), oracle.conv2d_bwd_data(mid, 7, d, dy, wt, native=True)),
            (B.approx_conv2d_bwd_weight_ex, (dx, ddy), oracle.conv2d_bwd_weight(mid, 7, d, x, dy, native=True))):
        assert_within_tolerance(host(fn(d, *ins, None, 7, multiply="native")), *ref, fn.__name__)
