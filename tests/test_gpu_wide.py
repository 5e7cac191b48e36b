"""GPU parity of the lane-decoded matrix-core GEMMs over every payload width.

Weights are random codes (the reserved pattern among them) with random scales
and admissible shapes; the bounds are elementwise and follow from the operand
formats, so that one wrong code, scale or row fails.
"""
import numpy as np
import pytest

from oracle import format as F
from tests._cases import act, say
from workloads import PRINTED_SHAPES, to_f16_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    import paper_2608_06763_amd as cq
    cq.lib()
    return torch


def random_weight(seed, n, k, bits, group, repeat=1):
    """(CQWeight of n * repeat rows, codes, scale, a, b of the n rows); a few
    fields hold the reserved pattern, whose code is given as 0."""
    import torch
    import paper_2608_06763_amd as cq
    g = np.random.Generator(np.random.PCG64(seed))
    m = F.max_code(bits)
    codes = g.integers(-m, m + 1, (n, k)) if bits > 1 else g.integers(0, 2, (n, k)) * 2 - 1
    fields = np.mod(codes, 1 << bits) if bits > 1 else (codes > 0).astype(np.int64)
    if bits > 1:
        reserved = g.random((n, k)) < 0.01
        fields[reserved] = 1 << (bits - 1)
        codes[reserved] = 0
    stream = ((fields[:, :, None] >> np.arange(bits)) & 1).astype(np.uint8).reshape(n, k * bits)
    packed = np.packbits(stream, axis=1, bitorder="little")
    ng = k // group
    scale = (0.02 * np.exp(0.5 * g.standard_normal((n, ng)))).astype(np.float32)
    shapes = np.array(PRINTED_SHAPES)[g.integers(0, len(PRINTED_SHAPES), (n, ng))]
    a, b = to_f16_bits(shapes[..., 0]), to_f16_bits(shapes[..., 1])
    rep = lambda v, dt: torch.from_numpy(np.ascontiguousarray(v).view(dt)).cuda().repeat(repeat, 1)
    w = cq.CQWeight(rep(packed, np.uint8), rep(scale, np.float32), rep(a, np.int16), rep(b, np.int16), bits, group,
                    n * repeat, k)
    return w, codes, scale, a, b


def model_dtype_bound(xv, wd, dtype):
    """Largest error of sum x w with the weight as hi + lo BF16 parts (hi and lo
    each rounded once, at most 2^-18 of the weight, and an FP32 level within
    2^-20) or as one FP16 operand (2^-11), plus the FP32 accumulation over K."""
    per_weight = 2.0 ** -17 if dtype == "bf16" else 2.0 ** -11 + 2.0 ** -20
    mass = np.abs(xv) @ np.abs(wd).T
    return (per_weight + 2.0 ** -24 * np.sqrt(xv.shape[1]) * 4) * mass + 1e-30


# m: one row block, a ragged tile of 64 and, with many weight rows, of 128, 160
# and 256 rows of x (test_wide_tile_heights of test_abi_host.py); K: several loop trips, an
# odd number of steps, an odd number of 32-code units where the width allows it
@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("group,k", [(32, 1152), (64, 1152), (128, 1152), (256, 1280), (512, 1536)])
@pytest.mark.parametrize("m,repeat", [(17, 1), (130, 1), (100, 214), (300, 104), (450, 104)])
def test_wide_model_dtype(torch_dev, bits, group, k, m, repeat):
    import paper_2608_06763_amd as cq
    if group == 32 and bits in (4, 8):
        k = 1056
    n = 131
    w, codes, scale, a, b = random_weight(900 + bits, n, k, bits, group, repeat)
    wd = F.decode(codes, bits, group, scale, a, b)
    # up to five bits the fixed heights, above them the conservative family
    families = ("gemm_mfma", "gemm_mfma_m128", "gemm_mfma_m256") if bits <= 5 else ("gemm_tiled",)
    for dtype in ("bf16", "fp16"):
        xb, xv = act(901 + m, m, k, dtype)
        x = torch_dev.from_numpy(xb.view(np.int16)).cuda().view(
            torch_dev.bfloat16 if dtype == "bf16" else torch_dev.float16)
        want, bound = xv @ wd.T, model_dtype_bound(xv, wd, dtype)
        for f in families:
            say("wide", bits, group, k, m, repeat, dtype, f)
            y = cq.cq_gemm_model_dtype_family(w, x, f, y_dtype=torch_dev.float32)
            assert torch_dev.equal(y, cq.cq_gemm_model_dtype_family(w, x, f, y_dtype=torch_dev.float32))
            got = y.view(m, repeat, n)
            assert torch_dev.equal(got[:, -1], got[:, 0])
            got = got[:, 0].cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - want) <= bound), f
            y16 = cq.cq_gemm_model_dtype_family(w, x, f)
            assert torch_dev.equal(y16, y.to(y16.dtype)), f


def whole_bound(xv, wd):
    """FP32 weights and products: coefficients rounded once and three Horner
    roundings, up to twice that where the curve's terms cancel (8 units of
    2^-24), and an FP32 sum over K."""
    return (2.0 ** -21 + 2.0 ** -24 * np.sqrt(xv.shape[1]) * 4) * (np.abs(xv) @ np.abs(wd).T) + 1e-30


# Up to 16 rows the split-K kernel stands in for the FP32 GEMV, which still runs
# calls of four rows: its FP32 outputs are no further from the 64-bit result
# (norm over 16 x 64 outputs; one chain of matrix instructions over all of K was
# 2.6 times further at this K).
@pytest.mark.parametrize("bits", [6, 7, 8])
@pytest.mark.parametrize("group", [32, 128, 512])
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_split_whole_precision(torch_dev, bits, group, dtype):
    import paper_2608_06763_amd as cq
    k, n, repeat, m = 8192, 64, 128, 16
    w, codes, scale, a, b = random_weight(970 + bits, n, k, bits, group, repeat)
    xb, xv = act(971 + group, m, k, dtype)
    x = torch_dev.from_numpy(xb.view(np.int16)).cuda().view(
        torch_dev.bfloat16 if dtype == "bf16" else torch_dev.float16)
    want = xv @ F.decode(codes, bits, group, scale, a, b).T
    say("split whole precision", bits, group, dtype)
    y = cq.cq_gemm_model_dtype(w, x, y_dtype=torch_dev.float32)[:, :n]
    base = torch_dev.cat([cq.cq_gemm_model_dtype_family(w, x[i:i + 4].contiguous(), "gemv_generic",
                                                        y_dtype=torch_dev.float32)[:, :n] for i in range(0, m, 4)])
    err, err_base = (np.linalg.norm(v.cpu().numpy().astype(np.float64) - want) for v in (y, base))
    assert not torch_dev.equal(y, base)  # the split kernel ran
    assert err <= err_base, (err, err_base)


# The split-K kernel: FP32-whole weights up to 16 rows (B >= 6, the generic
# family), the many-row operands above; K of 17 and 33 steps of 128
# codes over eight waves (some with one step more, the last with none or a part),
# ragged weight and activation rows.
@pytest.mark.parametrize("group,k", [(32, 2176), (64, 2176), (128, 4224), (256, 2304), (512, 4608)])
@pytest.mark.parametrize("m,bits", [(m, bits) for m in (12, 16, 17, 33, 64, 130) for bits in range(1, 9)
                                    if m > 32 or bits > 5])  # (else the slab kernels' rows)
def test_split_model_dtype(torch_dev, bits, group, k, m):
    import paper_2608_06763_amd as cq
    if group == 32 and bits in (4, 8):
        k = 2080  # a step with one unit
    n = 75
    w, codes, scale, a, b = random_weight(980 + bits, n, k, bits, group)
    wd = F.decode(codes, bits, group, scale, a, b)
    family = "gemv_generic" if m <= 16 else "gemm_mfma" if bits <= 5 else "gemm_tiled"
    for dtype in ("bf16", "fp16"):
        xb, xv = act(981 + m, m, k, dtype)
        x = torch_dev.from_numpy(xb.view(np.int16)).cuda().view(
            torch_dev.bfloat16 if dtype == "bf16" else torch_dev.float16)
        say("split", bits, group, k, m, dtype, family)
        y = cq.cq_gemm_model_dtype_family(w, x, family, y_dtype=torch_dev.float32)
        assert torch_dev.equal(y, cq.cq_gemm_model_dtype_family(w, x, family, y_dtype=torch_dev.float32))
        assert torch_dev.equal(y, cq.cq_gemm_model_dtype(w, x, y_dtype=torch_dev.float32))
        bound = whole_bound(xv, wd) if m <= 16 else model_dtype_bound(xv, wd, dtype)
        assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - xv @ wd.T) <= bound)
        y16 = cq.cq_gemm_model_dtype(w, x)
        assert torch_dev.equal(y16, y.to(y16.dtype))


# Infinities and NaNs of one activation row, on both sides of the row count from
# which the split-K kernel takes W6-W8: what FP32 products give (a zero weight
# against an infinity is NaN), and the other rows as without them.
@pytest.mark.parametrize("bits", [6, 7, 8])
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("group", [32, 128])
def test_few_rows_nonfinite(torch_dev, bits, dtype, group):
    import paper_2608_06763_amd as cq
    k, n, repeat, m = 4224, 64, 64, 16
    w, codes, scale, a, b = random_weight(975 + bits, n, k, bits, group, repeat)
    wd = F.decode(codes, bits, group, scale, a, b)
    xb, xv = act(976, m, k, dtype)
    x = torch_dev.from_numpy(xb.view(np.int16)).cuda().view(
        torch_dev.bfloat16 if dtype == "bf16" else torch_dev.float16)
    bad, inf = x.clone(), float("inf")
    # single infinities at the ends of K and inside, two in one row, a NaN
    marks = {1: {0: inf}, 2: {k - 1: -inf}, 6: {2000: inf}, 9: {5: inf, 4000: inf}, 11: {77: inf, 78: -inf},
             15: {3000: float("nan")}}
    for r, at in marks.items():
        for j, v in at.items():
            bad[r, j] = v
            xv[r, j] = v
    rows = sorted(marks)
    with np.errstate(invalid="ignore"):
        want = (xv[rows][:, None, :] * wd[None]).sum(-1)
    for rows_per_call in (16, 4):
        say("nonfinite", bits, dtype, group, rows_per_call)
        run = lambda v: torch_dev.cat([cq.cq_gemm_model_dtype_family(w, v[i:i + rows_per_call].contiguous(),
                                       "gemv_generic", y_dtype=torch_dev.float32)[:, :n]
                                       for i in range(0, m, rows_per_call)])
        clean, y = run(x), run(bad)
        if rows_per_call == 16:
            assert torch_dev.allclose(y, cq.cq_gemm_model_dtype(w, bad, y_dtype=torch_dev.float32)[:, :n], rtol=0,
                                      atol=0, equal_nan=True)
        others = [r for r in range(m) if r not in marks]
        assert torch_dev.equal(y[others], clean[others])
        got = y[rows].cpu().numpy().astype(np.float64)
        assert np.array_equal(got, want, equal_nan=True)


# A8: the wide kernel against the conservative one (whose partials dump keeps
# it) bit for bit, both rescale the exact INT32 partials in group order, and
# against the oracle's semantics.  Heights of 32 to 256 rows, K ending inside a
# step for the smaller groups, G above and below a step.
# (rows are whole 16-byte units, and one long-group size runs the tall tiles)
@pytest.mark.parametrize("bits,group,k,m,repeat", [
    (bits, group, 1056 if group == 32 and bits in (4, 8) else k, m, repeat)  # 1056: an odd number of units
    for bits in range(1, 9)
    for group, k in [(32, 1152), (64, 1152), (64, 1216), (128, 1152), (256, 1280), (512, 1536)]
    for m, repeat in [(2, 1), (16, 1), (2, 62), (16, 8), (17, 1), (64, 1), (130, 1),
                      (17, 256), (64, 128), (130, 52), (500, 104)]
    if (k * bits) % 128 == 0 and (repeat == 1 or group != 256)])
def test_wide_a8(torch_dev, bits, group, k, m, repeat):
    import paper_2608_06763_amd as cq
    from oracle import a8 as A8
    n = 131
    w, codes, scale, a, b = random_weight(950 + bits, n, k, bits, group, repeat)
    xb, xv = act(951 + m, m, k)
    x8_np, dx_np = A8.quantize_act(xv)
    x8, dx = torch_dev.from_numpy(x8_np).cuda(), torch_dev.from_numpy(dx_np.astype(np.float32)).cuda()
    families = ("gemm_tiled",)
    if bits in (3, 4) and group >= 64:
        families = ("gemm_tiled", "gemm_mfma_m128", "gemm_mfma_m256") + (("gemm_mfma",) if m > 32 else ())
    base, _ = cq.cq_gemm_a8(w, x8, dx, y_dtype=torch_dev.float32, want_partials=True) if m * n * repeat < 1 << 20 \
        else (None, None)
    ref = None
    if repeat == 1 or m <= 16:
        ref, _ = A8.gemm_a8(x8_np, dx_np, codes, bits, group, scale, a, b)
    # up to 16 rows few weight rows keep the generic GEMV, more take the split-K
    # kernel; only the latter's FP16 outputs round through FP32
    split = repeat > 1 or m > 16
    if m <= 16:
        # W3 and W4 with G >= 64 have other kernels here
        families = () if bits in (3, 4) and group >= 64 else ("gemv_generic",)
        base = None
    if m <= 64:
        # the load-time tables hold the same carriers
        tab = cq.cq_build_carriers(w)
        say("wide a8 carriers", bits, group, k, m)
        assert torch_dev.equal(cq.cq_gemm_a8_carriers(w, tab, x8, dx, y_dtype=torch_dev.float32),
                               cq.cq_gemm_a8(w, x8, dx, y_dtype=torch_dev.float32))
    for f in families:
        say("wide a8", bits, group, k, m, repeat, f)
        y = cq.cq_gemm_a8_family(w, x8, dx, f, y_dtype=torch_dev.float32)
        assert torch_dev.equal(y, cq.cq_gemm_a8_family(w, x8, dx, f, y_dtype=torch_dev.float32)), f
        # (on few tiles the built-in choice splits K, in another order)
        dumped = bits in (3, 4) and group >= 64 and (m > 64 or f == "gemm_tiled" and m <= 32)
        if base is not None and (f not in ("gemm_tiled", "gemm_mfma") or repeat > 1 or dumped):
            assert torch_dev.equal(y, base), f
        if repeat > 1 and m <= 16:
            got = y.view(m, repeat, n)
            assert torch_dev.equal(got[:, 0], got[:, -1])
            assert np.max(np.abs(got[:, 0].cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref)), f
        elif repeat > 1:
            got = y.view(m, repeat, n)
            one = cq.CQWeight(w.codes[:n], w.scale[:n], w.a[:n], w.b[:n], bits, group, n, k)
            small, _ = cq.cq_gemm_a8(one, x8, dx, y_dtype=torch_dev.float32, want_partials=True)
            assert torch_dev.equal(got[:, 0], small) and torch_dev.equal(got[:, -1], small), f
        else:
            assert np.max(np.abs(y.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref)), f
        for dt in (torch_dev.bfloat16, torch_dev.float16) if split else (torch_dev.bfloat16,):
            assert torch_dev.equal(cq.cq_gemm_a8_family(w, x8, dx, f, y_dtype=dt), y.to(dt)), f


# rows whose shapes put a carrier within 3e-4 of a half-integer: exact integer
# sums from every kernel that forms carriers
@pytest.mark.parametrize("bits,group", [(bits, group) for bits in range(3, 9) for group in (32, 64, 128, 256)
                                        if (2 * group * bits) % 128 == 0])
def test_wide_a8_near_ties(torch_dev, bits, group):
    import paper_2608_06763_amd as cq
    from tests._cases import carrier_probe
    codes, s, a, b, x8, dx, p = carrier_probe(bits, group)
    w = cq.CQWeight.from_codes(codes, s, a, b, bits, group)
    for m in (20, 70, 32970):  # split K, and more tiles than it takes
        x8_t = torch_dev.from_numpy(np.repeat(x8, m, axis=0)).cuda()
        dx_t = torch_dev.from_numpy(np.repeat(dx, m)).cuda()
        want = np.repeat(p.sum(axis=-1).astype(np.float64).reshape(1, -1), m, axis=0)
        for f in ("gemm_tiled",) + (("gemm_mfma_m128",) if bits <= 4 and group >= 64 else ()):
            say("wide near ties", bits, group, f, m)
            y = cq.cq_gemm_a8_family(w, x8_t, dx_t, f, y_dtype=torch_dev.float32).cpu().numpy().astype(np.float64)
            assert np.array_equal(y, want), f


# Groups that are no power of two, which the conservative kernels take at every
# row count on both paths (K: an odd number of 64-code steps at 96 and 160).
@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("group,k", [(96, 1152), (160, 1280), (480, 1920)])
@pytest.mark.parametrize("m", [1, 8, 40, 130])
def test_other_groups(torch_dev, bits, group, k, m):
    import paper_2608_06763_amd as cq
    from oracle import a8 as A8
    n = 131
    w, codes, scale, a, b = random_weight(990 + bits, n, k, bits, group)
    wd = F.decode(codes, bits, group, scale, a, b)
    for dtype in ("bf16", "fp16"):
        xb, xv = act(991 + m, m, k, dtype)
        x = torch_dev.from_numpy(xb.view(np.int16)).cuda().view(
            torch_dev.bfloat16 if dtype == "bf16" else torch_dev.float16)
        say("other groups", bits, group, k, m, dtype)
        y = cq.cq_gemm_model_dtype(w, x, y_dtype=torch_dev.float32)
        bound = whole_bound(xv, wd) if m <= 16 else model_dtype_bound(xv, wd, dtype)
        assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - xv @ wd.T) <= bound)
    xb, xv = act(992 + m, m, k)
    x8_np, dx_np = A8.quantize_act(xv)
    x8, dx = torch_dev.from_numpy(x8_np).cuda(), torch_dev.from_numpy(dx_np.astype(np.float32)).cuda()
    ref, parts = A8.gemm_a8(x8_np, dx_np, codes, bits, group, scale, a, b)
    say("other groups a8", bits, group, k, m)
    y = cq.cq_gemm_a8(w, x8, dx, y_dtype=torch_dev.float32)
    assert np.max(np.abs(y.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
    tab = cq.cq_build_carriers(w)
    assert torch_dev.equal(cq.cq_gemm_a8_carriers(w, tab, x8, dx, y_dtype=torch_dev.float32), y)
    y, p = cq.cq_gemm_a8(w, x8, dx, y_dtype=torch_dev.float32, want_partials=True)
    assert np.array_equal(p.cpu().numpy(), parts)
    assert np.max(np.abs(y.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
