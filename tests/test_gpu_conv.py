"""GPU parity: lp_conv_fwd / lp_fc_fwd against the CPU oracle, bit for bit (int64 accumulators,
requantized codes, zero counts), through the C ABI."""
import numpy as np
import pytest

import lp_inputs
import paper_1711_04713_amd as lp
from gpu_helpers import conv, fc, quantize

pytestmark = pytest.mark.gpu

QX, QW, QY = (16, 4, 12), (16, 1, 15), (16, 5, 11)


def _codes(rng, shape, n=16, zero_frac=0.0, full_range=True):
    if full_range:
        c = rng.integers(-(1 << (n - 1)), 1 << (n - 1), shape)
    else:
        c = np.clip(np.round(rng.standard_normal(shape) * (1 << (n - 3))), -(1 << (n - 1)), (1 << (n - 1)) - 1)
    c = c.astype(np.int32)
    if zero_frac:
        c[rng.random(shape) < zero_frac] = 0
    return c


def _check(oracle, x, w, qx, qw, qy, relu=True, bias=None, qb=None, stride=1, pad=1, expect_path=None,
           modes=("away",)):
    f_acc = qx[2] + qw[2]
    want_acc = oracle.conv(x, w, bias=bias, f_acc=f_acc, fb=qb[2] if qb else 0, stride=stride, pad=pad, threads=8)
    for mode in modes:
        r_gpu = lp.LP_ROUND_NEAREST_AWAY if mode == "away" else lp.LP_ROUND_NEAREST_EVEN
        r_cpu = oracle.ROUND_AWAY if mode == "away" else oracle.ROUND_EVEN
        got = conv(x, qx, w, qw, qy=qy, relu=relu, r=r_gpu, bias=bias, qb=qb, stride=stride, pad=pad)
        if expect_path is not None:
            assert got["info"]["path"] == expect_path
        assert np.array_equal(got["acc"], want_acc)
        want_y, want_z, want_s = oracle.act(want_acc, f_acc, qy[0], qy[1], qy[2], relu, r_cpu, with_sat=True)
        assert np.array_equal(got["y"], want_y)
        assert (got["zeros"], got["sats"]) == (want_z, want_s)        # zero codes, clipped values
    return got


def test_config1_single_layer(oracle):
    """Batch 1, 16->16 channels, 16x16, 3x3 pad 1; w ~N(0, 0.1) in Q1.15, x = ReLU(N(0,1)) in Q8.8,
    output Q8.8 with ReLU and zero count; seed 0."""
    xf, wf = lp_inputs.config1(seed=0)
    qx, qw, qy = (16, 8, 8), (16, 1, 15), (16, 8, 8)
    x, _, _ = quantize(xf, qx)
    w, _, _ = quantize(wf, qw)
    assert np.array_equal(x, oracle.quantize(xf, *qx)[0]) and np.array_equal(w, oracle.quantize(wf, *qw)[0])
    got = _check(oracle, x, w, qx, qw, qy, expect_path=1, modes=("away", "even"))
    assert 0.3 < got["zeros"] / got["y"].size < 0.7


@pytest.mark.parametrize("N,Cin,H,W,Cout,R,S,pad", [
    (2, 64, 20, 24, 64, 3, 3, 1),      # several tiles, ragged right/bottom edges
    (1, 64, 33, 17, 128, 3, 3, 1),
    (70, 64, 32, 32, 128, 3, 3, 1),    # grid large enough for 128-wide channel tiles (BN = 128)
    (3, 32, 14, 14, 64, 3, 3, 1),      # row strips that straddle images; half-filled channel chunk
    (2, 128, 9, 9, 192, 3, 3, 1),      # two chunks, ragged channel tiles
    (2, 192, 7, 7, 40, 3, 3, 1),       # three chunks, Cout < 64
    (1, 16, 40, 40, 16, 3, 3, 1),
    (5, 64, 2, 2, 64, 3, 3, 1),        # tiny images, many boundaries per tile
    (2, 64, 12, 12, 64, 1, 1, 0),      # 1x1
    (1, 32, 16, 16, 32, 5, 5, 2),      # Table 1 kernel sizes
    (1, 16, 18, 18, 32, 7, 7, 3),
    (2, 64, 10, 10, 64, 3, 3, 0),      # no padding
    (1, 32, 9, 30, 32, 3, 5, 2),       # non-square kernel, padding wider than (R-1)/2 vertically
])
def test_conv_two_limb_shapes(oracle, N, Cin, H, W, Cout, R, S, pad):
    rng = np.random.default_rng(N * 131 + Cin + H)
    x = _codes(rng, (N, Cin, H, W), zero_frac=0.5)
    w = _codes(rng, (Cout, Cin, R, S))
    _check(oracle, x, w, QX, QW, (16, 12, 4), pad=pad, expect_path=1)


def _random_shapes(count, seed):
    """Seeded draw of small layer shapes the MFMA path accepts: every kernel size of Table 1, odd
    widths and heights (tile widths of every kind, patches of many pitches), 1..3 channel chunks,
    ragged channel tiles, with and without padding."""
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < count:
        R = int(rng.choice([1, 3, 3, 3, 5, 7]))
        S = R if rng.random() < 0.8 else int(rng.choice([1, 3, 5]))
        pad = int(rng.integers(0, (max(R, S) + 1) // 2 + 1))
        H, W = int(rng.integers(max(R - 2 * pad, 1), 40)), int(rng.integers(max(S - 2 * pad, 1), 40))
        if H + 2 * pad < R or W + 2 * pad < S:
            continue
        Cin = int(rng.choice([16, 24, 32, 64, 72, 128, 136, 192]))
        Cout = int(rng.choice([8, 16, 40, 64, 100, 128, 192]))
        N = int(rng.integers(1, 6))
        if N * H * W * Cin * R * S * Cout > 6e9:          # keep the oracle under a few seconds
            continue
        out.append((N, Cin, H, W, Cout, R, S, pad))
    return out


@pytest.mark.parametrize("N,Cin,H,W,Cout,R,S,pad", _random_shapes(24, 2024))
def test_conv_random_shapes_16bit(oracle, N, Cin, H, W, Cout, R, S, pad):
    rng = np.random.default_rng(N * 7 + Cin + 3 * H + W)
    x = _codes(rng, (N, Cin, H, W), zero_frac=0.4)
    w = _codes(rng, (Cout, Cin, R, S))
    _check(oracle, x, w, QX, QW, (16, 13, 3), pad=pad, expect_path=1)          # int64 epilogue and raw sums
    xs = np.maximum(_codes(rng, (N, Cin, H, W), full_range=False), 0)
    ws = _codes(rng, (Cout, Cin, R, S), full_range=False) >> 3
    got = conv(xs, QX, ws, QW, qy=(16, 4, 12), pad=pad, want_acc=False)         # fused 32-bit epilogue
    acc = oracle.conv(xs, ws, pad=pad, threads=8)
    y, z, sat = oracle.act(acc, 27, 16, 4, 12, True, oracle.ROUND_AWAY, with_sat=True)
    assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


@pytest.mark.parametrize("N,Cin,H,W,Cout,R,S,pad", _random_shapes(10, 77))
def test_conv_random_shapes_8bit(oracle, N, Cin, H, W, Cout, R, S, pad):
    if Cin % 16:
        Cin += 16 - Cin % 16
    rng = np.random.default_rng(N + Cin + H + W)
    x = np.maximum(_codes(rng, (N, Cin, H, W), n=8), 0)
    w = _codes(rng, (Cout, Cin, R, S), n=8)
    qx, qw, qy = (8, 3, 5), (8, 1, 7), (8, 5, 3)
    got = conv(x, qx, w, qw, qy=qy, pad=pad, want_acc=False)
    acc = oracle.conv(x, w, pad=pad, threads=8)
    y, z, sat = oracle.act(acc, 12, *qy, True, oracle.ROUND_AWAY, with_sat=True)
    assert got["info"]["path"] == 1 and got["info"]["limbs"] == 1
    assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


@pytest.mark.parametrize("N,Cin,H,W,Cout,pad,fx,fy", [
    (2, 64, 20, 24, 64, 1, 12, 4),       # shift 15
    (1, 136, 9, 11, 40, 0, 12, 12),      # shift 7; three chunks, the last an eighth full, ragged channels
    (3, 72, 14, 14, 128, 1, 8, 0),       # shift 15, images straddled by tiles
    (1, 904, 7, 7, 72, 1, 12, 2),        # K = 8136: just inside the 32-bit epilogue; shift 17
    (1, 920, 6, 7, 64, 1, 12, 3),        # K = 8280: just past it; shift 16
    (70, 64, 32, 32, 128, 1, 12, 6),     # more whole tiles than fit at once
    (37, 128, 28, 24, 256, 1, 12, 6),    # whole tiles, and a last round of 16 cut into eight parts each
])
def test_conv_16bit_activations_8bit_weights(oracle, N, Cin, H, W, Cout, pad, fx, fy):
    """One-limb weights under two-limb activations: every code of both widths with the extremes forced,
    raw sums, both tie rules, the fused epilogue of every shift class."""
    rng = np.random.default_rng(Cin + H)
    x = _codes(rng, (N, Cin, H, W), zero_frac=0.3)
    w = _codes(rng, (Cout, Cin, 3, 3), n=8)
    x[0], w[0], w[-1] = -32768, -128, 127           # the largest sums of either sign
    qx, qw, qy = (16, 16 - fx, fx), (8, 1, 7), (16, 16 - fy, fy)
    acc = oracle.conv(x, w, pad=pad, threads=8)
    got = conv(x, qx, w, qw, qy=qy, r=lp.LP_ROUND_NEAREST_EVEN, pad=pad)
    info = got["info"]
    assert info["path"] == 1 and info["bn"] == 64 and np.array_equal(got["acc"], acc)
    if N > 3:
        cut = 8 * (info["items_per_die"] - info["whole_items_per_die"])
        assert (info["split"], cut, info["workgroups"]) == {70: (1, 0, 1120), 37: (8, 16, 896)}[N]
    y, z, sat = oracle.act(acc, fx + 7, *qy, True, oracle.ROUND_EVEN, with_sat=True)
    assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)
    bias = _codes(rng, (Cout,), n=8)
    acc = acc + (bias.astype(np.int64) << (fx + 7 - 5)).reshape(1, -1, 1, 1)
    got = conv(x, qx, w, qw, qy=qy, bias=bias, qb=(8, 3, 5), pad=pad, want_acc=False)
    y, z, sat = oracle.act(acc, fx + 7, *qy, True, oracle.ROUND_AWAY, with_sat=True)
    assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


def test_conv_realistic_values_and_bias(oracle):
    rng = np.random.default_rng(5)
    x = np.maximum(_codes(rng, (2, 64, 18, 18), full_range=False), 0)
    w = _codes(rng, (64, 64, 3, 3), full_range=False)
    bias = _codes(rng, (64,))
    for relu in (True, False):
        _check(oracle, x, w, QX, QW, (16, 9, 7), relu=relu, bias=bias, qb=(16, 3, 13), modes=("away", "even"))
    _check(oracle, x, w, QX, QW, (16, 9, 7), bias=(bias >> 8), qb=(8, 2, 6))      # 8-bit bias codes


def test_conv_extreme_codes(oracle):
    """All-minimum and all-maximum codes: the largest limb sums and int64 results the path can see."""
    for xv, wv in ((-32768, -32768), (32767, -32768), (-32768, 32767), (32767, 32767)):
        x = np.full((1, 512, 6, 6), xv, np.int32)
        w = np.full((64, 512, 3, 3), wv, np.int32)
        got = _check(oracle, x, w, QX, QW, (16, 15, 1), relu=False)
        assert abs(int(got["acc"][0, 0, 2, 2])) == 9 * 512 * abs(xv) * abs(wv)


@pytest.mark.parametrize("N,Cin,H,W,Cout", [(2, 64, 14, 14, 64), (1, 128, 28, 28, 128), (3, 48, 10, 12, 80), (2, 256, 7, 7, 64)])
def test_conv_int8_single_limb(oracle, N, Cin, H, W, Cout):
    rng = np.random.default_rng(Cin + H)
    x = np.maximum(_codes(rng, (N, Cin, H, W), n=8), 0)
    w = _codes(rng, (Cout, Cin, 3, 3), n=8)
    _check(oracle, x, w, (8, 3, 5), (8, 1, 7), (8, 4, 4), expect_path=1, modes=("away", "even"))
    _check(oracle, -x - 1, w, (8, 3, 5), (8, 1, 7), (8, 6, 2), relu=False, expect_path=1)


def test_conv_mixed_widths_and_direct_path(oracle):
    rng = np.random.default_rng(9)
    x16, x8 = _codes(rng, (2, 32, 9, 9)), _codes(rng, (2, 32, 9, 9), n=8)
    w16, w8 = _codes(rng, (24, 32, 3, 3)), _codes(rng, (24, 32, 3, 3), n=8)
    _check(oracle, x16, w8, QX, (8, 1, 7), (16, 10, 6), expect_path=1)       # 8-bit weights on the two-limb kernel
    _check(oracle, x8, w16, (8, 3, 5), QW, (16, 10, 6), expect_path=0)       # direct kernel
    _check(oracle, x16, w16, QX, QW, QY, stride=2, expect_path=0)
    x12, w12 = _codes(rng, (1, 12, 8, 8)), _codes(rng, (16, 12, 3, 3))      # neither chunkable nor tiny
    _check(oracle, x12, w12, QX, QW, QY, expect_path=0)
    x3, w3 = _codes(rng, (2, 3, 10, 10), n=8), _codes(rng, (8, 3, 3, 3), n=8)
    _check(oracle, x3, w3, (8, 3, 5), (8, 1, 7), (8, 7, 1), expect_path=0)


@pytest.mark.parametrize("N,Cin,H,W,Cout,R,S,pad,qy", [
    (2, 3, 20, 20, 64, 3, 3, 1, (8, 7, 1)),       # first VGG16 layer shape, 8-bit output codes
    (1, 3, 37, 29, 64, 3, 3, 1, (16, 12, 4)),
    (2, 1, 18, 18, 16, 7, 7, 3, (16, 12, 4)),     # K = 49: two K=32 steps
    (3, 4, 9, 9, 40, 3, 3, 1, (16, 12, 4)),       # K = 36
    (2, 5, 6, 6, 130, 1, 1, 0, (16, 12, 4)),      # K = 5
    (2, 7, 8, 8, 64, 3, 3, 0, (16, 12, 4)),       # K = 63
    (9, 3, 2, 2, 64, 3, 3, 1, (16, 12, 4)),       # tiles straddling many images
])
def test_conv_flat_window(oracle, N, Cin, H, W, Cout, R, S, pad, qy):
    """Tiny input-channel counts: the whole window is gathered as one slab (K <= 64)."""
    rng = np.random.default_rng(N + Cin * 10 + H)
    x, w = _codes(rng, (N, Cin, H, W), zero_frac=0.3), _codes(rng, (Cout, Cin, R, S))
    _check(oracle, x, w, QX, QW, qy, pad=pad, expect_path=1, modes=("away", "even"))
    _check(oracle, x, w, QX, QW, qy, relu=False, pad=pad, expect_path=1)


@pytest.mark.parametrize("N,Cin,H,W,Cout,R,S,pad", [
    (2, 16, 30, 30, 16, 7, 7, 1),      # Table 1, layer 2: 112 codes per window row, 4 pieces of which the last is half padding
    (1, 16, 20, 23, 32, 7, 7, 0),      # layer 3
    (3, 32, 12, 12, 64, 5, 5, 1),      # layer 4: both 32-channel blocks, 5 whole pieces per row
    (2, 48, 9, 11, 40, 3, 3, 1),       # 144 codes per row: 4.5 pieces; ragged second block
    (1, 16, 17, 9, 100, 1, 1, 0),      # 1x1: half a piece per row; two channel tiles
    (4, 32, 5, 5, 8, 3, 5, 2),         # non-square window, tiles straddling images, 8 channels
    (2, 16, 6, 40, 24, 5, 3, 2),       # three-piece rows, wide rows
    (1, 16, 12, 12, 16, 11, 11, 5),    # 44 pieces
])
def test_conv_window_row_kernel(oracle, N, Cin, H, W, Cout, R, S, pad):
    """16-bit codes with 16, 32 or 48 input channels: the reduction runs over window rows of a
    densely staged patch (positions past a row's S * Cin codes meet zero weight bytes)."""
    rng = np.random.default_rng(N * 17 + Cin + H * 3 + R)
    x, w = _codes(rng, (N, Cin, H, W), zero_frac=0.3), _codes(rng, (Cout, Cin, R, S))
    info = lp.lp_conv_plan_info(lp.ConvDesc(N, H, W, Cin, Cout, R, S, 1, pad), QX, QW)
    assert info["kernel"] == lp.LP_KERNEL_ROWS
    _check(oracle, x, w, QX, QW, (16, 12, 4), pad=pad, expect_path=1, modes=("away", "even"))
    _check(oracle, x, w, QX, QW, (8, 7, 1), relu=False, pad=pad, expect_path=1)
    # 8-bit weight codes with 16-bit inputs, bias, the 32-bit epilogue
    xs = np.maximum(_codes(rng, (N, Cin, H, W), full_range=False), 0)
    w8 = _codes(rng, (Cout, Cin, R, S), n=8)
    b = _codes(rng, (Cout,), n=16, full_range=False)
    got = conv(xs, QX, w8, (8, 1, 7), qy=(16, 6, 10), pad=pad, bias=b, qb=(16, 4, 12), want_acc=False)
    acc = oracle.conv(xs, w8, bias=b, f_acc=19, fb=12, pad=pad, threads=8)
    y, z, sat = oracle.act(acc, 19, 16, 6, 10, True, oracle.ROUND_AWAY, with_sat=True)
    assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


def test_conv_window_rows_too_large_for_lds_take_the_patch_kernel(oracle):
    """A 13x13 window over 48 channels: the dense patch of the window-row kernel would not leave
    room for three workgroups per CU; the planner keeps the patch kernel, same results."""
    N, Cin, H, W, Cout, R, S, pad = 1, 48, 40, 6, 32, 13, 13, 6
    info = lp.lp_conv_plan_info(lp.ConvDesc(N, H, W, Cin, Cout, R, S, 1, pad), QX, QW)
    assert info["kernel"] == lp.LP_KERNEL_PATCH
    rng = np.random.default_rng(99)
    x, w = _codes(rng, (N, Cin, H, W), zero_frac=0.3), _codes(rng, (Cout, Cin, R, S))
    _check(oracle, x, w, QX, QW, (16, 14, 2), pad=pad, expect_path=1)


@pytest.mark.parametrize("fo", [15, 14, 11, 10, 3, 0])
def test_conv_requantization_shift_sweep(oracle, fo):
    """Output formats that put the right shift f_acc - fo at 12, 13, 16, 17, 24 and 27 bits, with
    values scaled so that results spread over zero, mid-range and saturated codes."""
    rng = np.random.default_rng(40 + fo)
    f_acc = 27
    s = f_acc - fo
    x = np.maximum(_codes(rng, (2, 64, 12, 12), full_range=False), 0)
    w = (_codes(rng, (64, 64, 3, 3), full_range=False).astype(np.float64) * 2.0 ** min(0, s - 24)).astype(np.int32)
    bias = _codes(rng, (64,), n=12)
    for q16 in ((16, 16 - fo, fo), (8, 8 - fo, fo) if fo <= 7 else None):
        if q16 is None:
            continue
        _check(oracle, x, w, QX, QW, q16, bias=bias, qb=(16, 4, 12), expect_path=1)
        got = conv(x, QX, w, QW, qy=q16, bias=bias, qb=(16, 4, 12), want_acc=False)       # 32-bit epilogue
        acc = oracle.conv(x, w, bias=bias, f_acc=f_acc, fb=12)
        y, z, sat = oracle.act(acc, f_acc, *q16, True, oracle.ROUND_AWAY, with_sat=True)
        assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)
        assert 0 < z < y.size


@pytest.mark.parametrize("fo", [12, 11, 10, 7, 5, 4, 3])
def test_conv_requantization_short_form_boundaries(oracle, fo):
    """Right shifts 8, 9, 10, 13, 15, 16 and 17 (f_acc = 20): the edges of the range in which the
    fused epilogue uses its shorter 32-bit form, with codes on every side of the rounding
    boundaries, and with outputs whose top limb sum is far beyond what that form keeps (all-maximum
    and all-minimum weights against an all-maximum image: saturated and zero codes)."""
    rng = np.random.default_rng(70 + fo)
    qx, qw = (16, 8, 8), (16, 4, 12)
    f_acc = 20
    x = np.maximum(_codes(rng, (2, 64, 10, 12), full_range=False), 0)
    x[0] = 32767
    w = _codes(rng, (64, 64, 3, 3), full_range=False) >> 6
    w[0], w[1], w[2] = 32767, -32768, 1
    w[3] = 0
    w[3, 0, 1, 1] = 1 << (f_acc - fo - 1) if f_acc - fo - 1 < 15 else 1    # products that land on exact halves
    bias = _codes(rng, (64,), n=12)
    qy = (16, 16 - fo, fo)
    _check(oracle, x, w, qx, qw, qy, bias=bias, qb=(16, 8, 8), expect_path=1)
    got = conv(x, qx, w, qw, qy=qy, bias=bias, qb=(16, 8, 8), want_acc=False)          # 32-bit epilogue
    acc = oracle.conv(x, w, bias=bias, f_acc=f_acc, fb=8)
    y, z, sat = oracle.act(acc, f_acc, *qy, True, oracle.ROUND_AWAY, with_sat=True)
    assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)
    assert (y[0, 0] == 32767).all() and (y[0, 1] == 0).all() and 0 < z < y.size and sat >= y[0, 0].size


def test_conv_int8_wide_tiles(oracle):
    rng = np.random.default_rng(12)
    x = np.maximum(_codes(rng, (66, 64, 32, 32), n=8), 0)
    w = _codes(rng, (128, 64, 3, 3), n=8)
    got = conv(x, (8, 3, 5), w, (8, 1, 7), qy=(8, 5, 3), want_acc=False)
    assert got["info"]["bn"] == 128 and got["info"]["limbs"] == 1
    acc = oracle.conv(x, w, threads=16)
    y, z, sat = oracle.act(acc, 12, 8, 5, 3, True, oracle.ROUND_AWAY, with_sat=True)
    assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


def test_conv_only_codes_or_only_accumulators(oracle):
    rng = np.random.default_rng(10)
    x, w = _codes(rng, (1, 64, 8, 8)), _codes(rng, (64, 64, 3, 3))
    acc = oracle.conv(x, w)
    got = conv(x, QX, w, QW, qy=None, want_y=False)
    assert got["y"] is None and np.array_equal(got["acc"], acc) and got["zeros"] == 0
    got = conv(x, QX, w, QW, qy=QY, want_acc=False)
    y, z, sat = oracle.act(acc, 27, *QY, True, oracle.ROUND_AWAY, with_sat=True)
    assert got["acc"] is None and np.array_equal(got["y"], y) and got["zeros"] == z


def test_conv1_2_shaped_layer_small_batch(oracle):
    """The conv1_2-shaped workload (64->64, 3x3) on a 56x56 crop, formats from the dynamic range."""
    xf, wf = lp_inputs.config2(seed=1, batch=2, hw=56)
    mx, mw = oracle.range_float(xf, 16)[0], oracle.range_float(wf, 16)[0]
    qx, qw = (16, mx, 16 - mx), (16, mw, 16 - mw)
    x, w = oracle.quantize(xf, *qx)[0], oracle.quantize(wf, *qw)[0]
    acc = oracle.conv(x, w, threads=8)
    mo = oracle.range_acc(acc, qx[2] + qw[2], True, 16)[0]
    _check(oracle, x, w, qx, qw, (16, mo, 16 - mo), expect_path=1)


# ------------------------------------------------------------------------------------ fc

@pytest.mark.parametrize("M,K,Nout", [(4, 64, 10), (130, 200, 70), (256, 1024, 1000), (3, 4096, 129), (1, 8, 1)])
def test_fc_matches_oracle(oracle, M, K, Nout):
    rng = np.random.default_rng(M + K)
    x, w = _codes(rng, (M, K), zero_frac=0.5), _codes(rng, (Nout, K))
    bias = _codes(rng, (Nout,))
    want = oracle.fc(x, w, bias=bias, f_acc=27, fb=15, threads=8)
    for relu in (True, False):
        got = fc(x, QX, w, QW, qy=(16, 14, 2), relu=relu, bias=bias, qb=(16, 1, 15))
        assert np.array_equal(got["acc"], want)
        y, z, sat = oracle.act(want, 27, 16, 14, 2, relu, oracle.ROUND_AWAY, with_sat=True)
        assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


def test_fc_extreme_k(oracle):
    """K = 25088 with every code at the minimum: 25088 * 2^30 per output, the widest sum of the FC path."""
    K = 25088
    x = np.full((2, K), -32768, np.int32)
    w = np.full((64, K), -32768, np.int32)
    w[1] = 32767
    got = fc(x, QX, w, QW, qy=(16, 16, 0), relu=False)
    assert np.array_equal(got["acc"], oracle.fc(x, w, threads=8))
    assert got["acc"][0, 0] == K * (1 << 30)


def test_fc_int8(oracle):
    rng = np.random.default_rng(3)
    x, w = _codes(rng, (40, 512), n=8), _codes(rng, (100, 512), n=8)
    want = oracle.fc(x, w)
    got = fc(x, (8, 3, 5), w, (8, 1, 7), qy=(8, 8, 0), relu=True)
    assert np.array_equal(got["acc"], want)
    y, z, sat = oracle.act(want, 12, 8, 8, 0, True, oracle.ROUND_AWAY, with_sat=True)
    assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


@pytest.mark.parametrize("M", [1, 2, 31, 32, 33, 63, 64, 65])
@pytest.mark.parametrize("K,Nout", [(16, 1), (31, 10), (33, 33), (500, 64), (1537, 97), (2049, 40)])
def test_fc_few_rows(oracle, M, K, Nout):
    """The few-rows kernel's edges: one and two 32-row blocks and the first size past them, rows that
    start off a 4-byte boundary (odd K), reductions shorter than one turn of the waves and ending inside
    a K half, ragged columns; 16-bit and 8-bit codes, both epilogues' options."""
    rng = np.random.default_rng(M * 10007 + K)
    for n, qx, qw, qy in ((16, QX, QW, (16, 14, 2)), (8, (8, 3, 5), (8, 1, 7), (8, 8, 0))):
        x, w, bias = _codes(rng, (M, K), n=n, zero_frac=0.5), _codes(rng, (Nout, K), n=n), _codes(rng, (Nout,), n=n)
        f_acc, qb = qx[2] + qw[2], (n, 1, n - 1)
        want = oracle.fc(x, w, bias=bias, f_acc=f_acc, fb=n - 1)
        for relu, r_gpu, r_cpu in ((True, lp.LP_ROUND_NEAREST_AWAY, oracle.ROUND_AWAY), (False, lp.LP_ROUND_NEAREST_EVEN, oracle.ROUND_EVEN)):
            got = fc(x, qx, w, qw, qy=qy, relu=relu, r=r_gpu, bias=bias, qb=qb)
            assert np.array_equal(got["acc"], want)
            y, z, sat = oracle.act(want, f_acc, *qy, relu, r_cpu, with_sat=True)
            assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


@pytest.mark.parametrize("M,K,Nout,few", [
    (40, 801, 520, True), (64, 1001, 4100, True), (64, 1002, 2080, True),   # two blocks, more than one turn of the waves
    (64, 2500, 33, False), (20, 9001, 40, False), (1, 25087, 70, True),     # either side of the line between the kernels
])
def test_fc_kernels_of_up_to_64_rows(oracle, M, K, Nout, few):
    rng = np.random.default_rng(M + K)
    for n, qx, qw, qy in ((16, QX, QW, (16, 14, 2)), (8, (8, 3, 5), (8, 1, 7), (8, 8, 0))):
        x, w = _codes(rng, (M, K), n=n, zero_frac=0.5), _codes(rng, (Nout, K), n=n)
        assert (lp.lp_fc_workspace_bytes(M, K, Nout, qx, qw) == 256) == few
        want = oracle.fc(x, w, threads=8)
        got = fc(x, qx, w, qw, qy=qy)
        assert np.array_equal(got["acc"], want)
        y, z, sat = oracle.act(want, qx[2] + qw[2], *qy, True, oracle.ROUND_AWAY, with_sat=True)
        assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


@pytest.mark.parametrize("M,K,Nout", [(100, 1030, 40), (300, 520, 384), (100, 1030, 768), (100, 1030, 832)])
def test_fc_parts_of_few_and_of_many_tiles(oracle, M, K, Nout):
    """Both forms of the kernel that adds up the parts of a tile: a workgroup per column block up to 12
    tiles, one for both from 13 on (the last row), ragged rows and columns."""
    rng = np.random.default_rng(M + Nout)
    for n, qx, qw, qy in ((16, QX, QW, (16, 14, 2)), (8, (8, 3, 5), (8, 1, 7), (8, 8, 0))):
        x, w = _codes(rng, (M, K), n=n, zero_frac=0.5), _codes(rng, (Nout, K), n=n)
        assert lp.lp_fc_workspace_bytes(M, K, Nout, qx, qw) > 2 * 256 * 64 * (8 if n == 16 else 4)   # room for parts
        want = oracle.fc(x, w, threads=8)
        got = fc(x, qx, w, qw, qy=qy)
        assert np.array_equal(got["acc"], want)
        y, z, sat = oracle.act(want, qx[2] + qw[2], *qy, True, oracle.ROUND_AWAY, with_sat=True)
        assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (z, sat)


def test_zero_count_needs_workspace_and_accumulates(oracle):
    import torch
    from gpu_helpers import to_dev

    rng = np.random.default_rng(11)
    x, w = _codes(rng, (1, 64, 8, 8), zero_frac=0.5), _codes(rng, (64, 64, 3, 3))
    d = lp.ConvDesc(1, 8, 8, 64, 64, 3, 3, 1, 1)
    xd = to_dev(x.transpose(0, 2, 3, 1).astype(np.int16))
    wd = to_dev(w.transpose(0, 2, 3, 1).astype(np.int16))
    packed = torch.empty(lp.lp_conv_packed_bytes(d, QX, QW), dtype=torch.uint8, device="cuda")
    lp.lp_conv_pack_weights(d, QX, QW, wd, packed)
    y = torch.empty((1, 8, 8, 64), dtype=torch.int16, device="cuda")
    z = torch.full((1,), 1000, dtype=torch.int64, device="cuda")
    with pytest.raises(lp.LpError) as e:
        lp.lp_conv_fwd(d, xd, QX, packed, QW, qy=QY, y_codes=y, zero_count=z)      # no workspace
    assert e.value.status == 3
    ws = torch.empty(lp.lp_conv_workspace_bytes(d, QX, QW), dtype=torch.uint8, device="cuda")
    for _ in range(2):                                                             # counters are added to
        lp.lp_conv_fwd(d, xd, QX, packed, QW, qy=QY, y_codes=y, zero_count=z, workspace=ws)
    torch.cuda.synchronize()
    _, want = oracle.act(oracle.conv(x, w), 27, *QY, True, oracle.ROUND_AWAY)
    assert int(z.item()) == 1000 + 2 * want


@pytest.mark.parametrize("shape", [(2, 12, 12, 256, 64), (1, 20, 16, 128, 192), (3, 8, 8, 192, 64)])
def test_split_reduction_matches_single_workgroup_tiles(oracle, shape):
    """With a workspace the tail tiles are cut along the reduction and merged by the finishing
    kernel; without one every tile is reduced by a single workgroup.  Both must give the
    oracle's codes, zero count (where counted) and raw accumulators."""
    import torch
    from gpu_helpers import to_dev

    N, H, W, Cin, Cout = shape
    rng = np.random.default_rng(17)
    x, w = _codes(rng, (N, Cin, H, W), zero_frac=0.4), _codes(rng, (Cout, Cin, 3, 3))
    d = lp.ConvDesc(N, H, W, Cin, Cout, 3, 3, 1, 1)
    assert lp.lp_conv_plan_info(d, QX, QW)["split"] > 1
    xd = to_dev(x.transpose(0, 2, 3, 1).astype(np.int16))
    wd = to_dev(w.transpose(0, 2, 3, 1).astype(np.int16))
    packed = torch.empty(lp.lp_conv_packed_bytes(d, QX, QW), dtype=torch.uint8, device="cuda")
    lp.lp_conv_pack_weights(d, QX, QW, wd, packed)
    want_acc = oracle.conv(x, w)
    want_y, want_z, want_s = oracle.act(want_acc, 27, *QY, True, oracle.ROUND_AWAY, with_sat=True)
    for use_ws in (False, True):
        ws = torch.full((lp.lp_conv_workspace_bytes(d, QX, QW),), 0x5A, dtype=torch.uint8, device="cuda") if use_ws else None
        y = torch.full((N, H, W, Cout), -7, dtype=torch.int16, device="cuda")
        acc = torch.full((N, H, W, Cout), -7, dtype=torch.int64, device="cuda")
        z = torch.zeros(1, dtype=torch.int64, device="cuda") if use_ws else None
        sc = torch.zeros(1, dtype=torch.int64, device="cuda") if use_ws else None
        lp.lp_conv_fwd(d, xd, QX, packed, QW, qy=QY, y_codes=y, zero_count=z, workspace=ws, sat_count=sc)   # fast epilogue
        lp.lp_conv_fwd(d, xd, QX, packed, QW, acc_out=acc, workspace=ws)                            # raw accumulators
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().transpose(0, 3, 1, 2), want_y)
        assert np.array_equal(acc.cpu().numpy().transpose(0, 3, 1, 2), want_acc)
        if use_ws:
            assert int(z.item()) == want_z and int(sc.item()) == want_s and want_s > 0


@pytest.mark.parametrize("shape", [(2, 16, 16, 64, 64), (3, 16, 24, 32, 40), (1, 8, 32, 16, 128), (5, 4, 4, 64, 64)])
def test_fused_maxpool_matches_conv_act_pool(oracle, shape):
    """d.pool = 1: the stored codes are the 2x2 maxima of LPAct(conv) and the zero count is
    that of the unpooled codes, as if lp_maxpool2x2 had followed."""
    import torch
    from gpu_helpers import to_dev

    N, H, W, Cin, Cout = shape
    rng = np.random.default_rng(23)
    x, w = _codes(rng, (N, Cin, H, W), zero_frac=0.4), _codes(rng, (Cout, Cin, 3, 3))
    d = lp.ConvDesc(N, H, W, Cin, Cout, 3, 3, 1, 1, 1)
    info = lp.lp_conv_plan_info(d, QX, QW)
    assert info["tile_rows"] % 2 == 0 and info["tile_cols"] in (2, 4, 8, 16)
    xd = to_dev(x.transpose(0, 2, 3, 1).astype(np.int16))
    wd = to_dev(w.transpose(0, 2, 3, 1).astype(np.int16))
    packed = torch.empty(lp.lp_conv_packed_bytes(d, QX, QW), dtype=torch.uint8, device="cuda")
    lp.lp_conv_pack_weights(d, QX, QW, wd, packed)
    ws = torch.full((lp.lp_conv_workspace_bytes(d, QX, QW),), 0x3C, dtype=torch.uint8, device="cuda")
    y = torch.full((N, H // 2, W // 2, Cout), -7, dtype=torch.int16, device="cuda")
    z = torch.zeros(1, dtype=torch.int64, device="cuda")
    sc = torch.zeros(1, dtype=torch.int64, device="cuda")
    lp.lp_conv_fwd(d, xd, QX, packed, QW, qy=QY, y_codes=y, zero_count=z, workspace=ws, sat_count=sc)
    torch.cuda.synchronize()
    codes, zeros, sats = oracle.act(oracle.conv(x, w), 27, *QY, True, oracle.ROUND_AWAY, with_sat=True)
    assert np.array_equal(y.cpu().numpy().transpose(0, 3, 1, 2), oracle.maxpool2x2(codes))
    assert int(z.item()) == zeros and int(sc.item()) == sats and sats > 0      # both counted before pooling
    # the fused form has conditions: raw accumulators, no ReLU, 8-bit codes and odd sizes are refused
    acc = torch.empty((N, H, W, Cout), dtype=torch.int64, device="cuda")
    with pytest.raises(lp.LpError) as e:
        lp.lp_conv_fwd(d, xd, QX, packed, QW, acc_out=acc, workspace=ws)
    assert e.value.status == 2
    with pytest.raises(lp.LpError) as e:
        lp.lp_conv_fwd(d, xd, QX, packed, QW, qy=QY, y_codes=y, relu=False, workspace=ws)
    assert e.value.status == 2
    with pytest.raises(lp.LpError) as e:
        lp.lp_conv_plan_info(lp.ConvDesc(N, H + 1, W, Cin, Cout, 3, 3, 1, 1, 1), QX, QW)
    assert e.value.status == 2


FINISH_FORMS = [
    # (N, H, W, Cin, Cout, kernel, activation bits, weight bits; parts per cut tile, cut tiles, channels per tile)
    (1, 12, 10, 256, 64, 3, 16, 16, 8, 8, 64),       # few tiles: a workgroup per unit, all parts requested at once
    (1, 12, 10, 256, 72, 3, 16, 8, 8, 8, 64),        # one weight limb, ragged channels
    (1, 12, 10, 256, 64, 3, 8, 8, 8, 8, 64),         # one limb
    (2, 20, 20, 128, 16, 7, 16, 16, 8, 8, 64),       # the row sums of other windows than 3x3
    (20, 5, 5, 64, 40, 5, 16, 16, 7, 16, 64),
    (3, 9, 11, 1024, 24, 1, 16, 16, 8, 8, 64),
    (20, 5, 5, 64, 32, 5, 8, 8, 8, 8, 64),
    (55, 28, 28, 128, 384, 3, 8, 8, 8, 8, 128),      # 128-channel tiles, behind whole ones
    (1, 28, 28, 512, 512, 3, 16, 16, 4, 56, 64),     # four units side by side; parts of three wave groups
    (1, 28, 28, 512, 512, 3, 16, 8, 4, 56, 64),
    (7, 14, 14, 512, 512, 3, 16, 16, 5, 88, 64),     # five and seven parts: a second batch of requests
    (4, 28, 28, 192, 128, 3, 8, 8, 7, 56, 64),
    (46, 28, 28, 320, 512, 3, 8, 8, 4, 128, 128),    # the most tiles with two workgroups each
    (20, 28, 28, 512, 512, 3, 16, 16, 3, 240, 64),   # every tile in one workgroup, two trips
    (22, 14, 14, 512, 512, 3, 16, 8, 2, 280, 64),
    (32, 14, 14, 512, 512, 3, 8, 8, 2, 400, 64),
    (72, 28, 28, 512, 384, 3, 8, 8, 3, 304, 128),
]


@pytest.mark.parametrize("form", FINISH_FORMS)
def test_merged_parts_equal_whole_tiles(form):
    """Tiles cut along the reduction and merged by the finishing kernel give what one workgroup per tile
    gives (no workspace, the form the oracle tests cover): codes, accumulators; the counters
    equal counts of those codes."""
    import torch

    N, H, W, Cin, Cout, k, nx, nw, parts, cut, bn = form
    qx, qw, qy = (nx, 4, nx - 4), (nw, 1, nw - 1), (nx, 6, nx - 6)
    d = lp.ConvDesc(N, H, W, Cin, Cout, k, k, 1, k // 2)
    info = lp.lp_conv_plan_info(d, qx, qw)
    assert (info["path"], info["split"], info["bn"]) == (1, parts, bn)
    assert 8 * (info["items_per_die"] - info["whole_items_per_die"]) == cut
    gen = torch.Generator(device="cuda")
    gen.manual_seed(71)
    dt = torch.int16 if nx > 8 else torch.int8
    top = 1 << (nx - 1)
    x = torch.randint(-top, top, (N, H, W, Cin), device="cuda", generator=gen).to(dt)
    x[..., : Cin // 4] = top - 1                                                    # the row sums reach their largest
    w = torch.randint(-(1 << (nw - 1)), 1 << (nw - 1), (Cout, k, k, Cin), device="cuda", generator=gen).to(torch.int16 if nw > 8 else torch.int8)
    packed = torch.empty(lp.lp_conv_packed_bytes(d, qx, qw), dtype=torch.uint8, device="cuda")
    lp.lp_conv_pack_weights(d, qx, qw, w, packed)
    shape = (N, H, W, Cout)
    y0, y1, y2 = (torch.full(shape, -7, dtype=dt, device="cuda") for _ in range(3))
    acc0, acc1 = (torch.full(shape, -7, dtype=torch.int64, device="cuda") for _ in range(2))
    count = torch.full((4,), 1000, dtype=torch.int64, device="cuda")
    ws = torch.full((lp.lp_conv_workspace_bytes(d, qx, qw),), 0x5A, dtype=torch.uint8, device="cuda")
    lp.lp_conv_fwd(d, x, qx, packed, qw, qy=qy, y_codes=y0)
    lp.lp_conv_fwd(d, x, qx, packed, qw, acc_out=acc0)
    lp.lp_conv_fwd(d, x, qx, packed, qw, qy=qy, y_codes=y1, zero_count=count[0:1], sat_count=count[1:2], workspace=ws)
    lp.lp_conv_fwd(d, x, qx, packed, qw, qy=qy, y_codes=y2, acc_out=acc1, zero_count=count[2:3], sat_count=count[3:4], workspace=ws)
    assert torch.equal(y0, y1) and torch.equal(y0, y2) and torch.equal(acc0, acc1)
    zeros = int((y0 == 0).sum().item())
    s = qx[2] + qw[2] - qy[2]
    sats = int((((acc0.clamp(min=0) + (1 << (s - 1))) >> s) > top - 1).sum().item())
    assert count.tolist() == [1000 + zeros, 1000 + sats] * 2 and sats > 0


@pytest.mark.parametrize("shape,R,qx,qw,split", [
    ((3, 72, 17, 13, 200), 5, QX, QW, False),                    # 25 taps over three groups, a last chunk of 8 channels
    ((3, 72, 17, 13, 200), 5, QX, (8, 1, 7), False),             # one weight limb
    ((3, 80, 17, 13, 200), 5, (8, 4, 4), (8, 1, 7), False),      # one limb each
    ((24, 384, 7, 7, 132), 3, QX, QW, True),                     # tiles that straddle images, parts of whole chunks
    ((1, 448, 28, 28, 200), 3, QX, (8, 1, 7), True),
    ((19, 448, 14, 14, 256), 3, QX, QW, False),                  # 120 whole tiles
])
def test_three_wave_groups_per_workgroup(oracle, shape, R, qx, qw, split):
    """Grids of at most a tile per CU with a long reduction: three wave groups share a staged patch and add their
    sums up in LDS (seen by the LDS the exchange takes), whole or cut into parts of whole chunks."""
    N, Cin, H, W, Cout = shape
    info = lp.lp_conv_plan_info(lp.ConvDesc(N, H, W, Cin, Cout, R, R, 1, R // 2), qx, qw)
    assert info["lds_bytes"] > 65536 and (info["split"] > 1) == split
    rng = np.random.default_rng(N + Cin + R)
    x, w = _codes(rng, (N, Cin, H, W), n=qx[0], zero_frac=0.5), _codes(rng, (Cout, Cin, R, R), n=qw[0])
    _check(oracle, x, w, qx, qw, (16, 12, 4), pad=R // 2, expect_path=1)


@pytest.mark.parametrize("shape,k", [
    ((2, 9, 11, 64, 12), 3), ((2, 9, 11, 64, 20), 3), ((1, 13, 13, 32, 48), 3), ((3, 8, 8, 64, 100), 3),   # 64-wide channel tiles
    ((2, 9, 11, 16, 64), 5), ((1, 17, 19, 128, 200), 1),
    ((70, 32, 32, 16, 128), 1), ((70, 32, 32, 16, 120), 1), ((70, 31, 33, 16, 112), 1),                    # 128-wide ones
    ((1, 28, 28, 256, 512), 3), ((1, 28, 28, 256, 500), 3), ((1, 28, 28, 256, 498), 3),                    # three wave groups
])
@pytest.mark.parametrize("qx,qw,n", [((8, 4, 4), (8, 1, 7), 8), ((16, 4, 12), (16, 1, 15), 16), ((16, 4, 12), (8, 1, 7), 16), ((16, 4, 12), (16, 1, 15), 8)])
def test_codes_and_counts_of_the_short_epilogue(oracle, shape, k, qx, qw, n):
    """Codes alone (the 32-bit epilogue) with output formats that clip nothing, a few values and most of them; channel
    counts on both sides of what whole 16-byte pieces take."""
    N, H, W, Cin, Cout = shape
    rng = np.random.default_rng(N * 100 + Cout + k + n)
    x = np.maximum(_codes(rng, (N, Cin, H, W), qx[0], full_range=False), 0)
    w = _codes(rng, (Cout, Cin, k, k), qw[0], full_range=False)
    f_acc = qx[2] + qw[2]
    acc = oracle.conv(x, w, f_acc=f_acc, pad=k // 2, threads=8)
    top = int(acc.max()).bit_length() - f_acc + 1          # integer bits (with sign) that hold every value
    for m in (top, top - 2, top - 5):
        m = min(max(m, 1), n)
        qy = (n, m, n - m)
        if not 1 <= f_acc - qy[2] <= 31:
            continue
        got = conv(x, qx, w, qw, qy=qy, pad=k // 2, want_acc=False)
        assert (got["info"]["lds_bytes"] > 65536) == (Cin == 256)
        y, zeros, sats = oracle.act(acc, f_acc, *qy, True, oracle.ROUND_AWAY, with_sat=True)
        assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (zeros, sats)


def _flat_codes_launch(info, Cin, Cout, k, pool):
    """(the several-tiles kernel takes a call that wants 16-bit codes alone, workgroups it starts at most): the dispatch's rule."""
    K, tiles = k * k * Cin, info["tiles_m"]
    late = max(0, -(-info["patch_rows"] * info["patch_cols"] * Cin // 256) - 3)
    cap = 256 * (3 if Cout > 32 and K > 32 else 4)
    if Cout > 32:
        return tiles > 256 * (48 if late >= 5 and not pool else 6 if late >= 4 and not pool else 3 if K > 32 else 1.5), cap
    saved = 350 - 54 * late - 4 * K - (122 - 21 * -(-Cout // 8) if pool else 0)
    return tiles > 384 and saved * tiles > 1150 * 256, cap


def _spread_codes(rng, shape, zero_frac):
    """Codes of every magnitude, so that small and large shifts both leave values between zero and the clip."""
    return _codes(rng, shape, zero_frac=zero_frac) >> rng.integers(0, 13, shape).astype(np.int32)


@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("N,Cin,H,W,Cout,k,pad,n,pool", [
    (12, 3, 112, 113, 64, 3, 1, 16, 0),      # ragged tiles at the right edge
    (3, 3, 288, 192, 16, 1, 0, 16, 1),       # K = 3, half of the 32-channel block, pooled
    (3, 3, 256, 208, 64, 3, 1, 16, 1),       # both blocks, pooled
    (760, 3, 13, 13, 36, 3, 1, 16, 0),       # tiles straddle images; a group of four channels without its neighbour
    (17, 3, 100, 99, 32, 3, 1, 16, 0),       # one whole block
    (27, 7, 64, 64, 64, 3, 1, 16, 0),        # K = 63: two K = 32 halves; more of a patch than is under way at a time
    (11, 7, 96, 104, 40, 3, 1, 16, 1),       # the same pooled, ten of sixteen groups of channels
    (290, 1, 30, 30, 20, 7, 3, 12, 0),       # K = 49, one block, 12-bit codes
    (340, 2, 32, 32, 32, 5, 2, 16, 1),       # K = 50, pooled
    (3, 1, 47, 1100, 4, 1, 0, 16, 0),        # K = 1
    (1, 3, 224, 224, 64, 3, 1, 16, 0),       # one tile per workgroup
])
def test_flat_window_workgroups_of_several_tiles(oracle, N, Cin, H, W, Cout, k, pad, n, pool, plain):
    """Codes alone of more tiles than the launch has workgroups (but for the last case): shifts at both ends and in between, biases
    whose upper part is clamped, formats that clip, weights in both limb forms."""
    rng = np.random.default_rng(N + 10 * Cin + k)
    qw = (16, 1, 15)
    x, w = _spread_codes(rng, (N, Cin, H, W), 0.3), np.minimum(_spread_codes(rng, (Cout, Cin, k, k), 0.0), 32639)
    if plain:
        w[Cout // 2, 0, 0, 0] = 32767
    bias = _codes(rng, (Cout,))
    for qx, fb, fos in (((16, 8, 8), None, (14, 10, 6, 3)), ((16, 8, 8), 0, (14, 13, 9, 3)), ((16, 1, 15), 6, (15, 12, 10))):
        f = qx[2] + qw[2]                                          # 23 or 30; biases shifted by 23 or 24: up to 2^39
        b = None if fb is None else bias
        acc = oracle.conv(x, w, bias=b, f_acc=f, fb=fb or 0, pad=pad, threads=8)
        for fo in sorted({min(fo, n - 1) for fo in fos}):
            qy = (n, n - fo, fo)
            y, zeros, sats = oracle.act(acc, f, *qy, True, oracle.ROUND_AWAY, with_sat=True)
            got = conv(x, qx, w, qw, qy=qy, pad=pad, want_acc=False, bias=b, qb=None if fb is None else (16, 16 - fb, fb), pool=pool)
            taken, cap = _flat_codes_launch(got["info"], Cin, Cout, k, pool)
            assert got["info"]["kernel"] == lp.LP_KERNEL_FLAT and got["info"]["tiles_n"] == 1 and 9 <= f - fo <= 20 and taken
            assert (got["info"]["tiles_m"] > cap) == (N > 1)
            assert np.array_equal(got["y"], oracle.maxpool2x2(y) if pool else y)
            assert (got["zeros"], got["sats"]) == (zeros, sats)


@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("N,Cin,H,W,Cout,k", [(1, 3, 370, 370, 36, 3), (1, 7, 320, 320, 36, 3)])
def test_flat_window_shifts(oracle, N, Cin, H, W, Cout, k, plain):
    """Every shift the several-tiles kernel takes, 9 to 20 bits, and the two on each side of them, which run one tile per workgroup."""
    rng = np.random.default_rng(Cin)
    qx, qw = (16, 8, 8), (16, 1, 15)
    x, w = _spread_codes(rng, (N, Cin, H, W), 0.3), np.minimum(_spread_codes(rng, (Cout, Cin, k, k), 0.0), 32639)
    if plain:
        w[-1, 0, 0, 0] = 32640
    acc = oracle.conv(x, w, f_acc=23, pad=1, threads=8)
    for s in range(8, 23):
        fo = 23 - s
        y, zeros, sats = oracle.act(acc, 23, 16, 16 - fo, fo, True, oracle.ROUND_AWAY, with_sat=True)
        got = conv(x, qx, w, qw, qy=(16, 16 - fo, fo), want_acc=False)
        taken, cap = _flat_codes_launch(got["info"], Cin, Cout, k, 0)
        assert got["info"]["kernel"] == lp.LP_KERNEL_FLAT and taken and got["info"]["tiles_m"] > cap
        assert np.array_equal(got["y"], y), s
        assert (got["zeros"], got["sats"]) == (zeros, sats), s


@pytest.mark.parametrize("N,Cin,H,W,Cout,k,pool", [(1, 3, 224, 224, 32, 3, 0), (4, 7, 112, 112, 64, 3, 0), (16, 15, 56, 56, 32, 1, 1)])
def test_flat_window_layers_beside_the_line(oracle, N, Cin, H, W, Cout, k, pool):
    """Enough tiles for the several-tiles kernel with other channels or windows, not with these: one tile per workgroup."""
    rng = np.random.default_rng(Cout + Cin)
    x, w = _spread_codes(rng, (N, Cin, H, W), 0.3), _spread_codes(rng, (Cout, Cin, k, k), 0.0)
    acc = oracle.conv(x, w, f_acc=23, pad=k // 2, threads=8)
    y, zeros, sats = oracle.act(acc, 23, 16, 6, 10, True, oracle.ROUND_AWAY, with_sat=True)
    got = conv(x, (16, 8, 8), w, (16, 1, 15), qy=(16, 6, 10), pad=k // 2, want_acc=False, pool=pool)
    assert got["info"]["tiles_m"] > 384 and not _flat_codes_launch(got["info"], Cin, Cout, k, pool)[0]
    assert np.array_equal(got["y"], oracle.maxpool2x2(y) if pool else y) and (got["zeros"], got["sats"]) == (zeros, sats)


def _weights_of_both_forms(rng, shape, top):
    """Codes over the whole range of the signed limb form; top: the largest one, planted in the second tile of 64 channels (and
    in the only one of fewer), once."""
    w = rng.integers(-32768, 32640, shape).astype(np.int32)
    w.reshape(shape[0], -1)[min(shape[0] - 1, 70), -1] = top
    return w


@pytest.mark.parametrize("top", [32639, 32640, 32767])
@pytest.mark.parametrize("N,Cin,H,W,Cout,k", [
    (2, 64, 12, 11, 130, 3),       # patch kernel: three channel tiles, the second in the other form
    (1, 72, 9, 9, 40, 5),          # half-filled second chunk, window sums of 25 pixels
    (1, 256, 12, 10, 96, 3),       # parts of tiles
    (1, 512, 28, 28, 256, 3),      # three wave groups
    (2, 3, 20, 20, 72, 3),         # flat window
    (1, 3, 420, 420, 24, 3),       # flat window, several tiles per workgroup
    (2, 16, 17, 19, 80, 7),        # window rows
    (2, 48, 9, 9, 20, 3),
])
def test_weight_limb_forms(oracle, top, N, Cin, H, W, Cout, k):
    """The largest code whose low limb can be signed, the smallest that cannot, and the largest of all, beside the smallest code."""
    rng = np.random.default_rng(top + Cin + k)
    x = _codes(rng, (N, Cin, H, W), zero_frac=0.3)
    w = _weights_of_both_forms(rng, (Cout, Cin, k, k), top)
    acc = oracle.conv(x, w, pad=k // 2, threads=8)
    got = conv(x, QX, w, QW, pad=k // 2, want_y=False)
    assert np.array_equal(got["acc"], acc)
    for fo in (11, 9):
        qy = (16, 16 - fo, fo)
        y, zeros, sats = oracle.act(acc, 27, *qy, True, oracle.ROUND_AWAY, with_sat=True)
        got = conv(x, QX, w, QW, qy=qy, pad=k // 2, want_acc=False)
        assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (zeros, sats)


@pytest.mark.parametrize("top", [32639, 32640, 32767])
@pytest.mark.parametrize("N,Cin,H,W,Cout,k", [(2, 64, 16, 16, 136, 3), (1, 256, 16, 16, 96, 3), (2, 3, 32, 32, 72, 3), (2, 16, 32, 32, 80, 5)])
def test_weight_limb_forms_with_bias_and_pool(oracle, top, N, Cin, H, W, Cout, k):
    """The same codes beside a bias and through the fused pool, on the patch (whole tiles and parts), flat-window and window-row kernels."""
    rng = np.random.default_rng(top + Cin)
    x = _codes(rng, (N, Cin, H, W), zero_frac=0.3)
    w, bias, qb = _weights_of_both_forms(rng, (Cout, Cin, k, k), top), _codes(rng, (Cout,)), (16, 8, 8)
    acc = oracle.conv(x, w, bias=bias, f_acc=27, fb=8, pad=k // 2, threads=8)
    y, zeros, sats = oracle.act(acc, 27, 16, 6, 10, True, oracle.ROUND_AWAY, with_sat=True)
    for pool in (0, 1):
        got = conv(x, QX, w, QW, qy=(16, 6, 10), pad=k // 2, want_acc=False, bias=bias, qb=qb, pool=pool)
        assert np.array_equal(got["y"], oracle.maxpool2x2(y) if pool else y) and (got["zeros"], got["sats"]) == (zeros, sats)


@pytest.mark.parametrize("top", [32639, 32640, 32767])
@pytest.mark.parametrize("M,K,Nout", [(1, 1000, 130), (40, 333, 70), (64, 515, 100), (130, 700, 200), (300, 4100, 128)])
def test_fc_weight_limb_forms(oracle, top, M, K, Nout):
    rng = np.random.default_rng(top + M)
    x, w = _codes(rng, (M, K)), _weights_of_both_forms(rng, (Nout, K), top)
    got = fc(x, QX, w, QW)
    acc = x.astype(np.int64) @ w.astype(np.int64).T
    assert np.array_equal(got["acc"], acc)
    y, zeros, sats = oracle.act(acc, 27, *QY, True, oracle.ROUND_AWAY, with_sat=True)
    got = fc(x, QX, w, QW, qy=QY, want_acc=False)
    assert np.array_equal(got["y"], y) and (got["zeros"], got["sats"]) == (zeros, sats)
