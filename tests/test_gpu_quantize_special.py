"""Quantisers on NaN, infinity, rounding ties and the ends of the reachable range of exponents, bit for bit against the
decisions of the formats written out in fp32 below (the oracle's conversion is defined for finite values only).

Maxima and minima skip a NaN (fmaxf, fminf), and it converts to +-6; a block of 32 that is NaN throughout - a group of
NaN, or any group whose pair table breaks Def. 1 - must not turn into plausible numbers: it gets the largest scale,
2^126, so that a linear on it overflows."""
import numpy as np
import pytest

import oracle
import paro_inputs as pin

pytestmark = pytest.mark.gpu
f32 = np.float32


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2511_10645_amd as paro
    return paro


def mxfp4_definition(v):
    """fp32 rows -> codes (magnitude and sign of a NaN's code as of its bits), scale bytes."""
    v = v.astype(f32)
    rows, c = v.shape
    amax = np.fmax.reduce(np.abs(v).reshape(rows, c // 32, 32), axis=2)
    e = np.maximum((amax.view(np.uint32) >> 23).astype(np.int32) - 127 - 2, -127)
    with np.errstate(all="ignore"):
        r = np.ldexp(v.reshape(rows, c // 32, 32).astype(np.float64), -e[:, :, None]).reshape(rows, c)
    a = np.abs(r)
    code = np.full(v.shape, 7, dtype=np.uint8)            # saturated, and what no comparison below is true for: NaN
    for k, top in ((6, a <= 5.0), (5, a < 3.5), (4, a <= 2.5), (3, a < 1.75), (2, a <= 1.25), (1, a < 0.75), (0, a <= 0.25)):
        code[top] = k
    return code | (np.signbit(v).astype(np.uint8) << 3), (e + 127).astype(np.uint8)


def int4_definition(v):
    """fp32 rows -> codes [R][C], scales fp16 [R][G], zero points [R][G] (Eq. 1)."""
    v = v.astype(f32)
    rows, c = v.shape
    g = v.reshape(rows, c // 128, 128)
    with np.errstate(all="ignore"):
        mn, mx = np.fmin.reduce(g, axis=2), np.fmax.reduce(g, axis=2)
        s = ((mx - mn) / f32(15)).astype(f32)
        s16 = np.where(s >= f32(2.0 ** -14), s, f32(2.0 ** -14)).astype(np.float16)
        s = s16.astype(f32)
        z = np.fmin(np.fmax(-np.rint((mn / s).astype(f32)), f32(0)), f32(15))
        q = np.fmin(np.fmax(np.rint((g / s[:, :, None]).astype(f32)) + z[:, :, None], f32(0)), f32(15))
    return q.reshape(rows, c).astype(np.uint8), s16, z.astype(np.uint8)


def _nibbles(words):
    w = words.cpu().numpy().view(np.uint32)
    return ((w[:, :, None] >> np.arange(0, 32, 4, dtype=np.uint32)) & 15).astype(np.uint8).reshape(w.shape[0], -1)


def _empty_rotation(P, c_in, scale, n_layers):
    """A transform whose layers name no channel (i == j): x' = scale * x, exactly, for powers of two."""
    pairs = np.zeros((c_in // 128, n_layers, 64, 2), dtype=np.int16)
    rot = P.Rotation(pairs, np.zeros(pairs.shape[:3], dtype=np.float32), scale)
    P.paro_rotation_plan_build(rot)
    return rot


def special_rows():
    """8 rows x 256 channels of fp16, each block of 32 a case of its own."""
    rng = np.random.default_rng(11)
    x = rng.standard_normal((8, 256)).astype(np.float16)
    x[0, :32] = np.nan                                     # a block of NaN
    x[0, 32:64] = np.array([np.nan, -np.nan] * 16, dtype=np.float16)
    x[0, 64] = np.nan                                      # one among numbers
    x[0, 100], x[0, 101] = np.inf, np.nan
    x[1, 3] = np.inf
    x[1, 40] = -np.inf
    x[1, 70:72] = [np.inf, -np.inf]
    x[1, 128:256] = np.inf                                 # a group of infinities
    x[2, :128] = np.nan                                    # a group of NaN
    x[2, 128:160], x[2, 160:192] = 0.0, -0.0
    x[3, :128] = 65504.0                                   # a constant group
    x[3, 128:256] = np.where(np.arange(128) % 2, 65504.0, -65504.0)
    x[4, :] = np.float16(2.0 ** -24) * rng.integers(-8, 9, 256).astype(np.float16)      # subnormals
    ties = np.array([.25, .75, 1.25, 1.75, 2.5, 3.5, 5.0, 6.0, 7.0, .5, 0.0, 4.0])
    for b in range(24):                                    # ties and their neighbours in rows 5..7, exponents -17..12
        t = np.resize(np.concatenate([ties, -ties]), 32).astype(np.float16)
        t = np.where(np.arange(32) < 24, t, np.nextafter(np.roll(t, 5), np.float16(0 if b % 2 else 100)))
        t[11] = 4.0
        x[5 + b // 8, (b % 8) * 32:(b % 8) * 32 + 32] = np.ldexp(t, int(np.linspace(-17, 12, 24)[b]))
    return x


def _same(got, want, v):
    assert np.array_equal(got, want), [(tuple(i), v[tuple(i)], int(got[tuple(i)]), int(want[tuple(i)])) for i in np.argwhere(got != want)[:8]]


def test_mxfp4_weights_without_transform(P):
    import torch
    print("special values, MXFP4 weight side", flush=True)
    x = special_rows()
    codes, scales = mxfp4_definition(x)
    q = P.paro_mxfp4_quantize_weight(None, torch.as_tensor(x).cuda())
    assert np.array_equal(q.scales.cpu().numpy(), scales)
    _same(_nibbles(q.codes), codes, x)
    assert scales[0, 0] == 253 and (codes[0, :32] & 7 == 7).all()


def _activations(P, n_layers, exponent):
    """fp16 times a power of two, 2^-38 to 2^31; the transform, the values behind it and the inputs."""
    x = special_rows()
    rot = _empty_rotation(P, 256, np.full(256, 2.0 ** exponent, dtype=np.float16), n_layers)
    if n_layers:                                           # an empty slot turns by cos 0 and sin 0: 0 * inf is NaN, so no infinities
        x = np.where(np.isinf(x), np.float16(60000.0), x)
        x[np.isnan(x).reshape(8, 2, 128).any(axis=2).repeat(128, axis=1)] = np.nan      # and a NaN stays in its pair: whole groups
    return rot, x.astype(f32) * f32(2.0 ** exponent), x


@pytest.mark.parametrize("n_layers", [0, 1, 8])
@pytest.mark.parametrize("exponent", [-14, 0, 15])
def test_mxfp4_activations(P, n_layers, exponent):
    import torch
    print(f"special values, MXFP4 activations, layers={n_layers} scale=2^{exponent}", flush=True)
    rot, v, x = _activations(P, n_layers, exponent)
    codes, scales = mxfp4_definition(v)
    gc, gs = P.paro_rotate_scale_quantize_mxfp4(rot, torch.as_tensor(x).cuda())
    assert np.array_equal(gs.cpu().numpy(), scales)
    got, unsigned = _nibbles(gc), np.isnan(v) | (v == 0)   # the sign of a zero or a NaN is not kept by the sums of a layer
    _same(np.where(unsigned, got & 7, got), np.where(unsigned, codes & 7, codes), v)


@pytest.mark.parametrize("T,bad", [(3, "activation"), (70, "activation"), (5, "pairs")])
def test_nan_stays_visible_behind_the_mxfp4_linear(P, T, bad):
    import torch
    print(f"NaN through the MXFP4 linear T={T} {bad}", flush=True)
    li = pin.make_custom(6400 + T, T, 1024, 64)
    pairs, x = li.pairs.copy(), li.x.copy()
    if bad == "pairs":
        pairs[2, 3, 5, 1] = pairs[2, 3, 6, 0]              # a channel in two pairs of a layer: the group has no defined transform
    else:
        x[1, 256:384] = np.nan
    rot = P.Rotation(pairs, li.theta, li.ch_scale)
    P.paro_rotation_plan_build(rot)
    dense = np.abs(pin.make_dense_weight(6500, 64, 1024))  # one sign: the overflowing products cannot cancel
    w = P.paro_mxfp4_quantize_weight(None, torch.as_tensor(dense).cuda())
    P.paro_mxfp4_repack(w)
    ws = torch.empty(P.paro_workspace_bytes_mxfp4(1024, T), dtype=torch.uint8, device="cuda")
    y = P.paro_rotated_linear_mxfp4(rot, w, torch.as_tensor(x).cuda(), ws).cpu().numpy().astype(np.float64)
    hit = np.ones(T, dtype=bool) if bad == "pairs" else np.arange(T) == 1
    lost, spread = int(np.isfinite(y[hit]).sum()), int((~np.isfinite(y[~hit])).sum())
    assert lost == 0 and spread == 0


def test_int4_weights_without_transform(P):
    import torch
    print("special values, INT4 weight side", flush=True)
    x = special_rows()
    codes, scales, zeros = int4_definition(x)
    q = P.paro_w4_quantize(None, torch.as_tensor(x).cuda())
    assert np.array_equal(q.scales.cpu().numpy().view(np.uint16), scales.T.view(np.uint16))
    assert np.array_equal(oracle.unpack_zeros(q.qzeros.cpu().numpy().view(np.uint32)), zeros.T)
    _same(_nibbles(q.qweight), codes, x)


@pytest.mark.parametrize("n_layers", [0, 1, 8])
@pytest.mark.parametrize("exponent", [-14, 0, 15])
def test_int4_activations(P, n_layers, exponent):
    """At 2^15 there are ranges above 15 * 65504, whose stored scale is infinite."""
    import torch
    print(f"special values, INT4 activations, layers={n_layers} scale=2^{exponent}", flush=True)
    rot, v, x = _activations(P, n_layers, exponent)
    codes, scales, zeros = int4_definition(v)
    assert exponent < 15 or (np.isinf(scales) & np.isfinite(v).reshape(8, 2, 128).all(axis=2)).any()
    gc, gs, gz = P.paro_rotate_scale_quantize_int4(rot, torch.as_tensor(x).cuda())
    assert np.array_equal(gs.cpu().numpy().view(np.uint16), scales.view(np.uint16)) and np.array_equal(gz.cpu().numpy(), zeros)
    _same(_nibbles(gc), codes, v)
