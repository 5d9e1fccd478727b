"""Weight-side quantisers on large weights: numbers of rows that no run or tile divides, few and many layers, both scale orders, special
values, and a row's independence of the others."""
import numpy as np
import pytest

import oracle
import paro_inputs as pin
from test_gpu_quantize_special import _nibbles, int4_definition, mxfp4_definition

pytestmark = pytest.mark.gpu
f32 = np.float32


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2511_10645_amd as paro
    return paro


def _rot(P, pairs, theta, scale, order=0):
    rot = P.Rotation(pairs, theta, scale, scale_order=order)
    P.paro_rotation_plan_build(rot)
    return rot


@pytest.mark.parametrize("N,C,n_layers,order", [(240008, 128, 8, 0), (26680, 1152, 1, 1), (2144, 14464, 5, 0), (1120, 27648, 8, 1)])
def test_transformed_rows(P, N, C, n_layers, order):
    """Codes and scales against the fp64 transform: fp32 sums move a value by less than 2^-18 of its group's norm (the bound of
    the other quantiser tests), so a code is within half a step plus that, and few differ at all."""
    import torch
    print(f"weight quantiser N={N} C={C} layers={n_layers} order={order}", flush=True)
    li = pin.make_custom(6600 + n_layers, 1, C, 16, n_layers=n_layers)
    wide = torch.zeros((N, C + 6), dtype=torch.float16, device="cuda")                # rows that are only 4-byte aligned
    wide[:, 2:C + 2] = 0.02 * torch.randn((N, C), generator=torch.Generator(device="cuda").manual_seed(N), device="cuda").half()
    W = wide[:, 2:C + 2]
    W[:, 5::311] *= 20
    rot = _rot(P, li.pairs, li.theta, li.ch_scale, order)
    q, mx = P.paro_w4_quantize(rot, W), P.paro_mxfp4_quantize_weight(rot, W)
    n = min(N, 40 + 400000 // C)                           # rows looked at: both ends
    rows = np.r_[0:n, N - n:N]
    at = torch.as_tensor(rows).cuda()
    v = oracle.weight_transform(W[at].cpu().numpy(), li.pairs, li.theta, li.ch_scale, scale_order=order).reshape(len(rows), C // 128, 128)
    norm = np.linalg.norm(v, axis=2, keepdims=True)
    s = q.scales[:, at].cpu().numpy().T.astype(np.float64)[:, :, None]
    z = oracle.unpack_zeros(q.qzeros.cpu().numpy().view(np.uint32)).T[rows].astype(np.float64)[:, :, None]
    s_def = np.maximum((v.max(axis=2) - v.min(axis=2)) / 15, 2.0 ** -14)[:, :, None]
    assert (np.abs(s - s_def) <= 2.0 ** -11 * s_def * 1.001 + 2.0 ** -18 * norm / 7).all()
    code = _nibbles(q.qweight[at]).reshape(v.shape).astype(np.float64)
    tol = 0.5 + 2.0 ** -18 * norm / s + 2.0 ** -18
    assert (np.abs(z - np.clip(-v.min(axis=2, keepdims=True) / s, 0, 15)) <= tol).all()
    assert (np.abs(code - np.clip(v / s + z, 0, 15)) <= tol).all()
    assert (code != np.clip(np.rint(v / s) + z, 0, 15)).mean() < 1e-4
    codes, scales = mxfp4_definition(v.reshape(len(rows), C).astype(f32))
    assert (mx.scales[at].cpu().numpy() != scales).mean() < 1e-4 and (_nibbles(mx.codes[at]) & 7 != codes & 7).mean() < 1e-4


def _tiled(a, rows, cols):
    return np.tile(a, (rows, cols))


@pytest.mark.parametrize("span", [10, 11, 29])
@pytest.mark.parametrize("order", [0, 1])
def test_a_nan_stays_in_its_pair(P, span, order):
    """Layers that name no channel and factors that are powers of two, up to 2^29 apart: exact; a NaN stays in its filler pair and must not
    reach the other channels or rows."""
    import torch
    print(f"weight quantiser, NaN in a pair, factors 2^{span} apart, order={order}", flush=True)
    R, G = 16, 108                                         # the pattern of 72 rows x 256 channels, repeated
    rng = np.random.default_rng(span)
    W = rng.integers(-60, 61, (72, 256)).astype(np.float16)
    W[3, 37], W[40, 200], W[71, 128:256] = np.nan, np.nan, np.nan
    e = rng.integers(-14, -14 + span + 1, 256)
    e[[0, 1]] = -14, -14 + span
    scale = np.ldexp(1.0, e).astype(np.float16)
    pairs = np.zeros((2 * G, 8, 64, 2), dtype=np.int16)
    rot = _rot(P, pairs, np.zeros(pairs.shape[:3], dtype=f32), np.tile(scale, G), order)
    v = W.astype(f32) / scale.astype(f32)
    for r, c in ((3, 37), (40, 200)):
        v[r, c // 2 * 2:c // 2 * 2 + 2] = np.nan
    d = torch.as_tensor(_tiled(W, R, G)).cuda()
    q, mx = P.paro_w4_quantize(rot, d), P.paro_mxfp4_quantize_weight(rot, d)
    codes, scales, zeros = int4_definition(v)
    assert np.array_equal(q.scales.cpu().numpy().view(np.uint16), _tiled(scales.T, G, R).view(np.uint16))
    assert np.array_equal(oracle.unpack_zeros(q.qzeros.cpu().numpy().view(np.uint32)), _tiled(zeros.T, G, R))
    assert np.array_equal(_nibbles(q.qweight), _tiled(codes, R, G))
    codes, scales = mxfp4_definition(v)
    unsigned = _tiled(np.isnan(v) | (v == 0), R, G)
    got, codes = _nibbles(mx.codes), _tiled(codes, R, G)
    assert np.array_equal(mx.scales.cpu().numpy(), _tiled(scales, R, G))
    assert np.array_equal(np.where(unsigned, got & 7, got), np.where(unsigned, codes & 7, codes))


def test_infinities_and_broken_tables(P):
    """A row with an infinity leaves the others as they are; a group whose table breaks Def. 1 is NaN on every row."""
    import torch
    print("weight quantiser, infinities, broken table", flush=True)
    li = pin.make_custom(6800, 1, 27648, 16)
    pairs = li.pairs.copy()
    pairs[1, 2, 5, 1] = pairs[1, 2, 6, 0]
    good, broken = _rot(P, li.pairs, li.theta, li.ch_scale), _rot(P, pairs, li.theta, li.ch_scale)
    W = torch.randn((1128, 27648), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda").half()
    bad = W.clone()
    bad[5, 17], bad[1034, 130] = float("inf"), float("-inf")
    others = torch.tensor([r for r in range(1128) if r not in (5, 1034)]).cuda()
    a, b = P.paro_w4_quantize(good, W), P.paro_w4_quantize(good, bad)
    c, d = P.paro_mxfp4_quantize_weight(good, W), P.paro_mxfp4_quantize_weight(good, bad)
    assert torch.equal(a.qweight[others], b.qweight[others]) and torch.equal(a.scales[:, others], b.scales[:, others])
    assert torch.equal(c.codes[others], d.codes[others]) and torch.equal(c.scales[others], d.scales[others])
    assert torch.equal(a.qweight[5, 16:], b.qweight[5, 16:])              # the row's other groups
    few = P.paro_w4_quantize(good, bad[:8].contiguous())
    assert torch.equal(b.qweight[5, :16], few.qweight[5, :16]) and torch.equal(b.scales[0, 5:6], few.scales[0, 5:6])
    m = P.paro_mxfp4_quantize_weight(broken, W)
    assert (m.scales[:, 4:8] == 253).all() and torch.equal(m.codes[:, :16], c.codes[:, :16])


def test_rows_without_a_transform(P):
    """Many rows equal the same rows few at a time (which go through the other kernel), special values among them."""
    import torch
    from test_gpu_quantize_special import special_rows
    print("weight quantiser, many rows without a transform", flush=True)
    W = torch.randn((12328, 256), generator=torch.Generator(device="cuda").manual_seed(4), device="cuda").half()
    W[4096:4104], W[12320:] = torch.as_tensor(special_rows()).cuda(), torch.as_tensor(special_rows()).cuda()
    whole = P.paro_w4_quantize(None, W)
    for r in range(0, 12328, 8 * 67):
        r = min(r, 12320)
        part = P.paro_w4_quantize(None, W[r:r + 8].contiguous())
        assert torch.equal(whole.qweight[r:r + 8], part.qweight) and torch.equal(whole.qzeros[:, r // 8:r // 8 + 1], part.qzeros)
        assert torch.equal(whole.scales[:, r:r + 8], part.scales)
    codes, scales, zeros = int4_definition(special_rows())
    for r in (4096, 12320):
        assert np.array_equal(_nibbles(whole.qweight[r:r + 8]), codes) and np.array_equal(whole.scales[:, r:r + 8].cpu().numpy().view(np.uint16), scales.T.view(np.uint16))


@pytest.mark.parametrize("n_layers,slots", [(8, 64), (1, 64), (8, 8), (1, 8)])
@pytest.mark.parametrize("order", [0, 1])
def test_a_row_does_not_depend_on_how_many_there_are(P, n_layers, slots, order):
    """A weight quantised whole and in shards of rows, as ranks of a parallel layer do it: the same bits, which also says that
    the whole is decided with the rounding errors of a shard."""
    import torch
    print(f"weight quantiser in shards, {n_layers} layers of {slots} pairs, order={order}", flush=True)
    li = pin.make_custom(6700 + n_layers, 1, 4096, 16, n_layers=n_layers, pairs_per_layer=slots)
    rot = _rot(P, li.pairs, li.theta, li.ch_scale, order)
    W = 0.02 * torch.randn((8192, 4096), generator=torch.Generator(device="cuda").manual_seed(slots), device="cuda")
    W = W.half()
    whole, mx = P.paro_w4_quantize(rot, W), P.paro_mxfp4_quantize_weight(rot, W)
    for lo in range(0, 8192, 1024):
        part, mpart = P.paro_w4_quantize(rot, W[lo:lo + 1024]), P.paro_mxfp4_quantize_weight(rot, W[lo:lo + 1024])
        assert torch.equal(whole.qweight[lo:lo + 1024], part.qweight) and torch.equal(whole.scales[:, lo:lo + 1024], part.scales)
        assert torch.equal(whole.qzeros[:, lo // 8:lo // 8 + 128], part.qzeros)
        assert torch.equal(mx.codes[lo:lo + 1024], mpart.codes) and torch.equal(mx.scales[lo:lo + 1024], mpart.scales)
