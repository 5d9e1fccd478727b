"""The quantisers' runs of rows (four at a time, up to 32 per wave): a row's codes, scales and zero points must not depend on
how many rows are quantised with it or on its place in the batch, and must equal what the format's definition gives for the
same values (no rotation, so the values are the inputs)."""
import numpy as np
import pytest

import oracle
import paro_inputs as pin

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2511_10645_amd as paro
    return paro


def _rot(P, li, order=0):
    rot = P.Rotation(li.pairs, li.theta, li.ch_scale, scale_order=order)
    P.paro_rotation_plan_build(rot)
    return rot


@pytest.mark.parametrize("T", [1, 3, 4, 5, 31, 32, 33, 130])
@pytest.mark.parametrize("n_layers", [8, 3])
def test_activation_rows_do_not_depend_on_their_batch(P, T, n_layers):
    import torch
    print(f"quantise rows T={T} layers={n_layers}", flush=True)
    li = pin.make_custom(6100 + T, T, 640, 16, n_layers=n_layers, n_outlier=3)
    rot = _rot(P, li, order=T % 2)
    x = torch.as_tensor(li.x).cuda()
    wide = torch.zeros((T, 640 + 6), dtype=torch.float16, device="cuda")
    wide[:, 2:642] = x                                # rows that are only 4-byte aligned
    for fn in (P.paro_rotate_scale_quantize_int4, P.paro_rotate_scale_quantize_mxfp4):
        whole = fn(rot, x)
        strided = fn(rot, wide[:, 2:642])
        for a, b in zip(whole, strided):
            assert torch.equal(a, b)
        for t in sorted({0, T // 2, T - 1}):
            for a, b in zip(whole, fn(rot, x[t:t + 1].contiguous())):
                assert torch.equal(a[t], b[0]), (fn.__name__, t)


@pytest.mark.parametrize("T", [1023, 1025, 2051, 43693])
def test_rows_side_by_side_equal_rows_alone(P, T):
    """Below 3072 (row, group) pairs a wave has one row, above four side by side and runs of 4, .. 32 of them."""
    import torch
    print(f"quantise rows side by side T={T}", flush=True)
    li = pin.make_custom(6150, 8, 384, 16, n_outlier=3)
    rot = _rot(P, li)
    x = torch.randn((T, 384), generator=torch.Generator(device="cuda").manual_seed(T), device="cuda").half()
    for fn in (P.paro_rotate_scale_quantize_int4, P.paro_rotate_scale_quantize_mxfp4):
        whole = fn(rot, x)
        for t0 in (0, T // 2, T - 7):                     # seven rows at a time are 21 pairs
            for a, b in zip(whole, fn(rot, x[t0:t0 + 7])):
                assert torch.equal(a[t0:t0 + 7], b), (fn.__name__, t0)
    w = x[:T // 8 * 8]
    whole = P.paro_mxfp4_quantize_weight(rot, w)
    part = P.paro_mxfp4_quantize_weight(rot, w[8:64])
    assert torch.equal(whole.codes[8:64], part.codes) and torch.equal(whole.scales[8:64], part.scales)


@pytest.mark.parametrize("N", [8, 24, 32, 40, 264])
def test_weight_rows(P, N):
    import torch
    print(f"quantise weight N={N}", flush=True)
    W = pin.make_dense_weight(6200 + N, N, 384)
    W[1, :128] = 0.0                                  # a constant group: the scale's floor
    W[2, 5] = np.float16(60000.0)
    li = pin.make_custom(6300 + N, 1, 384, 16)
    rot, d = _rot(P, li), torch.as_tensor(W).cuda()
    plain = P.paro_w4_quantize(None, d)
    codes, scales, zeros = oracle.rtn_quantize(W.astype(np.float64))
    got = oracle.unpack_codes(plain.qweight.cpu().numpy().view(np.uint32))
    assert np.array_equal(plain.scales.cpu().numpy().view(np.uint16), scales.view(np.uint16))
    assert np.array_equal(oracle.unpack_zeros(plain.qzeros.cpu().numpy().view(np.uint32)), zeros) and np.array_equal(got, codes)
    whole, mx = P.paro_w4_quantize(rot, d), P.paro_mxfp4_quantize_weight(rot, d)
    for n0 in sorted({0, N // 16 * 8, N - 8}):        # 8 rows share a word of zero points
        part, mxp = P.paro_w4_quantize(rot, d[n0:n0 + 8].contiguous()), P.paro_mxfp4_quantize_weight(rot, d[n0:n0 + 8].contiguous())
        assert torch.equal(whole.qweight[n0:n0 + 8], part.qweight)
        assert torch.equal(whole.scales[:, n0:n0 + 8], part.scales)
        assert torch.equal(whole.qzeros[:, n0 // 8:n0 // 8 + 1], part.qzeros)
        assert torch.equal(mx.codes[n0:n0 + 8], mxp.codes) and torch.equal(mx.scales[n0:n0 + 8], mxp.scales)
