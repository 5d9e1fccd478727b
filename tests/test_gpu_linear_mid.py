"""The W4A16 linear between the streaming decode kernels and the GEMM (linear_tile.hip) and on weights in the interchange
layout (linear_ic.hip up to 32 tokens, linear_tile.hip above), against the oracle's contraction of the same fp16
activations.

Both kernels multiply q - z exactly, apply the group's scale to fp32 sums and round once, so every output must lie within
half an fp16 ulp of the oracle's fp64 value plus the fp32 rounding of its sums:
    |err| <= 2^-11 |y| 1.001 + (C + 64) 2^-24 sum |x w^| + 2^-25
(one rounding of at most 2^-24 of the running sum per accumulated product, per group scale and per combined partial sum)."""
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


def _weight(P, li, bias, form):
    import torch
    w = P.W4Weight(li.qweight, li.scales, li.qzeros, bias=bias)
    if form == "packed":
        P.paro_w4_repack(w)
        w.drop_interchange()
    elif form == "scales_odd":                        # scales not 4-byte aligned: the kernels' dword loads do not apply
        buf = torch.zeros(w.scales.numel() + 1, dtype=torch.float16, device="cuda")
        buf[1:] = w.scales.flatten()
        w.scales = buf[1:].view(w.scales.shape)
        w.c.scales = w.scales.data_ptr()
    return w


CASES = [
    # interchange layout: blocks of 16 tokens, the last group of a round missing, outputs that end inside a block
    (1, 512, 528, "plain"), (1, 1152, 144, "plain"),       # one token, few short rows
    (1, 640, 48, "plain"), (1, 11008, 272, "plain"), (16, 128, 16, "plain"), (17, 1920, 80, "plain"), (32, 640, 528, "plain"),
    (24, 2176, 4112, "plain"), (33, 128, 16, "plain"), (33, 640, 144, "plain"), (64, 1152, 2064, "plain"),
    # up to 32 tokens: fewer groups than a stage has, a last stage moved back, every split of the tokens into requests, 16 to 64
    # outputs per block with tiles beyond the last output, K split (the last two, rotated)
    (3, 384, 16, "plain"), (8, 896, 32064, "plain"), (4, 1664, 16400, "plain"), (9, 1152, 8240, "plain"), (16, 3712, 2064, "plain"), (25, 2688, 8208, "plain"),
    (6, 2944, 9744, "plain"), (5, 896, 6080, "plain"), (14, 2176, 6096, "plain"), (29, 5760, 4144, "plain"), (21, 640, 20544, "plain"), (13, 11008, 272, "plain"), (24, 11008, 272, "plain"),
    # every instantiation with more stages than its rings hold, the last one moved back (test_linear_plans.py), and the split of 11008 -> 4096
    (4, 7296, 16, "plain"), (12, 6272, 16, "plain"), (23, 6272, 16, "plain"), (29, 3200, 16, "plain"), (4, 3200, 4112, "plain"), (15, 3712, 4192, "plain"),
    (22, 3200, 4128, "plain"), (27, 3200, 4144, "plain"), (2, 1664, 8304, "plain"), (9, 2688, 8208, "plain"), (19, 2176, 8208, "plain"), (28, 1664, 8288, "plain"),
    (1, 1664, 16688, "plain"), (24, 11008, 4096, "plain"),
    # many outputs on few channels: every wave on its own, one and two blocks of 16 tokens, waves with no, one and many groups, ragged tokens and outputs
    (2, 128, 39280, "plain"), (16, 640, 19088, "plain"), (5, 640, 8208, "plain"), (1, 2432, 17424, "plain"), (13, 2560, 16400, "plain"), (25, 384, 51168, "plain"), (32, 128, 27312, "plain"),
    (65, 1920, 272, "plain"), (129, 4096, 1040, "plain"), (200, 2176, 1296, "plain"), (5, 640, 80, "scales_odd"), (40, 640, 80, "scales_odd"),
    # repacked: 64-token tiles, K split and not, ragged tokens and outputs
    (33, 4096, 4112, "packed"), (64, 4096, 6144, "packed"), (64, 512, 16400, "packed"), (80, 2048, 2064, "packed"),
    (128, 4096, 2048, "packed"), (129, 1536, 4112, "packed"), (193, 4096, 1552, "packed"), (40, 13824, 1040, "packed"),
    # streaming kernel behind a rotation: one and two blocks of 16 tokens, K split between blocks (operand order from 17 tokens on, up to 8192 channels)
    (8, 512, 16, "packed"), (9, 512, 16, "packed"), (12, 13824, 528, "packed"), (16, 4096, 4112, "packed"), (17, 4096, 2064, "packed"), (31, 13824, 1040, "packed"),
    (32, 2560, 528, "packed"), (19, 6656, 1040, "packed"), (32, 8192, 528, "packed"),
    # few outputs behind a rotation (operand order): one wave without groups, ragged blocks of 32 tokens and 32 / 64 outputs, K split
    (33, 512, 16, "packed"), (47, 512, 4112, "packed"), (64, 4096, 4096, "packed"), (64, 13824, 4096, "packed"), (65, 2560, 2064, "packed"), (97, 1536, 1040, "packed"),
    (176, 1024, 3088, "packed"), (255, 2048, 80, "packed"), (256, 512, 528, "packed"),
    # 128-token tiles: interchange layout and repacked, unsplit with a bias, and (behind a rotation, bare) with K split;
    # the last behind a rotation: operand order with 64 outputs per block and K split
    (65, 640, 16400, "plain"), (66, 2560, 6160, "plain"), (67, 512, 16400, "packed"), (66, 14336, 4112, "packed"), (64, 14336, 2064, "packed"),
    (127, 8704, 1040, "packed"),
    # 128-token tiles, groups that do not come in whole pairs of steps, ragged last slices and tiles of 16 outputs
    (66, 5248, 8208, "plain"), (129, 1152, 12304, "plain"), (66, 4608, 8208, "packed"), (129, 2560, 12304, "packed"), (383, 1536, 6160, "packed"),
    (65, 1664, 18400, "plain"), (105, 512, 17424, "packed"),
    # interchange layout above 32 tokens: blocks of 17..32 tokens at once, the last with one token and with all, K split and not, outputs that end inside a
    # block; and 64-token tiles with K split
    (33, 256, 400, "plain"), (97, 2944, 80, "plain"), (129, 1280, 1040, "plain"), (256, 384, 2064, "plain"), (65, 13824, 144, "plain"), (225, 896, 4112, "plain"),
    (64, 5248, 4112, "plain"),
]


@pytest.mark.parametrize("T,c_in,c_out,form", CASES)
@pytest.mark.parametrize("rotated", [False, True])
def test_linear_against_oracle(P, T, c_in, c_out, form, rotated):
    _check_linear(P, T, c_in, c_out, form, rotated)


# The least that calls have always needed: nothing for a bare linear whose GEMM does not split, the transformed activations
# (exchange header in front for repacked weights) otherwise.  Partial tiles that only save time are not insisted on.
@pytest.mark.parametrize("T,c_in,c_out,form,rotated,least", [
    (600, 2048, 528, "packed", False, 0), (24, 11008, 272, "plain", True, 24 * 11008 * 2), (600, 2048, 528, "packed", True, 256 + 600 * 2048 * 2),
    # the tiled kernel with fewer slices than it would like, none or those that the GEMM's room holds (test_linear_plans.py)
    (568, 1536, 672, "packed", False, 0), (568, 1536, 672, "packed", True, 256 + 568 * 1536 * 2), (901, 2048, 688, "packed", False, 0),
    (655, 13312, 672, "packed", False, 7386880), (200, 2176, 1296, "plain", True, 200 * 2176 * 2), (129, 4096, 1040, "plain", True, 129 * 4096 * 2),
])
def test_least_workspace(P, T, c_in, c_out, form, rotated, least):
    _check_linear(P, T, c_in, c_out, form, rotated, least)


# the rotation that writes operand order: every number of layers, the scale before and after them, whole and ragged blocks
@pytest.mark.parametrize("n_layers", range(9))
@pytest.mark.parametrize("T,c_in,c_out,order", [(19, 512, 80, 0), (32, 512, 48, 1), (48, 512, 48, 0), (61, 1024, 80, 1)])
def test_operand_order_of_every_rotation(P, T, c_in, c_out, order, n_layers):
    _check_linear(P, T, c_in, c_out, "packed", True, n_layers=n_layers, order=order)


def _check_linear(P, T, c_in, c_out, form, rotated, least=None, n_layers=8, order=0):
    import torch
    print(f"linear T={T} {c_in}->{c_out} {form} rotated={rotated} layers={n_layers} order={order}", flush=True)
    li = pin.make_custom(4000 + T + c_in, T, c_in, c_out, n_layers=n_layers, n_outlier=2)
    bias = pin.make_bias(8, 8, c_out) if T % 2 else None
    w = _weight(P, li, bias, form)
    rot = None
    if rotated:
        rot = P.Rotation(li.pairs, li.theta, li.ch_scale, scale_order=order)
        P.paro_rotation_plan_build(rot)
    want = P.paro_workspace_bytes(rot, w, T)
    assert least is None or least < want
    ws = P.Workspace(want if least is None else least)
    xbuf = torch.full((T, c_in + 24), 3.0, dtype=torch.float16, device="cuda")
    x = xbuf[:, 8:8 + c_in]                            # rows with a stride of their own
    x.copy_(torch.as_tensor(li.x))
    ybuf = torch.full((T, c_out + 24), 7.0, dtype=torch.float16, device="cuda")
    if rotated:
        P.paro_rotated_linear(rot, w, x, ws, Y=ybuf[:, 8:8 + c_out])
        u = P.paro_rotate_scale(rot, x).cpu().numpy().astype(np.float64) if T > 4 or form != "packed" else None   # what the linear read
    else:
        P.paro_w4a16_linear(w, x, ws if ws.nbytes else None, Y=ybuf[:, 8:8 + c_out])
        u = li.x.astype(np.float64)
    got = ybuf.cpu().numpy().astype(np.float64)
    assert (got[:, :8] == 7.0).all() and (got[:, 8 + c_out:] == 7.0).all()      # padding untouched
    y = oracle.linear(u, li.qweight, li.scales, li.qzeros, bias)
    g = c_in // 128
    what = (li.codes.reshape(c_out, g, 128).astype(np.float64) - li.zeros.T[:, :, None]) * li.scales.T.astype(np.float64)[:, :, None]
    mass = np.abs(u) @ np.abs(what.reshape(c_out, c_in)).T
    allowed = 2.0 ** -11 * np.abs(y) * 1.001 + (c_in + 64) * 2.0 ** -24 * mass + 2.0 ** -25
    worst = float((np.abs(got[:, 8:8 + c_out] - y) / allowed).max())
    print(f"  worst err/allowed = {worst:.3f}", flush=True)
    assert worst <= 1.0
