"""One token on repacked weights: the K-major kernel and the one whose waves each transform their own K-slice, on either side of
every line between them, against the oracle; and the second on a buffer that has no room for the first's partial sums.
Tolerance: 5e-3 ||w_n|| ||u|| / sqrt(C), the oracle's u in fp64 against fp16 activations (2^-11 each) and one fp16 result."""
import numpy as np
import pytest

import oracle
import paro_inputs as pin
from paro_tol import linear_allowed

pytestmark = pytest.mark.gpu

# (c_in, c_out): 1 slice, short and long; 2..4 slices, one output tile to several per wave; 5..8; 9..12 on both sides of 44 slices of
# tiles per compute unit; 2, 3, 4 and 7 blocks along K on both sides of theirs
CASES = [(512, 16), (512, 16400), (1024, 16), (1024, 4112), (1024, 24592), (1536, 528), (1536, 12304), (2048, 2064), (2048, 16400), (2560, 4112),
         (3584, 12304), (4608, 16400), (4608, 20496), (5632, 16400), (6144, 15008), (7168, 8208), (8192, 7952), (9216, 4112), (9216, 7520), (12288, 5440),
         (14336, 3264), (14336, 3664), (27648, 1424), (27648, 1456)]
TIGHT = [(7168, 8208, 2), (9216, 4752, 3), (14336, 3264, 4)]        # c_in, c_out, blocks along K


def _check(c_in, c_out, nbytes=None):
    import torch
    import paper_2511_10645_amd as P
    print(f"one token {c_in} -> {c_out}, workspace {nbytes}", flush=True)
    li = pin.make_custom(700 + c_in, 1, c_in, c_out, n_outlier=2)
    bias = pin.make_bias(7, 7, c_out) if c_out % 32 else None
    rot, w = P.Rotation(li.pairs, li.theta, li.ch_scale), P.W4Weight(li.qweight, li.scales, li.qzeros, bias=bias)
    P.paro_rotation_plan_build(rot)
    P.paro_w4_repack(w)
    need = P.paro_workspace_bytes(rot, w, 1)
    assert nbytes is None or nbytes < need
    ws = P.Workspace(nbytes or need)
    x = torch.as_tensor(li.x).cuda()
    ys = [P.paro_rotated_linear(rot, w, x, ws) for _ in range(2)]
    u = oracle.rotate_scale(li.x, li.pairs, li.theta, li.ch_scale)
    y = oracle.linear(u, li.qweight, li.scales, li.qzeros, bias)
    allowed = linear_allowed(oracle.row_sqnorms(li.qweight, li.scales, li.qzeros), u)
    assert float((np.abs(ys[0].cpu().numpy().astype(np.float64) - y) / allowed).max()) <= 1.0
    assert (ys[0] == ys[1]).all() and ws.partials_clean() and ws.error_word() == 0


@pytest.mark.parametrize("c_in,c_out", CASES)
def test_one_token_against_oracle(c_in, c_out):
    _check(c_in, c_out)


@pytest.mark.parametrize("c_in,c_out,blocks", TIGHT)
def test_no_room_for_all_partial_sums(c_in, c_out, blocks):
    _check(c_in, c_out, 256 + (blocks * c_out * 4 + 255) // 256 * 256)


# K-major; transforms per wave, K in one block (8 and 10 waves) and in several; two launches
@pytest.mark.parametrize("T,c_in,c_out", [(1, 512, 64), (1, 4096, 4096), (1, 1024, 64), (1, 4096, 28672), (1, 5120, 40960), (1, 14336, 4112), (7, 1024, 64)])
@pytest.mark.parametrize("angle", [float("nan"), float("inf"), float("-inf")])
def test_angles_that_are_not_finite(T, c_in, c_out, angle):
    """Cosine and sine of such an angle are NaN, hence every output of the call, whichever kernel it takes; an empty slot's angle counts for
    nothing."""
    import torch
    import paper_2511_10645_amd as P
    print(f"angle {angle}, T={T} {c_in} -> {c_out}", flush=True)
    li = pin.make_custom(760, T, c_in, 16)
    words = lambda *s: torch.randint(-(1 << 31), 1 << 31, s, generator=torch.Generator(device="cuda").manual_seed(c_out), device="cuda", dtype=torch.int32)
    w = P.W4Weight.from_device(words(c_out, c_in // 8), torch.full((c_in // 128, c_out), 0.01, dtype=torch.float16, device="cuda"), words(c_in // 128, c_out // 8))
    P.paro_w4_repack(w)
    for empty in (False, True):
        pairs, theta = li.pairs.copy(), li.theta.copy()
        theta[c_in // 128 - 1, 3, 9] = angle
        if empty:
            pairs[c_in // 128 - 1, 3, 9] = 0
        rot = P.Rotation(pairs, theta, li.ch_scale)
        P.paro_rotation_plan_build(rot)
        y = P.paro_rotated_linear(rot, w, torch.as_tensor(li.x).cuda(), P.Workspace(P.paro_workspace_bytes(rot, w, T)))
        assert (torch.isfinite(y) if empty else torch.isnan(y)).all()
