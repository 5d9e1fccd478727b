"""128-token tiles of linear_tile.hip where a block's groups do not fill its steps: what LDS holds in place of the missing ones
reaches no output, be it NaN from an earlier launch or infinities of the call's own earlier steps; and outputs whose rows begin
anywhere."""
import numpy as np
import pytest

import paro_inputs as pin
from test_gpu_linear_mid import P, _check_linear, _weight  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,c_in,c_out", [(512, 128, 16384), (300, 256, 16400), (140, 384, 16400), (129, 1152, 12304), (200, 2176, 8208)])
def test_missing_groups_after_a_launch_on_nan(P, T, c_in, c_out):
    import torch
    li = pin.make_custom(71, 512, 1280, 16384, n_layers=0)
    w = _weight(P, li, None, "plain")
    y = P.paro_w4a16_linear(w, torch.full((512, 1280), float("nan"), dtype=torch.float16, device="cuda"))
    assert torch.isnan(y).all()
    _check_linear(P, T, c_in, c_out, "plain", False)


def test_infinite_activations_stay_infinite_beside_missing_groups(P):
    """1152 channels are 9 groups, five steps of two: the sixth step and the second half of the fifth read what groups 5, 6 and 7
    left in LDS."""
    import torch
    T, c_in, c_out = 129, 1152, 12304
    li = pin.make_custom(72, T, c_in, c_out, n_layers=0)
    w = _weight(P, li, None, "plain")
    x = li.x.copy()
    at = {5: 5 * 128 + 60, 70: 6 * 128 + 3, 128: 7 * 128 + 127}
    for row, c in at.items():
        x[row, c] = np.inf
    y = P.paro_w4a16_linear(w, torch.as_tensor(x).cuda()).cpu().numpy()
    assert np.isfinite(np.delete(y, list(at), axis=0)).all()
    for row, c in at.items():
        q = li.codes.reshape(c_out, c_in)[:, c].astype(int) - li.zeros[c // 128].astype(int)
        assert np.isnan(y[row][q == 0]).all() and (y[row][q > 0] == np.inf).all() and (y[row][q < 0] == -np.inf).all(), row


@pytest.mark.parametrize("T,c_in,c_out", [(64, 512, 16384), (200, 512, 16384), (383, 1536, 6144)])
def test_outputs_are_the_same_wherever_their_rows_begin(P, T, c_in, c_out):
    """Rows that are whole cache lines are stored another way than others: 64-token tiles, 128-token tiles of both widths."""
    import torch
    li = pin.make_custom(73, T, c_in, c_out, n_layers=0)
    w = _weight(P, li, pin.make_bias(8, 8, c_out), "packed")
    x = torch.as_tensor(li.x).cuda()
    lines = P.paro_w4a16_linear(w, x)
    buf = torch.full((T, c_out + 24), 7.0, dtype=torch.float16, device="cuda")
    P.paro_w4a16_linear(w, x, Y=buf[:, 8:8 + c_out])
    assert torch.equal(lines, buf[:, 8:8 + c_out])
    assert (buf[:, :8] == 7.0).all() and (buf[:, 8 + c_out:] == 7.0).all()
    _check_linear(P, T, c_in, c_out, "packed", False)
