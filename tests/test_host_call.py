"""The native half of the Python linear calls: what it refuses without a GPU, and that outputs, streams, strides and errors are
those of the call."""
import threading

import numpy as np
import pytest

import paro_inputs as pin


@pytest.fixture(scope="module")
def P():
    import paper_2511_10645_amd as paro
    paro.lib()
    return paro


def test_refusals_need_no_gpu(P):
    import torch
    li = pin.make_custom(6900, 3, 512, 64)
    rot, w = P.Rotation(li.pairs, li.theta, li.ch_scale, device="cpu"), P.W4Weight(li.qweight, li.scales, li.qzeros, device="cpu")
    x = torch.zeros((3, 512), dtype=torch.float16)
    ws = P.Workspace(4096, device="cpu")
    for bad in (x.float(), x[0], x.reshape(1, 3, 512), x.t(), torch.zeros((3, 1024), dtype=torch.float16)[:, ::2]):
        for call in (lambda: P.paro_rotated_linear(rot, w, bad, ws), lambda: P.paro_w4a16_linear(w, bad), lambda: P.paro_rotate_scale(rot, bad),
                     lambda: P.paro_rotated_linear(rot, w, x, ws, bad), lambda: P.paro_rotate_scale(rot, x, bad)):
            with pytest.raises(AssertionError):
                call()
    with pytest.raises(TypeError):
        P.paro_w4a16_linear(w, li.x)                       # an array, not a tensor
    with pytest.raises(TypeError):
        P.paro_rotate_scale(w, x)                          # a weight, not a transform
    rot.c_out = 64
    with pytest.raises(TypeError):
        P.paro_rotated_linear(w, rot, x, ws)


@pytest.mark.gpu
@pytest.mark.parametrize("T", [1, 5, 40])
def test_calls(P, T):
    import torch
    print(f"host call T={T}", flush=True)
    li = pin.make_custom(6910 + T, T, 1024, 272)
    rot, w = P.Rotation(li.pairs, li.theta, li.ch_scale), P.W4Weight(li.qweight, li.scales, li.qzeros)
    P.paro_rotation_plan_build(rot)
    P.paro_w4_repack(w)
    x = torch.as_tensor(li.x).cuda()
    ws = P.Workspace(P.paro_workspace_bytes(rot, w, T))
    y = P.paro_rotated_linear(rot, w, x, ws)
    assert y.dtype == torch.float16 and y.shape == (T, 272) and y.is_contiguous() and not y.requires_grad
    out = torch.full((T, 280), 7.0, dtype=torch.float16, device="cuda")[:, :272]
    wide = torch.zeros((T, 1040), dtype=torch.float16, device="cuda")
    wide[:, 8:1032] = x
    assert P.paro_rotated_linear(rot, w, wide[:, 8:1032], ws, out) is out and torch.equal(out, y)
    xr = P.paro_rotate_scale(rot, x)
    assert P.paro_rotate_scale(rot, x, xr) is xr
    bare_ws = P.Workspace(P.paro_workspace_bytes(None, w, T))
    bare = P.paro_w4a16_linear(w, xr, bare_ws)
    assert torch.allclose(bare.float(), y.float(), rtol=4e-3, atol=4e-3 * float(y.float().abs().max()))
    with pytest.raises(P.binding.ParoError) as e:          # workspace too small
        P.paro_rotated_linear(rot, w, x, P.Workspace(0))
    assert e.value.status == 6
    with pytest.raises(P.binding.ParoError):               # no tokens
        P.paro_rotated_linear(rot, w, x[:0], ws)
    side, results = torch.cuda.Stream(), []

    def work():                                            # another thread, on a stream of its own
        with torch.cuda.stream(side):
            z = torch.zeros((T, 1024), dtype=torch.float16, device="cuda")
            torch.cuda._sleep(2000000)
            z.copy_(x)                                     # the call has to wait for this copy: it runs on the same stream
            results.append(P.paro_rotated_linear(rot, w, z, P.Workspace(P.paro_workspace_bytes(rot, w, T))))
    torch.cuda.synchronize()
    t = threading.Thread(target=work)
    t.start(); t.join()
    side.synchronize()
    assert torch.equal(results[0], y)
    assert np.isfinite(y.cpu().numpy()).all()
