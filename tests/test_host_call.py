"""The native half of the Python linear calls, and the same steps through ctypes: what they refuse without a GPU, and that outputs, streams,
strides and errors are those of the call."""
import os
import shutil
import subprocess
import sys
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


def test_libparo_alone_is_enough(P, tmp_path):
    """Without paro_host.so, or with one that does not load, and without any compiler: the library loads and the calls take the same
    steps through ctypes."""
    package = os.path.dirname(P.binding.__file__)
    for broken in (False, True):
        copy = tmp_path / str(broken) / "paper_2511_10645_amd"
        copy.mkdir(parents=True)
        for name in os.listdir(package):
            if name.endswith(".py") or name == "libparo.so":
                shutil.copy(os.path.join(package, name), copy / name)
        if broken:
            (copy / "paro_host.so").write_bytes(b"not a library")
        code = """
import torch, paper_2511_10645_amd as P
assert P.paro_version() == 110
w = P.W4Weight.from_device(torch.zeros((64, 64), dtype=torch.int32), torch.zeros((4, 64), dtype=torch.float16), torch.zeros((4, 8), dtype=torch.int32))
try:
    P.paro_w4a16_linear(w, torch.zeros((1, 512)))
except AssertionError:
    print("refused")
"""
        env = {**{k: v for k, v in os.environ.items() if k != "PYTHONPATH"}, "PATH": "/nonexistent", "HIPCC": "/nonexistent"}
        r = subprocess.run([sys.executable, "-W", "ignore", "-c", code], cwd=tmp_path / str(broken), env=env, capture_output=True, text=True)
        assert r.returncode == 0 and r.stdout == "refused\n", r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("T", [1, 5, 40])
def test_calls(P, T, native, monkeypatch):
    import torch
    print(f"host call T={T} native={native}", flush=True)
    if not native:
        monkeypatch.setattr(P.binding, "_host", P.binding._CtypesCalls)
    assert (P.binding._native().__name__ == "paper_2511_10645_amd.paro_host") == native
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
