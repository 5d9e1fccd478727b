"""Which kernel an MXFP4 linear runs on, asked of the library's own dispatch on the host: the shapes of test_gpu_mxfp4_linear.py
reach both widths of the GEMM in the forms that they are there for, and calls measured to be faster on one kernel stay on it."""
import ctypes

import paper_2511_10645_amd as paro
import test_gpu_mxfp4_linear as gpu
from paper_2511_10645_amd.binding import _CMxfp4Weight

STREAM = 0


def plan(T, c_in, c_out):
    f = paro.lib().paro_internal_mxfp4_plan
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_int32]
    return f(ctypes.byref(_CMxfp4Weight(c_in, c_out, None, None, None, None)), T)


def test_cases_reach_both_widths_of_the_gemm():
    (mark,) = [m for m in gpu.test_mxfp4_linear_against_oracle.pytestmark if m.name == "parametrize"]
    have = set()
    for case in mark.args[1]:
        T, C, N = case["T"], case["C"], case["N"]
        outputs = plan(T, C, N)
        wide = (N + case.get("pad", 0)) % 8 == 0      # rows of whole 16-byte stores
        have.add((outputs, wide, outputs > 0 and N % outputs != 0, outputs > 0 and C // 512 > 3))
    for outputs in (128, 256):                        # whole and ragged tiles, less and more than a period of the weights' ring
        assert {(outputs, True, ragged, long) for ragged in (False, True) for long in (False, True)} <= have, (outputs, sorted(have))
        assert any(h[:2] == (outputs, False) for h in have), outputs
    assert any(h[0] == STREAM for h in have)


def test_calls_take_the_kernel_that_is_faster():
    """Behind the quantiser, streaming kernel against GEMM, us: 34.0 / 45.8, 36.0 / 40.5, 15.1 / 16.8, 8.3 / 9.0; 39.1 / 9.2,
    54.8 / 37.5, 22.2 / 15.3, 12.9 / 9.0."""
    for T, c_in, c_out in ((48, 19456, 3536), (83, 15360, 3136), (92, 5632, 1872), (40, 2048, 11616)):
        assert plan(T, c_in, c_out) == STREAM, (T, c_in, c_out)
    for T, c_in, c_out in ((99, 1024, 35776), (160, 14848, 176), (172, 4608, 496), (120, 3072, 1344)):
        assert plan(T, c_in, c_out) != STREAM, (T, c_in, c_out)
