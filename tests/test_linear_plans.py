"""The shapes of test_gpu_linear_mid.py reach every instantiation that they are there for: asked of the library's own
dispatch on the host, so that a change of a fitted constant cannot take a kernel out of the tests unnoticed."""
import ctypes

import paper_2511_10645_amd as paro
from paper_2511_10645_amd.binding import _CRotation, _CW4Weight
from test_gpu_linear_mid import CASES

FAKE = 0x10000                                        # never dereferenced
HOSTED, STREAM, GEMM, TILE, OPERAND, ROWS, GENERIC = range(7)


def plan(T, c_in, c_out, form, rotated):
    f = paro.lib().paro_internal_linear_plan
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    scales = FAKE + 2 * (form == "scales_odd")
    w = _CW4Weight(c_in, c_out, 128, None, None, None, None, FAKE) if form == "packed" else _CW4Weight(c_in, c_out, 128, FAKE, scales, FAKE, None, None)
    rot = _CRotation(c_in, 128, 8, 64, FAKE, FAKE, None, 0, FAKE)
    tile, k_slices = ctypes.c_int32(), ctypes.c_int32()
    kernel = f(ctypes.byref(rot) if rotated else None, ctypes.byref(w), T, ctypes.byref(tile), ctypes.byref(k_slices))
    return kernel, tile.value, k_slices.value


def test_cases_reach_every_kernel():
    have = set()
    for T, c_in, c_out, form in CASES:
        for rotated in (False, True):
            kernel, tile, k = plan(T, c_in, c_out, form, rotated)
            have.add((kernel, form == "packed", 16 if kernel == ROWS and T <= 16 else tile, k > 1))
    want = {(TILE, packed, tokens, split) for packed in (False, True) for tokens in (64, 128) for split in (False, True)}
    want |= {(OPERAND, True, outputs, split) for outputs in (32, 64) for split in (False, True)}
    want |= {(ROWS, False, tokens, split) for tokens in (16, 0) for split in (False, True)}
    want |= {(STREAM, True, operand, False) for operand in (0, 1)} | {(GENERIC, False, 0, False)}
    assert want <= have, sorted(want - have)


def test_rotations_of_every_depth_are_read_in_operand_order():
    for T, c_in, c_out in ((19, 512, 80), (32, 512, 48), (48, 512, 48), (61, 1024, 80)):
        kernel, tile, _ = plan(T, c_in, c_out, "packed", True)
        assert kernel == OPERAND or (kernel, tile) == (STREAM, 1), (T, c_in, c_out, kernel)


def test_the_tiled_kernel_is_not_taken_where_it_is_slower():
    """Calls whose last round of GEMM tiles is a small tail, and two short passes of the streaming kernel on few outputs
    (measured, tiled kernel against the one expected here: 246 / 198, 317 / 275, 453 / 335 and 16.2 / 14.9 us)."""
    for T, c_in, c_out, want in ((946, 6144, 16496, GEMM), (888, 8704, 17328, GEMM), (910, 11264, 16480, GEMM), (42, 20992, 672, STREAM)):
        assert plan(T, c_in, c_out, "packed", False)[0] == want, (T, c_in, c_out)


def test_long_rows_at_64_tokens_stay_on_the_tiled_kernel():
    """Rotated 14336 -> 4096 on weights that no cache holds: operand order 27.0 us, the tiled kernel 24.5."""
    assert plan(64, 14336, 4096, "packed", True)[0] == TILE
    assert plan(64, 4096, 4096, "packed", True)[0] == OPERAND
