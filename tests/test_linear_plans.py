"""The shapes of test_gpu_linear_mid.py reach every instantiation that they are there for: asked of the library's own
dispatch on the host, so that a change of a fitted constant cannot take a kernel out of the tests unnoticed."""
import ctypes

import paper_2511_10645_amd as paro
from paper_2511_10645_amd.binding import _CRotation, _CW4Weight
import test_gpu_multi
from test_gpu_linear_mid import CASES

FAKE = 0x10000                                        # never dereferenced
HOSTED, STREAM, GEMM, TILE, OPERAND, ROWS, GENERIC = range(7)
SEPARATE, K_MAJOR, PER_WAVE, TWO_LAUNCHES = range(4)


def plan(T, c_in, c_out, form, rotated):
    f = paro.lib().paro_internal_linear_plan
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    scales = FAKE + 2 * (form == "scales_odd")
    w = _CW4Weight(c_in, c_out, 128, None, None, None, None, FAKE) if form == "packed" else _CW4Weight(c_in, c_out, 128, FAKE, scales, FAKE, None, None)
    rot = _CRotation(c_in, 128, 8, 64, FAKE, FAKE, None, 0, FAKE)
    tile, k_slices = ctypes.c_int32(), ctypes.c_int32()
    kernel = f(ctypes.byref(rot) if rotated else None, ctypes.byref(w), T, ctypes.byref(tile), ctypes.byref(k_slices))
    return kernel, tile.value, k_slices.value


def plan_in(T, c_in, c_out, form, rotated, ws_bytes):
    f = paro.lib().paro_internal_linear_plan_in
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_void_p]
    w = _CW4Weight(c_in, c_out, 128, None, None, None, None, FAKE) if form == "packed" else _CW4Weight(c_in, c_out, 128, FAKE, FAKE, FAKE, None, None)
    rot = _CRotation(c_in, 128, 8, 64, FAKE, FAKE, None, 0, FAKE)
    tile, k_slices = ctypes.c_int32(), ctypes.c_int32()
    kernel = f(ctypes.byref(rot) if rotated else None, ctypes.byref(w), T, ws_bytes, ctypes.byref(tile), ctypes.byref(k_slices))
    return kernel, tile.value, k_slices.value


def multi_plan(T, c_in, outs, n_layers=8):
    """The route, and what the two workspace queries give."""
    L = paro.lib()
    f = L.paro_internal_multi_plan
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32]
    rot = _CRotation(c_in, 128, n_layers, 64, FAKE, FAKE, None, 0, FAKE)
    ws = [_CW4Weight(c_in, n, 128, None, None, None, None, FAKE) for n in outs]
    rots = (ctypes.c_void_p * len(outs))(*[ctypes.addressof(rot)] * len(outs))
    weights = (ctypes.c_void_p * len(outs))(*[ctypes.addressof(w) for w in ws])
    return f(len(outs), rots, weights, T), L.paro_workspace_bytes_multi(len(outs), rots, weights, T), L.paro_workspace_exchange_bytes_multi(len(outs), rots, weights, T)


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


def test_little_workspace_does_not_cost_precision():
    """Calls without room for the slices of K that the tiled kernel would like run on it all the same, unsplit or with the slices
    there is room for (the GEMM's own partial tiles), not on the GEMM, which rounds the weights to fp16."""
    for T, c_in, c_out, least, k in ((568, 1536, 672, 0, 1), (901, 2048, 688, 0, 1), (666, 1536, 544, 0, 1), (959, 2048, 656, 0, 1),
                                     (565, 20480, 976, 9447936, 3), (655, 13312, 672, 7386880, 3)):
        assert plan_in(T, c_in, c_out, "packed", False, least) == (TILE, 64, k), (T, c_in, c_out)
        header = 0 if least else 256                  # the bare call's least workspace has the exchange header, or is empty
        assert plan_in(T, c_in, c_out, "packed", True, header + least + T * c_in * 2) == (TILE, 64, k), (T, c_in, c_out)
        assert plan(T, c_in, c_out, "packed", False)[2] > k


def test_calls_without_room_are_planned_unsplit():
    """Bare calls on interchange weights have no room for partial tiles: the tile is the one that is faster unsplit (64 tokens;
    measured 86, 63 and 93 us, with 128-token tiles 139, 106 and 158), not the one that would be with K split."""
    for T, c_in, c_out in ((92, 17664, 14640), (757, 13696, 1936), (121, 20736, 9856)):
        assert plan(T, c_in, c_out, "plain", False) == (TILE, 64, 1), (T, c_in, c_out)
        assert plan(T, c_in, c_out, "plain", True)[1:] > (64, 1)


def test_cases_reach_128_token_tiles_of_either_width():
    """64 x 32 per wave up to 11 groups per block, 64 x 64 from 12 on (measured on 28 shapes: 300 tokens 256 -> 16400 13.3 against
    18.7 us, 105 tokens 512 -> 17424 9.9 against 10.7); K is not split into slices of few groups of repacked weights."""
    have = set()
    for T, c_in, c_out, form in CASES:
        for rotated in (False, True):
            kernel, tile, k = plan(T, c_in, c_out, form, rotated)
            groups = min(c_in // 128, -(-(-(-(c_in // 128) // max(k, 1))) // 4) * 4)     # per block
            if kernel == TILE and tile == 128:
                have.add((form, groups >= 12, k > 1))
    want = {(form, wide, split) for form in ("plain", "packed") for wide in (False, True) for split in (False, True)}
    assert want - {("packed", False, True)} <= have, have


def test_two_pairs_of_steps_are_not_split():
    """1024 channels are two pairs of steps: in two slices, with a launch to sum them, slower but for very few outputs."""
    for T, c_out, k in ((97, 128, 1), (126, 208, 1), (69, 144, 1), (80, 16, 2), (202, 48, 2)):
        assert plan(T, 1024, c_out, "packed", False) == (TILE, 64, k), (T, c_out)


def rows_plan(T, c_in, c_out, room):
    """outputs per block (0: every wave on its own), slices of K, instantiation, stages of a slice, the deeper of its rings"""
    f = paro.lib().paro_internal_rows_plan
    f.restype, f.argtypes = None, [ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t, ctypes.c_void_p]
    out = (ctypes.c_int32 * 5)()
    f(ctypes.byref(_CW4Weight(c_in, c_out, 128, FAKE, FAKE, FAKE, None, None)), T, room, out)
    return tuple(out)


def test_cases_refill_the_rings_of_every_interchange_instantiation():
    wrap, split, direct = set(), set(), set()
    for T, c_in, c_out, form in CASES:
        for rotated in (False, True):
            if plan(T, c_in, c_out, form, rotated)[0] != ROWS:
                continue
            outputs, k, config, stages, ring = rows_plan(T, c_in, c_out, 1 << 40 if rotated else 0)
            if not outputs:
                direct.add(T > 16)
                continue
            groups = -(-(c_in // 128) // k)
            if stages > ring and groups % (8 if outputs == 16 else 4):
                wrap.add(config)                      # a slot is requested anew, and the last stage is moved back
            if k > 1 and stages > ring:
                split.add(outputs)
    assert wrap == set(range(13)), sorted(wrap)
    assert split >= {64} and direct == {False, True}, (split, direct)
    assert rows_plan(24, 11008, 4096, 1 << 40) == (64, 4, 10, 6, 4)


def test_many_outputs_on_few_channels_leave_the_staged_kernel():
    """Bare interchange calls, every wave on its own against staged through LDS, us: 9.7 / 14.2, 6.8 / 11.8, 7.1 / 8.8, 13.7 / 15.1;
    6.0 / 5.4, 6.8 / 6.3, 12.6 / 12.6, 9.0 / 8.5."""
    for T, c_in, c_out in ((4, 1024, 43280), (10, 128, 49216), (16, 640, 19072), (25, 384, 51168)):
        assert rows_plan(T, c_in, c_out, 0)[0] == 0, (T, c_in, c_out)
    for T, c_in, c_out in ((3, 256, 31184), (8, 1536, 12160), (24, 1152, 26784), (20, 512, 22304)):
        assert rows_plan(T, c_in, c_out, 0)[0] > 0, (T, c_in, c_out)


def test_interchange_weights_are_planned_with_their_own_times():
    """Several rounds of blocks, where the wide kernel's step costs more on interchange weights (64- / 128-token tiles, us: 157 / 162,
    240 / 249, 319 / 333; 356 / 338)."""
    for T, c_in, c_out, tokens in ((464, 5888, 16944, 64), (414, 5376, 36048, 64), (731, 13184, 11728, 64), (952, 4480, 29152, 128)):
        assert plan(T, c_in, c_out, "plain", False) == (TILE, tokens, 1), (T, c_in, c_out)


def test_many_tokens_on_few_outputs():
    """Above 1024 tokens the tiled kernel takes what leaves the GEMM's tiles few (measured, GEMM / tiled: 55.8 / 25.2, 70.1 / 43.2,
    124 / 98 us) and nothing else (211 / 219, 65 / 70 us), up to 4096 tokens."""
    for T, c_in, c_out in ((1250, 3584, 736), (4096, 4096, 512), (2048, 14336, 1024)):
        assert plan(T, c_in, c_out, "packed", False)[0] == plan(T, c_in, c_out, "packed", True)[0] == TILE
    for T, c_in, c_out in ((1283, 8192, 8240), (1229, 3584, 5296), (2048, 4096, 4096), (4097, 4096, 512)):
        assert plan(T, c_in, c_out, "packed", False)[0] == plan(T, c_in, c_out, "packed", True)[0] == GEMM


def test_few_outputs_on_interchange_weights_take_the_staged_kernel():
    """Above 32 tokens; bare, this against the tiled kernel, us: 15.5 / 45.9, 9.2 / 22.8, 4.3 / 9.4; but 56 / 42, 11.3 / 7.6, and it ends at 256."""
    for T, c_in, c_out, want in ((48, 9600, 2272, ROWS), (64, 4096, 4096, ROWS), (128, 1024, 208, ROWS), (200, 4224, 9408, TILE), (256, 256, 5840, TILE), (257, 1024, 208, TILE)):
        assert plan(T, c_in, c_out, "plain", False)[0] == want, (T, c_in, c_out)


def test_several_transforms_reach_the_wide_kernel():
    """Every case that test_gpu_multi.py has there, and with them every form of the two launches: K in one block and in several, one token
    and more."""
    assert all(multi_plan(*case)[0] == PER_WAVE for case in test_gpu_multi.PER_WAVE)
    assert all(multi_plan(*case)[0] == TWO_LAUNCHES for case in test_gpu_multi.TWO_LAUNCHES)
    assert all(multi_plan(*case)[0] == K_MAJOR for case in test_gpu_multi.SHORT_OF_IT)
    for cases, forms in ((test_gpu_multi.PER_WAVE, {(True, True), (True, False)}),
                         (test_gpu_multi.TWO_LAUNCHES, {(one, split) for one in (True, False) for split in (True, False)})):
        assert forms <= {(case[0] == 1, case[1] > 6144) for case in cases}


def test_rows_of_weights_that_are_quantised_32_to_a_wave():
    """The sizes of test_gpu_quantize_weight.test_rows_without_a_transform, whole and in parts."""
    pays = paro.lib().paro_internal_quantize_plan
    assert pays(12328, 256) == 1 and pays(8, 256) == 0


def test_several_transforms_need_no_scratch():
    """1..4 tokens: whatever the route, the workspace is the exchange part of the K-major kernel, which the other routes share."""
    seen = set()
    for T in (1, 2, 3, 4):
        for c_in in (512, 1024, 3584, 4096, 6144, 6656, 8192, 27648):
            for outs in ((64,), (4096, 1024, 1024), (14336, 14336), (16 * 900, 16 * 899, 16 * 31, 48)):
                for layers in (8, 3):
                    route, total, exchange = multi_plan(T, c_in, outs, layers)
                    seen.add(route)
                    slices = c_in // 512
                    k_major = sum((slices * T * n * 4 + 255) // 256 * 256 for n in outs) if slices > 1 else 0
                    assert total == exchange == 256 + k_major, (T, c_in, outs, layers)
    assert seen == {K_MAJOR, PER_WAVE, TWO_LAUNCHES}
