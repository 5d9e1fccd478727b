"""Workspaces that hold what their calls cannot do without (largest exchange part plus largest scratch part, without room
for the partial tiles that only make a call faster) and serve several calls: no call may leave anything in the exchange
part of another, whose kernels take any non-zero word there for a partial sum that has arrived.

The least scratch part is the transformed activations, T * c_in * 2 bytes, plus the partial tiles of the GEMM's own split
(slices * T * c_out * 4 bytes above 16 tokens).  Each case asserts that the full scratch part of one call does reach into
the exchange part of the other, so that it would show if the call left its partial tiles there."""
import numpy as np
import pytest

import oracle
import paro_inputs as pin
from paro_tol import linear_allowed
from test_linear_plans import TWO_LAUNCHES, multi_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2511_10645_amd as paro
    return paro


def _part(P, seed, c_in, c_out, packed=True):
    li = pin.make_custom(seed, 1, c_in, c_out)
    rot = P.Rotation(li.pairs, li.theta, li.ch_scale)
    P.paro_rotation_plan_build(rot)
    w = P.W4Weight(li.qweight, li.scales, li.qzeros)
    if packed:
        P.paro_w4_repack(w)
        w.drop_interchange()
    return li, rot, w


def _x(seed, T, c_in):
    return pin.make_custom(seed, T, c_in, 16, n_outlier=3).x


def _want(li, x):
    u = oracle.rotate_scale(x, li.pairs, li.theta, li.ch_scale)
    return oracle.linear(u, li.qweight, li.scales, li.qzeros), linear_allowed(oracle.row_sqnorms(li.qweight, li.scales, li.qzeros), u)


def _close(y, want, label):
    ref, allowed = want
    worst = float((np.abs(y.cpu().numpy().astype(np.float64) - ref) / allowed).max())
    print(f"  {label}: worst err/allowed = {worst:.3f}", flush=True)
    assert worst <= 1.0, label


def _sizes(P, rot, w, T):
    total, exchange = P.paro_workspace_bytes(rot, w, T), P.paro_workspace_exchange_bytes(rot, w, T)
    return exchange, total - exchange


# T, c_in, outputs of the two parts, most columns of the GEMM's partial tiles (slices x outputs)
@pytest.mark.parametrize("T,c_in,outs,columns", [(9, 8192, (4096, 512), 0), (17, 5120, (5120, 2048), 8 * 5120), (24, 4608, (5120, 4096), 15 * 4096)])
@pytest.mark.parametrize("reverse", [False, True])
def test_multi_with_the_least_workspace(P, T, c_in, outs, columns, reverse):
    import torch
    print(f"multi T={T} {c_in} -> {outs} reverse={reverse}", flush=True)
    outs = outs[::-1] if reverse else outs
    parts = [_part(P, 9100 + 7 * k + T, c_in, n) for k, n in enumerate(outs)]
    rots, weights = [p[1] for p in parts], [p[2] for p in parts]
    x = _x(9150 + T, T, c_in)
    exchange = max(_sizes(P, r, w, T)[0] for r, w in zip(rots, weights))
    assert exchange == P.paro_workspace_exchange_bytes_multi(rots, weights, T)
    ws = P.Workspace(exchange + T * c_in * 2 + columns * T * 4)
    want = [_want(p[0], x) for p in parts]
    xd = torch.as_tensor(x).cuda()
    for i in range(2):
        ys = P.paro_rotated_linear_multi(rots, weights, xd, ws)
        for k in range(2):
            _close(ys[k], want[k], f"call {i} part {k}")
        assert ws.partials_clean(exchange) and ws.error_word() == 0


# a call that exchanges partial sums between blocks, and one whose partial tiles would reach into them: interchange layout
# up to 32 tokens and above, repacked at a token count where the GEMM does not split K
@pytest.mark.parametrize("T,c_in,c_out,packed", [(24, 11008, 272, False), (40, 2176, 528, False), (600, 2048, 48, True)])
def test_single_calls_sharing_the_least_workspace(P, T, c_in, c_out, packed):
    import torch
    print(f"shared T={T} {c_in} -> {c_out} packed={packed}", flush=True)
    la, rot_a, wa = _part(P, 9200, 9216, 4112)
    lb, rot_b, wb = _part(P, 9210 + T, c_in, c_out, packed)
    xa, xb = _x(9201, 16, 9216), _x(9211 + T, T, c_in)
    (ea, _), (eb, full_b) = _sizes(P, rot_a, wa, 16), _sizes(P, rot_b, wb, T)
    nbytes = max(ea, eb) + max(16 * 9216 * 2, T * c_in * 2)
    assert eb + full_b <= nbytes and nbytes - full_b < ea
    ws = P.Workspace(nbytes)
    want_a, want_b = _want(la, xa), _want(lb, xb)
    da, db = torch.as_tensor(xa).cuda(), torch.as_tensor(xb).cuda()
    for i in range(2):
        _close(P.paro_rotated_linear(rot_a, wa, da, ws), want_a, f"exchanging call {i}")
        _close(P.paro_rotated_linear(rot_b, wb, db, ws), want_b, f"splitting call {i}")
        assert ws.partials_clean(ea) and ws.error_word() == 0


@pytest.mark.parametrize("T,c_in,c_out", [(17, 1024, 2064), (31, 512, 528), (33, 512, 1040), (47, 1024, 2064), (201, 1024, 528), (255, 512, 80)])
def test_nothing_is_written_behind_a_ragged_last_block(P, T, c_in, c_out):
    """Activations in operand order take T rows' room at the end of the buffer, whatever T is."""
    import torch
    print(f"guard T={T} {c_in} -> {c_out}", flush=True)
    li, rot, w = _part(P, 9300 + T, c_in, c_out)
    x = _x(9301 + T, T, c_in)
    need, guard = P.paro_workspace_bytes(rot, w, T), 1 << 20
    ws = P.Workspace(need + guard)
    ws.buf[need:] = 0x5A
    ws.nbytes = need
    _close(P.paro_rotated_linear(rot, w, torch.as_tensor(x).cuda(), ws), _want(li, x), "guarded")
    assert bool((ws.buf[need:] == 0x5A).all())


def _random_part(P, seed, c_in, c_out, n_layers=8):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    words = lambda *s: torch.randint(-(1 << 31), 1 << 31, s, generator=g, device="cuda", dtype=torch.int32)
    w = P.W4Weight.from_device(words(c_out, c_in // 8), (0.005 + 0.015 * torch.rand((c_in // 128, c_out), generator=g, device="cuda")).half(),
                               words(c_in // 128, c_out // 8))
    P.paro_w4_repack(w)
    li = pin.make_custom(seed, 1, c_in, 16, n_layers=n_layers)
    rot = P.Rotation(li.pairs, li.theta, li.ch_scale)
    P.paro_rotation_plan_build(rot)
    return rot, w


# several transforms of 1..4 tokens that run as one launch for the transforms and one for the products (K in one block and in two, one token
# and several), beside a call whose exchange part is the larger
@pytest.mark.parametrize("T,c_in,outs,n_layers", [(3, 4096, (8192, 8208), 8), (4, 4096, (6160, 4096, 4112), 5), (2, 7168, (16384, 2064), 8),
                                                  (1, 7168, (14336, 14352), 3)])
def test_transforms_of_several_linears_leave_nothing_behind(P, T, c_in, outs, n_layers):
    """The rows that the first launch hands to the second lie in the buffer: none of their words may be left in the exchange part
    of another call, whatever the buffer's size."""
    import torch
    print(f"multi in two launches T={T} {c_in} -> {outs}", flush=True)
    assert multi_plan(T, c_in, outs, n_layers)[0] == TWO_LAUNCHES
    parts = [_random_part(P, 9400 + 10 * k + T, c_in, n, n_layers) for k, n in enumerate(outs)]
    rots, weights = [p[0] for p in parts], [p[1] for p in parts]
    x = torch.as_tensor(_x(9450 + T, T, c_in)).cuda()
    total, exchange = P.paro_workspace_bytes_multi(rots, weights, T), P.paro_workspace_exchange_bytes_multi(rots, weights, T)
    want = P.paro_rotated_linear_multi(rots, weights, x, P.Workspace(total))
    _, other = _random_part(P, 9490, 27648, 5120)
    xo = torch.as_tensor(_x(9491, 16, 27648)).cuda()
    larger = P.paro_workspace_exchange_bytes(None, other, 16)
    assert larger > max(total, exchange)
    for nbytes in (larger, larger + 4096):
        ws = P.Workspace(nbytes)
        first = P.paro_w4a16_linear(other, xo, ws)
        for _ in range(2):
            ys = P.paro_rotated_linear_multi(rots, weights, x, ws)
            assert ws.partials_clean(nbytes) and ws.error_word() == 0
            assert all(torch.equal(a, b) for a, b in zip(ys, want))
            assert torch.equal(P.paro_w4a16_linear(other, xo, ws), first)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ys = P.paro_rotated_linear_multi(rots, weights, x, ws)
    for _ in range(3):                                     # replays, with eager calls on the same buffer between them
        for y in ys:
            y.fill_(float("nan"))
        graph.replay()
        assert torch.equal(P.paro_w4a16_linear(other, xo, ws), first)
        assert all(torch.equal(a, b) for a, b in zip(ys, want)) and ws.partials_clean(larger) and ws.error_word() == 0
