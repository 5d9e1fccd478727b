"""The prefill GEMM over numbers of tiles that no round of blocks or band of token tiles divides: every output against fp64."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2511_10645_amd as paro
    return paro


@pytest.mark.parametrize("T,c_in,c_out", [(1100, 512, 2320),        # 9 x 10 tiles of 128 tokens: a band and one more
                                          (2100, 512, 8208),        # 9 x 33 of 256: a round, a second band
                                          (4100, 512, 5136),        # 17 x 21: a tail of half-size tiles behind
                                          (700, 4096, 3088),        # 256-token tiles, K in two
                                          (513, 1024, 16),          # one output tile
                                          (1250, 3584, 736),        # few outputs: the kernel beside the GEMM, K split
                                          (4096, 512, 528)])        # at its largest number of tokens
def test_every_tile(P, T, c_in, c_out):
    """Bound: half an fp16 ulp of the result and one fp32 rounding per product of the fp16 weights that the GEMM multiplies."""
    import torch
    print(f"gemm tiles T={T} {c_in} -> {c_out}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T)
    words = lambda *s: torch.randint(-(1 << 31), 1 << 31, s, generator=g, device="cuda", dtype=torch.int32)
    scales = (0.005 + 0.015 * torch.rand((c_in // 128, c_out), generator=g, device="cuda")).half()
    w = P.W4Weight.from_device(words(c_out, c_in // 8), scales, words(c_in // 128, c_out // 8))
    P.paro_w4_repack(w)
    dense = P.paro_w4_dequant(w).double()
    x = torch.randn((T, c_in), generator=g, device="cuda").half()
    y = P.paro_w4a16_linear(w, x, P.Workspace(P.paro_workspace_bytes(None, w, T))).double()
    want, size = x.double() @ dense.t(), x.double().abs() @ dense.abs().t()
    # (the kernel beside the GEMM keeps q - z exact and scales fp32 sums: within one rounding of each weight)
    bound = 2.0 ** -11 * want.abs() * 1.001 + (c_in * 2.0 ** -24 + 2.0 ** -11) * size + 2.0 ** -25
    assert ((y - want).abs() <= bound).all()
