"""The tiled kernel's partial last sub-tile (a contraction length that is not a multiple of 32), against the oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
import rtp_workloads as wl
from paper_2311_01635_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# one sub-tile cut short, a K of whole sub-tiles plus 8, 16, 24; where K counts rows, any number of them
SHAPES = [(8, 8, 8), (304, 520, 200), (520, 264, 688), (256, 256, 40)]
ODD = {B.LAYOUT_NT: [(301, 76, 72)], B.LAYOUT_NN: [(33, 72, 40)], B.LAYOUT_TN: [(72, 264, 301), (136, 72, 37), (136, 72, 1)]}


# 5, 6, 7: tile heights 256, 192, 128
@pytest.mark.parametrize("variant", [5, 6, 7])
@pytest.mark.parametrize("layout", [B.LAYOUT_NT, B.LAYOUT_NN, B.LAYOUT_TN])
def test_partial_sub_tile(layout, variant):
    for i, (M, N, K) in enumerate(SHAPES + ODD[layout]):
        rng = np.random.default_rng(100 * layout + i)
        sa, sb = {B.LAYOUT_NT: ((M, K), (N, K)), B.LAYOUT_NN: ((M, K), (K, N)), B.LAYOUT_TN: ((K, M), (K, N))}[layout]
        a, b = (wl._store(rng.standard_normal(s, dtype=np.float32), "bf16") for s in (sa, sb))
        ref = np.zeros((M, N))
        {B.LAYOUT_NT: orc.gemm_nt, B.LAYOUT_NN: orc.gemm_nn, B.LAYOUT_TN: orc.gemm_tn}[layout](
            np.ascontiguousarray(a, dtype=np.float64), np.ascontiguousarray(b, dtype=np.float64), ref)
        # NaN behind the operands: what lies past K must not be read as data
        pad = lambda x: torch.cat([torch.from_numpy(np.ascontiguousarray(x)).to(DEV, torch.bfloat16).reshape(-1),
                                   torch.full((65536,), float("nan"), device=DEV, dtype=torch.bfloat16)])
        c = torch.ones(M, N, device=DEV, dtype=torch.float32)
        print(f"gemm layout={layout} variant={variant} M={M} N={N} K={K}", flush=True)
        B.rtp_gemm(layout, B.RTP_BF16, B.RTP_F32, True, pad(a), sa[1], pad(b), sb[1], c, N, M, N, K, variant)
        torch.cuda.synchronize()
        got = c.cpu().numpy().astype(np.float64) - 1.0
        # fp32 sums of at most 688 products of 8-bit significands: 688 * 2^-24 ~ 4e-5 of the largest
        assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max(), (M, N, K)


@pytest.mark.parametrize("layout", [B.LAYOUT_NT, B.LAYOUT_NN, B.LAYOUT_TN])
def test_every_tile_adds_up_in_the_order_of_k(layout):
    """Which tile runs a problem is the planner's choice and must not show in the result: the tall tiles (5, 6, 7)
    and the 64 x 128 one (8) give the bits of the register-staged kernel (2), partial sub-tile or not."""
    for M, N, K in SHAPES + ODD[layout] + [(136, 264, 32), (136, 264, 72), (136, 264, 104), (136, 264, 136), (136, 264, 1992)]:
        g = torch.Generator(device=DEV).manual_seed(M + N + K)
        sa, sb = {B.LAYOUT_NT: ((M, K), (N, K)), B.LAYOUT_NN: ((M, K), (K, N)), B.LAYOUT_TN: ((K, M), (K, N))}[layout]
        a, b = (torch.randn(*s, generator=g, device=DEV).bfloat16() for s in (sa, sb))
        out = {}
        for variant in (2, 5, 6, 7, 8):
            print(f"gemm layout={layout} variant={variant} M={M} N={N} K={K}", flush=True)
            out[variant] = torch.empty(M, N, device=DEV, dtype=torch.float32)
            B.rtp_gemm(layout, B.RTP_BF16, B.RTP_F32, False, a, sa[1], b, sb[1], out[variant], N, M, N, K, variant)
            torch.cuda.synchronize()
        for variant in (5, 6, 7, 8):
            assert torch.equal(out[variant], out[2]), (variant, M, N, K)


def test_gradients_of_a_ragged_batch_repeat():
    """fp32 `C += A B` over 1990 tokens into few tiles: the same bits on every run (and those of the unsplit tiles)."""
    M, N, K = 384, 768, 1990
    g = torch.Generator(device=DEV).manual_seed(3)
    a, b = (torch.randn(*s, generator=g, device=DEV).bfloat16() for s in ((K, M), (K, N)))
    c0 = torch.randn(M, N, generator=g, device=DEV)
    runs = []
    for variant in (2, 4, 4, 4):
        c = c0.clone()
        print(f"gemm TN variant={variant} M={M} N={N} K={K} accumulate", flush=True)
        B.rtp_gemm(B.LAYOUT_TN, B.RTP_BF16, B.RTP_F32, True, a, M, b, N, c, N, M, N, K, variant)
        torch.cuda.synchronize()
        runs.append(c)
    assert all(torch.equal(c, runs[0]) for c in runs)
