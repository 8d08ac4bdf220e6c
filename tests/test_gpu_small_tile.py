"""The 64 x 128 tile (four waves fetch, four multiply) at the edges of its tiles and sub-tiles, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
import rtp_workloads as wl
from paper_2311_01635_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SMALL_TILE = 8
# one partial tile and sub-tile; whole ones; one row / column group past a tile; the ring wraps an odd and an even
# number of times; K a multiple of neither 64 nor 32 (bf16)
SHAPES = [(8, 8, 8), (64, 128, 64), (72, 136, 128), (200, 768, 320), (136, 264, 704), (56, 120, 40), (128, 256, 1000)]
ODD = {B.LAYOUT_NT: [(33, 76, 72), (1, 128, 200)], B.LAYOUT_NN: [(65, 72, 40)], B.LAYOUT_TN: [(72, 264, 301), (136, 72, 1)]}


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("layout", [B.LAYOUT_NT, B.LAYOUT_NN, B.LAYOUT_TN])
def test_small_tile(layout, dtype):
    td, bd = {"bf16": (torch.bfloat16, B.RTP_BF16), "f16": (torch.float16, B.RTP_F16)}[dtype]
    for i, (M, N, K) in enumerate(SHAPES + ODD[layout]):
        if dtype == "f16" and K % 32:
            continue
        rng = np.random.default_rng(100 * layout + i)
        sa, sb = {B.LAYOUT_NT: ((M, K), (N, K)), B.LAYOUT_NN: ((M, K), (K, N)), B.LAYOUT_TN: ((K, M), (K, N))}[layout]
        a, b = (wl._store(rng.standard_normal(s, dtype=np.float32), dtype) for s in (sa, sb))
        ref = np.zeros((M, N))
        {B.LAYOUT_NT: orc.gemm_nt, B.LAYOUT_NN: orc.gemm_nn, B.LAYOUT_TN: orc.gemm_tn}[layout](
            np.ascontiguousarray(a, dtype=np.float64), np.ascontiguousarray(b, dtype=np.float64), ref)
        # NaN behind the operands and around the result: what lies past an edge is neither read nor written
        pad = lambda x: torch.cat([torch.from_numpy(np.ascontiguousarray(x)).to(DEV, td).reshape(-1),
                                   torch.full((65536,), float("nan"), device=DEV, dtype=td)])
        for accumulate, ldc in ((True, N), (False, N + 5)):
            c = torch.full((M + 1, ldc), float("nan"), device=DEV, dtype=torch.float32)
            c[:M, :N] = 1.0
            print(f"gemm layout={layout} dtype={dtype} M={M} N={N} K={K} accumulate={accumulate}", flush=True)
            B.rtp_gemm(layout, bd, B.RTP_F32, accumulate, pad(a), sa[1], pad(b), sb[1], c, ldc, M, N, K, SMALL_TILE)
            torch.cuda.synchronize()
            got = c[:M, :N].cpu().numpy().astype(np.float64) - (1.0 if accumulate else 0.0)
            # fp32 sums of at most 1000 products of 8- or 11-bit significands: 1000 * 2^-24 = 6e-5 of the largest
            assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max(), (M, N, K, accumulate)
            assert torch.isnan(c[M:]).all() and torch.isnan(c[:, N:]).all(), (M, N, K, accumulate)
