"""The tiles of two workgroups a compute unit (9, 10, 11: 128 x 128, 64 x 128, 64 x 64) and the 128 x 128 one that has a unit
to itself (12) against the tall tiles, bit for bit: every tile adds up an element's products in the order of K and shares
the epilogues."""
import pytest
import torch

import gemm_internal as G
from paper_2311_01635_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TD = {"bf16": torch.bfloat16, "f16": torch.float16}
TILES = [9, 10, 11, 12]
# one fragment of one tile; a tile and its neighbours by one unit; K of one sub-tile of 64, of none whole, of an odd and
# an even number of them, of more than the LDS ring holds; an edge in both directions
SHAPES = [(8, 8, 8), (64, 64, 64), (72, 136, 72), (136, 264, 128), (120, 56, 200), (200, 328, 448), (264, 136, 1000)]
LAYOUTS = [B.LAYOUT_NT, B.LAYOUT_NN, B.LAYOUT_TN]


def operands(layout, M, N, K, dtype, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    sa, sb = {B.LAYOUT_NT: ((M, K), (N, K)), B.LAYOUT_NN: ((M, K), (K, N)), B.LAYOUT_TN: ((K, M), (K, N))}[layout]
    # NaN behind the operands: what lies past K must not be read as data
    pad = lambda s: torch.cat([torch.randn(s[0] * s[1], generator=g, device=DEV).to(TD[dtype]),
                               torch.full((65536,), float("nan"), device=DEV, dtype=TD[dtype])])
    return pad(sa), sa[1], pad(sb), sb[1]


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_the_bits_are_the_tall_tiles(layout, tile, dtype):
    for M, N, K in SHAPES:
        if dtype == "f16":
            K = (K + 31) // 32 * 32  # fp16 contractions are whole sub-tiles of 32
        a, lda, b, ldb = operands(layout, M, N, K, dtype, M + N + K)
        for accumulate in (False, True):
            out, spare = [], torch.zeros(M + 1, N + 8, device=DEV)
            for variant in (7, tile):
                print(f"gemm {dtype} layout={layout} variant={variant} M={M} N={N} K={K} accumulate={accumulate}", flush=True)
                full = torch.full((M + 1, N + 8), 0.5, device=DEV)
                # (a leading dimension past the columns: what lies beside the result stays)
                # (a sum whose result is said to go elsewhere is not cut along K)
                args = G.GemmArgs(A=a.data_ptr(), B=b.data_ptr(), lda=lda, ldb=ldb, M=M, N=N, K=K, C=(spare if accumulate else full).data_ptr(), ldc=N + 8, c_is_f32=1,
                                  epi=G.EPI_ACC_ADD if accumulate else G.EPI_STORE, ws=full.data_ptr(), ldws=N + 8, elem=G.ELEM[dtype])
                assert G.launch(layout, args, variant) == 0
                torch.cuda.synchronize()
                out.append(full)
            assert not torch.isnan(out[1]).any()
            assert torch.equal(out[0], out[1]) and not spare.any(), (M, N, K, accumulate)


@pytest.mark.parametrize("tile,pad", [(9, 8), (10, 8), (11, 8), (12, 8), (12, 5)])  # 16-byte accesses; the element-wise form
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("epi", range(10))
def test_every_epilogue(epi, dtype, tile, pad):
    if tile == 11 and epi == G.EPI_SWIGLU_FWD:
        pytest.skip("a wave of the 64 x 64 tile holds one fragment column: no gate / up pairs")
    td = TD[dtype]
    backward = epi >= G.EPI_GELU_ERF_BWD
    layout = B.LAYOUT_NN if backward else B.LAYOUT_TN if 1 <= epi <= 3 else B.LAYOUT_NT
    paired = epi in (G.EPI_SWIGLU_FWD, G.EPI_SWIGLU_BWD)
    for M, N in ((8, 8), (72, 136), (200, 264)):
        cols = 2 * N if epi == G.EPI_SWIGLU_FWD else N
        a, lda, b, ldb = operands(layout, M, cols, 192, dtype, 7 * epi + M)
        g = torch.Generator(device=DEV).manual_seed(epi)
        old, aux0 = torch.randn(M, N, generator=g, device=DEV), torch.randn(M, 2 * N, generator=g, device=DEV).to(td)
        bias = torch.randn(cols, generator=g, device=DEV).to(td)
        for f32 in (0, 1) if epi in (G.EPI_STORE, G.EPI_ACC_LAST) else (0,):
            got = []
            for variant in (7, tile):
                print(f"epilogue {epi} {dtype} variant={variant} M={M} N={N} f32={f32}", flush=True)
                width = 2 * N if epi == G.EPI_SWIGLU_BWD else N
                c = torch.full((M + 1, width + pad), 3.0, device=DEV, dtype=torch.float32 if f32 else td)
                ws, aux = old.clone(), aux0.clone()
                args = G.GemmArgs(A=a.data_ptr(), B=b.data_ptr(), lda=lda, ldb=ldb, M=M, N=cols, K=192, epi=epi, C=c.data_ptr(),
                                  ldc=width + pad, ws=ws.data_ptr(), ldws=N, aux=aux.data_ptr(), ldaux=2 * N, half=N if paired else 0,
                                  c_is_f32=f32, elem=G.ELEM[dtype])
                if epi == G.EPI_STORE or (not backward and not 1 <= epi <= 3):
                    args.bias = bias.data_ptr()
                if 1 <= epi <= 3:  # a piece of a bias: `ldaux` entries for the columns from `half` on
                    args.bias, args.half, args.ldaux = bias.data_ptr(), 4, 4
                assert G.launch(layout, args, variant) == 0
                torch.cuda.synchronize()
                got.append((c, ws, aux))
            for x, y in zip(*got):
                assert torch.equal(x, y), (epi, M, N, f32)


def test_what_the_tiles_do_not_take_is_refused():
    a, lda, b, ldb = operands(B.LAYOUT_NT, 64, 128, 64, "bf16", 1)
    c, aux = torch.zeros(64, 136, device=DEV, dtype=torch.bfloat16), torch.zeros(64, 128, device=DEV, dtype=torch.bfloat16)
    args = G.GemmArgs(A=a.data_ptr(), B=b.data_ptr(), lda=lda, ldb=ldb, M=64, N=128, K=64, epi=G.EPI_STORE, C=c.data_ptr(), ldc=129)
    assert G.launch(B.LAYOUT_NT, args, 9) != 0  # an odd leading dimension: the element-wise form is the tall tiles'
    args.epi, args.ldc, args.half, args.aux, args.ldaux = G.EPI_SWIGLU_FWD, 136, 64, aux.data_ptr(), 128
    assert G.launch(B.LAYOUT_NT, args, 10) == 0 and G.launch(B.LAYOUT_NT, args, 11) != 0
    torch.cuda.synchronize()
    with pytest.raises(B.RtpError):  # they are the launcher's own choice, not the caller's
        B.rtp_gemm(B.LAYOUT_NT, B.RTP_BF16, B.RTP_BF16, False, a, lda, b, ldb, c, 136, 64, 128, 64, 9)
