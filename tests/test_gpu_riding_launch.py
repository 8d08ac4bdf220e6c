"""A backward launch with everything it may hold: both layouts, a weight gradient cut along K, transfers behind the tiles and
column sums in front of them.  Small integers throughout, so that every order of a sum gives the same bits."""
import pytest
import torch

import gemm_internal as G
from paper_2311_01635_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TD = {"bf16": torch.bfloat16, "f16": torch.float16}
SQUARE, D128, D64, D64S = G.SMALL_128X128, G.DUO_128X128, G.DUO_64X128, G.DUO_64X64
# dW [M, N] over K tokens beside dX [K, N]: the tile dW gets and the chunks its sum is cut in.  Rows and columns end inside a
# tile (fp16 contractions are of whole 32s); the last chunk of K is shorter than the others, unless listed below
CASES = [(96, 88, 736, D64S, 2), (352, 152, 512, D64S, 2), (224, 80, 2048, D64S, 8), (96, 1032, 5344, D64, 4), (160, 1848, 4224, D64, 2),
         (1632, 144, 4992, D128, 8), (96, 1744, 7328, D128, 4), (224, 1680, 4608, D128, 4), (1760, 200, 6272, SQUARE, 4),
         (1760, 496, 2816, SQUARE, 2), (160, 1512, 736, 64, 2), (480, 920, 5248, 128, 8), (672, 1688, 4448, 192, 4), (1632, 1168, 5152, 256, 4)]
SAME_LENGTH = {(352, 152, 512), (224, 80, 2048), (160, 1848, 4224), (224, 1680, 4608), (1760, 496, 2816)}


def ints(seed, *shape, dtype=torch.float32):
    return torch.randint(-2, 3, shape, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV).to(dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("M,N,K,tile,chunks", CASES)
def test_split_sums_transfers_and_column_sums(M, N, K, tile, chunks, dtype):
    td, elem = TD[dtype], G.ELEM[dtype]
    units = 5000  # 16-byte units of a transfer: some whole workgroups' and a part of one
    assert G.riding_plan([(B.LAYOUT_NN, K, N, M, G.EPI_ACC_ADD), (B.LAYOUT_TN, M, N, K, G.EPI_ACC_ADD)])[1] == (tile, chunks)
    made, span = G.chunks(K, tile, chunks, B.LAYOUT_TN)
    assert made == chunks and (K == made * span) == ((M, N, K) in SAME_LENGTH)

    dY, X, W = ints(1, K, M, dtype=td), ints(2, K, N, dtype=td), ints(3, M, N, dtype=td)
    # (a row and columns of NaN around each result: what lies beside it stays)
    into = lambda seed, r, c: torch.nn.functional.pad(ints(seed, r, c), (0, 8, 0, 1), value=float("nan"))
    dW, acc = into(4, M, N), into(5, K, N)
    dX = torch.zeros(K, N, device=DEV, dtype=td)  # (the step is not the last: unused)
    args = [G.GemmArgs(A=dY.data_ptr(), lda=M, B=W.data_ptr(), ldb=N, M=K, N=N, K=M, epi=G.EPI_ACC_ADD, C=dX.data_ptr(), ldc=N,
                       ws=acc.data_ptr(), ldws=N + 8, elem=elem, cu_share=2),
            G.GemmArgs(A=dY.data_ptr(), lda=M, B=X.data_ptr(), ldb=N, M=M, N=N, K=K, epi=G.EPI_ACC_ADD, C=dW.data_ptr(), ldc=N + 8,
                       ws=dW.data_ptr(), ldws=N + 8, c_is_f32=1, elem=elem, cu_share=2)]
    home, buf, slot = (ints(6 + i, units * 4) for i in range(3))
    bias_in, bias_out = [ints(9, M), ints(10, N)], [torch.full((M + 8,), float("nan"), device=DEV), torch.full((N + 8,), float("nan"), device=DEV)]
    r = G.Riders(count=1, sums=2)
    r.seg[0] = G.RideSeg(home.data_ptr(), buf.data_ptr(), slot.data_ptr(), 16 * units)
    for i, y in enumerate((dY, X)):
        r.sum[i] = G.RideSum(elem, y.data_ptr(), y.shape[1], K, y.shape[1], bias_in[i].data_ptr(), bias_out[i].data_ptr())
    want = dict(dW=dW[:M, :N] + (dY.double().T @ X.double()).float(), dX=acc[:K, :N] + (dY.double() @ W.double()).float(), home=buf.clone(),
                buf=slot.clone(), sum0=bias_in[0] + dY.float().sum(0), sum1=bias_in[1] + X.float().sum(0))
    torch.cuda.synchronize()
    print(f"riding launch {dtype} M={M} N={N} K={K} tile={tile} chunks={chunks}", flush=True)
    assert G.launch_riding([B.LAYOUT_NN, B.LAYOUT_TN], args, r) == 0
    torch.cuda.synchronize()
    got = dict(dW=dW[:M, :N], dX=acc[:K, :N], home=home, buf=buf, sum0=bias_out[0][:M], sum1=bias_out[1][:N])
    for key in want:
        assert torch.equal(got[key], want[key]), key
    for t, rows, cols in ((dW, M, N), (acc, K, N)):
        assert torch.isnan(t[rows:]).all() and torch.isnan(t[:, cols:]).all()
    assert all(torch.isnan(t[-8:]).all() for t in bias_out) and not dX.any()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_a_split_sum_of_square_tiles_on_the_streams(dtype):
    M, N, K = 1080, 472, 6464
    assert G.plan(B.LAYOUT_TN, M, N, K, G.EPI_ACC_ADD, cu_share=2) == (SQUARE, 4) and G.chunks(K, SQUARE, 4, B.LAYOUT_TN)[1] * 4 != K
    dY, X, dW = ints(1, K, M, dtype=TD[dtype]), ints(2, K, N, dtype=TD[dtype]), ints(4, M, N)
    want = dW + (dY.double().T @ X.double()).float()
    args = G.GemmArgs(A=dY.data_ptr(), lda=M, B=X.data_ptr(), ldb=N, M=M, N=N, K=K, epi=G.EPI_ACC_ADD, C=dW.data_ptr(), ldc=N,
                      ws=dW.data_ptr(), ldws=N, c_is_f32=1, elem=G.ELEM[dtype], cu_share=2)
    torch.cuda.synchronize()
    assert G.launch(B.LAYOUT_TN, args, 4) == 0
    torch.cuda.synchronize()
    assert torch.equal(dW, want)
