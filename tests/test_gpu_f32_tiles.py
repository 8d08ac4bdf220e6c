"""The fp32 GEMM's two tiles: edges, rows that no 16-byte load fits, and the same bits from both."""
import pytest
import torch

from paper_2311_01635_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LAYOUTS = {"nt": B.LAYOUT_NT, "nn": B.LAYOUT_NN, "tn": B.LAYOUT_TN}


def operands(layout, M, N, K, pad, off):
    """A and B as views with `pad` more elements a row, `off` elements past a 16-byte boundary."""
    out = []
    for seed, (r, c) in ((1, (K, M) if layout == "tn" else (M, K)), (2, (N, K) if layout == "nt" else (K, N))):
        flat = torch.randn(r * (c + pad) + off, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV)
        out.append(flat[off:].view(r, c + pad)[:, :c])
    return out


def product(layout, a, b, M, N, K, C0=None):
    c = torch.full((M, N), float("nan"), device=DEV) if C0 is None else C0.clone()
    B.rtp_gemm(LAYOUTS[layout], B.RTP_F32, B.RTP_F32, C0 is not None, a, a.stride(0), b, b.stride(0), c, N, M, N, K)
    torch.cuda.synchronize()
    return c


@pytest.mark.parametrize("pad,off", [(0, 0), (4, 0), (1, 0), (0, 1), (3, 2)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (16, 32, 64), (15, 31, 63), (17, 33, 65), (64, 128, 256), (33, 70, 130), (8, 200, 5)])
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_small_tile(layout, M, N, K, pad, off):
    a, b = operands(layout, M, N, K, pad, off)
    A, Bm = (a.double().T if layout == "tn" else a.double()), (b.double().T if layout == "nt" else b.double())
    C0 = torch.randn(M, N, generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    # a chain of K fused multiply-adds and one addition, each rounded once
    bound = (K + 1) * 2.0 ** -24 * (A.abs() @ Bm.abs() + C0.double().abs()) + 1e-30
    assert ((product(layout, a, b, M, N, K).double() - A @ Bm).abs() <= bound).all()
    assert ((product(layout, a, b, M, N, K, C0).double() - (C0.double() + A @ Bm)).abs() <= bound).all()


@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_both_tiles_give_the_same_bits(layout):
    M, N, K = 1024, 2048, 100                   # 4096 small tiles, the most there may be; one row more takes the large tile
    a, b = operands(layout, M + 1, N, K, 3, 0)
    C0 = torch.randn(M + 1, N, generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    head = a[:, :M] if layout == "tn" else a[:M]
    assert torch.equal(product(layout, head, b, M, N, K), product(layout, a, b, M + 1, N, K)[:M])
    assert torch.equal(product(layout, head, b, M, N, K, C0[:M].contiguous()), product(layout, a, b, M + 1, N, K, C0)[:M])
