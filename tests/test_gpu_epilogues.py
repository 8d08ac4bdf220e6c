"""Every epilogue of the GEMM launcher on every kernel that can be asked for by number, against 64-bit arithmetic.

Which kernel a layer's GEMM runs on follows from its sizes, so the layers' own tests cover an epilogue on a tile only
where the planner happens to choose it; here the kernel is given.  1, 2: register-staged (bf16); 5, 6, 7: tile heights
256, 192, 128; 8: the 64 x 128 tile."""
import math

import pytest
import torch

import gemm_internal as G
from paper_2311_01635_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TD = {"bf16": torch.bfloat16, "f16": torch.float16}
ROUND = {"bf16": 2.0 ** -8, "f16": 2.0 ** -10}   # twice the half unit in the last place of 8 and 11 significant bits
# one tile and a bit of the small tile in both directions; several of it, and a bit of the 128- and 192-high ones
SHAPES = [(72, 136), (200, 264)]
FORWARD = [G.EPI_STORE, G.EPI_GELU_ERF_FWD, G.EPI_GELU_TANH_FWD, G.EPI_SWIGLU_FWD]
SUMS = [G.EPI_ACC_FIRST, G.EPI_ACC_ADD, G.EPI_ACC_LAST]
BACKWARD = [G.EPI_GELU_ERF_BWD, G.EPI_GELU_TANH_BWD, G.EPI_SWIGLU_BWD]


def erf_gelu(x):
    return 0.5 * x * (1 + torch.erf(x / math.sqrt(2)))


def erf_gelu_grad(x):
    return 0.5 * (1 + torch.erf(x / math.sqrt(2))) + x * torch.exp(-0.5 * x * x) / math.sqrt(2 * math.pi)


def tanh_gelu(x):
    return 0.5 * x * (1 + torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3)))


def tanh_gelu_grad(x):
    th = torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3))
    return 0.5 * (1 + th) + 0.5 * x * (1 - th * th) * math.sqrt(2 / math.pi) * (1 + 3 * 0.044715 * x * x)


def silu(x):
    return x * torch.sigmoid(x)


def silu_grad(x):
    s = torch.sigmoid(x)
    return s * (1 + x * (1 - s))


class Matrix:
    """rows x cols inside a larger buffer of NaN: whatever is written outside shows."""

    def __init__(self, rows, cols, pad, dtype, data=None):
        self.ld = cols + pad
        self.full = torch.full((rows + 1, self.ld), float("nan"), device=DEV, dtype=dtype)
        self.view = self.full[:rows, :cols]
        if data is not None:
            self.view.copy_(data)

    def check(self, ref, rel, what, scale=None):
        got = self.view.double()
        # fp32 sums of at most 200 products: 200 * 2^-24 = 1.2e-5 of the largest, through one activation of slope < 1.2
        bound = rel * ref.abs() + 2e-5 * (ref.abs().max() if scale is None else scale)
        assert bool(((got - ref).abs() <= bound).all()), (what, float(((got - ref).abs() - bound).max()))
        assert torch.isnan(self.full[self.view.shape[0]:]).all() and torch.isnan(self.full[:, self.view.shape[1]:]).all(), what


@pytest.mark.parametrize("pad", [8, 5])           # 16-byte accesses; the element-wise form
@pytest.mark.parametrize("epi", FORWARD + SUMS + BACKWARD)
@pytest.mark.parametrize("variant,dtype", [(1, "bf16"), (2, "bf16"), (5, "bf16"), (6, "bf16"), (7, "bf16"), (8, "bf16"), (7, "f16"), (8, "f16")])
def test_epilogue(variant, dtype, epi, pad):
    td, K = TD[dtype], 200 if dtype == "bf16" else 192
    layout = B.LAYOUT_NN if epi in BACKWARD else B.LAYOUT_TN if epi in SUMS else B.LAYOUT_NT
    for M, N in SHAPES:
        g = torch.Generator(device=DEV).manual_seed(M + 10 * epi)
        normal = lambda *s: torch.randn(*s, generator=g, device=DEV)
        cols = 2 * N if epi == G.EPI_SWIGLU_FWD else N          # columns of the product
        sa, sb = {B.LAYOUT_NT: ((M, K), (cols, K)), B.LAYOUT_NN: ((M, K), (K, cols)), B.LAYOUT_TN: ((K, M), (K, cols))}[layout]
        a, b = normal(*sa).to(td), (normal(*sb) / math.sqrt(K)).to(td)
        ad, bd = a.double(), b.double()
        acc = ad @ bd.T if layout == B.LAYOUT_NT else ad @ bd if layout == B.LAYOUT_NN else ad.T @ bd
        args = G.GemmArgs(A=a.data_ptr(), B=b.data_ptr(), lda=sa[1], ldb=sb[1], M=M, N=cols, K=K, epi=epi, elem=G.ELEM[dtype])
        bias = normal(cols).to(td) if epi in FORWARD else None
        if bias is not None:
            args.bias = bias.data_ptr()
            acc = acc + bias.double()
        what = (variant, dtype, epi, pad, M, N)
        print(f"epilogue {epi} variant={variant} dtype={dtype} pad={pad} M={M} N={N} K={K}", flush=True)

        def run():
            assert G.launch(layout, args, variant) == 0, what
            torch.cuda.synchronize()

        if epi == G.EPI_STORE:
            for out, rel in ((td, ROUND[dtype]), (torch.float32, 0.0)):
                c = Matrix(M, N, pad, out)
                args.C, args.ldc, args.c_is_f32 = c.full.data_ptr(), c.ld, int(out == torch.float32)
                run()
                c.check(acc, rel, what)
        elif epi in SUMS:
            for out in (td, torch.float32) if epi == G.EPI_ACC_LAST else (None,):
                w0 = normal(M, N)
                ws = Matrix(M, N, pad, torch.float32, w0)
                args.ws, args.ldws = ws.full.data_ptr(), ws.ld
                if out is not None:
                    c = Matrix(M, N, pad, out)
                    args.C, args.ldc, args.c_is_f32 = c.full.data_ptr(), c.ld, int(out == torch.float32)
                run()
                if out is not None:
                    c.check(w0.double() + acc, 0.0 if out == torch.float32 else ROUND[dtype], what)
                    assert torch.equal(ws.view, w0), what
                else:
                    ws.check(acc if epi == G.EPI_ACC_FIRST else w0.double() + acc, 0.0, what)
        elif epi in BACKWARD:
            gated = epi == G.EPI_SWIGLU_BWD
            aux = Matrix(M, (2 if gated else 1) * N, pad, td, normal(M, (2 if gated else 1) * N) * 2)
            z = aux.view.double()
            if gated:
                ref = torch.cat([acc * z[:, N:] * silu_grad(z[:, :N]), acc * silu(z[:, :N])], 1)
                args.half = N
            else:
                ref = acc * (erf_gelu_grad if epi == G.EPI_GELU_ERF_BWD else tanh_gelu_grad)(z)
            c = Matrix(M, ref.shape[1], pad, td)
            args.aux, args.ldaux, args.C, args.ldc = aux.full.data_ptr(), aux.ld, c.full.data_ptr(), c.ld
            run()
            c.check(ref, ROUND[dtype], what)
        else:
            gated = epi == G.EPI_SWIGLU_FWD
            ref = silu(acc[:, :N]) * acc[:, N:] if gated else (erf_gelu if epi == G.EPI_GELU_ERF_FWD else tanh_gelu)(acc)
            aux, c = Matrix(M, cols, pad, td), Matrix(M, N, pad, td)
            args.half = N if gated else 0
            args.aux, args.ldaux, args.C, args.ldc = aux.full.data_ptr(), aux.ld, c.full.data_ptr(), c.ld
            run()
            aux.check(acc, ROUND[dtype], what)
            c.check(ref, ROUND[dtype], what, scale=max(float(ref.abs().max()), float(acc.abs().max())))


@pytest.mark.parametrize("pad", [8, 5])
@pytest.mark.parametrize("epi", SUMS)
@pytest.mark.parametrize("variant,dtype", [(1, "bf16"), (2, "bf16"), (5, "bf16"), (6, "bf16"), (7, "bf16"), (8, "bf16"), (7, "f16"), (8, "f16")])
def test_a_piece_of_a_bias_joins_the_sum(variant, dtype, epi, pad):
    """ldaux entries from column `half` on: inside a tile, across the edges of every tile's fragments, up to the last column
    and past none; what lies beside the piece in the bias is never added, the other columns are those without one."""
    td, K = TD[dtype], 200 if dtype == "bf16" else 192
    M, N = 72, 264
    g = torch.Generator(device=DEV).manual_seed(epi)
    normal = lambda *s: torch.randn(*s, generator=g, device=DEV)
    a, b = normal(M, K).to(td), (normal(N, K) / math.sqrt(K)).to(td)
    acc = a.double() @ b.double().T
    args = G.GemmArgs(A=a.data_ptr(), B=b.data_ptr(), lda=K, ldb=K, M=M, N=N, K=K, epi=epi, elem=G.ELEM[dtype])
    for half, width in ((0, 8), (16, 8), (28, 8), (60, 72), (120, 16), (128, 128), (252, 12), (0, 264)):
        bias = torch.full((width + 8,), float("nan"), device=DEV, dtype=td)
        bias[:width] = normal(width).to(td)
        args.bias, args.half, args.ldaux = bias.data_ptr(), half, width
        piece = torch.zeros(N, device=DEV, dtype=torch.float64)
        piece[half:half + width] = bias[:width].double()
        for out in (td, torch.float32) if epi == G.EPI_ACC_LAST else (None,):
            what = (variant, dtype, epi, pad, half, width, out)
            print(f"piece {what}", flush=True)
            w0 = normal(M, N)
            ws = Matrix(M, N, pad, torch.float32, w0)
            args.ws, args.ldws = ws.full.data_ptr(), ws.ld
            if out is not None:
                c = Matrix(M, N, pad, out)
                args.C, args.ldc, args.c_is_f32 = c.full.data_ptr(), c.ld, int(out == torch.float32)
            assert G.launch(B.LAYOUT_NT, args, variant) == 0, what
            torch.cuda.synchronize()
            want = piece + acc if epi == G.EPI_ACC_FIRST else w0.double() + piece + acc
            if out is None:
                ws.check(want, 0.0, what)
            else:
                c.check(want, 0.0 if out == torch.float32 else ROUND[dtype], what)
                assert torch.equal(ws.view, w0), what
