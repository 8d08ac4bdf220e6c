"""The GEMM launcher behind the layers, which the C ABI does not expose: its argument block and entry points,
so that a test can ask which tile a shape gets and run an epilogue on a chosen kernel."""
import ctypes as C

from paper_2311_01635_amd import binding as B

EPI_STORE, EPI_ACC_FIRST, EPI_ACC_ADD, EPI_ACC_LAST = 0, 1, 2, 3
EPI_GELU_ERF_FWD, EPI_GELU_TANH_FWD, EPI_SWIGLU_FWD = 4, 5, 6
EPI_GELU_ERF_BWD, EPI_GELU_TANH_BWD, EPI_SWIGLU_BWD = 7, 8, 9
ELEM = {"bf16": 0, "f16": 1}


class GemmArgs(C.Structure):
    _fields_ = [("A", C.c_void_p), ("B", C.c_void_p), ("lda", C.c_int64), ("ldb", C.c_int64), ("M", C.c_int), ("N", C.c_int),
                ("K", C.c_int), ("epi", C.c_int), ("C", C.c_void_p), ("ldc", C.c_int64), ("ws", C.c_void_p), ("ldws", C.c_int64),
                ("aux", C.c_void_p), ("ldaux", C.c_int64), ("bias", C.c_void_p), ("half", C.c_int), ("c_is_f32", C.c_int),
                ("elem", C.c_int), ("cu_share", C.c_int), ("sync", C.c_void_p), ("sync_signal", C.c_int), ("sync_wait", C.c_int)]


_plan = getattr(B.lib, "_ZN3rtp17gemm_bf16_pp_planEiPKNS_8GemmArgsEiPKiPiS5_")
_plan.restype = None
_plan.argtypes = [C.c_int, C.POINTER(GemmArgs), C.c_int, C.POINTER(C.c_int), C.POINTER(C.c_int), C.POINTER(C.c_int)]
_plan_riding = getattr(B.lib, "_ZN3rtp24gemm_bf16_pp_plan_ridingEPKiPKNS_8GemmArgsEiPi")
_plan_riding.restype = None
_plan_riding.argtypes = [C.POINTER(C.c_int), C.POINTER(GemmArgs), C.c_int, C.POINTER(C.c_int)]
_launch = getattr(B.lib, "_ZN3rtp16launch_gemm_bf16EiRKNS_8GemmArgsEiP12ihipStream_t")
_launch.restype = C.c_int
_launch.argtypes = [C.c_int, C.POINTER(GemmArgs), C.c_int, C.c_void_p]


def plan(layout, M, N, K, epi=EPI_STORE, half=0, f32=False, dtype="bf16", cu_share=1, force=0, sync=False):
    """(tile, K split) the launcher picks for one GEMM.  Needs no GPU: an fp32 sum lives at a made-up address."""
    a = GemmArgs(M=M, N=N, K=K, epi=epi, half=half, c_is_f32=int(f32), elem=ELEM[dtype], cu_share=cu_share, C=0x1000, ldc=N)
    if epi in (EPI_ACC_FIRST, EPI_ACC_ADD):
        a.ws, a.ldws, a.c_is_f32 = 0x1000, N, 1
    if sync:
        a.sync = 0x2000
    bm, ks = C.c_int(0), C.c_int(0)
    _plan(layout, C.byref(a), 1, C.byref(C.c_int(force)), C.byref(bm), C.byref(ks))
    return bm.value, ks.value


def riding_split(M, N, K, dx, cu_share=2):
    """Chunks of K of a weight gradient [M, N] over K in the launch it shares with the input gradient `dx` = (M, N, K, epi)."""
    w = GemmArgs(M=M, N=N, K=K, epi=EPI_ACC_ADD, c_is_f32=1, cu_share=cu_share, C=0x1000, ws=0x1000, ldc=N, ldws=N, lda=M, ldb=N)
    x = GemmArgs(M=dx[0], N=dx[1], K=dx[2], epi=dx[3], cu_share=cu_share, C=0x3000, ws=0x5000, ldc=dx[1], ldws=dx[1], lda=dx[2], ldb=dx[1])
    ks = (C.c_int * 2)(1, 1)
    _plan_riding((C.c_int * 2)(B.LAYOUT_NN, B.LAYOUT_TN), (GemmArgs * 2)(x, w), 2, ks)
    return ks[1]


_riding_tiles = getattr(B.lib, "_ZN3rtp25gemm_bf16_pp_riding_tilesEPKiPKNS_8GemmArgsEiPiS5_")
_riding_tiles.restype = None
_riding_tiles.argtypes = [C.POINTER(C.c_int), C.POINTER(GemmArgs), C.c_int, C.POINTER(C.c_int), C.POINTER(C.c_int)]


def riding_plan(group, ldc_pad=0):
    """(tile, K split) of each problem of a riding launch of (layout, M, N, K, epi) problems."""
    args = (GemmArgs * len(group))()
    for a, (layout, M, N, K, epi) in zip(args, group):
        sum_ = layout == B.LAYOUT_TN and epi == EPI_ACC_ADD  # a weight gradient: fp32, in place
        a.M, a.N, a.K, a.epi, a.half, a.C, a.ws, a.aux = M, N, K, epi, N // 2 if epi == EPI_SWIGLU_FWD else N, 0x1000 if sum_ else 0x3000, 0x1000, 0x2000
        a.ldc = a.ldws = (a.half if epi == EPI_SWIGLU_FWD else N) + ldc_pad
        a.ldaux, a.cu_share, a.c_is_f32 = 2 * N, 2, int(sum_)
    tiles, ks = (C.c_int * len(group))(), (C.c_int * len(group))()
    _riding_tiles((C.c_int * len(group))(*[g[0] for g in group]), args, len(group), tiles, ks)
    return list(zip(tiles, ks))


def riding_tiles(group, ldc_pad=0):
    """Its tiles alone."""
    return [tile for tile, _ in riding_plan(group, ldc_pad)]


SMALL_128X128, DUO_128X128, DUO_64X128, DUO_64X64 = 1000, 1024, 1025, 1026


def chunks(K, tile, ks, layout):
    """(chunks, K of each but the last) of a contraction over K that `tile` cuts in `ks`."""
    bk = 32 if tile in (256, 192, 128) or (tile == DUO_128X128 and layout == B.LAYOUT_TN) else 64
    subs = -(-K // bk)
    each = -(-subs // ks)
    return -(-subs // each), each * bk if ks > 1 else 0


def launch(layout, args, variant, stream=None):
    """launch_gemm_bf16 with the given arguments on kernel `variant`; the HIP status."""
    return _launch(layout, C.byref(args), variant, stream)


class RideSeg(C.Structure):
    _fields_ = [("out", C.c_void_p), ("buf", C.c_void_p), ("in_", C.c_void_p), ("bytes", C.c_size_t)]


class RideSum(C.Structure):
    _fields_ = [("elem", C.c_int), ("Y", C.c_void_p), ("ld", C.c_int64), ("rows", C.c_int), ("cols", C.c_int), ("in_", C.c_void_p), ("out", C.c_void_p)]


class Riders(C.Structure):
    _fields_ = [("count", C.c_int), ("sums", C.c_int), ("seg", RideSeg * 8), ("sum", RideSum * 2)]


_launch_riding = getattr(B.lib, "_ZN3rtp26launch_gemm_bf16_pp_ridingEPKiPKNS_8GemmArgsEiRKNS_6RidersEP12ihipStream_t")
_launch_riding.restype = C.c_int
_launch_riding.argtypes = [C.POINTER(C.c_int), C.POINTER(GemmArgs), C.c_int, C.POINTER(Riders), C.c_void_p]


def launch_riding(layouts, args, riders, stream=None):
    """One riding launch; the HIP status."""
    return _launch_riding((C.c_int * len(layouts))(*layouts), (GemmArgs * len(args))(*args), len(args), C.byref(riders), stream)


_colsum = getattr(B.lib, "_ZN3rtp13launch_colsumEiPKvliiPKfPfP12ihipStream_t")
_colsum.restype = C.c_int
_colsum.argtypes = [C.c_int, C.c_void_p, C.c_int64, C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_void_p]


def colsum(elem, Y, ld, rows, cols, into, out, stream=None):
    """out[c] = into[c] + sum over rows of Y[r, c]; elem -1: fp32.  Tensors must be on the GPU."""
    return _colsum(elem, Y.data_ptr(), ld, rows, cols, into.data_ptr(), out.data_ptr(), stream)
