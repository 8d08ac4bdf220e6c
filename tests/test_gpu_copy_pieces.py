"""The staging copy at the edges of its 32 KB pieces (64 KB beside long steps, 16 KB where nothing runs beside it): every unit arrives, nothing beyond them is touched."""
import ctypes as C

import pytest
import torch

from paper_2311_01635_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PIECE = 2048                                     # 16-byte units


@pytest.mark.parametrize("units", [1, 255, PIECE // 2 - 1, PIECE // 2, PIECE // 2 + 1, PIECE - 1, PIECE, PIECE + 1,
                                   2 * PIECE - 1, 2 * PIECE, 2 * PIECE + 1, 3 * PIECE, 6 * PIECE, 6 * PIECE + 257])
def test_copy(units):
    one = getattr(B.lib, "_ZN3rtp11launch_copyEPvPKvmP12ihipStream_tP11ihipEvent_t")
    one.restype, one.argtypes = C.c_int, [C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p, C.c_void_p]
    long, alone = (getattr(B.lib, f"_ZN3rtp{len(name)}{name}EPvPKvmP12ihipStream_tP11ihipEvent_t") for name in ("launch_copy_long", "launch_copy_alone"))
    for f in (long, alone):
        f.restype, f.argtypes = one.restype, one.argtypes
    many = getattr(B.lib, "_ZN3rtp17launch_copy_multiEPKPvPKPKvPKmiP12ihipStream_tP11ihipEvent_t")
    many.restype = C.c_int
    many.argtypes = [C.POINTER(C.c_void_p), C.POINTER(C.c_void_p), C.POINTER(C.c_size_t), C.c_int, C.c_void_p, C.c_void_p]
    stream = torch.cuda.current_stream().cuda_stream
    for call, count in ((one, 1), (one, 3), (long, 1), (alone, 1)):
        src = [torch.randint(0, 2 ** 31, (units * 4 + 8,), dtype=torch.int32, device=DEV) for _ in range(count)]
        dst = [torch.full_like(s, 7) for s in src]
        print(f"copy of {units} units, {count} segments", flush=True)
        if count == 1:
            assert call(dst[0].data_ptr() + 16, src[0].data_ptr() + 16, units * 16, stream, None) == 0
        else:
            at = lambda ts: (C.c_void_p * count)(*[t.data_ptr() + 16 for t in ts])
            assert many(at(dst), at(src), (C.c_size_t * count)(*[units * 16] * count), count, stream, None) == 0
        torch.cuda.synchronize()
        for d, s in zip(dst, src):
            assert torch.equal(d[4:-4], s[4:-4]) and (d[:4] == 7).all() and (d[-4:] == 7).all()
