"""The bias gradient's column sums, past one trip of the main loop and at its remainders, against 64-bit sums."""
import pytest
import torch

import gemm_internal as G

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TD = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_column_sums(dtype):
    elem = G.ELEM.get(dtype, -1)
    # 16-byte loads: 256 row groups, four in flight: the main loop starts at 769 rows; single elements: 32, at 97 rows
    for rows in (0, 1, 31, 97, 128, 255, 257, 768, 769, 1024, 1056, 1990, 2080):
        for cols, pad, shift in ((8, 0, 0), (40, 8, 0), (384, 0, 0), (72, 0, 8), (31, 1, 0), (100, 4, 0), (64, 0, 1)):
            g = torch.Generator(device=DEV).manual_seed(rows + cols)
            ld = cols + pad
            flat = torch.full((shift + rows * ld + 2048,), float("nan"), device=DEV, dtype=TD[dtype])
            Y = flat[shift:shift + rows * ld].view(rows, ld)
            Y[:, :cols] = torch.randn(rows, cols, generator=g, device=DEV).to(TD[dtype])
            into = torch.randn(cols, generator=g, device=DEV)
            out = torch.full((cols + 1,), float("nan"), device=DEV)
            print(f"colsum {dtype} rows={rows} cols={cols} ld={ld} shift={shift}", flush=True)
            assert G.colsum(elem, flat[shift:], ld, rows, cols, into, out) == 0
            torch.cuda.synchronize()
            y = Y[:, :cols].double()
            # at most ceil(2080 / 32) + 32 + 32 additions in a chain, each rounding a partial sum below sum |y|
            bound = 130 * 2.0 ** -24 * (y.abs().sum(0) + into.double().abs()) + 1e-12
            assert bool(((out[:cols].double() - (into.double() + y.sum(0))).abs() <= bound).all()), (rows, cols, ld, shift)
            assert torch.isnan(out[cols]), (rows, cols)
            again = into.clone()                       # in place, as a shard that stays where it is; the same bits
            assert G.colsum(elem, flat[shift:], ld, rows, cols, again, again) == 0
            torch.cuda.synchronize()
            assert torch.equal(again, out[:cols]), (rows, cols, ld, shift)
