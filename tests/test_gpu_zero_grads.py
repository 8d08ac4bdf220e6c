"""rtp_ring_zero_grads clears every byte of the gradient store and none beside it."""
import pytest
import torch

from paper_2311_01635_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# a slot of one 16-byte unit, stores around one and two workgroups of 256 units, and one of many
@pytest.mark.parametrize("n,units", [(1, 1), (1, 255), (1, 256), (1, 257), (3, 171), (2, 256), (5, 20001)])
def test_the_store_and_nothing_else(n, units):
    gb, guard = 16 * units, 4096
    whole = torch.full((2 * guard + n * gb,), 0xA5, dtype=torch.uint8, device=DEV)
    store = whole[guard:guard + n * gb]
    new = lambda size: torch.empty(size, dtype=torch.uint8, device=DEV)
    streams = [torch.cuda.Stream(DEV) for _ in range(2)]
    torch.cuda.synchronize()
    ring = B.Ring(n, 0, B.RTP_DOUBLE_BUFFER, 16, gb, new(16 * n), store, [new(16), new(16)], [new(gb), new(gb)], *streams)
    ring.zero_grads()
    ring.sync()
    assert int(whole[guard:guard + n * gb].count_nonzero()) == 0
    assert bool((whole[:guard] == 0xA5).all()) and bool((whole[guard + n * gb:] == 0xA5).all())
    ring.close()
