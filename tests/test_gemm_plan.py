"""Which tile, and how many chunks of K, the launcher picks for a shape (needs no GPU)."""
import random

import pytest

import gemm_internal as G
from paper_2311_01635_amd import binding as B


@pytest.mark.parametrize("cu_share", [1, 2])
def test_gradients_of_a_ragged_batch_or_a_narrow_shard_are_not_split(cu_share):
    """The chunks of a split sum meet through atomic adds and do not repeat bit for bit: only sums over whole sub-tiles
    into outputs of at least 64 x 64 may be split, and only where the tall tiles alone would be."""
    for K in (200, 301, 1000, 1990, 5000):
        assert K % 32
        for M, N in ((384, 768), (128, 264), (688, 4096), (64, 64), (32, 768)):
            assert G.plan(B.LAYOUT_TN, M, N, K, G.EPI_ACC_ADD, cu_share=cu_share)[1] == 1, (M, N, K)
    for M, N in ((16, 768), (56, 4096), (768, 16), (768, 56)):
        for K in (256, 1024, 8192):
            assert G.plan(B.LAYOUT_TN, M, N, K, G.EPI_ACC_ADD, cu_share=cu_share)[1] == 1, (M, N, K)
    for M, N, K in ((64, 1376, 1024), (96, 1376, 1024), (128, 1376, 512)):
        assert G.plan(B.LAYOUT_TN, M, N, K, G.EPI_ACC_ADD, cu_share=cu_share)[1] == 1, (M, N, K)
    assert G.plan(B.LAYOUT_TN, 384, 768, 8192, G.EPI_ACC_ADD, cu_share=cu_share)[1] > 1, "a narrow shard's long sum is"


@pytest.mark.parametrize("N,K", [(256, 2048), (384, 768), (768, 384), (768, 2048), (1376, 4096)])
def test_a_prompt_runs_on_the_small_tile_whatever_its_length(N, K):
    """Few rows: the small tile is the fastest at every one of them, one row into a tall tile or eight past one."""
    for M in (8, 32, 56, 64, 72, 96, 128, 130, 136, 192, 200, 224, 256, 264, 270, 400, 512):
        assert G.plan(B.LAYOUT_NT, M, N, K) == (64, 1), M


def test_a_machine_full_of_tall_tiles_keeps_them():
    assert G.plan(B.LAYOUT_NT, 8192, 768, 2048)[0] == 128 and G.plan(B.LAYOUT_NT, 8192, 768, 384)[0] == 128
    assert G.plan(B.LAYOUT_NN, 4096, 4096, 2752)[0] == 256


def test_a_height_that_is_not_built_is_picked():
    shape = (B.LAYOUT_NT, 512, 768, 1024)
    for force in (1, 32, 96, 160, 512, -1):
        assert G.plan(*shape, force=force) == G.plan(*shape), force
    # a producer or consumer of a fused step counts tall tiles' rows: the small tile is not for it, forced or not
    assert G.plan(*shape, sync=True)[0] in (256, 192, 128)
    assert G.plan(*shape, force=64, sync=True) == G.plan(*shape, sync=True)
    for force in (256, 192, 128, 64):
        assert G.plan(*shape, force=force)[0] == force


def test_the_unit_tests_reach_the_small_tile():
    """The GEMMs of the units the GPU tests compare with the oracle (200 and 288 tokens) run on it, not only forced ones."""
    for epi, half, N in ((G.EPI_GELU_ERF_FWD, 0, 136), (G.EPI_SWIGLU_FWD, 136, 272)):
        assert G.plan(B.LAYOUT_NT, 200, N, 136, epi, half)[0] == 64
    for dtype in ("bf16", "f16"):
        assert G.plan(B.LAYOUT_NT, 288, 128, 160, G.EPI_GELU_TANH_FWD, dtype=dtype)[0] == 64
        assert G.plan(B.LAYOUT_NT, 288, 256, 160, G.EPI_SWIGLU_FWD, 128, dtype=dtype)[0] == 64
        assert G.plan(B.LAYOUT_NN, 288, 128, 96, G.EPI_GELU_TANH_BWD, dtype=dtype)[0] == 64
        assert G.plan(B.LAYOUT_NN, 288, 128, 96, G.EPI_SWIGLU_BWD, 128, dtype=dtype)[0] == 64


def test_a_riding_launch_does_not_split_a_sum_that_repeats_on_the_streams():
    """One chunk stays one, two stay at most two (they repeat onto zeros), whatever the machine to itself would favour."""
    rng = random.Random(5)
    chunks = set()
    shapes = [(544, 2560, 2208), (384, 768, 1024), (1792, 864, 5120), (1344, 1248, 3520), (960, 256, 1664)]
    shapes += [(32 * rng.randint(2, 48), 64 * rng.randint(4, 64), 32 * rng.randint(1, 256)) for _ in range(150)]
    for M, N, K in shapes:
        alone = G.plan(B.LAYOUT_TN, M, N, K, G.EPI_ACC_ADD, cu_share=2)[1]
        for dx in ((K, N, M, G.EPI_ACC_ADD), (K, M, N, G.EPI_GELU_ERF_BWD)):
            riding = G.riding_split(M, N, K, dx)
            assert riding <= alone or alone > 2, (M, N, K, dx, alone, riding)
            chunks.add(riding)
    assert 1 in chunks and 2 in chunks and max(chunks) > 2


SMALL_128X128, DUO_128X128, DUO_64X128, DUO_64X64 = 1000, 1024, 1025, 1026


def test_which_kernel_a_riding_launch_runs_on():
    """Few or short tiles: two workgroups a compute unit; a machine full of long ones: the tall tiles."""
    duo, tall = (DUO_128X128, DUO_64X128, DUO_64X64), (256, 192, 128, 64)
    for M, N, K in ((200, 768, 2048), (32, 768, 2048), (512, 2048, 1024), (1024, 384, 768)):
        assert G.riding_tiles([(B.LAYOUT_NT, M, N, K, G.EPI_STORE)])[0] in duo, (M, N, K)
    for M, N, K in ((4096, 4096, 4096), (8192, 2048, 2048)):
        assert G.riding_tiles([(B.LAYOUT_NT, M, N, K, G.EPI_STORE)])[0] in tall, (M, N, K)
    # a machine that 128 x 128 tiles fill about once, and taller ones do not
    assert G.riding_tiles([(B.LAYOUT_NT, 1990, 1376, 4096, G.EPI_SWIGLU_FWD), (B.LAYOUT_NT, 1990, 4096, 688, G.EPI_ACC_ADD)])[0] == SMALL_128X128
    for last in (G.EPI_GELU_TANH_BWD, G.EPI_ACC_LAST):
        assert all(t in duo for t in G.riding_tiles([(B.LAYOUT_NN, 1024, 384, 768, last), (B.LAYOUT_TN, 768, 384, 1024, G.EPI_ACC_LAST)]))


def test_a_riding_launch_is_of_one_kernel_and_of_tiles_that_take_the_problem():
    rng = random.Random(11)
    seen = set()
    for _ in range(300):
        T, w, I = 8 * rng.randint(1, 1024), 8 * rng.randint(1, 200), 8 * rng.randint(16, 1000)
        epi = rng.choice([G.EPI_STORE, G.EPI_ACC_ADD, G.EPI_SWIGLU_FWD, G.EPI_GELU_ERF_FWD])
        group = [(B.LAYOUT_NT, T, 2 * w if epi == G.EPI_SWIGLU_FWD else w, I, epi), (B.LAYOUT_NT, T, I, w, G.EPI_ACC_ADD)]
        tiles = G.riding_tiles(group, ride_bytes=4.0 * w * I)
        seen.update(tiles)
        assert len({t >= DUO_128X128 for t in tiles}) == 1, (group, tiles)
        assert epi != G.EPI_SWIGLU_FWD or tiles[0] != DUO_64X64, (group, tiles)
        # an odd leading dimension takes the element-wise epilogue, which the tall tiles have
        assert all(t < DUO_128X128 for t in G.riding_tiles(group, ldc_pad=1)), group
    assert seen >= {DUO_128X128, DUO_64X128, DUO_64X64, 256}
