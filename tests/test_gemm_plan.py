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


# Weight gradients [M, N] over K and the input gradient of their launch (columns, K, epilogue) -> how many chunks the sum is
# cut in and the K of each but the last, 0 for one: in a riding launch, in a launch of its own, beside another GEMM.
CUTS = [
    (384, 768, 8192, 768, 384, 2, 2, 4096, 4, 2048, 4, 2048),
    (768, 384, 8192, 384, 768, 7, 8, 1024, 4, 2048, 4, 2048),
    (576, 832, 5056, 832, 576, 2, 2, 2560, 4, 1280, 4, 1280),
    (1344, 576, 7904, 576, 1344, 7, 1, 0, 2, 3968, 2, 3968),
    (576, 1344, 7904, 1344, 576, 2, 1, 0, 2, 3968, 4, 1984),
    (832, 1120, 7904, 1120, 832, 2, 1, 0, 2, 3968, 2, 3968),
    (704, 2688, 5216, 2688, 704, 2, 1, 0, 1, 0, 1, 0),
    (2688, 352, 5216, 704, 2688, 9, 1, 0, 2, 2624, 2, 2624),
    (896, 1152, 7968, 1152, 896, 2, 2, 4032, 2, 4032, 2, 4032),
    (1152, 896, 7968, 896, 1152, 7, 1, 0, 2, 4032, 2, 4032),
    (1248, 2432, 2560, 2432, 1248, 2, 1, 0, 2, 1280, 1, 0),
    (2432, 1248, 2560, 1248, 2432, 7, 1, 0, 2, 1280, 1, 0),
    (1280, 2176, 3648, 2176, 1280, 2, 2, 1824, 4, 928, 2, 1824),
    (1024, 2432, 6496, 2432, 1024, 2, 2, 3264, 4, 1632, 4, 1632),
    (3200, 1280, 4512, 1280, 3200, 9, 1, 0, 2, 2272, 2, 2272),
    (928, 1856, 6464, 1856, 928, 2, 4, 1632, 1, 0, 4, 1632),
    (1856, 928, 6464, 928, 1856, 9, 2, 3232, 1, 0, 4, 1632),
    (928, 3392, 6144, 3392, 928, 2, 2, 3072, 2, 3072, 2, 3072),
    (3392, 928, 6144, 928, 3392, 9, 1, 0, 2, 3072, 2, 3072),
    (768, 2432, 5312, 2432, 768, 2, 1, 0, 1, 0, 2, 2656),
    (2432, 768, 5312, 768, 2432, 9, 2, 2656, 1, 0, 2, 2656),
    (512, 3904, 5408, 3904, 512, 2, 2, 2720, 1, 0, 4, 1376),
    (3904, 512, 5408, 512, 3904, 9, 4, 1376, 1, 0, 4, 1376),
    (704, 2432, 6336, 2432, 704, 2, 1, 0, 1, 0, 4, 1600),
    (2176, 1280, 3648, 1280, 2176, 7, 2, 1824, 4, 928, 2, 1824),
    (2432, 1024, 6496, 1024, 2432, 9, 2, 3264, 4, 1632, 4, 1632),
    (1344, 3776, 3872, 3776, 1344, 2, 1, 0, 2, 1952, 1, 0),
    (3776, 1344, 3872, 1344, 3776, 7, 1, 0, 2, 1952, 1, 0),
    (2944, 64, 6688, 64, 2944, 7, 2, 3392, 4, 1728, 4, 1728),
    (1248, 384, 1920, 384, 1248, 2, 2, 960, 4, 512, 2, 960),
    (384, 1248, 1920, 1248, 384, 9, 2, 960, 4, 512, 2, 960),
    (3584, 96, 7008, 96, 3584, 9, 2, 3520, 4, 1792, 4, 1792),
    (640, 800, 1728, 800, 640, 7, 1, 0, 2, 896, 1, 0),
    (3648, 1088, 4064, 1088, 3648, 9, 1, 0, 2, 2048, 1, 0),
    (3712, 96, 6208, 96, 3712, 9, 2, 3136, 4, 1600, 4, 1600),
    (1408, 3072, 5600, 3072, 1408, 2, 1, 0, 2, 2816, 1, 0),
    (3072, 1408, 5600, 1408, 3072, 7, 1, 0, 2, 2816, 1, 0),
    (192, 1920, 3456, 1920, 192, 2, 2, 1728, 4, 896, 2, 1728),
]


def test_which_sums_repeat_does_not_depend_on_the_tile():
    """Where a sum is cut decides its bits, and whether they repeat (one chunk always, two onto zeros).  The tall and the
    64 x 128 tiles' plans decide it: every tile cuts such a sum there.  More chunks do not repeat, and do not become more."""
    def same(want, got, what):
        assert got == want if want[0] <= 2 else 2 <= got[0] <= want[0], (what, want, got)

    for M, N, K, cols, depth, epi, rc, rk, ac, ak, sc, sk in CUTS:
        pair = [(B.LAYOUT_NN, K, cols, depth, epi), (B.LAYOUT_TN, M, N, K, G.EPI_ACC_ADD)]
        same((rc, rk), G.chunks(K, *G.riding_plan(pair)[1], B.LAYOUT_TN), ("riding", M, N, K))
        for share, want in ((1, (ac, ak)), (2, (sc, sk))):
            same(want, G.chunks(K, *G.plan(B.LAYOUT_TN, M, N, K, G.EPI_ACC_ADD, cu_share=share), B.LAYOUT_TN), (share, M, N, K))


def test_the_splits_asked_about_are_the_launchs():
    """A gradient's send is fused into the launch that completes it only where that launch does not split its sum."""
    rng = random.Random(17)
    shapes = [(384, 864, 2016, (2016, 864, 384, G.EPI_GELU_ERF_BWD)), (1472, 1728, 3008, (3008, 1728, 1472, G.EPI_ACC_ADD))]
    for _ in range(150):
        M, N, K = 32 * rng.randint(2, 48), 64 * rng.randint(4, 64), 32 * rng.randint(8, 256)
        shapes += [(M, N, K, (K, N, M, G.EPI_ACC_ADD)), (N, M, K, (K, M, N, G.EPI_GELU_ERF_BWD))]
    split = 0
    for M, N, K, dx in shapes:
        asked = G.riding_split(M, N, K, dx)
        launched = G.riding_plan([(B.LAYOUT_NN,) + dx, (B.LAYOUT_TN, M, N, K, G.EPI_ACC_ADD)])[1][1]
        assert launched == asked if asked <= 2 else 2 <= launched <= asked, (M, N, K, dx, asked, launched)
        split += asked > 2
    assert 5 < split < 100


def test_plans_are_not_kept_without_end():
    """An expert layer meets another number of tokens every step: 150 000 plans of 200 bytes and more would be 30 MB."""
    grown = []
    for at in range(4):
        for T in range(25000):
            G.plan(B.LAYOUT_NT, 8 + T, 64 + 8 * at, 64)
        with open("/proc/self/statm") as f:
            grown.append(int(f.read().split()[1]) * 4096)
    assert grown[3] - grown[0] < 8 << 20, grown


SMALL_128X128, DUO_128X128, DUO_64X128, DUO_64X64 = G.SMALL_128X128, G.DUO_128X128, G.DUO_64X128, G.DUO_64X64


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


def test_square_tiles_do_not_crowd_the_machine():
    """128 x 128 tiles are for problems that they fill the 256 compute units with one and a half times at most."""
    for layout, M, N, K, epi in ((B.LAYOUT_NN, 1160, 9600, 6176, G.EPI_STORE), (B.LAYOUT_TN, 1192, 9512, 1760, G.EPI_ACC_ADD),
                                 (B.LAYOUT_TN, 3480, 3448, 5440, G.EPI_STORE), (B.LAYOUT_NN, 6664, 1144, 2912, G.EPI_STORE)):
        assert G.plan(layout, M, N, K, epi)[0] != SMALL_128X128, (layout, M, N, K)
    assert G.plan(B.LAYOUT_TN, 1784, 1320, 2176)[0] == G.plan(B.LAYOUT_NT, 936, 4056, 1728)[0] == SMALL_128X128
    assert SMALL_128X128 not in G.riding_tiles([(B.LAYOUT_NN, 6488, 936, 2816, G.EPI_GELU_ERF_BWD), (B.LAYOUT_TN, 2816, 936, 6488, G.EPI_ACC_LAST)])[:1]
    rng = random.Random(29)
    for _ in range(400):
        M, N, K = 8 * rng.randint(8, 1000), 8 * rng.randint(8, 1200), 32 * rng.randint(2, 200)
        for layout, epi in ((B.LAYOUT_NT, G.EPI_STORE), (B.LAYOUT_TN, G.EPI_ACC_ADD)):
            tile, ks = G.plan(layout, M, N, K, epi)
            assert tile != SMALL_128X128 or -(-M // 128) * -(-N // 128) * ks <= 384, (layout, M, N, K)


def test_a_gated_prompt_keeps_a_compute_unit_to_a_tile():
    """Pairs of gate and up columns have no 64 x 64 tile: with the wider ones the forward pass of these units (tokens, inputs,
    units of a shard) takes up to a fifth longer, whatever rides in its launches."""
    for T, I, o in ((16, 2368, 1568), (64, 3072, 1808), (64, 3584, 1552), (96, 3392, 1600), (160, 2688, 1488), (320, 3456, 1640),
                    (384, 2496, 1360), (512, 2624, 1336), (768, 1344, 744)):
        group = [(B.LAYOUT_NT, T, 2 * o, I, G.EPI_SWIGLU_FWD), (B.LAYOUT_NT, T, I, o, G.EPI_ACC_ADD)]
        assert all(t < DUO_128X128 for g in (group, group[:1]) for t in G.riding_tiles(g)), (T, I, o)


def test_a_riding_launch_is_of_one_kernel_and_of_tiles_that_take_the_problem():
    rng = random.Random(11)
    seen = set()
    for _ in range(300):
        T, w, I = 8 * rng.randint(1, 1024), 8 * rng.randint(1, 200), 8 * rng.randint(16, 1000)
        epi = rng.choice([G.EPI_STORE, G.EPI_ACC_ADD, G.EPI_SWIGLU_FWD, G.EPI_GELU_ERF_FWD])
        group = [(B.LAYOUT_NT, T, 2 * w if epi == G.EPI_SWIGLU_FWD else w, I, epi), (B.LAYOUT_NT, T, I, w, G.EPI_ACC_ADD)]
        tiles = G.riding_tiles(group)
        seen.update(tiles)
        assert len({t >= DUO_128X128 for t in tiles}) == 1, (group, tiles)
        assert epi != G.EPI_SWIGLU_FWD or tiles[0] != DUO_64X64, (group, tiles)
        # an odd leading dimension takes the element-wise epilogue, which the tall tiles have
        assert all(t < DUO_128X128 for t in G.riding_tiles(group, ldc_pad=1)), group
    assert seen >= {DUO_128X128, DUO_64X128, DUO_64X64, 256}
