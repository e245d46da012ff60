"""Which kernel a call runs is host arithmetic (prices fitted to measured times): its choices without a GPU.

The library's internal functions say which way a call of given sizes would go on a device of `cus` compute units.
"""
import pytest

from tests import routes

CUS = 256
MAX_THREADS = 2 ** 32 - 1        # of a launch: a dispatch states its grid as 32-bit thread counts


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("scratch", [True, False])
@pytest.mark.parametrize("n,heads", [(64, 1 << 23), (33, 1 << 23), (96, (1 << 24) // 3), (256, 1 << 21), (32, (1 << 24) - 1)])
def test_attention_never_takes_a_grid_that_cannot_be_launched(n, heads, scratch, hd):
    """Millions of very short heads: the short kernel takes 256 threads for every 32 rows of a head."""
    threads = 256 * heads * -(-n // 32)
    assert threads <= MAX_THREADS or routes.attention_tiles(n, heads, hd, scratch, CUS).rows > 0


@pytest.mark.parametrize("hd", [64, 128])
def test_calls_of_up_to_32_tokens_stay_with_the_short_kernel(hd):
    """The one whose offsets hold tokens 2^27 elements apart; its grid can be launched for any number of heads then."""
    for n in (1, 2, 15, 31, 32):
        for heads in (1, 40, 5000, 1 << 20, (1 << 24) - 1):
            for scratch, split, cus in ((True, False, CUS), (False, True, CUS), (True, True, 8), (False, False, 304)):
                assert routes.attention_tiles(n, heads, hd, scratch, cus, split).rows == 0


@pytest.mark.parametrize("head_dim", [0, 64, 128])
@pytest.mark.parametrize("d_in", [64, 128, 512, 5120])
def test_gemm_never_takes_a_grid_that_cannot_be_launched(d_in, head_dim):
    """Tilings smaller than 256 x 256 are left out where they would need 2^32 threads; 256 x 256 takes the call."""
    for d_out in (128, 384, 1536, 15360, 1 << 20):
        for shift in range(10, 31):
            for n in (1 << shift, (1 << shift) - 77, 3 << (shift - 1)):
                way = routes.gemm(n, d_in, d_out, head_dim, CUS)
                assert way.workgroups * way.threads <= MAX_THREADS or (way.tile, way.cut) == ((256, 256), None), (n, d_out, way)


# us on 256 compute units with scratch memory of the short kernel / query tiles of 256 (whole or cut) / 192 / 128 rows, and the rows taken
# (0: short kernel)
@pytest.mark.parametrize("n,heads,hd,rows", [
    (225, 256, 128, 256),    # 28.5 / 20.1 / 25.3 / 21.0
    (200, 256, 128, 256),    # 25.3 / 18.9 / 24.1 / 20.1
    (200, 200, 128, 256),    # 21.6 / 17.0 / 23.6 / 19.0
    (160, 256, 128, 192),    # 18.7 / 15.0 / 12.9 / 17.2
    (384, 256, 128, 192),    # 47.5 / 38.5 / 32.7 / 34.4
    (257, 1000, 64, 0),      # 54.7 / 73.8 / 61.6 / 67.7
    (129, 2000, 64, 0),      # 47.6 / 62.3 / 52.6 / 74.3
    (300, 640, 64, 192),     # 42.6 / 48.9 / 41.4 / 47.7
    (600, 400, 64, 128),     # 74.1 / 67.4 / 70.9 / 64.8
    (850, 150, 64, 192),     # 49.4 / 49.2 / 41.5 / 50.2
    (200, 4, 64, 0),         # 5.0 / 10.3 / 9.0 / 7.6
    (1000, 12, 128, 0),      # 15.4 / 24.7 / 22.5 / 17.4
    (1000, 24, 128, 128),    # 24.3 / 26.7 / 23.2 / 18.3
    (900, 60, 64, 256),      # 24.3 / 19.1 / 27.2 / 22.5
    (2999, 16, 64, 192),     # 52.1 / 39.4 / 34.3 / 47.2
    (3780, 12, 128, 192),    # 121.6 / 75.0 / 68.6 / 95.2
    (4212, 12, 128, 256),    # 153.3 / 84.6 / 133.3 / 103.2
    (4500, 16, 128, 256),    # 209.0 / 130.8 / 142.1 / 161.7
])
def test_attention_takes_the_faster_way(n, heads, hd, rows):
    assert routes.attention_tiles(n, heads, hd, True, CUS).rows == rows


# us, whole / cut: 256-row query tiles of a last round that leaves few compute units idle, and of one that leaves most
@pytest.mark.parametrize("n,heads,hd,cut", [
    (4212, 12, 128, False),  # 84.6 / 94.7
    (4680, 12, 128, False),  # 99.6 / 114.1
    (4500, 16, 128, True),   # 178.8 / 130.8
    (4500, 16, 64, True),    # 110.6 / 80.8
    (5000, 2, 128, True),    # 88.4 / 39.7
    (2000, 70, 128, True),   # 140.0 / 121.2
])
def test_attention_cuts_the_tiles_of_a_last_round(n, heads, hd, cut):
    assert routes.attention_tiles(n, heads, hd, True, CUS) == (256, 0, cut)
    assert not routes.attention_tiles(n, heads, hd, False, CUS).cut


# us, short kernel / 256-row query tiles (whole or cut) / 192 / 128, of calls whose rows are split over cache lines (short kernel
# and the tiles taken with whole lines)
@pytest.mark.parametrize("n,heads,hd,rows", [
    (1628, 25, 64, 192),     # 45.2 / 26.6 / 23.0 / 35.8 (27.6, 21.7)
    (1542, 22, 64, 192),     # 35.6 / 25.3 / 21.3 / 34.2 (25.8, 20.9)
    (861, 201, 64, 192),     # 83.7 / 68.4 / 56.6 / 65.6 (65.8, 54.5)
    (1063, 73, 64, 192),     # 49.7 / 38.0 / 33.3 / 39.8 (36.9, 31.0)
    (1625, 38, 128, 128),    # 88.7 / 67.7 / 62.8 / 53.6 (77.6, 51.2)
    (1777, 17, 128, 128),    # 52.8 / 40.7 / 33.5 / 30.2 (44.0, 28.5)
    (2963, 11, 128, 192),    # 82.3 / 57.0 / 48.6 / 80.1 (68.0, 47.7)
])
def test_calls_of_split_rows_that_run_tiles(n, heads, hd, rows):
    for split in (False, True):
        assert routes.attention_tiles(n, heads, hd, True, CUS, split=split).rows == rows


# us, short kernel in whole lines / split, and the tiles taken from it where rows are split
@pytest.mark.parametrize("n,heads,hd,tiles", [
    (640, 32, 64, (128, 0, False)),      # 9.8 / 11.8, 10.2
    (2444, 6, 64, (128, 0, False)),      # 17.1 / 22.5, 21.0
    (1969, 8, 128, (128, 0, False)),     # 25.0 / 30.9, 26.1
    (582, 121, 64, (192, 0, False)),     # 23.5 / 28.2, 24.0
    (600, 75, 64, (256, 0, False)),      # 16.4 / 19.6, 16.1
    (3094, 3, 64, (256, 0, True)),       # 19.1 / 24.4, 22.7
])
def test_split_rows_keep_a_call_from_the_short_kernel(n, heads, hd, tiles):
    assert routes.attention_tiles(n, heads, hd, True, CUS).rows == 0
    assert routes.attention_tiles(n, heads, hd, True, CUS, split=True) == tiles


# us of split rows, token-major / head-major, short kernel and the best of the tiles: heads of few rounds of 128 keys lose little there, while
# tiles of 192 and 128 rows fetch more lines for every tile of keys
@pytest.mark.parametrize("n,heads,hd", [
    (153, 411, 64),          # 14.6 / 14.8, 16.1 / 18.6
    (295, 311, 64),          # 25.4 / 24.3, 27.4 / 28.1
    (261, 213, 64),          # 16.5 / 17.2, 18.7 / 19.3
    (189, 519, 64),          # 22.3 / 22.3, 24.7 / 27.4
    (260, 95, 64),           # 9.8 / 9.2, 10.5 / 10.2
    (154, 195, 64),          # 8.2 / 8.2, 9.0 / 9.1
    (174, 87, 64),           # 7.3 / 6.8, 7.8 / 7.5
])
def test_split_rows_of_few_keys_stay_with_the_short_kernel(n, heads, hd):
    assert routes.attention_tiles(n, heads, hd, True, CUS, split=True).rows == 0


def test_split_rows_leave_small_calls_with_the_short_kernel():
    for n, heads, hd in ((200, 4, 64), (600, 24, 64), (1000, 12, 128)):      # 10.0 / 16.7 and 17.8 / 27.8 us for the latter two
        assert routes.attention_tiles(n, heads, hd, True, CUS, split=True).rows == 0


@pytest.mark.parametrize("hd", [64, 128])
def test_which_rows_are_split(hd):
    base = 1 << 20
    one = lambda k=base, v=base, tok=3 * hd, head=hd, batch=0, heads=3, items=1: routes.rows_split(k, v, tok, head, batch, heads, items, hd)
    assert not one()
    assert one(k=base + 16) and one(v=base + 64) and not one(k=base + 128)
    assert one(tok=3 * hd + 8) and one(tok=3 * (hd + 8), head=hd + 8)
    assert not one(head=hd + 8, heads=1, tok=4 * hd)                         # no second head, no second item
    assert not one(batch=9 * hd + 8) and one(batch=9 * hd + 8, items=2)
    assert not one(k=base + 16, tok=hd, head=100 * hd)                       # head-major: one row directly behind the other
    assert not one(tok=hd + 8, head=100 * (hd + 8)) and one(tok=hd + 72, head=100 * (hd + 72))


# us on 256 compute units of the tiles taken / of 128 x 64 tiles: products of a short k, where a tile is little more than
# its first loads and its stores
@pytest.mark.parametrize("n,d_in,d_out,tiles", [
    (200000, 64, 1536, [(256, 256)]),              # 130 / 292
    (60000, 64, 3840, [(256, 256)]),               # 96 / 219
    (10000, 64, 13824, [(256, 256)]),              # 59 / 131
    (4096, 64, 5120, [(256, 256)]),                # 13 / 23
    (200000, 128, 640, [(256, 256)]),              # 78 / 162
    (6500, 128, 5120, [(256, 256)]),               # 22 / 39
    (60000, 256, 640, [(256, 256), (256, 128)]),   # 35 / 59
    (1500, 256, 5120, [(256, 256), (256, 128)]),   # 10 / 14
])
def test_gemm_of_a_short_k_takes_large_tiles(n, d_in, d_out, tiles):
    assert routes.gemm(n, d_in, d_out, 0, CUS).tile in tiles


# us of the tiles taken / of those with twice the features or tokens, or half: one round that fills half of the chip
@pytest.mark.parametrize("n,d_in,d_out,head_dim,tile", [
    (1271, 704, 1536, 0, (128, 64)),      # 6.7 / 8.1
    (5095, 1792, 384, 0, (128, 64)),      # 11.6 / 14.2
    (14871, 896, 128, 0, (128, 64)),      # 7.6 / 8.9
    (1327, 1344, 1408, 0, (128, 64)),     # 9.2 / 11.6
    (135, 1792, 3200, 0, (64, 32)),       # 6.5 / 8.2
    (572, 1216, 768, 0, (64, 32)),        # 5.3 / 6.4
    (532, 1024, 3072, 128, (128, 64)),    # 9.6 / 11.7
    (910, 512, 1536, 128, (128, 64)),     # 7.3 / 9.0
    (2420, 256, 768, 64, (128, 64)),      # 6.6 / 7.8
])
def test_gemm_fills_the_chip_with_the_smaller_tile(n, d_in, d_out, head_dim, tile):
    assert routes.gemm(n, d_in, d_out, head_dim, CUS).tile == tile


@pytest.mark.parametrize("n,d_in,d_out,tile,cut", [
    (520, 5120, 640, (64, 32), None), (13230, 5120, 5120, (256, 256), (128, 64)), (13230, 5120, 15360, (256, 256), (128, 128)),
    (3780, 1536, 4608, (256, 256), (128, 64)), (3780, 1536, 1536, (256, 128), None), (2737, 1024, 1024, (128, 128), None),
    (24000, 256, 5120, (256, 256), None),          # 87 us; 106 with the last round cut: short rounds take longer in the kernel of two tilings
    (300, 13824, 3840, (128, 64), None),           # 59 us; 77 in 64 x 64: two of them on one compute unit take twice as long
])
def test_gemm_tiles_of_the_block(n, d_in, d_out, tile, cut):
    way = routes.gemm(n, d_in, d_out, 0, CUS)
    assert (way.tile, way.cut) == (tile, cut)
