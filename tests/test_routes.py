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
    way = routes.attention(n, heads, hd, scratch, CUS)
    assert way == ("short" if threads <= MAX_THREADS else "whole")


@pytest.mark.parametrize("head_dim", [0, 64, 128])
@pytest.mark.parametrize("d_in", [64, 128, 512, 5120])
def test_gemm_never_takes_a_grid_that_cannot_be_launched(d_in, head_dim):
    """Tilings smaller than 256 x 256 are left out where they would need 2^32 threads; 256 x 256 takes the call."""
    for d_out in (128, 384, 1536, 15360, 1 << 20):
        for shift in range(10, 31):
            for n in (1 << shift, (1 << shift) - 77, 3 << (shift - 1)):
                way = routes.gemm(n, d_in, d_out, head_dim, CUS)
                assert way.workgroups * way.threads <= MAX_THREADS or (way.tile, way.cut) == ((256, 256), None), (n, d_out, way)


# us on 256 compute units, short kernel / 256-row query tiles (whole or cut), with scratch memory: calls of many heads and
# a few hundred tokens, where the dearer way costs 14 % and more
@pytest.mark.parametrize("n,heads,hd,way", [
    (225, 256, 128, "long"),     # 28.9 / 21.7
    (200, 256, 128, "long"),     # 25.5 / 19.8
    (200, 200, 128, "long"),     # 21.9 / 17.8
    (160, 256, 128, "long"),     # 19.1 / 16.0
    (384, 256, 128, "long"),     # 48.9 / 41.7
    (257, 1000, 64, "short"),    # 55.9 / 80.9
    (300, 640, 64, "short"),     # 42.6 / 55.9
    (129, 2000, 64, "short"),    # 51.0 / 66.9
    (600, 400, 64, "short"),     # 67.7 / 78.4
    (850, 150, 64, "short"),     # 48.4 / 55.6
    (200, 4, 64, "short"), (1000, 12, 128, "short"), (2999, 16, 64, "long"), (3780, 12, 128, "long"),
])
def test_attention_takes_the_faster_way(n, heads, hd, way):
    assert (routes.attention(n, heads, hd, True, CUS) == "short") == (way == "short")


# us, short kernel / 256-row query tiles, of calls whose rows are split over cache lines (short kernel with whole lines)
@pytest.mark.parametrize("n,heads,hd,whole_lines", [
    (1628, 25, 64, "short"),     # 49.0 / 30.1 (30.0)
    (1542, 22, 64, "short"),     # 36.5 / 28.2 (28.5)
    (861, 201, 64, "short"),     # 94.0 / 73.1
    (1063, 73, 64, "short"),     # 51.7 / 43.8
    (1625, 38, 128, "short"),    # 97.9 / 76.0 (87.9)
    (1777, 17, 128, "short"),    # 54.3 / 46.5 (49.3)
    (3427, 21, 64, "cut"), (2963, 11, 128, "cut"),
])
def test_split_rows_keep_a_call_from_the_short_kernel(n, heads, hd, whole_lines):
    assert routes.attention(n, heads, hd, True, CUS) == whole_lines
    assert routes.attention(n, heads, hd, True, CUS, split=True) in ("whole", "cut")


def test_split_rows_leave_small_calls_with_the_short_kernel():
    for n, heads, hd in ((200, 4, 64), (600, 24, 64), (1000, 12, 128)):      # 10.0 / 16.7 and 17.8 / 27.8 us for the latter two
        assert routes.attention(n, heads, hd, True, CUS, split=True) == "short"


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
