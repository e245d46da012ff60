"""The library's internal say on which way a call goes, for tests that are about one kernel."""
import ctypes as C
from collections import namedtuple

from paper_2512_07350_amd import binding as lp


class GemmWay(namedtuple("GemmWay", "tile cut workgroups threads")):
    def __str__(self):
        """Features x tokens of a tile, + those of the tiles that cut the last round."""
        return "%dx%d" % self.tile + ("+%dx%d" % self.cut if self.cut else "")


def _cus(cus):
    if cus is None:
        import torch
        cus = torch.cuda.get_device_properties(torch.cuda.current_device()).multi_processor_count
    return cus


class Tiles(namedtuple("Tiles", "rows last cut")):
    """Query rows of attention_kernel's tiles (0: the short kernel), of those of its last round where they are smaller
    (else 0), and whether tiles are cut and merged."""


def attention_tiles(n, all_heads, head_dim, scratch=True, cus=None, split=False):
    """What a call runs.  split: see rows_split."""
    fn = lp._lib().lp_internal_attention_tiles
    fn.argtypes, fn.restype = [C.c_int64] + [C.c_int32] * 5 + [C.POINTER(C.c_int32)], C.c_int
    t = (C.c_int32 * 3)()
    assert fn(n, all_heads, head_dim, _cus(cus), int(scratch), int(split), t) == 0
    return Tiles(t[0], t[1], bool(t[2]))


def rows_split(k, v, stride_tok, stride_head, stride_batch, heads, batch, head_dim):
    """Whether the rows of K or V (byte addresses k, v) lie split over cache lines, with other rows in between."""
    fn = lp._lib().lp_internal_attention_rows_split
    fn.argtypes, fn.restype = [C.c_uint64] * 2 + [C.c_int64] * 3 + [C.c_int32] * 3, C.c_int
    return bool(fn(k, v, stride_tok, stride_head, stride_batch, heads, batch, head_dim))


def gemm(n, d_in, d_out, head_dim=0, cus=None):
    """head_dim 0: lp_linear, else lp_qkv_projection (d_out = 3 d_in)."""
    fn = lp._lib().lp_internal_gemm_way
    fn.argtypes, fn.restype = [C.c_int64] + [C.c_int32] * 4 + [C.POINTER(C.c_int64)], C.c_int
    way = (C.c_int64 * 6)()
    assert fn(n, d_in, d_out, head_dim, _cus(cus), way) == 0
    return GemmWay((way[0], way[1]), (way[2], way[3]) if way[2] else None, way[4], way[5])
