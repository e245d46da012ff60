"""attention_kernel on each of the query tiles that it is compiled for: 128, 192 and 256 rows throughout, rounds of 256 with a
last one of 192, and 256 with the last round cut and merged.  Every case says which of them it runs."""
import numpy as np
import pytest

from oracle import lp_oracle as orc
from paper_2512_07350_amd import synth
from tests import routes

pytestmark = pytest.mark.gpu

# heads, rows of a tile, of those of the last round, cut, and lengths whose last key tile holds 1, 31 .. 33 or 63, 64 keys and whose
# last query tile holds 1 row or all
KINDS = [
    (40, 128, 0, False, (640, 641, 672, 673, 703, 767, 768)),
    (40, 192, 0, False, (769, 800, 801, 831, 960, 961, 1151, 1152)),
    (40, 256, 0, False, (1153, 1184, 1217, 1280, 1281, 1535, 1536)),
    (40, 256, 192, False, (2433, 2464, 2465, 2527, 2560, 2561, 2688, 2689, 2815, 2816)),
    (70, 256, 192, False, (1345, 1376, 1409, 1472, 1535, 1536)),
    (70, 256, 0, True, (1921, 1952, 1953, 2015, 2047, 2048)),
]
CASES = [(n, heads, hd, rows, last, cut) for heads, rows, last, cut, ns in KINDS for n in ns for hd in (64, 128)]
CASES += [(n, 150, 128, 128, 0, False) for n in (117, 127, 128)] + [(n, 150, 128, 192, 0, False) for n in (129, 160, 161, 191, 192)]
CASES += [(n, 150, 64, 128, 0, False) for n in (353, 384)] + [(n, 150, 64, 192, 0, False) for n in (417, 447, 448)]


def runs(n, heads, hd, rows, last, cut, **how):
    assert routes.attention_tiles(n, heads, hd, **how) == (rows, last, cut)


@pytest.mark.parametrize("n,heads,hd,rows,last,cut", CASES)
def test_tiles_at_their_edges(n, heads, hd, rows, last, cut):
    from tests import gpu_util as g
    runs(n, heads, hd, rows, last, cut)
    q, k, v = synth.qkv_bf16(6100 + 2 * n + hd, n, heads, hd)
    got = g.hip_attention(q, k, v)
    picked = synth.sample_rows(n, 48, seed=n, tile=rows)
    g.assert_attention_close(got[picked], orc.attention(q, k, v, rows=picked), "n=%d hd=%d tiles of %d" % (n, hd, rows))
    assert np.all(np.isfinite(got))


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("n,rows,last", [(700, 128, 0), (1000, 192, 0), (2500, 256, 192)])
def test_tiles_taken_again_for_scores_far_above_the_first_round(n, rows, last, hd):
    """Scores 2^256 above the first 32 keys' from key 40 on: every tile is walked a second time with a running maximum."""
    from tests import gpu_util as g
    heads = 40
    runs(n, heads, hd, rows, last, False)
    rng = np.random.default_rng(4321)
    base = np.where(rng.random((heads, hd)) < 0.5, -1.0, 1.0).astype(np.float32)
    level = np.where(np.arange(n) < 40, 0.0, 32.0).astype(np.float32)
    qf = np.broadcast_to(base[None] * np.float32(64.0 / hd), (n, heads, hd)).copy()
    q, k, v = (synth.f32_to_bf16_bits(a) for a in (qf, base[None] * level[:, None, None], rng.standard_normal((n, heads, hd)).astype(np.float32)))
    scale = 0.125 / np.log2(np.e)
    got = g.hip_attention(q, k, v, scale=scale)
    picked = synth.sample_rows(n, 48, seed=7, tile=rows)
    g.assert_attention_close(got[picked], orc.attention(q, k, v, scale=scale, rows=picked), "scores far above the first round")
    assert np.all(np.isfinite(got))


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("n,rows,last", [(700, 128, 0), (1001, 192, 0), (2497, 256, 192)])
@pytest.mark.parametrize("layout", ["token-padded", "head-major-padded", "items-side-by-side"])
def test_tiles_on_strided_layouts(layout, n, rows, last, hd):
    """40 heads in all; every gap of q, k, v and o holds NaN: nothing is read from it or written to it."""
    import torch
    from tests import gpu_util as g
    from paper_2512_07350_amd import binding as lp
    batch = 2 if layout.startswith("items") else 1
    heads = 40 // batch
    runs(n, 40, hd, rows, last, False, split=True)
    if layout == "token-padded":
        stride_head, stride_batch = hd + 8, 0
        stride_tok = heads * stride_head + 24
    elif layout == "head-major-padded":
        stride_tok, stride_batch = hd + 72, 0
        stride_head = n * stride_tok + 40
    else:
        stride_head = hd + 8
        stride_batch = heads * stride_head + 16
        stride_tok = batch * stride_batch + 8
    total = (batch - 1) * stride_batch + (n - 1) * stride_tok + (heads - 1) * stride_head + hd + 64
    where = (np.arange(batch)[:, None, None, None] * stride_batch + np.arange(n)[:, None, None] * stride_tok
             + np.arange(heads)[:, None] * stride_head + np.arange(hd))
    items = [synth.qkv_bf16(6700 + hd + b, n, heads, hd) for b in range(batch)]

    def pack(j):
        buf = np.full(total, 0x7fc0, dtype=np.uint16)
        buf[where] = np.stack([it[j] for it in items])
        return g.to_dev_bf16(buf)

    qd, kd, vd = pack(0), pack(1), pack(2)
    od = torch.full((total,), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws, ws_bytes = g.workspace(hd)
    lp.lp_attention_batch(qd, kd, vd, od, batch, n, heads, hd, stride_batch, stride_tok, stride_head, 0.0, ws, ws_bytes, g.stream())
    torch.cuda.synchronize()
    out = g.from_dev_bf16(od)
    got = out[where]
    assert np.all(np.isfinite(got))
    picked = synth.sample_rows(n, 48, seed=hd, tile=rows)
    for b, (q, k, v) in enumerate(items):
        g.assert_attention_close(got[b][picked], orc.attention(q, k, v, rows=picked), "%s item %d hd=%d" % (layout, b, hd))
    out[where] = np.nan
    assert np.all(np.isnan(out)), "wrote outside its rows"


def dead_keys(n, heads, hd, dead, far, seed):
    """q, k, v whose keys dead[0] .. dead[1] - 1 have score -inf; the scores of the first `far` of them all lie 4096 hd^-1/2 / ln 2 (522 or
    738) log2 units lower."""
    q, k, v = synth.qkv_bf16(seed, n, heads, hd)
    q[:, :, 3:5] = 0x3f80                                # 1.0
    k[dead[0]:dead[1], :, 3] = 0xff80                    # -inf
    k[:far, :, 4] = 0xc580                               # -4096
    return q, k, v


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("far", [0, 0.7, 1], ids=["scores near 0", "far below, then near 0", "scores far below"])
@pytest.mark.parametrize("n,heads,rows,last,cut,dead", [
    (1000, 24, 128, 0, False, (0, 32)), (1000, 24, 128, 0, False, (0, 999)), (700, 40, 128, 0, False, (5, 640)), (1001, 40, 192, 0, False, (0, 500)),
    (1500, 40, 256, 0, False, (0, 64)), (1500, 40, 256, 0, False, (64, 1000)), (2500, 40, 256, 192, False, (0, 33)), (2500, 40, 256, 192, False, (0, 2499)),
    (5000, 2, 256, 0, True, (0, 32)), (5000, 2, 256, 0, True, (0, 2600)), (5000, 2, 256, 0, True, (900, 4999)), (2000, 70, 256, 0, True, (0, 1100))])
def test_tiles_whose_first_keys_have_score_minus_infinity(n, heads, rows, last, cut, dead, far, hd):
    """Keys whose score is -inf count for nothing, also where they are all of the first round, of a part of a cut tile, or all but one."""
    from tests import gpu_util as g
    runs(n, heads, hd, rows, last, cut)
    q, k, v = dead_keys(n, heads, hd, dead, int(far * n), 6900 + n)
    got = g.hip_attention(q, k, v)
    picked = synth.sample_rows(n, 32, seed=3, tile=rows)
    g.assert_attention_close(got[picked], orc.attention(q, k, v, rows=picked), "n=%d dead %s" % (n, dead))
    assert np.all(np.isfinite(got))
