"""lp_attention_static (the entry point for callers that cannot allocate) against lp_attention.

Calls in a row on the one device-resident scratch array, each smaller than the one before it,
each compared with the workspace entry point on the same inputs (same kernels, same split of
the work: bit-identical) and with the oracle at the attention tolerance.
"""
import numpy as np
import pytest

from oracle import lp_oracle as orc
from paper_2512_07350_amd import synth
from tests import routes

pytestmark = pytest.mark.gpu


def _static(q, k, v):
    import torch
    from tests import gpu_util as g
    from paper_2512_07350_amd import binding as lp
    n, heads, d = q.shape
    qd, kd, vd = g.to_dev_bf16(q), g.to_dev_bf16(k), g.to_dev_bf16(v)
    od = torch.full((n, heads, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lp.lp_attention_static(qd, kd, vd, od, n, heads, d, heads * d, d, 0.0, g.stream())
    torch.cuda.synchronize()
    return g.from_dev_bf16(od)


def test_static_scratch_two_calls_second_smaller():
    from tests import gpu_util as g
    from paper_2512_07350_amd import binding as lp
    assert lp.lp_attention_static_scratch_bytes() >= lp.lp_attention_workspace_size(128)
    # few heads: all three run the short kernel, which leaves the scratch array alone
    for n, heads, hd, seed in ((3000, 3, 128, 811), (700, 2, 128, 812), (333, 5, 64, 813)):
        q, k, v = synth.qkv_bf16(seed, n, heads, hd)
        got = _static(q, k, v)
        ref = g.hip_attention(q, k, v, balanced=True)
        assert np.array_equal(got, ref), "n=%d: differs from lp_attention with a workspace" % n
        g.assert_attention_close(got, orc.attention(q, k, v), "static n=%d" % n)


@pytest.mark.parametrize("calls", [
    [(4500, 16, 128), (7410, 2, 128), (5000, 1, 128)],       # query tiles cut over 256 compute units: 32 left after a round; 58; 20, each in about ten parts
    [(3700, 40, 64), (4800, 4, 64), (5000, 2, 64)],          # 88 left after two rounds; 76; 40
    [(4800, 4, 64), (5000, 1, 128)],                         # the slots of the other head_dim lie elsewhere in the array
    [(7410, 2, 128), (5000, 2, 64)],
], ids=["128", "64", "64 then 128", "128 then 64"])
def test_static_scratch_carries_the_parts_of_shared_query_tiles(calls):
    """Calls whose query tiles are cut: every one finds the slots as the larger call before it left them."""
    from tests import gpu_util as g
    for n, heads, hd in calls:
        assert routes.attention_tiles(n, heads, hd).cut
    for i, (n, heads, hd) in enumerate(calls):
        q, k, v = synth.qkv_bf16(820 + i + n + hd, n, heads, hd)
        got = _static(q, k, v)
        ref = g.hip_attention(q, k, v, balanced=True)
        assert np.array_equal(got, ref), "n=%d: differs from lp_attention with a workspace" % n
        rows = synth.sample_rows(n, 96, seed=n, tile=256)
        g.assert_attention_close(got[rows], orc.attention(q, k, v, rows=rows), "static n=%d" % n)
