"""lp_linear with a long k: tiles of 256 features with one wavefront to a SIMD, whole and with the last round cut smaller."""
import numpy as np
import pytest

from oracle import lp_oracle as orc
from paper_2512_07350_amd import synth
from tests import routes
from tests.test_gpu_block import _bits, _close, _linear

pytestmark = pytest.mark.gpu


# threads 256: four wavefronts.  Lengths with one token or all in the last tile, d_out that 256 does or does not divide, the fewest
# k-tiles and odd numbers of them (two or three LDS stages)
@pytest.mark.parametrize("n,d_in,d_out,way,threads", [
    (1665, 2048, 3200, "256x128", 256), (4033, 2112, 1536, "256x128", 256), (4096, 4160, 1408, "256x128", 256),
    (4096, 1984, 1536, "256x128", 512),
    (2560, 4096, 6144, "256x256", 256), (2561, 4160, 3200, "256x256", 256), (2560, 4032, 6144, "256x256", 512),
    (4097, 2112, 4224, "256x256+128x128", 256), (4353, 2112, 4096, "256x256+128x64", 256), (6145, 2176, 3584, "256x256+256x128", 256),
])
def test_linear_of_a_long_k_on_sampled_tokens(n, d_in, d_out, way, threads):
    w_ = routes.gemm(n, d_in, d_out)
    assert (str(w_), w_.threads) == (way, threads)
    x = _bits(2200 + n, (n, d_in))
    w = _bits(2300 + n, (d_out, d_in), scale=d_in ** -0.5)
    b = synth.normal_f32(2400 + n, (d_out,))
    y = _linear(x, w, b)
    assert np.all(np.isfinite(y))
    rows = synth.sample_rows(n, 96, seed=31)
    _close(y[rows], orc.linear(x[rows], w, b), "linear %dx%d->%d" % (n, d_in, d_out))
