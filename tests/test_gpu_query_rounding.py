"""A query that the rotary embedding leaves in place is rounded once.  With a base of 1e38 the rotation angles of the upper features
are below 1e-18 rad, so their cosine is 1 and their sine vanishes in fp32; the query and key rows of all other features are zero.
Such a block must then give the bits of the same block without a rotary embedding, whose queries the product scales and rounds once:
a scale applied between two roundings shows in every score.  Few rows with the rotation in the product's epilogue and behind it,
LDS-staged tiles with whole query tiles and with tiles that queries share with keys, the register-staged kernel; with a cache and
without one."""
import numpy as np
import pytest

from paper_2605_11678_amd import configs as CFG
from tests.gpu_common import GpuStack

pytestmark = pytest.mark.gpu

# (d_model, Hq, Hkv, dh, tokens, cache)
CASES = [(256, 8, 2, 64, 19, 1), (256, 8, 2, 64, 50, 0), (256, 8, 2, 80, 19, 1), (256, 8, 2, 64, 200, 1), (256, 6, 3, 72, 200, 0),
         (1024, 16, 4, 128, 300, 1), (264, 4, 2, 64, 90, 1)]


@pytest.mark.parametrize("d,Hq,Hkv,dh,T,cache", CASES)
def test_still_queries_are_rounded_once(d, Hq, Hkv, dh, T, cache):
    bits = []
    for theta in (1e38, 0.0):
        c = CFG.ModuleConfig("dec", 1, d, Hq, Hkv, dh, 256, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, theta, max_seq=T + 3 if cache else 0,
                             seed_base=5800)
        w = {k: v.copy() for k, v in CFG.make_layer_weights(c, 0, 1.28).items()}
        half = dh // 2
        still = np.arange(dh) % half >= int(np.ceil(0.6 * half))        # 1e38^-0.6 = 1e-22.8 rad per position
        for k, heads in ((CFG.T_WQ, Hq), (CFG.T_WK, Hkv)):
            w[k][np.tile(~still, heads)] = 0
        g = GpuStack(c, max_tokens=T, cap_bytes=256 << 20, weights=lambda l: w)
        try:
            bits.append(g.forward_bits(CFG.make_tokens(T, d, seed=71)))
        finally:
            g.close()
    assert np.all(np.isfinite(bits[0].view(np.float32)))
    assert np.array_equal(bits[0], bits[1]), np.mean(bits[0] != bits[1])
