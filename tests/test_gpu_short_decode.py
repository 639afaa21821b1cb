"""Single-token attention over few cached positions (one launch, one workgroup per KV head) on both sides of the switch to the
two-launch form: one tile, ragged tiles, the last length and the largest head group that take it and the first that do not, for each
padded head dimension, grouped and ungrouped heads; against the oracle, the feed-forward zeroed."""
import numpy as np
import pytest

from oracle import forward as F
from paper_2605_11678_amd import configs as CFG
from tests.gpu_common import GpuStack

pytestmark = pytest.mark.gpu
TOL = 2e-2

# (Hq, Hkv, dh, cached positions before the token)
CASES = [(4, 4, 64, s) for s in (0, 1, 62, 63, 64, 200, 254, 255, 256)] + [(8, 2, 40, 129), (3, 3, 72, 63), (8, 2, 128, 200), (32, 1, 64, 255), (16, 1, 64, 62),
                                                                                       (17, 1, 64, 62), (32, 2, 64, 127), (32, 2, 64, 128), (32, 1, 32, 130), (32, 1, 8, 255)]


@pytest.mark.parametrize("Hq,Hkv,dh,prefix", CASES)
def test_token_over_short_cache(Hq, Hkv, dh, prefix):
    c = CFG.ModuleConfig("dec", 1, 256, Hq, Hkv, dh, 256, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, 1e4, max_seq=prefix + 3, seed_base=5400)
    full = CFG.make_layer_weights(c, 0, 1.28)
    w = {k: (np.zeros_like(v) if k == CFG.T_W_DOWN else v) for k, v in full.items()}
    x = CFG.make_tokens(prefix + 1, c.d_model, seed=51)
    want = F.stack_forward(c.as_dict(), lambda l: w, x)
    g = GpuStack(c, max_tokens=prefix + 1, cap_bytes=256 << 20, weights=lambda l: w)
    try:
        if prefix:
            g.forward(x[:prefix])
        got = g.forward(x[prefix:], pos0=prefix)
    finally:
        g.close()
    assert np.max(np.abs(got - want[prefix:])) / np.max(np.abs(want[prefix:] - x[prefix:])) <= TOL
