"""A normalised value past the largest bf16 in a product of few rows that normalises its rows itself: its row's outputs are infinite, not
NaN, also where wavefronts have fewer k-tiles than LDS stages or none; the other rows are the oracle's."""
import numpy as np
import pytest

from oracle import forward as F
from paper_2605_11678_amd import configs as CFG
from tests.gpu_common import GpuStack

pytestmark = pytest.mark.gpu
TOL = 2e-2
J = 3                                                      # the feature that overflows, in the first k-tile


# (d_model, tokens): one k-tile and none a wavefront, two and one, four; row tiles of 16, 32 and 64
@pytest.mark.parametrize("d,T", [(128, 5), (192, 16), (320, 9), (1024, 16), (128, 31), (320, 32), (128, 64), (256, 64)])
def test_row_overflows(d, T):
    c = CFG.ModuleConfig("dec", 1, d, 4, 2, 64, 256, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, 1e4, seed_base=6800)
    w = {k: v.copy() for k, v in CFG.make_layer_weights(c, 0, 1.28).items()}
    bf16 = lambda v: np.uint16(np.float32(v).view(np.uint32) >> 16)
    shaped = {t: w[t].reshape(shape) for t, shape, _ in CFG.layer_tensors(c)}
    shaped[CFG.T_NORM2_G][J] = bf16(3e38)
    shaped[CFG.T_W_GATE][:, J] = shaped[CFG.T_W_UP][:, J] = bf16(0.5)
    shaped[CFG.T_W_DOWN][...] &= 0x7FFF                    # a sum of positive terms
    shaped[CFG.T_WO][...] = 0
    x = CFG.make_tokens(T, d, seed=63)
    x[:, J] = 0.0
    x[0, J] = 40.0
    want = F.stack_forward(c.as_dict(), lambda l: shaped, x[1:])           # (without attention a row stands alone)
    g = GpuStack(c, max_tokens=T, cap_bytes=256 << 20, weights=lambda l: w)
    try:
        g.eng.ctx.set_kernel_timing(True)
        got = g.forward(x)
        assert g.eng.ctx.collect_kernel_times()["norm"]["launches"] == 0
    finally:
        g.close()
    assert got[0].min() == np.inf, got[0][:8]
    assert np.max(np.abs(got[1:] - want)) / np.max(np.abs(want - x[1:])) <= TOL
