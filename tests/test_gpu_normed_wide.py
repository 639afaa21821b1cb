"""Products of few rows that normalise their rows themselves, by their columns: both sides of every limit (one workgroup to a compute
unit, long rows, LayerNorm of long rows, more than 16 short rows); whole blocks against the oracle, judged on what they add to their
input (bf16 operands, bound of the other block tests).  Whether the launches are there is read from the kernel times."""
import numpy as np
import pytest

from oracle import forward as F
from paper_2605_11678_amd import configs as CFG
from tests.gpu_common import GpuStack

pytestmark = pytest.mark.gpu
TOL = 2e-2


# (d_model, tokens, columns of the feed-forward's first product, LayerNorm, normalised inside it); the QKV product has 512 columns
@pytest.mark.parametrize("d,T,cols,ln,inside", [
    (256, 16, 4096, False, True), (256, 16, 4160, False, False), (512, 9, 4096, False, True), (512, 2, 4160, False, False),
    (1024, 16, 2048, False, True), (1024, 16, 2112, False, False), (256, 32, 12288, False, True), (256, 17, 12352, False, False),
    (320, 17, 4160, False, False), (128, 64, 8192, False, True), (128, 16, 4112, True, False), (512, 16, 4096, True, True),
    (1024, 5, 512, True, True), (1024, 5, 528, True, False), (576, 16, 912, True, False), (256, 33, 8192, True, True)])
def test_columns(d, T, cols, ln, inside):
    if ln:
        c = CFG.ModuleConfig("n", 1, d, 4, 2, 64, cols, CFG.NORM_LN, CFG.ACT_GELU, 1, 0, 0.0, seed_base=6900)
    else:
        c = CFG.ModuleConfig("n", 1, d, 4, 2, 64, cols // 2, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, 1e4, seed_base=6900)
    w = CFG.make_layer_weights(c, 0, 1.28)
    x = CFG.make_tokens(T, d, seed=64)
    want = F.stack_forward(c.as_dict(), lambda l: w, x)
    g = GpuStack(c, max_tokens=T, cap_bytes=512 << 20, weights=lambda l: w)
    try:
        g.eng.ctx.set_kernel_timing(True)
        got = g.forward(x)
        assert g.eng.ctx.collect_kernel_times()["norm"]["launches"] == (0 if inside else 1)
    finally:
        g.close()
    assert np.max(np.abs(got - want)) / np.max(np.abs(want - x)) <= TOL
