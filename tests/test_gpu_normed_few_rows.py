"""Products of few rows that normalise their rows themselves: every row tile at its longest reduction and one past it (which keeps the
launch of its own), ragged rows, reductions of one to four k-tiles a wavefront, both normalisations and activations, with a rotary
embedding and without, the queries of a cross-attention; whole blocks against the oracle, judged on what they add to their input
(bf16 operands, bound of the other block tests).  Whether the launches are there is read from the kernel times."""
import numpy as np
import pytest

from oracle import forward as F
from paper_2605_11678_amd import configs as CFG
from tests.gpu_common import GpuStack

pytestmark = pytest.mark.gpu
TOL = 2e-2

# (d_model, tokens, normalised inside the products)
CASES = [(128, 2, True), (128, 64, True), (256, 64, True), (256, 33, True), (320, 33, False), (512, 32, True), (512, 17, True), (576, 32, False),
         (1024, 16, True), (1024, 5, True), (960, 9, True), (1088, 16, False), (192, 31, True), (448, 2, True), (256, 65, False)]


def compare(c, T, inside, n_ctx=0):
    w = CFG.make_layer_weights(c, 0, 1.28)
    x = CFG.make_tokens(T, c.d_model, seed=61)
    x = x * (1.0 + np.arange(T, dtype=np.float32)[:, None] / 8) + 0.25          # rows of different size, a mean
    ctx = CFG.make_tokens(n_ctx, c.d_ctx, seed=62) if n_ctx else None
    want = F.stack_forward(c.as_dict(), lambda l: w, x, ctx=ctx)
    g = GpuStack(c, max_tokens=T, cap_bytes=512 << 20, max_ctx=n_ctx, weights=lambda l: w)
    try:
        g.eng.ctx.set_kernel_timing(True)
        got = g.forward(x, ctx=ctx)
        n = g.eng.ctx.collect_kernel_times()["norm"]["launches"]
        g.eng.ctx.set_kernel_timing(False)
        again = g.forward(x, ctx=ctx)
    finally:
        g.close()
    assert n == (0 if inside else 2)
    assert np.array_equal(got.view(np.uint32), again.view(np.uint32))
    assert np.max(np.abs(got - want)) / np.max(np.abs(want - x)) <= TOL


@pytest.mark.parametrize("d,T,inside", CASES)
def test_decoder_block(d, T, inside):
    compare(CFG.ModuleConfig("dec", 1, d, 4, 2, 64, 256, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, 1e4, seed_base=6500), T, inside)


@pytest.mark.parametrize("d,T,inside", CASES)
def test_cross_attending_block(d, T, inside):
    compare(CFG.ModuleConfig("act", 1, d, 2, 2, 64, 384, CFG.NORM_LN, CFG.ACT_GELU, 1, 0, 0.0, d_ctx=256, seed_base=6600), T, inside, n_ctx=70)


def test_cache_without_rotation():
    """K goes to the cache in a launch of its own behind the normalising product."""
    c = CFG.ModuleConfig("dec", 1, 256, 4, 2, 64, 256, CFG.NORM_LN, CFG.ACT_GELU, 1, 1, 0.0, max_seq=40, seed_base=6700)
    compare(c, 19, True)
