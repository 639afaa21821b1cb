"""The V columns of a QKV (or cross-attention KV) product land as V^T rows straight from the product's epilogue: every kernel
that has one (few rows, LDS-staged tiles, register-staged tiles), V columns that start inside a column tile, ragged last rows
and columns, and chunks that start at an unaligned cache position; one attention block against the oracle, the feed-forward
zeroed, judged on what it adds to its input."""
import numpy as np
import pytest

from oracle import forward as F
from paper_2605_11678_amd import configs as CFG
from tests.gpu_common import GpuStack, tile_of

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 operands, as the other block tests


def attention_only(c):
    full = CFG.make_layer_weights(c, 0, 1.28)
    return {k: (np.zeros_like(v) if k in (CFG.T_W_DOWN, CFG.T_B_DOWN) else v) for k, v in full.items()}


# (d_model, Hq, Hkv, dh, tokens)
PLAIN = [(128, 2, 1, 72, 2), (128, 2, 1, 72, 17), (128, 2, 1, 72, 33), (128, 2, 1, 72, 64), (128, 36, 12, 88, 64), (128, 3, 1, 40, 67),
         (128, 4, 4, 72, 300), (256, 16, 16, 72, 517), (256, 16, 16, 72, 1300), (512, 12, 4, 120, 731), (72, 2, 1, 72, 19), (72, 4, 2, 40, 150)]


@pytest.mark.parametrize("d,Hq,Hkv,dh,T", PLAIN)
def test_encoder_block(d, Hq, Hkv, dh, T):
    c = CFG.ModuleConfig("enc", 1, d, Hq, Hkv, dh, 256, CFG.NORM_LN, CFG.ACT_GELU, 1, 0, 0.0, seed_base=5100)
    w = attention_only(c)
    x = CFG.make_tokens(T, d, seed=41)
    want = F.stack_forward(c.as_dict(), lambda l: w, x)
    g = GpuStack(c, max_tokens=T, cap_bytes=512 << 20, weights=lambda l: w)
    try:
        got = g.forward(x)
        few = g.forward(x[:2])                         # the few-rows or the register-staged kernel
    finally:
        g.close()
    assert np.max(np.abs(got - want)) / np.max(np.abs(want - x)) <= TOL
    want = F.stack_forward(c.as_dict(), lambda l: w, x[:2])
    assert np.max(np.abs(few - want)) / np.max(np.abs(want - x[:2])) <= TOL


@pytest.mark.parametrize("prefix,T", [(1, 2), (3, 19), (8, 64), (5, 67), (130, 131), (7, 517)])
def test_chunk_at_unaligned_position(prefix, T):
    _chunk(CFG.ModuleConfig("dec", 1, 128, 8, 2, 40, 256, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, 1e6, max_seq=prefix + T + 5, seed_base=5200), prefix, T)


# (d_model, Hq, Hkv, dh, prefix, tokens): column tiles that are all V, the last one ragged; their rows are stored from transposed
# accumulators
WHOLE = [(512, 6, 6, 40, 5, 67), (512, 6, 6, 72, 7, 300), (1024, 5, 5, 120, 3, 517), (1152, 16, 16, 72, 1, 731)]


@pytest.mark.parametrize("d,Hq,Hkv,dh,prefix,T", WHOLE)
def test_chunk_with_tiles_of_v_alone(d, Hq, Hkv, dh, prefix, T):
    n, v0 = (Hq + 2 * Hkv) * dh, (Hq + Hkv) * dh
    bn = tile_of(T, n, d, 0)[1]
    assert -(-v0 // bn) * bn < n and (n % bn or d == 1152)
    _chunk(CFG.ModuleConfig("dec", 1, d, Hq, Hkv, dh, 256, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, 1e6, max_seq=prefix + T + 5, seed_base=5250), prefix, T)


def _chunk(c, prefix, T):
    w = attention_only(c)
    x = CFG.make_tokens(prefix + T, c.d_model, seed=43)
    want = F.stack_forward(c.as_dict(), lambda l: w, x)
    g = GpuStack(c, max_tokens=prefix + T, cap_bytes=512 << 20, weights=lambda l: w)
    try:
        whole = g.forward(x)
        g.forward(x[:prefix])
        got = g.forward(x[prefix:], pos0=prefix)
    finally:
        g.close()
    scale = np.max(np.abs(want - x))
    assert np.max(np.abs(whole - want)) / scale <= TOL
    assert np.max(np.abs(got - want[prefix:])) / scale <= TOL


@pytest.mark.parametrize("n_ctx", [1, 2, 33, 65, 700])
def test_cross_attention_source(n_ctx):
    c = CFG.ModuleConfig("act", 1, 128, 2, 1, 72, 256, CFG.NORM_LN, CFG.ACT_GELU, 1, 0, 0.0, d_ctx=192, seed_base=5300)
    w = attention_only(c)
    x, src = CFG.make_tokens(9, c.d_model, seed=47), CFG.make_tokens(n_ctx, c.d_ctx, seed=48)
    want = F.stack_forward(c.as_dict(), lambda l: w, x, ctx=src)
    g = GpuStack(c, max_tokens=9, cap_bytes=512 << 20, max_ctx=n_ctx, weights=lambda l: w)
    try:
        got = g.forward(x, ctx=src)
    finally:
        g.close()
    assert np.max(np.abs(got - want)) / np.max(np.abs(want - x)) <= TOL
