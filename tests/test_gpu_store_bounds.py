"""What the products store stays inside their outputs: ragged last row tiles and last column tiles of the LDS-staged and the few-rows
kernels, in fp32, behind a GELU, and as V^T rows (workspace and cache), plus the values against the oracle.  The whole arena is
one tensor, so the bytes behind an output are looked at directly: buffers are sized for more rows than the pass has, filled with a
pattern, and must still hold it behind the last row."""
import numpy as np
import pytest

from oracle import forward as F
from oracle import pipeline as PL
from paper_2605_11678_amd import configs as CFG
from paper_2605_11678_amd.harness import Engine
from tests.gpu_common import GpuStack, rel_err

pytestmark = pytest.mark.gpu
TOL = 2e-2
PAT = 0x5A                       # 0x5A5A is a finite bf16 value
SPARE = 192                      # rows behind the pass


def align(n):
    return (n + 255) // 256 * 256


# both products on LDS-staged tiles (widths are multiples of 128) of many shapes, the second one with a ragged column tile as well
MLPS = [(67, 512, 640, 72), (67, 384, 128, 64), (131, 2176, 6144, 200), (197, 768, 8192, 296), (300, 640, 8320, 1096), (517, 896, 8192, 1096),
        (731, 896, 8320, 4104), (1000, 640, 4224, 1152), (1300, 1024, 6144, 3456), (2999, 896, 4224, 1000), (19, 256, 384, 48)]


@pytest.mark.parametrize("T,d_in,d_hid,d_out", MLPS)
def test_mlp_rows_behind_the_last(T, d_in, d_hid, d_out):
    w = CFG.make_mlp(d_in, d_hid, d_out, seed=977 + d_hid)
    x = CFG.make_tokens(T, d_in, seed=18)
    n = T + SPARE
    eng = Engine(4 * n * (d_in + d_out) + 2 * n * (d_in + d_hid) + 2 * (d_hid * d_in + d_out * d_hid + d_hid + d_out) + (64 << 20), device=0)
    try:
        m = eng.ctx.mlp_create(d_in, d_hid, d_out, *w, max_tokens=n)
        hid0 = eng.ctx.residency_budget()                # the hidden rows are the lowest block of the arena's top stack
        hid = eng.arena[hid0:hid0 + 2 * n * d_hid].view(n, 2 * d_hid)
        xp, xv = eng.alloc_f32(T * d_in)
        yp, yv = eng.alloc_f32(n * d_out)
        hid.fill_(PAT)
        yv.fill_(7.0)
        eng.torch.cuda.synchronize()
        eng.upload(xv, x)
        eng.ctx.mlp_forward(m, xp, yp, T)
        got = eng.download(yv).reshape(n, d_out)
        assert np.all(got[T:] == 7.0)
        assert bool((hid[T:] == PAT).all())
        assert not bool((hid[:T].view(T * 2 * d_hid) == PAT).all())
        rows = sorted({r for b in (0, 64, 128, 192, 256, 512, T - 1) for r in (b - 1, b, b + 1) if 0 <= r < T})
        assert rel_err(got[rows], PL.mlp(x[rows], *w)) <= TOL
    finally:
        eng.close()


# (d_model, Hq, Hkv, dh, tokens): the V columns end inside a column tile
BLOCKS = [(128, 2, 1, 72, 2), (128, 4, 4, 72, 300), (256, 16, 16, 72, 517), (1152, 16, 16, 72, 731), (512, 12, 4, 120, 731), (1152, 16, 16, 72, 517),
          (1024, 5, 5, 120, 1000)]


@pytest.mark.parametrize("d,Hq,Hkv,dh,T", BLOCKS)
def test_workspace_vt_rows(d, Hq, Hkv, dh, T):
    c = CFG.ModuleConfig("enc", 1, d, Hq, Hkv, dh, 256, CFG.NORM_LN, CFG.ACT_GELU, 1, 0, 0.0, seed_base=5100)
    w = {k: (np.zeros_like(v) if k in (CFG.T_W_DOWN, CFG.T_B_DOWN) else v) for k, v in CFG.make_layer_weights(c, 0, 1.28).items()}
    x = CFG.make_tokens(T, d, seed=41)
    n, dkv, n_qkv = T + SPARE, Hkv * dh, (Hq + 2 * Hkv) * dh
    g = GpuStack(c, max_tokens=n, cap_bytes=512 << 20, weights=lambda l: w)
    try:
        # workspace: normed rows, QKV rows, attention output, feed-forward rows, V^T; the last activation block lies behind it
        ws = g.eng.ctx.residency_budget()
        qkv0 = ws + align(2 * n * d)
        vt0 = qkv0 + align(2 * n * n_qkv) + align(2 * n * Hq * dh) + align(2 * n * 256)
        ld = (n + 63) // 64 * 64
        qkv = g.eng.arena[qkv0:qkv0 + 2 * n * n_qkv].view(n, 2 * n_qkv)
        vt = g.eng.arena[vt0:vt0 + 2 * dkv * ld].view(dkv, 2 * ld)
        assert vt0 + align(2 * dkv * ld) == g.np_ - g.eng.arena.data_ptr()
        qkv.fill_(PAT)
        vt.fill_(PAT)
        g.nv.fill_(7.0)
        g.eng.torch.cuda.synchronize()
        got = g.forward(x)
        assert bool((qkv[T:] == PAT).all()) and bool((vt[:, 2 * T:] == PAT).all()) and bool((g.nv == 7.0).all())
        assert bool((qkv[:T, 2 * (Hq + Hkv) * dh:] == PAT).all())              # V goes to V^T and nowhere else
        assert not bool((vt[:, 2 * T - 2:2 * T] == PAT).all(1).any()) or T < 3
    finally:
        g.close()
    rows = sorted({0, 1, T // 2, T - 1} | {r for r in (63, 64, 127, 128, 255, 256, 511, 512) if r < T})
    want = F.stack_forward(c.as_dict(), lambda l: w, x)
    assert np.max(np.abs(got - want)[rows]) / np.max(np.abs(want - x)) <= TOL


# (d_model, Hq, Hkv, dh, prefix, tokens): chunks at unaligned cache positions, V columns that end inside a column tile
CHUNKS = [(512, 6, 6, 40, 5, 67), (512, 6, 6, 72, 7, 300), (1024, 5, 5, 120, 3, 517), (128, 8, 2, 40, 9, 131), (1024, 5, 5, 72, 130, 64), (1152, 16, 16, 72, 1, 731)]


@pytest.mark.parametrize("d,Hq,Hkv,dh,prefix,T", CHUNKS)
def test_cache_rows(d, Hq, Hkv, dh, prefix, T):
    """Two layers: behind the first one's V^T rows lie the second one's keys.  Nothing but the chunk's own positions changes."""
    S = prefix + T + 21
    c = CFG.ModuleConfig("dec", 2, d, Hq, Hkv, dh, 256, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, 1e6, max_seq=S, seed_base=5900)
    x = CFG.make_tokens(prefix + T, d, seed=43)
    g = GpuStack(c, max_tokens=prefix + T, cap_bytes=512 << 20, weights=lambda l: CFG.make_layer_weights(c, l, 1.28))
    try:
        g.forward(x[:prefix])
        ld, dkv = (S + 63) // 64 * 64, Hkv * dh
        kb, vb = align(2 * dkv * S), align(2 * dkv * ld)
        kv0 = g.xp - g.eng.arena.data_ptr() + align(4 * (prefix + T) * d)        # the block above the activations
        kv = g.eng.arena[kv0:kv0 + 2 * (kb + vb)]
        before = kv.clone()
        assert not bool(before[2 * kb + 2 * vb - vb + 2 * dkv * ld:].any())
        g.forward(x[prefix:], pos0=prefix)
        changed = (kv != before).cpu().numpy()
        for l in range(2):
            o = l * (kb + vb)
            k = changed[o:o + 2 * dkv * S].reshape(Hkv, S, 2 * dh)
            v = changed[o + kb:o + kb + 2 * dkv * ld].reshape(dkv, ld, 2)
            assert k[:, prefix:prefix + T].any(2).all() and v[:, prefix:prefix + T].any(2).mean() > 0.99
            k[:, prefix:prefix + T] = False
            v[:, prefix:prefix + T] = False
        assert not changed.any()
    finally:
        g.close()


def test_rows_of_four_million():
    """An output whose rows are longer than 2^22 elements, on LDS-staged tiles, and the reduction over them.  The weights repeat 64 times,
    so one period is the oracle's."""
    T, d_in, period, reps, d_out = 66, 128, 65544, 64, 64
    w1, b1, w2, b2 = CFG.make_mlp(d_in, period, d_out, seed=4321)
    x = CFG.make_tokens(T, d_in, seed=18)
    d_hid = reps * period
    eng = Engine(2 * (d_hid * (d_in + d_out + 1) + T * (d_in + d_hid)) + 4 * T * (d_in + d_out) + (64 << 20), device=0)
    try:
        m = eng.ctx.mlp_create(d_in, d_hid, d_out, np.tile(w1, (reps, 1)), np.tile(b1, reps), np.tile(w2, (1, reps)), b2, max_tokens=T)
        xp, xv = eng.alloc_f32(T * d_in)
        yp, yv = eng.alloc_f32(T * d_out)
        eng.upload(xv, x)
        eng.ctx.mlp_forward(m, xp, yp, T)
        got = eng.download(yv).reshape(T, d_out)
    finally:
        eng.close()
    rows = [0, 1, 31, 32, 63, 64, 65]
    bias = F.widen(b2)
    want = reps * (PL.mlp(x[rows], w1, b1, w2, b2) - bias) + bias
    assert rel_err(got[rows], want) <= TOL
