"""Logits that reach the host by the kernel that chooses the token, up to 16384 of them, and by a copy of their own above that: the same as
a head whose rows are a prefix of the larger one gives, for every residue of a workgroup's stride, one call after the other, and no
value behind the last one touched; the token is the place of the largest."""
import numpy as np
import pytest

from paper_2605_11678_amd import configs as CFG
from tests.gpu_common import GpuStack

pytestmark = pytest.mark.gpu


def test_logits_on_both_ways():
    d, big = 64, 16392
    c0 = CFG.ModuleConfig("head", 1, d, 1, 1, 64, 64, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, 1e4, max_seq=8, vocab=big, seed_base=7000)
    head = CFG.make_head(c0)
    x = CFG.make_tokens(3, d, seed=71)
    rows = {}
    for vocab in (big, 16384, 8193, 1024, 1000, 64, 1):
        c = CFG.ModuleConfig("head", 1, d, 1, 1, 64, 64, CFG.NORM_RMS, CFG.ACT_SWIGLU, 0, 1, 1e4, max_seq=8, vocab=vocab, seed_base=7000)
        g = GpuStack(c, max_tokens=3, cap_bytes=64 << 20, head={k: (v[:vocab] if v.ndim == 2 else v) for k, v in head.items()})
        try:
            g.eng.upload(g.xv[:3 * d], x)
            for t in (0, 1, 2, 0):
                out = np.full(vocab + 16, np.float32(-7.5))
                tok = g.eng.ctx.logits_argmax(g.mid, g.xp + 4 * d * t, out[:vocab])
                assert np.all(out[vocab:] == np.float32(-7.5))
                rows.setdefault(t, out[:vocab].copy())                       # the largest head comes first
                assert np.array_equal(out[:vocab].view(np.uint32), rows[t][:vocab].view(np.uint32)), (vocab, t)
                assert tok == int(np.argmax(out[:vocab])) == g.eng.ctx.logits_argmax(g.mid, g.xp + 4 * d * t)
        finally:
            g.close()
