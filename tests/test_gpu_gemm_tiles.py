"""Tile shapes of the fast GEMM path at their edges, through the first product of the C-ABI's two-layer perceptron (GELU
epilogue; the second one, K not a multiple of 128, is the register-staged kernel's): ragged last row and column tiles, reductions of
as few k-tiles as the shape has LDS stages, and the remainders of k-tiles behind the whole turns of the stages.  192x256 and the split
last round are test_gpu_gemm_shapes' (larger products), fp32 outputs of these tiles test_gpu_store_bounds'.

All shapes add the products of a row up in the same order, so besides the oracle (sampled rows, bound of the other GEMM
tests) the first 66 rows of a pass are compared bit for bit with a pass over these rows alone, for which the dispatcher takes
another, smaller tile."""
import numpy as np
import pytest

from oracle import pipeline as PL
from paper_2605_11678_amd import configs as CFG
from paper_2605_11678_amd.harness import Engine
from tests.gpu_common import rel_err, tile_of

pytestmark = pytest.mark.gpu
TOL = 2e-2

# (tokens, d_hidden, k-tiles of 64, tile of the first product: rows, columns, LDS stages)
SHAPES = (
    [(67, 72, nk, (64, 64, 8)) for nk in (8, 10, 12, 14, 16, 18, 22)]
    + [(131, 6152, 6, (64, 128, 6))] + [(131, 8200, nk, (64, 128, 6)) for nk in (8, 10, 12)]
    + [(67, 72, 6, (128, 64, 6))] + [(67, 8200, nk, (128, 64, 6)) for nk in (8, 10, 12)] + [(131, 6152, 34, (128, 64, 6))]
    + [(197, 8200, nk, (128, 96, 5)) for nk in (14, 16, 18, 20, 22)]
    + [(197, 8200, nk, (128, 128, 5)) for nk in (6, 8, 10, 12)] + [(300, 8200, nk, (128, 128, 5)) for nk in (10, 12, 14)]
    + [(67, 72, 4, (128, 160, 4))] + [(1000, 4104, nk, (128, 160, 4)) for nk in (20, 22)]
    + [(517, 8200, nk, (192, 128, 4)) for nk in (14, 16)]
    + [(1000, 6152, 36, (128, 256, 3)), (731, 8200, 38, (128, 256, 3))]
    + [(1300, 6152, nk, (192, 192, 3)) for nk in (16, 18, 20)]
    + [(67, 72, 2, (128, 192, 2)), (1000, 8200, 14, (128, 192, 2)), (1300, 8200, 14, (128, 192, 2)), (1300, 6152, 14, (128, 192, 2))]
    + [(1000, 4104, nk, (128, 128, 2)) for nk in (4, 10, 12)] + [(731, 8200, nk, (128, 128, 2)) for nk in (12, 14, 16)]
    + [(517, 8200, 12, (128, 128, 2)), (1700, 6152, 38, (256, 192, 2)), (2999, 4104, 14, (256, 256, 2))]
)


@pytest.mark.parametrize("T,d_hid,nk,tile", SHAPES, ids=["%dx%d-on-%d-%d-%d" % (s[3] + (s[2], s[0])) for s in SHAPES])
def test_tile_shape(T, d_hid, nk, tile):
    d_in, d_out = 64 * nk, 96
    assert tile_of(T, d_hid, d_in, 3) == tile            # the shape this case is for
    w = CFG.make_mlp(d_in, d_hid, d_out, seed=977 + nk)
    x = CFG.make_tokens(T, d_in, seed=18)
    eng = Engine(4 * T * (d_in + d_out) + 2 * T * (d_in + d_hid) + 2 * (d_hid * d_in + d_out * d_hid + d_hid + d_out) + (64 << 20), device=0)
    try:
        ctx = eng.ctx
        m = ctx.mlp_create(d_in, d_hid, d_out, *w, max_tokens=T)
        xp, xv = eng.alloc_f32(T * d_in)
        yp, yv = eng.alloc_f32(T * d_out)
        eng.upload(xv, x)
        ctx.mlp_forward(m, xp, yp, T)
        got = eng.download(yv).reshape(T, d_out)
        rows = sorted({r for b in (0, 64, 128, 192, 256, 512, T - 1) for r in (b - 1, b, b + 1) if 0 <= r < T}
                      | set(np.random.default_rng(5).integers(0, T, 8).tolist()))
        assert np.all(np.isfinite(got))
        assert rel_err(got[rows], PL.mlp(x[rows], *w)) <= TOL
        yv.zero_()
        eng.torch.cuda.synchronize()
        ctx.mlp_forward(m, xp, yp, 66)
        few = eng.download(yv).reshape(T, d_out)
        assert np.array_equal(few[:66].view(np.uint32), got[:66].view(np.uint32))
        assert not few[66:].any()
    finally:
        eng.close()
