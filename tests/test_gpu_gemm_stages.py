"""The GEMM tiles with more LDS stages for one operand than for the other (192x256: four and two, 256x192: three and two), whose main loop is
left behind the last k-tile while its copies go on: fewer k-tiles than stages, as many, every remainder of a turn of the stages, and an
operand of more than 2 GB.  Through the C-ABI's two-layer perceptron, against the oracle (sampled rows, bound of the other GEMM tests), and
the first 66 rows bit for bit against a pass over these rows alone, which takes another tile."""
import numpy as np
import pytest

from oracle import pipeline as PL
from paper_2605_11678_amd import configs as CFG
from paper_2605_11678_amd.harness import Engine
from tests.gpu_common import rel_err, tile_of

pytestmark = pytest.mark.gpu
TOL = 2e-2


def check(T, d_in, d_hid, d_out, seed):
    w = CFG.make_mlp(d_in, d_hid, d_out, seed=seed)
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
        rows = sorted({r for b in (0, 64, 128, 192, 256, 512, T // 192 * 192, T - 1) for r in (b - 1, b, b + 1) if 0 <= r < T}
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


@pytest.mark.parametrize("T,N,nk", [(731, 12288, 2), (731, 12288, 4), (731, 12288, 6), (300, 24576, 2), (300, 24576, 8)])
def test_second_product_on_192x256(T, N, nk):
    assert tile_of(T, N, 64 * nk, 4) == (192, 256, 2)
    check(T, 64, 64 * nk, N, 650 + nk)


@pytest.mark.parametrize("T,N,nk", [(1000, 12288, 36), (1000, 12288, 38), (1000, 12288, 40), (1700, 6152, 42)])
def test_first_product_on_256x192(T, N, nk):
    assert tile_of(T, N, 64 * nk, 3) == (256, 192, 2)
    check(T, 64 * nk, N, 96, 660 + nk)


def test_operand_of_more_than_2_gb():
    T, K, N = 34000, 32768, 256
    assert 2 * T * K > 1 << 31 and tile_of(T, N, K, 4) == (192, 256, 2)
    check(T, 64, K, N, 671)
