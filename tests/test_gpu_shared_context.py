"""The cross-attention's keys and values of a whole inference, made once for all of its Euler steps in the decoder's workspace:
every buffer bit for bit as from separate calls, which make them anew each step.  Contexts of whole tiles of 64 positions and not,
a decoder whose workspace has to keep its zero padding, and an action stack whose keys and values do not fit there (both make them
each step as well); behind the inference the decoder's passes still give the same bits."""
import ctypes
import dataclasses

import numpy as np
import pytest

from paper_2605_11678_amd import binding as B
from paper_2605_11678_amd.harness import Engine, VlaPipeline
from tests import parity_cases as PC

pytestmark = pytest.mark.gpu

# (text tokens behind 8 visual ones, feed-forward width of the decoder, layers of the action stack)
CASES = [(9, None, None), (56, None, None), (57, None, 3), (120, None, None), (9, 1056, None), (9, None, 40)]


@pytest.mark.parametrize("n_text,d_ff,layers", CASES)
def test_shared_context_equals_separate_calls(n_text, d_ff, layers):
    vit, dec, act = PC.pipe_small_modules()
    if d_ff:
        dec = dataclasses.replace(dec, d_ff=d_ff)
    if layers:
        act = dataclasses.replace(act, n_layers=layers)
    eng = Engine(1 << 30, device=0)
    try:
        p = VlaPipeline(eng, vit, dec, act, n_patches=32, n_text=n_text, n_actions=7, matrix_gain=PC.PIPE_SMALL["gain"])
        assert p.n_prefill == 8 + n_text
        p.run(0, 3)
        got = [eng.download(v).view(np.uint32).copy() for v in (p.v_a, p.v_ain, p.v_vel, p.v_traj)]
        assert np.all(np.isfinite(got[3].view(np.float32)))
        eng.upload(p.v_a, p.a0)
        for s in range(3):
            eng.ctx.add_time_embedding(p.p_a, p.p_ain, float(np.float32(s) / np.float32(3)), 7, act.d_model)
            eng.ctx.forward(p.m_act, p.p_ain, p.p_vel, 7, 0, p.p_ctx, p.n_prefill)
            eng.ctx.axpy(p.p_a, float(np.float32(1) / np.float32(3)), p.p_vel, 7 * act.d_model)
        eng.ctx.mlp_forward(p.mlp_out, p.p_a, p.p_traj, 7)
        eng.ctx.sync()
        for a, v in zip(got, (p.v_a, p.v_ain, p.v_vel, p.v_traj)):
            assert np.array_equal(a, eng.download(v).view(np.uint32))
        p.run(0, 3)                                        # the decoder's workspace has held keys and values meanwhile
        for a, v in zip(got, (p.v_a, p.v_ain, p.v_vel, p.v_traj)):
            assert np.array_equal(a, eng.download(v).view(np.uint32))
    finally:
        eng.close()


def shared(p):
    """(whether the keys and values stay between the steps, arena offset, bytes of a layer)"""
    off, layer = ctypes.c_uint64(), ctypes.c_uint64()
    f = B.lib().dlk_shared_ctx
    f.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 3 + [ctypes.POINTER(ctypes.c_uint64)] * 2
    return f(p.eng.ctx._h, p.m_act, p.m_dec, p.n_prefill, ctypes.byref(off), ctypes.byref(layer)), off.value, layer.value


@pytest.mark.parametrize("case,share", list(zip(CASES, (1, 1, 1, 1, 0, 0))) + [((9, None, 3), 0)])
def test_which_cases_share(case, share):
    """And that an inference does so: the products of keys and values are there once, or in each step."""
    n_text, d_ff, layers = case
    vit, dec, act = PC.pipe_small_modules()
    dec, act = dataclasses.replace(dec, d_ff=d_ff or dec.d_ff), dataclasses.replace(act, n_layers=layers or act.n_layers)
    eng = Engine(1 << 30, device=0)
    try:
        p = VlaPipeline(eng, vit, dec, act, n_patches=32, n_text=n_text, n_actions=7, matrix_gain=PC.PIPE_SMALL["gain"])
        assert shared(p)[0] == share
        eng.ctx.set_kernel_timing(True, [B.DL_K_NAMES.index("cross")])
        flops = []
        for n in (1, 3):
            eng.ctx.collect_kernel_times()
            p.run(0, n)
            flops.append(eng.ctx.collect_kernel_times()["cross"]["flops"])
        kv = 2.0 * act.n_layers * p.n_prefill * 2 * act.n_kv_heads * act.d_head * act.d_ctx
        assert flops[1] == 3 * flops[0] - 2 * kv * share
    finally:
        eng.close()


@pytest.mark.parametrize("n_text,n_actions,layers", [(9, 7, 2), (60, 33, 3), (57, 7, 3), (100, 64, 2)])
def test_positions_behind_the_context(n_text, n_actions, layers):
    """Attention reads whole tiles of 64 positions: NaN in all of the memory that takes the keys and values, in a decoder whose workspace is
    much larger than its prefill needs, changes no bit."""
    vit, dec, act = PC.pipe_small_modules()
    act = dataclasses.replace(act, n_layers=layers)
    eng = Engine(1 << 30, device=0)
    try:
        p = VlaPipeline(eng, vit, dec, act, n_patches=32, n_text=n_text, n_actions=n_actions, matrix_gain=PC.PIPE_SMALL["gain"])
        eng.ctx.module_set_max_tokens(p.m_dec, dec.max_seq)
        share, off, layer = shared(p)
        # the prefill writes its normalised rows there, which end in front of the first layer's last V^T rows
        assert share == 1 and 2 * p.n_prefill * dec.d_model < layer - 128 <= 2 * dec.max_seq * dec.d_model - 128
        p.run(0, 3)
        want = [eng.download(v).view(np.uint32).copy() for v in (p.v_a, p.v_vel, p.v_traj)]
        for _ in range(2):
            eng.arena[off: off + layers * layer].fill_(0xFF)
            eng.torch.cuda.synchronize()
            p.run(0, 3)
            for a, v in zip(want, (p.v_a, p.v_vel, p.v_traj)):
                b = eng.download(v)
                assert np.all(np.isfinite(b)) and np.array_equal(a, b.view(np.uint32))
    finally:
        eng.close()
