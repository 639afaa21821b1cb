"""The cross-attention's keys and values of a whole inference, made once for all of its Euler steps in the decoder's workspace:
every buffer bit for bit as from separate calls, which make them anew each step.  Contexts of whole tiles of 64 positions and not,
a decoder whose workspace has to keep its zero padding, and an action stack whose keys and values do not fit there (both make them
each step as well); behind the inference the decoder's passes still give the same bits."""
import dataclasses

import numpy as np
import pytest

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
