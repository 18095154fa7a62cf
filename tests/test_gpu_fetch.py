"""Results fetched from a server into pinned memory."""

import ctypes

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu] {msg}", flush=True)


@pytest.mark.parametrize("D,T", [(16, 500), (701, 3003)])      # below and above the size that goes by chunks
def test_fetch_into_pinned_memory(D, T):
    from paper_2511_09165_amd import Server, plan_for_frame
    f = synth.random_frame(np.random.default_rng(D), 4, D, T, 3)
    _say(f"fetch into pinned memory D={D} T={T}")
    out = torch.full((D * T + 16,), 7.0, dtype=torch.float32, pin_memory=True)
    with plan_for_frame(f) as plan, Server(64 << 20, staging=16 << 20) as srv:
        ref = plan.envelope(torch.from_numpy(f.x_f32()).cuda()).cpu()
        t = srv.submit(plan, f.x_f32())
        srv.wait(t, 30.0)
        for _ in range(2):
            assert srv._lib.dmas_server_fetch(srv._h, t, ctypes.c_void_p(out.data_ptr() + 32)) == 0
            assert torch.equal(out[8:8 + D * T].view(D, T), ref)
            assert (out[:8] == 7.0).all() and (out[8 + D * T:] == 7.0).all()
        srv.release(t)
