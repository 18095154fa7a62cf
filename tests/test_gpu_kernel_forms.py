"""Forms of a call that the plan chooses between by size give the same bits as each other."""

import numpy as np
import pytest

import oracle
import synth
from _parity import check_t1

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu] {msg}", flush=True)


def _image(f, x, out=None, **kw):
    from paper_2511_09165_amd import plan_for_frame
    with plan_for_frame(f, **kw) as plan:
        y = plan.envelope(torch.from_numpy(np.ascontiguousarray(x)).cuda(), out=out)
        torch.cuda.synchronize()
        return y.cpu().numpy()


@pytest.mark.parametrize("L", [1, 63, 65, 67, 255])          # 65 is the last length with its taps in registers
@pytest.mark.parametrize("D,T", [(21, 1), (21, 33), (13, 2047), (13, 2048), (13, 2049), (9, 4100), (7, 5003),
                                 (2100, 70)])                # steps of 2048; more rows than workgroups
def test_envelope_in_two_passes_gives_the_fused_bits(L, D, T, monkeypatch):
    """The filter run over the RF image in place equals the beamformer's fused filter bit for bit,
    over one and several walk steps, rows on and off the 16-byte grid, and agrees with the oracle."""
    f = synth.random_frame(np.random.default_rng(31 * L + D + T), 6, D, T, 3)
    taps = np.random.default_rng(L).normal(size=L).astype(np.float32)
    _say(f"two-pass envelope L={L} D={D} T={T}")
    monkeypatch.setenv("DMAS_ENVELOPE_PASSES", "1")
    one = _image(f, f.x_f32(), fir_taps=taps)
    monkeypatch.setenv("DMAS_ENVELOPE_PASSES", "2")
    two = _image(f, f.x_f32(), fir_taps=taps)
    np.testing.assert_array_equal(two, one)
    if D <= 21:
        y_ref = oracle.frame_rows(f, x=f.x_f32().astype(np.float64))
        check_t1(two, oracle.envelope(y_ref, taps.astype(np.float64)))


def test_two_pass_envelope_in_an_unaligned_output(monkeypatch):
    """An output that starts off the 16-byte grid, and nothing written around it."""
    f = synth.random_frame(np.random.default_rng(77), 8, 10, 2064, 2)
    monkeypatch.setenv("DMAS_ENVELOPE_PASSES", "1")
    ref = _image(f, f.x_f32())
    monkeypatch.setenv("DMAS_ENVELOPE_PASSES", "2")
    _say("two-pass envelope, unaligned output")
    buf = torch.full((10 * 2064 + 8,), 7.0, dtype=torch.float32, device="cuda")
    got = _image(f, f.x_f32(), out=buf[3:3 + 10 * 2064].view(10, 2064))
    np.testing.assert_array_equal(got, ref)
    rest = torch.cat([buf[:3], buf[3 + 10 * 2064:]]).cpu().numpy()
    assert (rest == 7.0).all()
