"""The envelope filter in the beamforming kernel and in a pass of its own: non-finite pixels, and
workgroups that walk several long rows."""

import numpy as np
import pytest

import oracle
import synth
from _parity import check_t1

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu] {msg}", flush=True)


def _both(f, xs, monkeypatch, **kw):
    """Envelopes of the records xs with the filter in the kernel and as a second pass."""
    from paper_2511_09165_amd import plan_for_frame
    got = {}
    for passes in ("1", "2"):
        monkeypatch.setenv("DMAS_ENVELOPE_PASSES", passes)
        with plan_for_frame(f, **kw) as plan:
            got[passes] = [plan.envelope(torch.from_numpy(x).cuda()).cpu().numpy() for x in xs]
    return got["1"], got["2"]


# 255, 191, 127, 63: half a filter is one sample short of a multiple of 32, where a block of outputs
# reads one sample past its chunk; 61 and 65: not; segments of the fused kernel on and off the chunks
@pytest.mark.parametrize("L", [1, 3, 61, 63, 65, 127, 191, 255])
@pytest.mark.parametrize("segment", [None, 32, 480, 2048])
def test_both_forms_agree_where_pixels_are_not_finite(L, segment, monkeypatch):
    """Single NaN and infinite pixels at every offset around the ends of chunks, segments and walk
    steps: the same outputs are NaN in both forms, the others have the same bits, and outputs away
    from the pixels equal those of the record without them."""
    T, gap = 4100, 683                                       # a few pixels per record, far apart
    f = synth.random_frame(np.random.default_rng(L), 3, 4, T, 2)
    f.mic_pos = f.mic_pos * 1e-6                             # no delays: a sample is a pixel
    taps = np.random.default_rng(L).normal(size=L).astype(np.float32)
    if segment is not None:
        monkeypatch.setenv("DMAS_SEGMENT", str(segment))
    clean = f.x_f32()
    at = np.arange(0, gap)                                   # together every pixel of the record
    xs = [clean]
    for k in at[:: 1 if segment is None and L == 63 else 5]:
        x = clean.copy()
        x[0, k::gap] = np.where(np.arange(len(x[0, k::gap])) % 2, np.nan, np.inf)
        xs.append(x)
    _say(f"non-finite pixels L={L} segment={segment}: {len(xs)} records")
    one, two = _both(f, xs, monkeypatch, fir_taps=taps)
    for a, b in zip(one, two):
        np.testing.assert_array_equal(b, a)                  # NaN equal to NaN
    H = (L - 1) // 2
    for x, b in zip(xs[1:], two[1:]):
        t = np.flatnonzero(~np.isfinite(x[0]))
        away = np.ones(T, bool)
        for p in t:
            away[max(0, p - H - 17):p + H + 16] = False
        np.testing.assert_array_equal(b[:, away], two[0][:, away])
        assert all(np.isnan(b[:, max(0, p - H):p + H + 1]).all() for p in t[1::2])   # the NaN ones


# more rows than the pass has workgroups (eight a compute unit), of two steps and a little more: a
# workgroup goes from the end of one row to the start of another; rows on and off the 16-byte grid
@pytest.mark.parametrize("L", [1, 63, 255])
@pytest.mark.parametrize("D,T", [(2100, 2049), (4300, 2113), (2500, 4100), (4200, 2048)])
def test_workgroups_that_walk_several_long_rows(L, D, T, monkeypatch):
    """Rows of several steps, two or three a workgroup: the fused filter's bits in every row."""
    assert D > 8 * torch.cuda.get_device_properties(0).multi_processor_count
    f = synth.random_frame(np.random.default_rng(D + T + L), 2, D, T, 2)
    taps = np.random.default_rng(L).normal(size=L).astype(np.float32)
    x = f.x_f32()
    _say(f"rows of several steps D={D} T={T} L={L}")
    one, two = _both(f, [x, np.ascontiguousarray(x[:, ::-1])], monkeypatch, fir_taps=taps)
    for a, b in zip(one, two):
        np.testing.assert_array_equal(b, a)
    rows = [0, 1, D // 2, D - 1]
    g = synth.random_frame(np.random.default_rng(D + T + L), 2, D, T, 2)
    g.dirs = g.dirs[rows]
    y_ref = oracle.frame_rows(g, x=x.astype(np.float64))
    check_t1(two[0][rows], oracle.envelope(y_ref, taps.astype(np.float64)))
