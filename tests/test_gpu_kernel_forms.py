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


@pytest.mark.parametrize("L", [1, 63, 65, 67, 255])          # 63 and 65 keep their taps in registers
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


# (M, D, T, order): microphone blocks of one partial, one full, several; a record shorter than a
# window; a window tail shorter than a wave
DIRECT = [(3, 5, 40, 2), (8, 64, 1024, 2), (16, 9, 257, 3), (17, 30, 700, 4), (33, 21, 512, 5), (70, 12, 300, 8)]


@pytest.mark.parametrize("M,D,T,n", DIRECT)
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("nearfield", [False, True])
def test_roots_taken_while_staging_give_the_plane_bits(M, D, T, n, dtype, nearfield, monkeypatch):
    """Small frames take the signed roots while staging; the image and envelope equal, bit for bit,
    those of a plan that reads them from a root plane, and the plane-free call needs no scratch."""
    from paper_2511_09165_amd import plan_for_frame
    f = synth.random_frame(np.random.default_rng(M + D + T + n), M, D, T, n, nearfield=nearfield)
    x = f.x_f32()
    x[0, ::7] = 0.0
    x[M // 2, 3::11] = np.float32(1e-39)                     # below the FP32 normal range
    xt = torch.from_numpy(x).cuda().to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype])
    _say(f"direct roots M={M} D={D} T={T} n={n} {dtype} near={nearfield}")
    got = {}
    for direct in ("0", "1"):
        monkeypatch.setenv("DMAS_DIRECT_ROOTS", direct)
        with plan_for_frame(f, in_dtype=dtype) as plan:
            env = torch.empty((D, T), dtype=torch.float32, device="cuda")
            got[direct] = [plan.beamform(xt), plan.envelope(xt), plan.envelope_noalloc(xt, env)]
            torch.cuda.synchronize()
    for a, b in zip(got["0"], got["1"]):
        assert torch.equal(a, b)
    if dtype == "f32":
        check_t1(got["1"][0].cpu().numpy(), oracle.frame_rows(f, x=x.astype(np.float64)))


@pytest.mark.parametrize("accumulate", ["kahan", "f64"])
@pytest.mark.parametrize("n", [2, 5, 7])
def test_direct_roots_with_other_sums(accumulate, n, monkeypatch):
    """The same for the compensated and FP64 sums, with more microphones than one table block."""
    f = synth.random_frame(np.random.default_rng(9 + n), 21, 33, 900, n)
    _say(f"direct roots {accumulate} n={n}")
    got = {}
    for direct in ("0", "1"):
        monkeypatch.setenv("DMAS_DIRECT_ROOTS", direct)
        got[direct] = _image(f, f.x_f32(), accumulate=accumulate)
    np.testing.assert_array_equal(got["0"], got["1"])
    y_ref = oracle.frame_rows(f, x=f.x_f32().astype(np.float64))
    taps = oracle.lowpass_taps(63, 5000.0, f.fs).astype(np.float32).astype(np.float64)
    check_t1(got["1"], oracle.envelope(y_ref, taps))


@pytest.mark.parametrize("T", [1, 63, 900])
@pytest.mark.parametrize("spread", [0.004, 0.05, 0.15, 0.4])
@pytest.mark.parametrize("M", [3, 8, 9, 16, 25])
def test_direct_rows_and_record_ends(M, spread, T, monkeypatch):
    """No, one or two rows a wave, windows of one to several rounds of loads (five pieces of 64 and
    up), and records shorter than a window: the bits of the root plane. The first and last samples
    are not finite, so a sample taken from outside its place shows."""
    from paper_2511_09165_amd import plan_for_frame
    f = synth.random_frame(np.random.default_rng(100 * M + T), M, 19, T, 3)
    f.mic_pos = f.mic_pos * (spread / np.abs(f.mic_pos).max())
    x = f.x_f32().copy()
    x[0, 0], x[1, T - 1], x[M - 1, 0] = np.inf, np.nan, -np.inf
    _say(f"direct rows M={M} spread={spread} T={T}")
    got = {}
    for direct in ("0", "1"):
        monkeypatch.setenv("DMAS_DIRECT_ROOTS", direct)
        with plan_for_frame(f) as plan:
            xt = torch.from_numpy(x).cuda()
            got[direct] = [plan.beamform(xt).cpu().numpy(), plan.envelope(xt).cpu().numpy()]
    for a, b in zip(got["0"], got["1"]):
        np.testing.assert_array_equal(a, b)


def test_direct_plan_in_a_graph_and_on_two_streams():
    """A plan without a root plane replays from a graph, with eager calls between, and runs on two
    streams at once: every result equals the eager one."""
    from paper_2511_09165_amd import plan_for_frame
    f = synth.random_frame(np.random.default_rng(5), 12, 40, 1500, 3)
    _say("direct plan, graph and streams")
    with plan_for_frame(f) as plan:
        x = torch.from_numpy(f.x_f32()).cuda()
        ref = plan.envelope(x)
        out = torch.empty_like(ref)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            plan.envelope(x, out=out)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            plan.envelope(x, out=out)
        for _ in range(3):
            out.fill_(float("nan"))
            g.replay()
            with torch.cuda.stream(side):
                other = plan.envelope(x)
            torch.cuda.synchronize()
            assert torch.equal(out, ref) and torch.equal(other, ref)


def test_plane_rows_too_short_for_padding(monkeypatch):
    """A wide array on a short record keeps its root plane unpadded; windows that reach past the
    record then take the element-wise path: the same bits as roots taken while staging, and T1."""
    f = synth.random_frame(np.random.default_rng(15), 9, 20, 300, 3)
    f.mic_pos = f.mic_pos * (1.5 / np.abs(f.mic_pos).max())          # delays up to about 2000 samples
    _say("unpadded plane")
    got = {}
    for direct in ("0", "1"):
        monkeypatch.setenv("DMAS_DIRECT_ROOTS", direct)
        got[direct] = _image(f, f.x_f32())
    np.testing.assert_array_equal(got["0"], got["1"])
    taps = oracle.lowpass_taps(63, 5000.0, f.fs).astype(np.float32).astype(np.float64)
    check_t1(got["0"], oracle.envelope(oracle.frame_rows(f, x=f.x_f32().astype(np.float64)), taps))


def test_fixed_scratch_that_holds_only_the_unpadded_plane(monkeypatch):
    """dmas_envelope_noalloc at its limit: the plane fills the fixed scratch without padding, and
    gives the bits of the padded plane from the pool."""
    from paper_2511_09165_amd import plan_for_frame
    monkeypatch.setenv("DMAS_DIRECT_ROOTS", "0")
    f = synth.random_frame(np.random.default_rng(16), 64, 9, 32768, 2)
    _say("plane of exactly the fixed scratch")
    with plan_for_frame(f) as plan:
        x = torch.from_numpy(f.x_f32()).cuda()
        ref = plan.envelope(x)
        out = plan.envelope_noalloc(x, torch.empty_like(ref))
        torch.cuda.synchronize()
        assert torch.equal(ref, out)


@pytest.mark.parametrize("D,T", [(200, 700), (512, 1024), (640, 2048), (701, 3003)])
def test_fetch_moves_whole_results(D, T):
    """Results fetched from a server, below and above the size that goes by chunks (2 MiB exactly,
    whole chunks, a ragged tail), from several threads at once: the standalone call's bits."""
    import threading
    from paper_2511_09165_amd import Server, plan_for_frame
    f = synth.random_frame(np.random.default_rng(D + T), 4, D, T, 3)
    _say(f"fetch D={D} T={T}")
    with plan_for_frame(f) as plan, Server(256 << 20, staging=16 << 20) as srv:
        ref = plan.envelope(torch.from_numpy(f.x_f32()).cuda()).cpu().numpy()
        tickets = [srv.submit(plan, f.x_f32()) for _ in range(4)]
        for t in tickets:
            srv.wait(t, 30.0)
        got = {}

        def fetch(t):
            got[t] = [srv.fetch(t) for _ in range(3)]

        threads = [threading.Thread(target=fetch, args=(t,)) for t in tickets]
        for t in threads:
            t.start()
        for t in threads:
            t.join(60.0)
        assert len(got) == 4
        for images in got.values():
            for y in images:
                np.testing.assert_array_equal(y, ref)
        for t in tickets:
            srv.release(t)


def test_root_plane_of_more_rows_than_a_grid_dimension(monkeypatch):
    """More microphones than the root pass has workgroup rows: the bits of roots taken while
    staging, and T1."""
    f = synth.random_frame(np.random.default_rng(17), 70001, 9, 40, 2)
    _say("root plane of 70001 rows")
    got = {}
    for direct in ("0", "1"):
        monkeypatch.setenv("DMAS_DIRECT_ROOTS", direct)
        got[direct] = _image(f, f.x_f32())
    np.testing.assert_array_equal(got["0"], got["1"])
    taps = oracle.lowpass_taps(63, 5000.0, f.fs).astype(np.float32).astype(np.float64)
    check_t1(got["0"], oracle.envelope(oracle.frame_rows(f, x=f.x_f32().astype(np.float64)), taps))


@pytest.mark.parametrize("M,T", [(8, 255), (8, 257), (64, 3680), (64, 3681), (130, 40001)])
def test_root_plane_with_one_and_four_elements_a_thread(M, T, monkeypatch):
    """Planes below and above 2^18 elements, rows on and off the workgroups' blocks: the bits of
    roots taken while staging."""
    f = synth.random_frame(np.random.default_rng(M + T), M, 9, T, 3)
    f.x[0, 0], f.x[M - 1, T - 1] = np.inf, np.nan                    # the plane's first and last samples
    _say(f"root plane {M} x {T}")
    got = {}
    for direct in ("0", "1"):
        monkeypatch.setenv("DMAS_DIRECT_ROOTS", direct)
        got[direct] = _image(f, f.x_f32())
    np.testing.assert_array_equal(got["0"], got["1"])
