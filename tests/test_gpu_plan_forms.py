"""Which forms a plan's launches take, read from the line that DMAS_LOG prints."""

import re

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu] {msg}", flush=True)


def _logged(capfd, monkeypatch, f, **kw):
    """A plan for frame f and what its DMAS_LOG line says, as a dict of strings."""
    from paper_2511_09165_amd import plan_for_frame
    monkeypatch.setenv("DMAS_LOG", "1")
    capfd.readouterr()
    plan = plan_for_frame(f, **kw)
    lines = [ln for ln in capfd.readouterr().err.splitlines() if ln.startswith("[dmas] plan ")]
    assert len(lines) == 1
    return plan, dict(re.findall(r"(\w+)=(\S+)", lines[0]))


# the block of the tables (None: the plan's) and of the plane-free launch: the whole array, a
# multiple of it, a divisor of it, one that no smaller block divides
@pytest.mark.parametrize("M,block", [(9, None), (33, None), (64, None), (40, 24), (40, 20), (37, 23)])
@pytest.mark.parametrize("accumulate", ["kahan", "f64"])
def test_plane_free_calls_leave_the_other_launches_as_they_are(M, block, accumulate, monkeypatch, capfd):
    """Kahan and FP64 sums: whether single calls take the roots while staging does not change the
    tables, blocks and LDS of the plan's other launches (a server's); single calls and served
    frames give the bits of a plan that reads a root plane."""
    from paper_2511_09165_amd import Server
    f = synth.random_frame(np.random.default_rng(M), M, 21, 900, 3)
    x = f.x_f32()
    if block is not None:
        monkeypatch.setenv("DMAS_MIC_BLOCK", str(block))
    got, log = {}, {}
    for direct in ("0", "1"):
        monkeypatch.setenv("DMAS_DIRECT_ROOTS", direct)
        plan, log[direct] = _logged(capfd, monkeypatch, f, accumulate=accumulate)
        _say(f"M={M} block={block} {accumulate} direct={log[direct].get('direct')}")
        with plan, Server(64 << 20, staging=4 << 20) as srv:
            xt = torch.from_numpy(x).cuda()
            t = srv.submit(plan, x)
            srv.wait(t, 30.0)
            got[direct] = [plan.envelope(xt).cpu().numpy(), plan.beamform(xt).cpu().numpy(), srv.fetch(t)]
            srv.release(t)
    same = ("tables", "mb", "row", "lds", "occupancy", "seg", "nseg")
    assert {k: log["1"].get(k) for k in same} == {k: log["0"].get(k) for k in same}
    assert log["0"]["direct"] == "0" and 1 <= int(log["1"]["direct"]) <= 16
    assert log["1"]["tables"] == "mics"
    for a, b in zip(got["0"], got["1"]):
        np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(got["1"][2], got["1"][0])


@pytest.mark.parametrize("M", range(4, 20))
def test_plan_memory_that_a_budget_counts(M):
    """The device memory a plan reports: geometry, tiles, taps, 36 bytes of tables per tile and
    microphone and 64 spare; a server whose budget is exactly that and a frame's takes the frame."""
    from paper_2511_09165_amd import Server, plan_for_frame
    D, T = 16, 300
    f = synth.random_frame(np.random.default_rng(M), M, D, T, 3)
    up = lambda n: (n + 255) & ~255
    with plan_for_frame(f) as plan:
        info = plan.info()
        want = 24 * (M + D) + 32 * info["num_tiles"] + 4 * 64 + 36 * info["num_tiles"] * M + 64
        assert info["device_bytes"] == want
        _say(f"budget M={M}: {want} bytes of plan")
        with Server(up(4 * M * T) + up(4 * D * T) + up(8 * M * T) + up(want), staging=1 << 20) as srv:
            t = srv.submit(plan, f.x_f32())
            assert srv.wait(t, 30.0)["t_done"] > 0
            srv.release(t)


def test_rf_frames_are_packed_by_long_walks(monkeypatch, capfd):
    """A server counts an RF frame's workgroups as long walks, not as the short segments of single
    calls: two frames whose segments together exceed a launch's cap of two device rounds still
    share one, with the bits of the calls alone."""
    from paper_2511_09165_amd import Server, plan_for_frame
    monkeypatch.setenv("DMAS_SMALL_LAUNCH_WGS", "0")          # frames behind the first wait and are packed
    first = synth.random_frame(np.random.default_rng(1), 32, 4096, 16384, 5)
    f = synth.random_frame(np.random.default_rng(2), 16, 600, 4096, 3)
    plan, log = _logged(capfd, monkeypatch, f)
    tiles, walks = int(log["tiles"]), int(log["nseg"].split("/")[0])
    calls = -(-4096 // int(log["call"]))
    cap = 2 * 3 * torch.cuda.get_device_properties(0).multi_processor_count
    _say(f"packing: {tiles} tiles, {walks} walks, {calls} segments, cap {cap}")
    assert 2 * tiles * walks <= cap < 2 * tiles * calls
    with plan, plan_for_frame(first) as plan1, Server(4 << 30, staging=64 << 20) as srv:
        ref = plan.beamform(torch.from_numpy(f.x_f32()).cuda()).cpu().numpy()
        x1, x = first.x_f32(), f.x_f32()
        heads = [srv.submit(plan1, x1) for _ in range(2)]
        tickets = [srv.submit(plan, x, envelope=False) for _ in range(8)]
        infos = [srv.wait(t, 30.0) for t in tickets]
        assert max(i["batch_frames"] for i in infos) >= 2
        for t in tickets:
            np.testing.assert_array_equal(srv.fetch(t), ref)
        for t in tickets + heads:
            srv.wait(t, 30.0)
            srv.release(t)


@pytest.mark.parametrize("n", [3, 5])
@pytest.mark.parametrize("envelope", [False, True])
def test_resident_workers_take_two_workgroups_a_unit(n, envelope, monkeypatch, capfd):
    """Small windows would let three or four worker workgroups share a compute unit; each costs a
    descriptor read and a write-back per job, and two serve frames faster."""
    from paper_2511_09165_amd import Server, plan_for_frame
    monkeypatch.setenv("DMAS_LOG", "1")
    f = synth.random_frame(np.random.default_rng(n), 16, 200, 900, n)
    f.mic_pos = f.mic_pos * 0.1
    x = f.x_f32()
    _say(f"resident workgroups n={n} envelope={envelope}")
    with plan_for_frame(f) as plan, Server(64 << 20, staging=4 << 20, resident=True) as srv:
        xt = torch.from_numpy(x).cuda()
        ref = (plan.envelope(xt) if envelope else plan.beamform(xt)).cpu().numpy()
        capfd.readouterr()
        t = srv.submit(plan, x, envelope=envelope)
        srv.wait(t, 30.0)
        np.testing.assert_array_equal(srv.fetch(t), ref)
        srv.release(t)
    logged = re.findall(r"resident worker n=(\d) env=(\d) workgroups=(\d+)", capfd.readouterr().err)
    assert logged and logged[0][:2] == (str(n), str(int(envelope)))
    assert int(logged[0][2]) == 2 * torch.cuda.get_device_properties(0).multi_processor_count


def test_overrides_choose_the_forms(monkeypatch, capfd):
    """The overrides that the tests of equal forms rely on do choose the form, on either side of the
    plan's own choice; a form that cannot run is not chosen."""
    small = synth.random_frame(np.random.default_rng(3), 8, 20, 500, 3)
    large = synth.random_frame(np.random.default_rng(4), 64, 1200, 8192, 3)

    def forms(f, env, **kw):
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        plan, log = _logged(capfd, monkeypatch, f, **kw)
        plan.close()
        for k in env:
            monkeypatch.delenv(k)
        return log["direct"] != "0", int(log["passes"])

    _say("plan forms")
    assert forms(small, {}) == (True, 1)
    assert forms(large, {}) == (False, 2)
    for f in (small, large):
        for direct in (False, True):
            for passes in (1, 2):
                env = {"DMAS_DIRECT_ROOTS": str(int(direct)), "DMAS_ENVELOPE_PASSES": str(passes)}
                assert forms(f, env) == (direct, passes)
    force = {"DMAS_DIRECT_ROOTS": "1", "DMAS_ENVELOPE_PASSES": "2"}
    assert forms(small, force, env_decimation=2) == (True, 1)              # decimated: the fused filter
    assert forms(small, force, linear=True) == (False, 2)          # no roots
    assert forms(small, dict(force, DMAS_NO_DELAY_TABLE="1")) == (False, 2)
    assert forms(small, dict(force, DMAS_RING_SHARING="1")) == (False, 2)
    assert forms(small, dict(force, DMAS_BLOCK_TABLES="0")) == (False, 2)


def test_plane_free_plan_in_a_graph(monkeypatch, capfd):
    """A plan whose calls use no root plane, and one in two passes, replay from a graph with eager
    calls between the replays."""
    monkeypatch.setenv("DMAS_DIRECT_ROOTS", "1")
    monkeypatch.setenv("DMAS_ENVELOPE_PASSES", "2")
    f = synth.random_frame(np.random.default_rng(6), 12, 40, 2500, 3)
    plan, log = _logged(capfd, monkeypatch, f)
    assert log["direct"] != "0" and log["passes"] == "2"
    _say("plane-free two-pass plan in a graph")
    with plan:
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("place", ["start", "end", "before", "behind"])
def test_output_over_the_channels(place, dtype, monkeypatch, capfd):
    """A plan with roots reads its channels into a root plane before it writes, so an output may lie
    over them; a plan whose calls use no plane does so too, and where the two only touch it does
    not need to."""
    monkeypatch.setenv("DMAS_DIRECT_ROOTS", "1")
    f = synth.random_frame(np.random.default_rng(8), 48, 400, 4000, 3)
    plan, log = _logged(capfd, monkeypatch, f, in_dtype=dtype)
    assert log["direct"] != "0"
    _say(f"output over the channels: {place} {dtype}")
    xt = torch.from_numpy(f.x_f32()).cuda().to({"f32": torch.float32, "bf16": torch.bfloat16}[dtype])
    xb, yb = xt.numel() * xt.element_size(), 4 * f.num_dirs * f.num_samples
    x_at, y_at = {"start": (0, 0), "end": (yb - xb, 0), "before": (yb, 0), "behind": (0, xb)}[place]
    with plan:
        ref = [plan.beamform(xt), plan.envelope(xt)]
        for _ in range(5):
            for call, want in zip((plan.beamform, plan.envelope, plan.envelope_noalloc), ref + ref[1:]):
                buf = torch.zeros(xb + yb, dtype=torch.uint8, device="cuda")
                x = buf[x_at:x_at + xb].view(xt.dtype).view(xt.shape)
                y = buf[y_at:y_at + yb].view(torch.float32).view(want.shape)
                x.copy_(xt)
                call(x, y) if call == plan.envelope_noalloc else call(x, out=y)
                assert torch.equal(y, want)


def test_blocks_without_tables_do_not_depend_on_the_record(monkeypatch, capfd):
    """Without delay tables a block can hold 64 microphones: its size follows the occupancy alone,
    also where the record is too short to give every compute unit several workgroups."""
    monkeypatch.setenv("DMAS_NO_DELAY_TABLE", "1")
    _say("blocks without tables")
    mb = {}
    for D, T in ((240, 2048), (240, 60000)):
        f = synth.random_frame(np.random.default_rng(9), 512, 8, T, 4)
        f.dirs = synth.unit_vectors(np.linspace(-60, 60, D), np.zeros(D))
        plan, log = _logged(capfd, monkeypatch, f)
        plan.close()
        assert log["tables"] == "none"
        mb[T] = log["mb"]
    assert mb[2048] == mb[60000]


# sizes where reading a root plane was measured faster (by more than a tenth) or slower
@pytest.mark.parametrize("M,na,ne,T,n,L,accumulate,chosen", [
    (8, 64, 1, 1024, 2, 63, "f32", "ren"),
    (19, 181, 1, 3001, 3, 63, "f32", "ren"),
    (19, 77, 30, 1659, 8, 63, "kahan", "---"),
    (48, 52, 20, 1101, 2, 255, "f32", "r--"),
    (50, 71, 55, 303, 3, 255, "f32", "--"),                      # (RF images: either)
    (113, 10, 1, 13403, 4, 255, "f32", "--"),
    (32, 1035, 1, 8192, 3, 63, "f32", "---"),
])
def test_calls_without_a_root_plane(M, na, ne, T, n, L, accumulate, chosen, monkeypatch, capfd):
    """RF images, envelopes and envelopes that allocate nothing take the roots while staging where
    that is the faster for each."""
    f = synth.random_frame(np.random.default_rng(1), M, 8, T, n)
    A, B = np.meshgrid(np.linspace(-60, 60, na), np.linspace(-30, 30, ne) if ne > 1 else [0.0])
    f.dirs = synth.unit_vectors(A.ravel(), B.ravel())
    plan, log = _logged(capfd, monkeypatch, f, accumulate=accumulate, fir_len=L)
    plan.close()
    _say(f"plane-free calls M={M} T={T} n={n} L={L} {accumulate}: {log['plane_free']}")
    assert log["plane_free"].endswith(chosen)


# sizes where one pass, or two, were measured faster by 7 % and more
@pytest.mark.parametrize("M,na,ne,T,n,L,passes", [
    (64, 45, 23, 8192, 3, 63, 2),
    (17, 113, 56, 6131, 3, 63, 2),
    (7, 74, 48, 8580, 7, 31, 1),
    (12, 74, 48, 8580, 7, 63, 1),
    (12, 4032, 1, 4920, 6, 1, 1),
    (143, 70, 36, 8580, 7, 63, 2),
])
def test_passes_of_an_envelope(M, na, ne, T, n, L, passes, monkeypatch, capfd):
    """The plan takes the faster of the fused filter and a pass over the image."""
    f = synth.random_frame(np.random.default_rng(1), M, 8, T, n)
    A, B = np.meshgrid(np.linspace(-60, 60, na), np.linspace(-30, 30, ne) if ne > 1 else [0.0])
    f.dirs = synth.unit_vectors(A.ravel(), B.ravel())
    plan, log = _logged(capfd, monkeypatch, f, fir_len=L)
    plan.close()
    _say(f"passes M={M} D={na * ne} T={T} n={n} L={L}: {log['passes']}")
    assert int(log["passes"]) == passes


@pytest.mark.parametrize("M,D,T,n,L,passes", [(27, 275, 21826, 5, 101, 1), (157, 153, 7406, 8, 101, 2)])
def test_passes_of_few_long_rows(M, D, T, n, L, passes, monkeypatch, capfd):
    """The second pass walks a row step by step: with few rows that is weighed too."""
    f = synth.random_frame(np.random.default_rng(1), M, 8, T, n)
    f.dirs = synth.unit_vectors(np.linspace(-60, 60, D), np.zeros(D))
    plan, log = _logged(capfd, monkeypatch, f, fir_len=L)
    plan.close()
    _say(f"passes M={M} D={D} T={T} n={n} L={L}: {log['passes']}")
    assert int(log["passes"]) == passes


@pytest.mark.parametrize("M,D,T,n,L,accumulate", [(59, 96, 8192, 5, 57, "f64"), (19, 640, 1199, 4, 63, "f64"),
                                                  (10, 791, 12811, 3, 63, "kahan")])
def test_segments_of_plane_free_envelopes(M, D, T, n, L, accumulate, monkeypatch, capfd):
    """Kahan and FP64 sums: a plane-free launch that holds fewer workgroups takes longer segments;
    the image, fresh and with a fixed scratch, and a served frame keep the plane's bits."""
    from paper_2511_09165_amd import Server
    f = synth.random_frame(np.random.default_rng(2), M, 8, T, n)
    f.dirs = synth.unit_vectors(np.linspace(-60, 60, D), np.zeros(D))
    x, got, segments = f.x_f32(), {}, {}
    for direct in ("0", "1"):
        monkeypatch.setenv("DMAS_DIRECT_ROOTS", direct)
        plan, log = _logged(capfd, monkeypatch, f, accumulate=accumulate, fir_len=L)
        segments[direct] = int(log["nseg"].split("/")[1])
        _say(f"M={M} D={D} T={T} n={n} L={L} {accumulate} direct={direct}: {segments[direct]} segments")
        with plan, Server(256 << 20, staging=32 << 20) as srv:
            xt = torch.from_numpy(x).cuda()
            t = srv.submit(plan, x)
            srv.wait(t, 30.0)
            out = plan.envelope(xt)
            got[direct] = [out.cpu().numpy(), srv.fetch(t),
                           plan.envelope_noalloc(xt, torch.full_like(out, float("nan"))).cpu().numpy()]
            srv.release(t)
    assert segments["1"] <= segments["0"]
    for a in got["0"] + got["1"]:
        np.testing.assert_array_equal(a, got["0"][0])
