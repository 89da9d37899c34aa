"""The two-step launches that clbm_step chooses by itself for FP32 row-layout
lattices: the state ends in the buffer that single steps leave it in, with the
same bits, however the steps are split over calls, and a captured call of an
even number of steps can be replayed."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def clbm():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1908_05396_amd import clbm as c
    c.load()
    return c


def _box(nx, ny, nz, **kw):
    return W.cavity(64, 0.05, 0.8, 300.0).with_(nx=nx, ny=ny, nz=nz, **kw)


# shapes that the cost model pairs at 256 compute units
SHAPES = [(160, 160, 160), (62, 14, 4000), (201, 191, 221)]


def _kernels(fn):
    """Names of the step kernels that fn launches, in order."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    ev = [e for e in prof.events() if "stream_collide" in e.name]
    return [e.name for e in sorted(ev, key=lambda e: e.time_range.start)]


@pytest.mark.parametrize("shape", SHAPES)
def test_default_steps_run_in_two_step_launches(clbm, shape):
    print(f"[gpu] default kernels {shape}", flush=True)
    lat = clbm.Lattice(_box(*shape), storage="f32", track_residual=False)
    lat.init_rest()
    names = _kernels(lambda: lat.step(11))
    lat.close()
    two = ["stream_collide2" in n for n in names]
    assert two == [True] * 4 + [False] * 3


@pytest.mark.parametrize("shape", SHAPES)
def test_state_buffer_follows_the_step_count(clbm, shape):
    print(f"[gpu] default buffer {shape}", flush=True)
    lat = clbm.Lattice(_box(*shape), storage="f32", track_residual=False)
    lat.init_rest()
    done = 0
    for k in (2, 1, 3, 4, 6, 7, 2):
        lat.step(k)
        done += k
        assert lat.state() == (done % 2, done)
    lat.close()


@pytest.mark.parametrize("k", [2, 4, 6])
def test_captured_steps_replay(clbm, k):
    """k steps captured and replayed, with eager steps between the replays,
    against the same steps without a graph."""
    spec = _box(160, 160, 160)
    print(f"[gpu] captured step({k})", flush=True)
    f0 = W.perturbed_populations(spec, 4, 1e-2, device="cuda")
    ref = clbm.Lattice(spec, storage="f32", track_residual=False)
    lat = clbm.Lattice(spec, storage="f32", track_residual=False)
    for x in (ref, lat):
        x.init_populations(f0)
        x.step(k)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lat.step(k)
    for _ in range(3):
        graph.replay()
        ref.step(k)
        torch.cuda.synchronize()
        assert torch.equal(lat.state_view(), ref.state_view())
        for x in (ref, lat):
            x.step(2)
    torch.cuda.synchronize()
    assert torch.equal(lat.state_view(), ref.state_view())
    ref.close()
    lat.close()


LIDS = {W.LID_MX: (0.0, 0.03, 0.02), W.LID_PX: (0.0, 0.03, -0.02), W.LID_MY: (0.03, 0.0, 0.02),
        W.LID_PY: (0.05, 0.0, 0.0), W.LID_MZ: (0.03, 0.02, 0.0), W.LID_PZ: (0.03, -0.02, 0.0)}


@pytest.mark.parametrize("shape,periodic,lid",
                         [((160, 160, 160), (0, 0, 0), lid) for lid in LIDS] +
                         [((201, 191, 221), (1, 0, 0), W.LID_PY), ((201, 191, 221), (0, 1, 0), W.LID_MX),
                          ((160, 160, 160), (1, 1, 0), W.LID_MZ), ((62, 14, 4000), (1, 1, 0), W.LID_PZ),
                          ((160, 160, 160), (1, 1, 0), W.LID_NONE)])
def test_results_do_not_depend_on_the_split(clbm, shape, periodic, lid):
    """Eight steps in one call (two-step launches), in calls of 5 and 3, and one
    by one: the same operations with the same roundings, so the same bits."""
    spec = _box(*shape, periodic=periodic, lid_face=lid, lid_velocity=LIDS.get(lid, (0.0, 0.0, 0.0)))
    print(f"[gpu] default split {shape} periodic {periodic} lid {lid}", flush=True)
    f0 = W.perturbed_populations(spec, 6, 1e-2, device="cuda")
    outs = []
    for calls in ((8,), (5, 3), (1,) * 8):
        lat = clbm.Lattice(spec, storage="f32", track_residual=False)
        lat.init_populations(f0)
        for k in calls:
            lat.step(k)
        outs.append(lat.state_view().clone())
        lat.close()
    assert torch.equal(outs[0], outs[2]) and torch.equal(outs[1], outs[2])


def _launches(fn, tmp_path):
    """{(kernel, workgroups, threads)} of the step kernels that fn launches."""
    import json
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    path = tmp_path / "trace.json"
    prof.export_chrome_trace(str(path))
    events = json.loads(path.read_text())["traceEvents"]
    return {(e["name"], e["args"]["grid"][0], e["args"]["block"][0]) for e in events
            if e.get("cat") == "kernel" and "stream_collide" in e["name"]}


@pytest.mark.parametrize("shape,storage,steps", [((201, 191, 221), "f32", 4), ((201, 191, 221), "f32", 1),
                                                 ((300, 440, 440), "f32", 1), ((70, 50, 40), "f64", 1)])
def test_autotune_tries_the_default(clbm, tmp_path, shape, storage, steps):
    """The launches that steps take by default are among those that the tuner
    times: its choice is no worse than leaving it uncalled."""
    print(f"[gpu] autotune {shape} {storage}", flush=True)
    lat = clbm.Lattice(_box(*shape), storage=storage, track_residual=False)
    lat.init_rest()
    default = _launches(lambda: lat.step(steps), tmp_path)
    tried = _launches(lat.autotune, tmp_path)
    lat.close()
    assert len(default) == 1 and default <= tried
