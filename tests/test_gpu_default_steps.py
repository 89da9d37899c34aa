"""The two-step launches that clbm_step chooses by itself for FP32 row-layout
lattices: the state ends in the buffer that single steps leave it in, however
the steps are split over calls, and a captured call of an even number of steps
can be replayed."""
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
