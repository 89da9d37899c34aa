"""Row-layout lattices whose z layers lie beyond the reach of 32-bit offsets
(some 430 MB a layer and more), against the planes layout.  Node coordinates
and sources take 64-bit offsets there, one thread per node at any width; with a
wave per row, or a workgroup per row, the narrow ones among them would need more
than the 2^32 threads that a launch can have, and the runtime starts only the
remainder without an error."""
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


BYTES = {"f64": 8, "f32": 4, "f16": 2}
TOL = {"f64": 1e-13, "f32": 2e-6, "f16": 2e-3}      # as the other comparisons of the layouts


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("storage,nx,ny,nz,periodic,lid", [
    ("f64", 1, 4200000, 7, (0, 0, 0), W.LID_PZ),
    ("f64", 7, 420000, 10, (1, 0, 1), W.LID_PY),
    ("f64", 70, 42000, 10, (0, 1, 0), W.LID_MX),
    ("f32", 1, 5700000, 12, (0, 0, 1), W.LID_MY),
    ("f32", 20, 290000, 10, (0, 1, 0), W.LID_PX),
    ("f32", 300, 20000, 10, (1, 1, 0), W.LID_MZ),
    ("f16", 20, 580000, 10, (1, 1, 1), W.LID_NONE),
])
def test_wide_layers_match_planes(clbm, storage, nx, ny, nz, periodic, lid, in_place):
    layer = 19 * BYTES[storage] * nx * ny
    assert layer * 5 >= 2 ** 31 and layer * (nz + 1) >= 2 ** 32
    u = [0.02, 0.03, -0.01]
    if lid:
        u[(lid - 1) // 2] = 0.0
    spec = W.LatticeSpec(nx=nx, ny=ny, nz=nz, K=0.02, n=0.8, periodic=periodic, lid_face=lid,
                         lid_velocity=tuple(u) if lid else (0.0, 0.0, 0.0), name="wide")
    print(f"[gpu] wide {storage} {nx}x{ny}x{nz} in_place={in_place}", flush=True)
    f0 = W.perturbed_populations(spec, 8, 1e-2, device="cuda")
    outs = []
    for layout in ("rows", "planes"):
        lat = clbm.Lattice(spec, storage=storage, track_residual=False, layout=layout, in_place=in_place)
        lat.init_populations(f0)
        lat.step(2)
        outs.append(lat.state_view())
        lat.close()
    for k in range(19):
        scale = outs[1][k].abs().max().double().item()
        diff = (outs[0][k].double() - outs[1][k].double()).abs().max().item()
        assert diff <= TOL[storage] * scale, (k, diff, scale)
    del f0, outs
    torch.cuda.empty_cache()
