"""Paths of the row-layout kernels that only certain sizes and boundaries take:
the two-step launch with its loads a plane ahead on periodic x and y axes and
under a lid on each face, a wave per run of a row beyond 4 GiB, and 32-bit
offsets between 2 and 4 GiB.  Bounds as in the two-step and layout tests."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

TOL_U = {"f64": 1e-12, "f32": 1e-5, "f16": 2e-3}            # velocity against the oracle
REL = {"f64": 1e-13, "f32": 1e-5, "f16": 2e-2}              # two steps against one, of the largest deviation
TOL = {"f64": 1e-13, "f32": 2e-6, "f16": 2e-3}              # rows against planes, of the direction's largest deviation


@pytest.fixture(scope="module")
def clbm():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1908_05396_amd import clbm as c
    c.load()
    return c


LIDS = {W.LID_NONE: (0.0, 0.0, 0.0), W.LID_MX: (0.0, 0.03, 0.02), W.LID_PX: (0.0, 0.03, -0.02),
        W.LID_MY: (0.03, 0.0, 0.02), W.LID_PY: (0.03, 0.0, -0.02), W.LID_MZ: (0.03, 0.02, 0.0),
        W.LID_PZ: (0.03, -0.02, 0.0)}


def _spec(nx, ny, nz, periodic, lid):
    return W.LatticeSpec(nx=nx, ny=ny, nz=nz, K=0.02, n=0.8, periodic=periodic, lid_face=lid, lid_velocity=LIDS[lid],
                         name="path")


GEOMETRIES = [((1, 0, 0), W.LID_MY), ((1, 0, 0), W.LID_PZ), ((0, 1, 0), W.LID_PX), ((0, 1, 0), W.LID_MZ),
              ((1, 1, 0), W.LID_MZ), ((1, 1, 0), W.LID_NONE), ((0, 0, 0), W.LID_PX), ((0, 0, 0), W.LID_MY),
              ((0, 0, 0), W.LID_MZ)]


@pytest.mark.parametrize("periodic,lid", GEOMETRIES)
@pytest.mark.parametrize("storage,rows", [("f32", 8), ("f32", 12), ("f32", 16), ("f64", 8), ("f16", 16)])
def test_two_step_boundaries_over_several_patches(clbm, storage, rows, periodic, lid):
    """130 x 40 x 11: three patches along x, three to seven along y, three z chunks."""
    spec = _spec(130, 40, 11, periodic, lid)
    print(f"[gpu] two-step {storage} rows={rows} periodic {periodic} lid {lid}", flush=True)
    f0 = W.perturbed_populations(spec, 12, 1e-2)
    steps, got = 6, {}
    for launch in ({"fuse_steps": 1}, {"fuse_steps": 2, "fuse_rows": rows, "fuse_planes": 4}):
        lat = clbm.Lattice(spec, storage=storage, track_residual=False, layout="rows", launch=launch)
        lat.init_populations(f0.to("cuda"))
        lat.step(steps)
        got[launch["fuse_steps"]] = (lat.state_view().double(), lat.macroscopic()[1].cpu().numpy())
        lat.close()
    scale = got[1][0].abs().max().item()
    assert (got[2][0] - got[1][0]).abs().max().item() <= REL[storage] * scale
    _, u_ref = oracle.macroscopic(spec, oracle.run(spec, f0.numpy(), steps))
    assert np.abs(got[2][1] - u_ref).max() <= TOL_U[storage] * np.abs(u_ref).max()


def _against_planes(clbm, spec, storage, steps, flags=None, **kw):
    f0 = W.perturbed_populations(spec, 13, 1e-2, device="cuda")
    outs = []
    for layout in ("rows", "planes"):
        lat = clbm.Lattice(spec, storage=storage, track_residual=False, layout=layout, flags=flags, **kw)
        lat.init_populations(f0)
        lat.step(steps)
        outs.append(lat.state_view())
        lat.close()
    for k in range(19):
        scale = outs[1][k].abs().max().double().item()
        diff = (outs[0][k].double() - outs[1][k].double()).abs().max().item()
        assert diff <= TOL[storage] * scale, (k, diff, scale)
    del f0, outs
    torch.cuda.empty_cache()


@pytest.mark.parametrize("nx,ny,nz,periodic,lid", [(500, 340, 341, (0, 0, 0), W.LID_PX), (500, 340, 341, (1, 0, 0), W.LID_PZ),
                                                   (511, 337, 340, (0, 1, 1), W.LID_MX), (65, 941, 941, (1, 1, 1), W.LID_NONE),
                                                   (65, 941, 941, (0, 0, 1), W.LID_MY), (512, 335, 341, (0, 0, 0), W.LID_PY)])
def test_wave_per_row_beyond_4_gib(clbm, nx, ny, nz, periodic, lid):
    """One FP32 step per launch beyond the reach of 32-bit offsets: a wave takes
    64 columns of one row."""
    spec = _spec(nx, ny, nz, periodic, lid)
    assert 19 * 4 * spec.nodes > 2 ** 32
    print(f"[gpu] wave per row {nx}x{ny}x{nz} periodic {periodic} lid {lid}", flush=True)
    _against_planes(clbm, spec, "f32", 2, launch={"fuse_steps": 1})


@pytest.mark.parametrize("storage,nz", [("f64", 34003), ("f32", 69001), ("f16", 135001)])
@pytest.mark.parametrize("form", ["two_buffers", "in_place", "flagged"])
def test_offsets_between_2_and_4_gib(clbm, storage, nz, form):
    nx, ny = 70, 9
    size = {"f64": 8, "f32": 4, "f16": 2}[storage]
    spec = _spec(nx, ny, nz, (1, 0, 1), W.LID_PY)
    assert 3 * 2 ** 30 < 19 * size * spec.nodes < 2 ** 32 - 2 ** 25
    print(f"[gpu] 2 to 4 GiB {form} {storage}", flush=True)
    flags = None
    if form == "flagged":
        flags = torch.zeros((nz, ny, nx), dtype=torch.uint8, device="cuda")
        flags[0, 2:4, 10:20] = 1
        flags[nz - 1, 5:7, 30:50] = 2
        flags[nz - 1010:nz - 1000, 1:3, 60:70] = 1
    kw = {"launch": {"fuse_steps": 1}} if form == "two_buffers" else {}
    _against_planes(clbm, spec, storage, 2, flags=flags, in_place=form == "in_place", **kw)
