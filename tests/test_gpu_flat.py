"""The row layout's flat kernels at the edges of their addressing, the default
pairs of steps, and the reductions at the edges of their block counts.

The flat kernel takes 64 consecutive nodes per wave and addresses sources by
32-bit offsets: from the start of the state below 1 GiB (FP32, FP64), else from
the layer of the wave's first node, where the lanes that pull across a periodic
z face address in 64 bits.  The planes layout runs the same arithmetic through
another kernel, so the two agree to the compiler's choice of fused
multiply-adds (bounds of the layout tests).
"""
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


def _state(clbm, spec, storage, layout, steps):
    lat = clbm.Lattice(spec, storage=storage, track_residual=False, layout=layout)
    lat.init_populations(W.perturbed_populations(spec, 5, 1e-2, device="cuda"))
    lat.step(steps)
    st = lat.state_view().clone()
    lat.close()
    return st


@pytest.mark.parametrize("periodic", [(0, 0, 0), (1, 0, 1), (1, 1, 1)])
@pytest.mark.parametrize("storage,nx,ny,nz,tol", [("f64", 70, 9, 12001, 1e-13), ("f32", 50, 9, 33003, 2e-6),
                                                  ("f64", 3, 2, 65, 1e-13), ("f32", 1, 67, 3, 2e-6),
                                                  ("f32", 63, 1, 5, 2e-6), ("f16", 65, 3, 2, 2e-3)])
def test_flat_step_matches_planes(clbm, storage, nx, ny, nz, tol, periodic):
    lid = W.LID_PY if not periodic[1] else W.LID_NONE
    spec = W.LatticeSpec(nx=nx, ny=ny, nz=nz, K=0.02, n=0.8, periodic=periodic, lid_face=lid,
                         lid_velocity=(0.04, 0.0, 0.01) if lid else (0.0, 0.0, 0.0), name="flat")
    print(f"[gpu] flat {nx}x{ny}x{nz} {storage} periodic {periodic}", flush=True)
    a = _state(clbm, spec, storage, "rows", 3)
    b = _state(clbm, spec, storage, "planes", 3)
    worst = max((a[k].double() - b[k].double()).abs().max().item() for k in range(19))
    assert worst <= tol * b.abs().max().item()


@pytest.mark.parametrize("nodes", [1, 64, 256, 257, 255 * 256 + 1, 256 * 256, 257 * 256, 1024 * 256, 1025 * 256 + 3])
def test_reductions_at_block_edges(clbm, nodes):
    """nodes = nx x 1 x 1: from one reduction block to more than the 1024 a
    lattice uses.  Sums of N FP64 terms in another order differ by at most
    about N eps times the sum of their magnitudes."""
    spec = W.LatticeSpec(nx=nodes, ny=1, nz=1, K=0.02, n=0.8, periodic=(1, 1, 1), name="line")
    print(f"[gpu] reduce {nodes}", flush=True)
    lat = clbm.Lattice(spec, storage="f64", layout="rows")
    lat.init_populations(W.perturbed_populations(spec, 9, 1e-2, device="cuda"))
    lat.step(1)
    r = lat.reduce()
    out = torch.empty(8, dtype=torch.float64, device="cuda")
    lat.reduce_noalloc(out)
    rho, u = lat.macroscopic()
    eps = nodes * 2.0 ** -52
    assert abs(r["mass"] - rho.sum().item()) <= eps * rho.sum().item()
    for k, c in enumerate("xyz"):
        m = rho * u[k]
        assert abs(r[f"momentum_{c}"] - m.sum().item()) <= (eps + 2.0 ** -50) * m.abs().sum().item()
    kin = 0.5 * rho * (u * u).sum(0)
    assert abs(r["kinetic"] - kin.sum().item()) <= (eps + 2.0 ** -50) * kin.sum().item()
    assert abs(r["umax"] - (u * u).sum(0).max().sqrt().item()) <= 2.0 ** -50 * r["umax"]
    assert r["nonfinite"] == 0.0
    again = dict(zip(r, out.cpu().tolist()))
    for k in ("mass", "momentum_x", "momentum_y", "momentum_z", "umax", "kinetic"):
        assert again[k] == r[k]         # the same order of additions
    lat.close()


@pytest.mark.parametrize("shape,steps", [((248, 238, 240), 5), ((187, 169, 250), 4)])
def test_default_pairs_of_steps_match_single_steps(clbm, shape, steps):
    """FP32 lattices large enough that pairs of steps run as two-step launches
    by default (an odd remainder as one step), against one step per launch: the
    operations of both are the same up to the compiler's choice of fused
    multiply-adds (bound of the two-step tests)."""
    nx, ny, nz = shape
    spec = W.cavity(64, 0.05, 0.8, 300.0).with_(nx=nx, ny=ny, nz=nz)
    print(f"[gpu] default pairs {shape}", flush=True)
    f0 = W.perturbed_populations(spec, 3, 1e-2, device="cuda")
    outs = []
    for launch in (None, {"fuse_steps": 1}):
        lat = clbm.Lattice(spec, storage="f32", track_residual=False, launch=launch)
        lat.init_populations(f0)
        lat.step(steps)
        idx, done = lat.state()
        assert done == steps and idx == ((steps + 1) // 2 if launch is None else steps) % 2
        outs.append(lat.state_view().clone())
        lat.close()
    worst = max((outs[0][k] - outs[1][k]).abs().max().item() for k in range(19))
    assert worst <= 1e-5 * outs[1].abs().max().item()


@pytest.mark.parametrize("form", ["flagged", "in_place"])
def test_far_addressing_of_flagged_and_one_buffer_lattices(clbm, form):
    """A state beyond 4 GiB with a periodic z axis: offsets from the wave's own
    layer, and 64-bit addresses across the z faces, against the planes layout."""
    nx, ny, nz = 70, 9, 45003
    spec = W.LatticeSpec(nx=nx, ny=ny, nz=nz, K=0.02, n=0.8, periodic=(1, 0, 1), lid_face=W.LID_PY,
                         lid_velocity=(0.04, 0.0, 0.01), name="far")
    assert 19 * 8 * spec.nodes > 2 ** 32
    kw = {}
    if form == "flagged":
        flags = torch.zeros((nz, ny, nx), dtype=torch.uint8, device="cuda")
        flags[0, 2:4, 10:20] = 1            # solid nodes on both z faces: sources across the wrap
        flags[nz - 1, 5:7, 30:50] = 2
        flags[1000:1010, 1:3, 60:70] = 1
        kw = dict(flags=flags)
    else:
        kw = dict(in_place=True)
    print(f"[gpu] far {form}", flush=True)
    f0 = W.perturbed_populations(spec, 8, 1e-2, device="cuda")
    outs = []
    for layout in ("rows", "planes"):
        lat = clbm.Lattice(spec, storage="f64", track_residual=False, layout=layout, **kw)
        lat.init_populations(f0)
        lat.step(4)
        outs.append(lat.state_view().clone())
        lat.close()
    scale = max(outs[1][k].abs().max().item() for k in range(19))
    worst = max((outs[0][k] - outs[1][k]).abs().max().item() for k in range(19))
    assert worst <= 1e-13 * scale
