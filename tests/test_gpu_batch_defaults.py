"""Defaults of large batches, and which entries of a tune cache apply."""
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


@pytest.mark.parametrize("count", [8, 18])
def test_default_grid_gives_each_wave_one_item(clbm, count):
    """FP32 row-layout batches take 256 threads per workgroup while 1024
    workgroups per CU of them cover the items (64 nodes each), else 512."""
    spec = W.cavity(160, 0.05, 0.8, 300.0)
    print(f"[gpu] batch of {count} cavities 160^3", flush=True)
    b = clbm.Batch([spec] * count, storage="f32")
    cfg = b.get_config()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    items = count * (160 ** 3 // 64)
    assert cfg["blocks_per_cu"] == 1024
    assert cfg["bx"] == (256 if items <= 1024 * cus * 4 else 512)
    assert items <= 1024 * cus * (cfg["bx"] // 64)
    b.init_rest()
    b.step(3)
    first, last = b.populations(0), b.populations(count - 1)
    b.close()
    lat = clbm.Lattice(spec, storage="f32", track_residual=False)
    lat.init_rest()
    lat.step(3)
    ref = lat.populations()
    lat.close()
    assert torch.equal(first, ref) and torch.equal(last, ref)


def _fnv1a(h, data):
    for c in data:
        h = ((h ^ c) * 1099511628211) & (2 ** 64 - 1)
    return h


def test_tune_cache_entries_apply_to_their_own_kernels(clbm, tmp_path):
    """An entry applies to the layout it was tuned for; entries with the keys of
    earlier kernels (storage, collision form and sizes alone) are passed over."""
    import struct
    specs = [W.cavity(12, 0.05, 0.8, 100.0), W.cavity(17, 0.05, 1.2, 100.0)]
    cache = tmp_path / "tune.txt"
    print("[gpu] tune cache keys", flush=True)

    def config(layout, path=None):
        b = clbm.Batch(specs, storage="f32", layout=layout, tune_cache=path)
        cfg = b.get_config()
        b.close()
        return cfg

    b = clbm.Batch(specs, storage="f32", layout="planes", tune_cache=str(cache))
    b.init_rest()
    b.autotune()
    b.close()
    key = cache.read_text().split()[0]
    entry = "64 1 7 3 1 0"
    tuned = dict(bx=64, by=1, blocks_per_cu=7, graph_steps=3, nt_stores=1, passes=0)
    cache.write_text(f"{key} {entry}\n")
    assert config("planes", str(cache)) == tuned
    assert config("rows", str(cache)) == config("rows")
    h = _fnv1a(1469598103934665603, struct.pack("<iii", clbm.STORAGE["f32"], 0, len(specs)))
    for s in specs:
        h = _fnv1a(h, struct.pack("<iii", s.nx, s.ny, s.nz))
    old = key.rsplit("-", 1)[0] + f"-{h:016x}"
    cache.write_text(f"{old} {entry}\n")
    for layout in ("rows", "planes"):
        assert config(layout, str(cache)) == config(layout)


@pytest.mark.parametrize("layout", ["rows", "planes"])
@pytest.mark.parametrize("storage,L", [("f32", 48), ("f16", 50), ("f64", 96)])
def test_step_each_launches_what_a_lattice_does(clbm, tmp_path, storage, L, layout):
    """One launch per instance: the kernel, workgroups and store hint that the
    instance takes as a lattice of its own (kernels read from a trace)."""
    import json
    from torch.profiler import ProfilerActivity, profile
    spec = W.cavity(L, 0.05, 0.8, 100.0)
    print(f"[gpu] step_each {storage} {layout} {L}", flush=True)

    def launches(fn):
        with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
            fn()
            torch.cuda.synchronize()
        path = tmp_path / "trace.json"
        prof.export_chrome_trace(str(path))
        return {(e["name"], e["args"]["grid"][0], tuple(e["args"]["block"]))
                for e in json.loads(path.read_text())["traceEvents"]
                if e.get("cat") == "kernel" and "stream_collide" in e["name"]}

    b = clbm.Batch([spec], storage=storage, layout=layout)
    lat = clbm.Lattice(spec, storage=storage, layout=layout, track_residual=False)
    for x in (b, lat):
        x.init_rest()
    each, one = launches(lambda: b.step_each(1)), launches(lambda: lat.step(1))
    b.close()
    lat.close()
    assert each == one and len(one) == 1
