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
