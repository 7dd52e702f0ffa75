"""Key buffers far larger than a frame's keys, and frames of more keys than one
sweep of a bounded grid takes (67 M in the sort, 33 M in the emission): the same
lists in the global order."""
import numpy as np
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from test_gpu_bins import check, front_scene

pytestmark = pytest.mark.gpu


@pytest.fixture
def r():
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    x = Renderer(0)
    assert capi.dgs_set_list_order(x.ctx, capi.DGS_LIST_ORDER_GLOBAL) == capi.DGS_OK
    yield x
    x.close()


@pytest.mark.parametrize("keys", [16384 * 4096, 16384 * 4096 + 1, 1 << 28])
def test_large_buffer(r, keys):
    r.reserve(keys)
    s, cam = front_scene(3000, 333, 300, 1.2, 60.0, 2)
    check(r, s, cam)


def test_more_keys_than_one_sweep(r):
    from paper_2508_03180_amd.renderer import DeviceScene
    n, size = 16_500, 1024
    s, cam = front_scene(n, size, size, 0.2, 1.0, 4)
    s["cell_scale"] = np.full((n, 3), 1.5 * size * 4.0 / 100.0, np.float32)  # each covers the image
    tiles = (size // 16) ** 2
    assert n * tiles > 16384 * 4096
    r.render(DeviceScene.from_numpy(s, "cuda:0"), cam)
    keys, vals, ranges = r.read_lists(tiles)
    assert keys.numel() == n * tiles
    _, depth, _ = r.read_prims(n)
    depth = depth.long() & 0xffffffff
    want = torch.argsort(depth, stable=True)
    assert torch.equal(ranges, torch.arange(tiles, device="cuda", dtype=torch.int32)[:, None] * n
                       + torch.tensor([0, n], device="cuda", dtype=torch.int32))
    assert bool((vals.view(tiles, n) == want.int()).all())
    tile = torch.arange(tiles, device="cuda")[:, None] << 32
    assert bool((keys.view(tiles, n) == (tile | depth[want])).all())
