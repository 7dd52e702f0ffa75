"""Tile lists of the global order at the sizes where its key emission changes:
primitives around a block of offsets, keys around a workgroup's, one primitive
of many workgroups' keys, culled primitives, more blocks than one step of their
scan takes, and a key buffer that is too small.  Lists are compared with the
oracle's bit for bit."""
import numpy as np
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from test_gpu_bins import check, front_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def r():
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    x = Renderer(0)
    assert capi.dgs_set_list_order(x.ctx, capi.DGS_LIST_ORDER_GLOBAL) == capi.DGS_OK
    yield x
    x.close()


@pytest.mark.parametrize("n", [1, 2, 255, 1023, 1024, 1025, 2047, 2048, 2049, 4097, 70_001])
def test_one_tile(r, n):
    """A key per primitive: blocks and workgroups end together."""
    s, cam = front_scene(n, 16, 16, 0.5, 2.0, n)
    check(r, s, cam)


@pytest.mark.parametrize("n", [1, 5, 300, 1500])
@pytest.mark.parametrize("size", [(1, 130), (333, 300), (1025, 40), (2100, 1100)])
def test_large_and_culled_primitives(r, size, n):
    """Up to the whole screen (9,108 tiles) per primitive, half of them behind
    the camera."""
    s, cam = front_scene(n, *size, 1.2, 0.8 * max(size), n + size[0])
    s["cell_pos"][::2, 2] *= -1.0 if n > 5 else 1.0
    s["means"] = np.repeat(s["cell_pos"], 2, 0)
    check(r, s, cam)


def test_nothing_visible(r):
    s, cam = front_scene(3000, 100, 100, 1.0, 5.0, 1)
    s["cell_pos"][:, 2] *= -1.0
    s["means"] = np.repeat(s["cell_pos"], 2, 0)
    check(r, s, cam)


def test_blocks_beyond_one_step(r):
    """More than 4096 blocks of 1024 primitives."""
    s, cam = front_scene(4096 * 1024 + 5, 64, 48, 1.0, 3.0, 2)
    check(r, s, cam)


def test_key_buffer_too_small():
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    s, cam = front_scene(3000, 2100, 1100, 1.2, 2000.0, 7)
    x = Renderer(0)
    try:
        assert capi.dgs_set_list_order(x.ctx, capi.DGS_LIST_ORDER_GLOBAL) == capi.DGS_OK
        ds = DeviceScene.from_numpy(s, "cuda:0")
        out = x.render(ds, cam, check=False)
        assert x.sync() == capi.DGS_ERR_CAPACITY
        need = x.stats()["num_keys"]
        out = x.render(ds, cam)  # reserves what the frame reported and renders again
        assert x.stats()["num_keys"] == need and torch.isfinite(out["color"]).all()
    finally:
        x.close()
