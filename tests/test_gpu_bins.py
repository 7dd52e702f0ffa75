"""Tile lists made by counting (the per-tile order), at the sizes where the
walk changes: run lengths around what a wavefront and a workgroup sort, tile
grids of one to a few rows per band, primitives of up to the whole screen,
chunk remainders, and a grid too large for the counters.  Lists are compared
with the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_03180_amd import _capi as capi
from paper_2508_03180_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def r():
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    x = Renderer(0)
    assert capi.dgs_set_list_order(x.ctx, capi.DGS_LIST_ORDER_PER_TILE) == capi.DGS_OK
    yield x
    x.close()


def front_scene(n, width, height, spread, size, seed):
    """n cells (two members each) in front of an unrotated camera, centres
    over `spread` of the image, radii up to `size` pixels, every third depth
    the same."""
    rng = np.random.default_rng(seed)
    s = scenes.make_tiny_scene(seed, n_cells=n, K=2)
    f = 100.0
    z = rng.uniform(2.0, 4.0, n)
    z[::3] = 3.0
    x = (rng.uniform(-0.5, 0.5, n) * spread * width) * z / f
    y = (rng.uniform(-0.5, 0.5, n) * spread * height) * z / f
    s["cell_pos"] = np.stack([x, y, z], 1).astype(np.float32)
    rad = size * rng.uniform(0.01, 1.0, n) ** 3 * z / f
    s["cell_scale"] = np.repeat(rad[:, None], 3, 1).astype(np.float32)
    s["means"] = np.repeat(s["cell_pos"], 2, 0)
    cam = dict(viewmat=np.eye(4, dtype=np.float32), fx=f, fy=f, cx=width / 2, cy=height / 2, width=width,
               height=height, z_near=0.2)
    return s, cam


def check(r, s, cam):
    from paper_2508_03180_amd.renderer import DeviceScene
    W, H = cam["width"], cam["height"]
    tiles = ((W + 15) // 16) * ((H + 15) // 16)
    d = oracle.cells_discrete(s, cam)
    ids, otiles, oranges = oracle.build_lists(d["visible"], d["depth_bits"], d["rect"], W, H)
    r.render(DeviceScene.from_numpy(s, "cuda:0"), cam)
    keys, vals, ranges = r.read_lists(tiles)
    torch.cuda.synchronize()
    assert keys.numel() == len(ids)
    np.testing.assert_array_equal(ranges.cpu().numpy(), oranges)
    np.testing.assert_array_equal(vals.cpu().numpy(), ids)
    want = (otiles.astype(np.uint64) << np.uint64(32)) | d["depth_bits"][ids].astype(np.uint64)
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64), want)
    return oranges


@pytest.mark.parametrize("n", [1, 2, 16, 17, 32, 33, 64, 65, 128, 129, 256, 257, 512, 513, 1023, 1024, 1025, 2048,
                               2049, 4097, 9000])
def test_run_lengths(r, n):
    s, cam = front_scene(n, 16, 16, 0.5, 2.0, n)
    rg = check(r, s, cam)
    assert int(rg[0, 1]) == n


@pytest.mark.parametrize("size", [(16, 16), (1, 130), (300, 15), (257, 129), (333, 300), (1025, 40), (40, 1025)])
@pytest.mark.parametrize("n", [1, 255, 257, 1500])
def test_grids_and_rectangles(r, size, n):
    s, cam = front_scene(n, *size, 1.2, 0.8 * max(size), n + size[0])
    check(r, s, cam)


def test_chunk_remainders(r):
    """More primitives than one per thread and chunk (64 chunks of 256)."""
    s, cam = front_scene(64 * 256 + 77, 200, 150, 1.1, 6.0, 3)
    check(r, s, cam)


def test_grid_too_large_for_the_counters(r):
    s, cam = front_scene(500, 16400, 2500, 1.0, 60.0, 4)
    check(r, s, cam)


@pytest.mark.parametrize("mode", ["duplex", "alpha"])
@pytest.mark.parametrize("n", [9, 31, 32, 33, 50, 64])
def test_quarters_change_no_result(mode, n):
    """A tile that is walked in quarters (it holds more than the frame's
    entries per SIMD) gives the pixels it gives in halves or whole (the same
    tile beside others that hold enough)."""
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    s, cam = front_scene(n, 16, 16, 0.6, 2.0, n)
    extra = 170000
    rng = np.random.default_rng(n)
    wide = dict(s)
    z = rng.uniform(2.0, 4.0, extra)
    px, py = rng.uniform(60, 1000, extra), rng.uniform(-8, 8, extra)
    pos = np.stack([(px - 8) * z / 100.0, py * z / 100.0, z], 1).astype(np.float32)
    t = scenes.make_tiny_scene(9, n_cells=extra, K=2)
    t["cell_pos"], t["means"] = pos, np.repeat(pos, 2, 0)
    t["cell_scale"] = np.full((extra, 3), 0.005, np.float32)
    t["scales"] = np.full((2 * extra, 3), 0.01, np.float32)
    for k in ("cell_pos", "cell_scale", "cell_rot", "cell_v_sh", "means", "scales", "rots", "opacities", "sh"):
        wide[k] = np.concatenate([s[k], t[k]])
    wcam = dict(cam, width=1024)
    r = Renderer(0)
    try:
        a = r.render(DeviceScene.from_numpy(s, "cuda:0"), cam, mode=mode)
        b = r.render(DeviceScene.from_numpy(wide, "cuda:0"), wcam, mode=mode)
        assert r.stats()["num_keys"] > 1024 * 2 * n  # no quarters for a list of up to 2 n entries
        for k in ("color", "D", "T", "last"):
            assert torch.equal(a[k], b[k][..., :16]), k
    finally:
        r.close()
