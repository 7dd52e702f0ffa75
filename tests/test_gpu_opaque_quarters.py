"""A walk ends once its pixels are opaque, however few of the
entries behind touch its part of the tile: the compositor's time for a list of
ten times the entries is about the same."""
import numpy as np
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from paper_2508_03180_amd import scenes

pytestmark = pytest.mark.gpu


def scene(n, share, front, width=64, height=64):
    """`front` opaque Gaussians over the whole image, behind them small ones of
    which `share` lie in the first quarter of their tile."""
    rng = np.random.default_rng(1)
    s = scenes.make_tiny_scene(1, n_cells=n, K=1)
    f = 100.0
    z = rng.uniform(2.0, 4.0, n)
    z[:front] = 1.0 + 0.001 * np.arange(front)
    quarter = np.where(rng.random(n) < share, 0, rng.integers(1, 4, n))
    px = rng.integers(0, width // 16, n) * 16 + quarter % 2 * 8 + rng.uniform(2, 6, n)
    py = rng.integers(0, height // 16, n) * 16 + quarter // 2 * 8 + rng.uniform(2, 6, n)
    x, y = (px - width / 2) * z / f, (py - height / 2) * z / f
    x[:front] = y[:front] = 0.0
    s["cell_pos"] = s["means"] = np.stack([x, y, z], 1).astype(np.float32)
    scale = 0.2 / f * z
    scale[:front] = 4.0 * width / f
    s["cell_scale"] = s["scales"] = np.repeat(scale[:, None], 3, 1).astype(np.float32)
    s["opacities"] = np.full(n, 0.6, np.float32)
    s["opacities"][:front] = 0.98
    cam = dict(viewmat=np.eye(4, dtype=np.float32), fx=f, fy=f, cx=width / 2, cy=height / 2, width=width,
               height=height, z_near=0.2)
    return s, cam


def compositor_us(n, share, mode, front):
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    s, cam = scene(n, share, front)
    r = Renderer(0)
    try:
        ds, out, best = DeviceScene.from_numpy(s, "cuda:0"), r.alloc_image(cam), np.inf
        r.render(ds, cam, out=out, mode=mode, v_one=True)
        assert float(out["T"].max()) < 1e-4
        capi.dgs_set_timing(r.ctx, True)
        for _ in range(10):
            r.render(ds, cam, out=out, mode=mode, v_one=True)
            ms, frames = capi.dgs_get_timing(r.ctx)
            best = min(best, 1e3 * ms[-1] / frames)
        return best
    finally:
        r.close()


@pytest.mark.parametrize("mode", ["alpha", "duplex"])
@pytest.mark.parametrize("front", [3, 8])
@pytest.mark.parametrize("share", [1 / 3, 1 / 8, 1 / 16, 0.0])
def test_time_does_not_grow_with_the_list(share, mode, front):
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    few, many = compositor_us(20_000, share, mode, front), compositor_us(200_000, share, mode, front)
    assert many < 3 * few + 10, (few, many)
