"""Quarters of a tile with opaque pixels below transparent ones: members whose
boxes hold opaque pixels only are not walked, and leaving them out changes no
bit of the image."""
import numpy as np
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from paper_2508_03180_amd import scenes

pytestmark = pytest.mark.gpu

KEYS = ("cell_pos", "cell_scale", "cell_rot", "cell_v_sh", "means", "scales", "rots", "opacities", "sh")


def scene(px, py, z, sx, sy, opacity, width, height, f=100.0):
    """Gaussians (a cell each) at pixel px, py and depth z with standard
    deviations of sx, sy pixels (before the screen's low pass), axes upright."""
    n = len(z)
    s = scenes.make_tiny_scene(1, n_cells=n, K=1)
    s["cell_pos"] = s["means"] = np.stack([(px - width / 2) * z / f, (py - height / 2) * z / f, z],
                                          1).astype(np.float32)
    s["cell_scale"] = s["scales"] = np.stack([sx * z / f, sy * z / f, np.full(n, 1e-4)], 1).astype(np.float32)
    up = np.zeros((n, 4), np.float32)
    up[:, 0] = 1.0
    s["cell_rot"] = s["rots"] = up
    s["opacities"] = np.asarray(opacity, np.float32)
    cam = dict(viewmat=np.eye(4, dtype=np.float32), fx=f, fy=f, cx=width / 2, cy=height / 2, width=width,
               height=height, z_near=0.2)
    return s, cam


def compositor_us(n, row, mode, layers=300, size=64):
    """Opaque bands over rows 4 to 7 of each 8, n faint Gaussians behind them
    centred at `row` of 8."""
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    rng = np.random.default_rng(1)
    bands, m = size // 8, size // 8 * layers
    px = np.concatenate([np.full(m, size / 2), rng.uniform(2, size - 2, n)])
    py = np.concatenate([np.tile(np.arange(bands) * 8 + 6.0, layers), rng.integers(0, bands, n) * 8 + row])
    z = np.concatenate([np.linspace(1.0, 1.1, m), rng.uniform(2.0, 4.0, n)])
    sx = np.concatenate([np.full(m, 4.0 * size), np.full(n, 0.1)])
    sy = np.concatenate([np.full(m, 0.25), np.full(n, 0.1)])
    s, cam = scene(px, py, z, sx, sy, np.concatenate([np.full(m, 0.98), np.full(n, 0.03)]), size, size)
    r = Renderer(0)
    try:
        ds, out, best = DeviceScene.from_numpy(s, "cuda:0"), r.alloc_image(cam), np.inf
        r.render(ds, cam, out=out, mode=mode, v_one=True)
        T = out["T"].reshape(bands, 8, size)
        assert float(T[:, 4:].max()) < 1e-4 and float(T[:, :2].min()) > 1e-3
        capi.dgs_set_timing(r.ctx, True)
        for _ in range(10):
            r.render(ds, cam, out=out, mode=mode, v_one=True)
            ms, frames = capi.dgs_get_timing(r.ctx)
            best = min(best, 1e3 * ms[-1] / frames)
        return best
    finally:
        r.close()


@pytest.mark.parametrize("mode", ["alpha", "duplex"])
def test_members_below_the_skyline_are_not_walked(mode):
    """The same list costs less with its members hidden than in the open: by
    columns alone 0.98 and 1.00 of it, by pixels 0.52 (alpha) and 0.73 (duplex,
    whose cells of one member are looked at one by one all the same)."""
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    hidden, open_ = compositor_us(100_000, 6.0, mode), compositor_us(100_000, 2.0, mode)
    assert hidden < 0.87 * open_, (hidden, open_)


@pytest.mark.parametrize("mode", ["alpha", "duplex", "lcwsr"])
@pytest.mark.parametrize("seed", range(6))
def test_skyline_changes_no_result(mode, seed):
    """A tile walked in quarters and (beside tiles that hold enough) in halves."""
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    rng = np.random.default_rng(seed)
    m, n, extra = 40, 30, 170000
    # across the tile or upright, so that edges between opaque and open pixels
    # cut the quarters either way; behind them boxes of 1 to 12 pixels
    narrow = rng.choice([0.3, 0.5, 0.8], m)
    across = seed % 2 == 0
    at = rng.choice([3.0, 7.5, 12.0], 2, replace=False)[rng.integers(0, 2, m)] + rng.uniform(-0.5, 0.5, m)
    px = np.concatenate([np.full(m, 8.0) if across else at, rng.uniform(0, 16, n)])
    py = np.concatenate([at if across else np.full(m, 8.0), rng.uniform(0, 16, n)])
    sx = np.concatenate([np.full(m, 40.0) if across else narrow, rng.uniform(0.05, 2.0, n)])
    sy = np.concatenate([narrow if across else np.full(m, 40.0), rng.uniform(0.05, 2.0, n)])
    z = np.concatenate([np.linspace(1.0, 1.1, m), rng.uniform(2.0, 4.0, n)])
    o = np.concatenate([np.full(m, 0.98), rng.uniform(0.1, 0.9, n)])
    s, cam = scene(px, py, z, sx, sy, o, 16, 16)
    zt = rng.uniform(2.0, 4.0, extra)
    t, _ = scene(rng.uniform(60, 1000, extra), rng.uniform(0, 16, extra), zt, np.full(extra, 0.1),
                 np.full(extra, 0.1), np.full(extra, 0.5), 16, 16)
    wide = {k: np.concatenate([s[k], t[k]]) if k in KEYS else v for k, v in s.items()}
    r = Renderer(0)
    try:
        a = r.render(DeviceScene.from_numpy(s, "cuda:0"), cam, mode=mode, v_one=True, tau=8.0)
        b = r.render(DeviceScene.from_numpy(wide, "cuda:0"), dict(cam, width=1024), mode=mode, v_one=True,
                     tau=8.0)
        assert r.stats()["num_keys"] > 1024 * (m + n)  # no quarters for a list of up to m + n entries
        if mode != "lcwsr":
            assert float(a["T"].min()) < 1e-3 and float(a["T"].max()) > 0.2
        for k in ("color", "D", "T", "last"):
            assert torch.equal(a[k], b[k][..., :16]), k
    finally:
        r.close()
