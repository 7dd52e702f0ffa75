"""A quarter's walk takes the members of a cell in groups: for member counts
around the groups' sizes, a tile walked in quarters gives bit for bit the
pixels it gives in halves or whole."""
import numpy as np
import pytest
import torch

from paper_2508_03180_amd import scenes
from test_gpu_bins import front_scene

pytestmark = pytest.mark.gpu


def with_members(s, K, seed):
    """The scene's cells with K members each, spread over the cell."""
    n = len(s["cell_pos"])
    rng = np.random.default_rng(seed)
    t = scenes.make_tiny_scene(seed, n_cells=n, K=K)
    t.update({k: s[k] for k in ("cell_pos", "cell_scale", "cell_rot", "cell_v_sh")})
    rad = np.repeat(s["cell_scale"][:, :1], K, 0)
    t["means"] = (np.repeat(s["cell_pos"], K, 0) + rad * rng.uniform(-0.4, 0.4, (n * K, 3))).astype(np.float32)
    t["scales"] = (rad * rng.uniform(0.1, 0.4, (n * K, 3))).astype(np.float32)
    return t


@pytest.mark.parametrize("mode", ["duplex", "lcwsr"])
@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 7, 8, 9])
def test_member_groups(mode, K):
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    n, extra = 40, 170000
    s, cam = front_scene(n, 16, 16, 0.6, 8.0, K)
    s = with_members(s, K, K)
    rng = np.random.default_rng(n)
    z = rng.uniform(2.0, 4.0, extra)
    px, py = rng.uniform(60, 1000, extra), rng.uniform(-8, 8, extra)
    pos = np.stack([(px - 8) * z / 100.0, py * z / 100.0, z], 1).astype(np.float32)
    t = scenes.make_tiny_scene(9, n_cells=extra, K=K)
    t["cell_pos"], t["means"] = pos, np.repeat(pos, K, 0)
    t["cell_scale"] = np.full((extra, 3), 0.005, np.float32)
    t["scales"] = np.full((K * extra, 3), 0.01, np.float32)
    wide = dict(s)
    for k in ("cell_pos", "cell_scale", "cell_rot", "cell_v_sh", "means", "scales", "rots", "opacities", "sh"):
        wide[k] = np.concatenate([s[k], t[k]])
    r = Renderer(0)
    try:
        a = r.render(DeviceScene.from_numpy(s, "cuda:0"), cam, mode=mode, tau=8.0)
        b = r.render(DeviceScene.from_numpy(wide, "cuda:0"), dict(cam, width=1024), mode=mode, tau=8.0)
        assert r.stats()["num_keys"] > 1024 * 2 * n  # no quarters for a list of up to 2 n entries
        assert float(a["D"].max()) > 0
        for k in ("color", "D", "T", "last"):
            assert torch.equal(a[k], b[k][..., :16]), k
    finally:
        r.close()
