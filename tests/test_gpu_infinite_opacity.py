"""An infinite opacity is clamped to alpha_max like any other above it: the
image is the one of a large finite opacity, also where a tile is walked in
quarters, four Gaussians at a time, and their number is no multiple of four."""
import numpy as np
import pytest
import torch

from test_gpu_bins import front_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["alpha", "duplex"])
@pytest.mark.parametrize("n", [9, 11, 13, 15, 33])
def test_infinite_opacity(mode, n):
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    s, cam = front_scene(n, 16, 16, 0.3, 20.0, n)
    s["cell_scale"] = np.full_like(s["cell_scale"], 0.3)
    s["scales"] = np.full_like(s["scales"], 0.3)
    r = Renderer(0)
    try:
        out = []
        for big in (1e30, np.inf):
            s["opacities"] = np.full_like(s["opacities"], 0.05)
            s["opacities"][2 * int(np.argmin(s["cell_pos"][:, 2]))] = big  # in front of all others but its twin
            out.append({k: v.clone() for k, v in r.render(DeviceScene.from_numpy(s, "cuda:0"), cam, mode=mode, no_et=True).items()})
    finally:
        r.close()
    assert int(out[0]["last"].max()) > 8
    for k in out[0]:
        assert torch.equal(out[0][k], out[1][k]), k
