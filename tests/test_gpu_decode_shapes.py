"""The neural decode at the edges of its kernels: feature and hidden sizes
around the register capacities (32, 64 hidden units) and the feature blocks,
members per cell around the rounds through the output buffer, the largest
weights, and cell counts that leave a wavefront's last lanes empty.  Centres,
scales and quaternions bit for bit, opacity and colour within 1e-6, as in the
other decode tests."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_03180_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,F,H,K", [(70, 1, 1, 1), (130, 7, 31, 32), (257, 33, 32, 3), (100, 64, 64, 32),
                                     (300, 32, 33, 20), (65, 9, 8, 17), (500, 32, 32, 5), (64, 16, 64, 6)])
def test_decode_shapes(n, F, H, K):
    from paper_2508_03180_amd.renderer import NeuralDeviceScene, Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    s, d = scenes.make_neural_scene(11, n_cells=n, K=K, F=F, H=H)
    cam = scenes.orbit_cameras(12, 160, 120)[3]
    r = Renderer(0)
    try:
        r.render_neural(NeuralDeviceScene.from_numpy(s, d, "cuda:0"), cam)
        got = {k: v.cpu().numpy() for k, v in r.read_decoded(n * K).items()}
    finally:
        r.close()
    ref = oracle.decode(s, d, cam)
    g = np.repeat(oracle.cells_discrete(s, cam)["visible"].astype(bool), K)
    assert g.any()
    for k in ("means", "scales", "rots"):
        np.testing.assert_array_equal(got[k][g], ref[k][g], err_msg=k)
    np.testing.assert_allclose(got["opacities"][g], ref["opacity64"][g], atol=1e-6)
    np.testing.assert_allclose(got["colors"][g], ref["color64"][g], atol=1e-6)
