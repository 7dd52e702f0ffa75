"""The loss at the edges of its strips: rows around one strip's, strips of more
rows where there are many columns, a last strip of one row, and 64 columns and
one more.  Bounds as in test_gpu_loss: 2e-6 for the loss, 5e-4 of the largest
entry for the gradient."""
import numpy as np
import pytest
import torch

from oracle import loss as L

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def r():
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    return Renderer(0)


@pytest.mark.parametrize("shape", [(1, 11, 64), (1, 12, 65), (2, 13, 64), (1, 25, 129), (1024, 67, 1), (2048, 70, 2),
                                   (1500, 24, 65)])
def test_strips(r, shape):
    rng = np.random.default_rng(sum(shape))
    x = torch.tensor(rng.random(shape), dtype=torch.float32, device="cuda")
    y = torch.tensor(rng.random(shape), dtype=torch.float32, device="cuda")
    loss, g = r.loss_l1_ssim(x, y, 0.2)
    alone, _ = r.loss_l1_ssim(x, y, 0.2, grad=False)
    torch.cuda.synchronize()
    lo, go, _ = L.l1_ssim_loss(x.double().cpu().numpy(), y.double().cpu().numpy(), 0.2)
    assert abs(float(loss) - lo) <= 2e-6 and float(alone) == float(loss)
    assert np.abs(g.double().cpu().numpy() - go).max() <= 5e-4 * max(np.abs(go).max(), 1.0 / x.numel())
