"""The loss gradient where the images are equal and flat (a background that is
already right): the terms of dL/dx cancel there, and only the last addition
rounds.  It adds -2 x m and 2 x m for m = lambda / (n b2), b2 >= c2 = 0.03^2
less the rounding of the variances, one product rounded: half a unit in the last
place of 2 x m, plus 1e-7 / n for terms without 1 / b2."""
import pytest
import torch

pytestmark = pytest.mark.gpu

LAM, C2 = 0.2, 0.03 ** 2


@pytest.mark.parametrize("shape", [(1, 40, 70), (3, 97, 150)])
@pytest.mark.parametrize("value", [0.1, 0.3, 0.7, 0.95, 1.0])
def test_equal_flat_images(shape, value):
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    x = torch.full(shape, value, device="cuda")
    r = Renderer(0)
    try:
        loss, g = r.loss_l1_ssim(x, x.clone(), LAM)
        torch.cuda.synchronize()
    finally:
        r.close()
    bound = 2.0 ** -24 * 2 * value * LAM / (C2 - 2.0 ** -20) + 1e-7
    assert float(g.abs().max()) * x.numel() <= bound
