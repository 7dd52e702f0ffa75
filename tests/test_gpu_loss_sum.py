"""The loss without its gradient is summed by a kernel of its own: the same bits
as the loss that comes with one, with strips on either side of the 64 and 4096
that it takes at a time."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 11, 64), (63, 12, 64), (64, 12, 64), (65, 12, 64), (4095, 9, 7),
                                   (4096, 9, 7), (4097, 9, 7), (8193, 5, 3), (3, 843, 178), (16, 300, 400)])
def test_loss_alone_is_the_loss_with_its_gradient(shape):
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    x, y = torch.rand(shape, device="cuda", generator=g), torch.rand(shape, device="cuda", generator=g)
    r = Renderer(0)
    try:
        alone, none = r.loss_l1_ssim(x, y, 0.2, grad=False)
        both, grad = r.loss_l1_ssim(x, y, 0.2, grad=True)
        torch.cuda.synchronize()
        assert none is None and grad is not None
        assert torch.equal(alone, both)
    finally:
        r.close()
