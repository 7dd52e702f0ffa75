"""Long tile runs where most keys are in them: run lengths around the chunks and
merges of the launch that sorts them by larger workgroups, taken by a context's
first frame and whenever the last one had many long runs, and the same runs in
the other kernel, after a frame without any.  Lists against the oracle's, bit
for bit."""
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from test_gpu_bins import check, front_scene
from test_gpu_long_runs import covering

pytestmark = pytest.mark.gpu


@pytest.fixture
def make():
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    made = []

    def f():
        made.append(Renderer(0))
        assert capi.dgs_set_list_order(made[-1].ctx, capi.DGS_LIST_ORDER_PER_TILE) == capi.DGS_OK
        return made[-1]
    yield f
    for r in made:
        r.close()


@pytest.mark.parametrize("n", [2049, 4096, 4097, 6145, 8191, 8192, 8193, 20_001])
def test_long_runs(make, n):
    s, cam = covering(n, 40, 24, n)
    r = make()
    for _ in range(2):  # no load known, then many long runs known (from 4097 on)
        check(r, s, cam)
    light, lcam = front_scene(50, 40, 24, 0.5, 2.0, 1)
    check(r, light, lcam)
    check(r, s, cam)  # none known


def test_saved_frame_of_long_runs(make):
    """The ids of a saved frame are copied by both launches."""
    from paper_2508_03180_amd.renderer import DeviceScene
    s, cam = front_scene(15_000, 130, 100, 1.0, 60.0, 6)
    r, ds, grads = make(), DeviceScene.from_numpy(s, "cuda:0"), []
    light, lcam = front_scene(50, 40, 24, 0.5, 2.0, 1)
    for first in (True, False):
        if not first:
            check(r, light, lcam)
        out = r.render(ds, cam, save=True)
        grads.append({k: v.clone() for k, v in r.render_backward(ds, out["frame"], torch.ones_like(out["color"])).items()})
        out["frame"].release()
    for k, v in grads[0].items():
        scale = v.abs().max()
        assert torch.isfinite(v).all() and scale > 0
        assert float((v - grads[1][k]).abs().max()) <= 1e-4 * float(scale), k  # sums in a free order
