"""Frames on either side of the size from which the members are projected on
the second stream (96 MB at 112 bytes per member of SH degree 0): the same bits
with the overlap on and off, and from a captured frame replayed between eager
ones."""
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from paper_2508_03180_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [89_800, 89_900])
def test_overlap_changes_no_result(cells):
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    assert (cells * 10 * 112 > 96 << 20) == (cells == 89_900)
    s = scenes.make_tiny_scene(1, n_cells=cells, K=10)
    cams = [scenes.tiny_camera(), scenes.orbit_cameras(12, 256, 256, radius=3.0)[4]]
    side = torch.cuda.Stream()
    r = Renderer(0, stream=side)
    try:
        ds = DeviceScene.from_numpy(s, "cuda:0")
        assert ds.struct().sh_degree == 0
        with torch.cuda.stream(side):
            capi.dgs_set_overlap(r.ctx, 0)
            ref = [{k: v.clone() for k, v in r.render(ds, c).items()} for c in cams]
            capi.dgs_set_overlap(r.ctx, 1)
            on = [{k: v.clone() for k, v in r.render(ds, c).items()} for c in cams]
            out = r.alloc_image(cams[0])
            side.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=side):
                r.render(ds, cams[0], out=out, check=False)
        for a, b in zip(ref, on):
            assert all(torch.equal(a[k], b[k]) for k in a)
        for rep in range(3):
            for v in out.values():
                v.fill_(0)
            g.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(out[k], ref[0][k]) for k in ref[0]), rep
            with torch.cuda.stream(side):
                o = r.render(ds, cams[1])
            torch.cuda.synchronize()
            assert torch.equal(o["color"], ref[1]["color"])
    finally:
        r.close()
