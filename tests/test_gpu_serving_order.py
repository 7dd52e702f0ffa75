"""A server's captured frames follow the list order that suits what the shape's
frames hold: the choice is made before every frame, and a shape has a graph for
each order that it took.  Images are those of dgs_render."""
import numpy as np
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from test_gpu_bins import front_scene

pytestmark = pytest.mark.gpu


def test_graphs_of_both_orders():
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    from paper_2508_03180_amd.serving import Server
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    s, near = front_scene(20_000, 160, 120, 0.3, 2.0, 7)  # all cells in a few tiles: long runs
    far = dict(near, viewmat=np.array([[1, 0, 0, 3.0], [0, 1, 0, 0], [0, 0, 1, 0], [0, 0, 0, 1]], np.float32))
    ds, r = DeviceScene.from_numpy(s, "cuda:0"), Renderer(0)
    try:
        ref, runs = {}, {}
        for name, cam in (("near", near), ("far", far)):
            ref[name] = r.render(ds, cam)["color"].clone()
            _, _, rg = r.read_lists(80)
            ln = (rg[:, 1] - rg[:, 0]).cpu().numpy()
            runs[name] = (int(ln.sum()), int(ln[ln > 4096].sum()))
        assert runs["far"][0] > 0 and runs["far"][1] == 0  # few cells, short runs
        assert 64 * runs["near"][1] > runs["near"][0]
        with Server(0, num_slots=1, use_graphs=True) as srv:
            sid = srv.add_scene(ds)
            seq, captures, replayed = ["far", "far", "far", "near", "near", "near", "far", "far", "near"], [], []
            for name in seq:
                info, img = srv.wait(srv.submit(sid, near if name == "near" else far), timeout=60)
                assert info["state"] == capi.DGS_REQ_DONE
                torch.cuda.synchronize()
                assert torch.equal(img, ref[name]), (name, len(captures))
                captures.append(srv.stats()["graph_captures"])
            # the first frame expects a key per cell (per tile), and so does the first of
            # the near ones; the next knows its load (global); both graphs serve the rest
            assert captures == [1] * 4 + [2] * (len(seq) - 4), captures
            assert srv.stats()["graph_replays"] == len(seq) - 2
    finally:
        r.close()
