"""The backward's own list of work items: around the length from which a tile
is walked in halves, where the forward takes the tile whole, in halves or in
quarters, in both list orders and with few or many tiles.  The gradients of a
tile's cells are the same bits whatever the rest of the image holds (each sum
has at most two terms from the tile's halves, so their order does not matter)."""
import numpy as np
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from paper_2508_03180_amd import scenes
from test_gpu_bins import front_scene

pytestmark = pytest.mark.gpu

KEYS = ("cell_pos", "cell_scale", "cell_rot", "cell_v_sh", "means", "scales", "rots", "opacities", "sh")


def beside(s, extra, seed):
    """The scene with `extra` small cells to the right of its 16 columns."""
    rng = np.random.default_rng(seed)
    z = rng.uniform(2.0, 4.0, extra)
    px, py = rng.uniform(60, 1000, extra), rng.uniform(-8, 8, extra)
    pos = np.stack([(px - 8) * z / 100.0, py * z / 100.0, z], 1).astype(np.float32)
    t = scenes.make_tiny_scene(9, n_cells=extra, K=2)
    t["cell_pos"], t["means"] = pos, np.repeat(pos, 2, 0)
    t["cell_scale"] = np.full((extra, 3), 0.005, np.float32)
    t["scales"] = np.full((2 * extra, 3), 0.01, np.float32)
    return dict(s, **{k: np.concatenate([s[k], t[k]]) for k in KEYS})


def grads(order, s, cam, n, height=None):
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    r = Renderer(0)
    try:
        assert capi.dgs_set_list_order(r.ctx, order) == capi.DGS_OK
        ds = DeviceScene.from_numpy(s, "cuda:0")
        cam = dict(cam, height=height or cam["height"])
        out = r.render(ds, cam, save=True)
        gc = torch.zeros_like(out["color"])
        g = torch.Generator(device="cuda").manual_seed(5)
        gc[:, :16, :16] = torch.randn((3, 16, 16), device="cuda", generator=g)
        res = []
        for _ in range(2):  # the queue is rewound
            gr = r.render_backward(ds, out["frame"], gc, torch.zeros_like(out["D"]))
            res.append({k: v[..., :n if k.startswith("cell") else 2 * n].clone() for k, v in gr.items()})
        for k in res[0]:
            assert torch.equal(res[0][k], res[1][k]), k
        out["frame"].release()
        return res[0]
    finally:
        r.close()


@pytest.mark.parametrize("order", [capi.DGS_LIST_ORDER_PER_TILE, capi.DGS_LIST_ORDER_GLOBAL])
@pytest.mark.parametrize("n", [4, 9, 31, 32, 33, 64])
def test_gradients_do_not_depend_on_the_other_items(order, n):
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    s, cam = front_scene(n, 16, 16, 0.6, 2.0, n)
    alone = grads(order, s, cam, n)
    assert float(alone["means"].abs().max()) > 0
    wide = beside(s, 4000, n)
    for other in (grads(order, wide, dict(cam, width=1024), n),  # 64 tiles
                  grads(order, wide, dict(cam, width=1024), n, height=304),  # 1216: more than a workgroup per CU
                  grads(order, wide, dict(cam, width=1024), n, height=1024)):  # 4096 tiles: tickets
        for k in alone:
            assert torch.equal(alone[k], other[k]), k
