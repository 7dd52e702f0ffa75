"""More than 2^32 list entries: the frame reports a full key buffer, and the
runs that fit in the buffer hold their tile's entries all the same."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_03180_amd import _capi as capi
from test_gpu_bins import front_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [capi.DGS_LIST_ORDER_PER_TILE, capi.DGS_LIST_ORDER_GLOBAL])
def test_more_entries_than_32_bits_count(order):
    from paper_2508_03180_amd.renderer import DeviceScene, Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    n, size = 66_000, 4096
    s, cam = front_scene(n, size, size, 0.2, 1.0, 3)
    s["cell_scale"] = np.full((n, 3), 1.5 * size * 4.0 / 100.0, np.float32)  # each covers the image
    tiles = (size // 16) ** 2
    assert n * tiles > 2 ** 32
    d = oracle.cells_discrete(s, cam)
    assert d["visible"].all()
    assert (d["rect"] == d["rect"][0]).all() and list(d["rect"][0]) == [0, size - 1, 0, size - 1]
    want = np.lexsort((np.arange(n), d["depth_bits"]))
    r = Renderer(0)
    try:
        assert capi.dgs_set_list_order(r.ctx, order) == capi.DGS_OK
        r.render(DeviceScene.from_numpy(s, "cuda:0"), cam, check=False)
        assert r.sync() == capi.DGS_ERR_CAPACITY
        st = r.stats()
        cap = st["key_capacity"]
        assert st["num_keys"] == 2 ** 32 - 1 and cap > 8 * n
        dv = torch.empty(cap, dtype=torch.int32, device="cuda")
        dr = torch.empty((tiles, 2), dtype=torch.int32, device="cuda")
        capi.dgs_read_lists(r.ctx, None, dv.data_ptr(), dr.data_ptr())
        torch.cuda.synchronize()
        vals, ranges = dv.cpu().numpy(), dr.cpu().numpy()
    finally:
        r.close()
    if order == capi.DGS_LIST_ORDER_GLOBAL:  # cut off in depth order: the nearest primitives in every tile
        whole = cap // tiles
        assert (ranges[:, 1] - ranges[:, 0] >= whole).all()
        for t in range(0, tiles, 997):
            np.testing.assert_array_equal(vals[ranges[t, 0]:][:whole], want[:whole])
    else:  # cut off in tile order: the first tiles, whole
        assert ranges[:, 1].max() == cap
        for t in range(cap // n):
            assert list(ranges[t]) == [t * n, (t + 1) * n]
            np.testing.assert_array_equal(vals[t * n:(t + 1) * n], want)
