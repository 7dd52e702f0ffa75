"""The per-tile order with key buffers that hold few counters: many primitives
take the global way (it has the depth's four digits more), the same ones in a
larger buffer, or fewer, are counted.  Lists against the oracle's, bit for bit."""
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from test_gpu_bins import check, front_scene

pytestmark = pytest.mark.gpu

WORDS = 8 * 128 * 16  # counters of a chunk: 128 x 128 tiles in eight bands


@pytest.mark.parametrize("n,chunks,counted", [(15_000, 1, True), (15_700, 1, False), (31_000, 2, True), (32_000, 2, False),
                                              (66_000, 4, True), (67_000, 4, False), (67_000, 5, True),
                                              (300_000, 16, True), (300_000, 12, False), (300_000, 64, True)])
def test_route(n, chunks, counted):
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    r = Renderer(0)
    try:
        assert capi.dgs_set_list_order(r.ctx, capi.DGS_LIST_ORDER_PER_TILE) == capi.DGS_OK
        r.reserve(chunks * WORDS // 2)
        s, cam = front_scene(n, 2048, 2048, 30.0, 4.0, n)  # one cell in 900 in the image
        check(r, s, cam)
        st = r.stats()
        assert st["key_capacity"] == chunks * WORDS // 2
        assert st["sort_passes"] == (2 if counted else 6)
    finally:
        r.close()
