"""The radix sort around the sizes where its passes change: one partition,
whole and ragged partitions, the counts' table summed by the scatter or by its
own launch, small and large partitions, and more partitions than one step of
the table's scan holds; and tile lists made between sorts of the same context."""
import numpy as np
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from paper_2508_03180_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def r():
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    x = Renderer(0)
    yield x
    x.close()


def check_sort(r, k, bits):
    n = len(k)
    # one element into its allocation: 8- and 4-byte aligned only
    kt = torch.from_numpy(np.concatenate([np.zeros(1, np.uint64), k]).view(np.int64)).cuda()[1:]
    vt = torch.arange(-1, n, dtype=torch.int32, device="cuda")[1:]
    r.sort_pairs(kt, vt, bits)
    order = np.argsort(k, kind="stable")
    np.testing.assert_array_equal(kt.cpu().numpy().view(np.uint64), k[order])
    np.testing.assert_array_equal(vt.cpu().numpy(), order)


@pytest.mark.parametrize("n", [63, 1023, 1024, 1025, 9 * 1024 - 1, 64 * 1024, 64 * 1024 + 1, (1 << 19) - 1, 1 << 19,
                               (1 << 19) + 4097, 1024 * 4096 + 1])
@pytest.mark.parametrize("bits", [16, 40, 64])
def test_partition_edges(r, n, bits):
    rng = np.random.default_rng(n + bits)
    k = rng.integers(0, 1 << 63, n, dtype=np.int64).astype(np.uint64) * np.uint64(2) >> np.uint64(64 - bits)
    k[rng.random(n) < 0.3] = k[0]  # one key a third of the time: stability, and one digit that dominates
    check_sort(r, k, bits)


def test_lists_between_sorts(r):
    """The sort's counts and the tile lists' look-back words share a buffer."""
    from paper_2508_03180_amd.renderer import DeviceScene
    s = scenes.make_tiny_scene(3, n_cells=3000, K=2)
    cam = scenes.pinhole(scenes.look_at((0, 0, 3), (0, 0, 0)), 333, 217)
    ds = DeviceScene.from_numpy(s, "cuda:0")
    ref = {}
    for i, order in enumerate((capi.DGS_LIST_ORDER_PER_TILE, capi.DGS_LIST_ORDER_GLOBAL) * 3):
        check_sort(r, np.random.default_rng(i).integers(0, 1 << 40, 150_000 + i).astype(np.uint64), 40)
        assert capi.dgs_set_list_order(r.ctx, order) == capi.DGS_OK
        out = {k: v.cpu().numpy() for k, v in r.render(ds, cam).items() if torch.is_tensor(v)}
        ref = ref or out
        for k in ref:
            np.testing.assert_array_equal(out[k], ref[k])
    capi.dgs_set_list_order(r.ctx, capi.DGS_LIST_ORDER_AUTO)
