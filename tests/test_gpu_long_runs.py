"""Tile runs that the counting lists for workgroups of their own: run lengths
around the limit, several in one image, more of them than workgroups, and runs
cut off by the key capacity.  Lists are compared with the oracle's bit for bit."""
import numpy as np
import pytest
import torch

from paper_2508_03180_amd import _capi as capi
from test_gpu_bins import check, front_scene

pytestmark = pytest.mark.gpu


def renderer():
    from paper_2508_03180_amd.renderer import Renderer
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    x = Renderer(0)
    assert capi.dgs_set_list_order(x.ctx, capi.DGS_LIST_ORDER_PER_TILE) == capi.DGS_OK
    return x


@pytest.fixture(scope="module")
def r():
    x = renderer()
    yield x
    x.close()


def covering(n, width, height, seed):
    """n cells that each cover the whole image."""
    s, cam = front_scene(n, width, height, 0.2, 1.0, seed)
    s["cell_scale"] = np.full((n, 3), 0.5 * max(width, height) * 4.0 / 100.0, np.float32)
    return s, cam


@pytest.mark.parametrize("n", [2047, 2048, 2049, 2050])
@pytest.mark.parametrize("size", [(16, 16), (64, 48)])
def test_limit(r, n, size):
    s, cam = covering(n, *size, n)
    rg = check(r, s, cam)
    assert (rg[:, 1] - rg[:, 0] == n).all()


def test_more_runs_than_workgroups(r):
    s, cam = covering(2100, 640, 464, 5)
    rg = check(r, s, cam)
    assert len(rg) == 1160 and (rg[:, 1] - rg[:, 0] == 2100).all()


def test_mixed_lengths(r):
    s, cam = front_scene(15_000, 130, 100, 1.0, 60.0, 6)
    rg = check(r, s, cam)
    ln = rg[:, 1] - rg[:, 0]
    assert (ln > 2048).sum() > 4 and (ln <= 2048).sum() > 4


def test_capacity():
    """The frame that overflows the key buffer reports it; the retry is right."""
    x = renderer()
    try:
        s, cam = covering(2100, 640, 464, 5)
        check(x, s, cam)  # 2.4 M keys in a buffer of 1 M at first
    finally:
        x.close()
