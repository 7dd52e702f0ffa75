"""Decoders whose weights and output buffer come to within a kilobyte of the
64 KB of LDS that a workgroup takes at most.  Compared as in
test_gpu_decode_shapes."""
import pytest

from test_gpu_decode_shapes import test_decode_shapes as decode_shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,F,H,K", [(130, 45, 64, 32), (70, 41, 64, 32), (70, 49, 64, 30), (70, 44, 64, 32),
                                     (70, 46, 64, 32)])
def test_near_the_limit(n, F, H, K):
    decode_shape(n, F, H, K)
