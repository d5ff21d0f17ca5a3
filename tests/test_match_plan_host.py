"""Which kernel a match is given to, and its tiles (host only: no GPU call)."""
import pytest

from tests.match_plan import F32S, KERNEL, plan


@pytest.mark.parametrize("b,n,d,k", [(49, 1000, 1536, 5), (100, 1000, 768, 10), (256, 2000, 768, 10), (96, 5000, 384, 10),
                                     (48, 16384, 256, 10), (64, 300, 64, 32), (256, 2400, 64, 32)])
def test_small_float32_caches_have_their_kernel(b, n, d, k):
    """The tiled kernel takes 1.1 to 4 times as long there."""
    assert plan("f32", b, n, d, k).kernel == F32S


@pytest.mark.parametrize("b,n,d,k", [(128, 10000, 768, 10), (256, 5000, 768, 10), (49, 16384, 384, 5), (256, 2401, 64, 32),
                                     (257, 1000, 768, 5), (16, 16385, 768, 5), (16, 1000, 768, 33), (16, 1000, 100, 5)])
def test_other_float32_caches_are_tiled(b, n, d, k):
    assert KERNEL[plan("f32", b, n, d, k).kernel] == "k_tile"
