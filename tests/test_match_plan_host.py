"""Which kernel a match is given to, and its tiles (host only: no GPU call)."""
import pytest

from tests.match_plan import F32S, KERNEL, TILE, plan


@pytest.mark.parametrize("b,n,d,k", [(49, 1000, 1536, 5), (100, 1000, 768, 10), (256, 2000, 768, 10), (96, 5000, 384, 10),
                                     (48, 16384, 256, 10), (64, 300, 64, 32), (256, 2400, 64, 32)])
def test_small_float32_caches_have_their_kernel(b, n, d, k):
    """The tiled kernel takes 1.1 to 4 times as long there."""
    assert plan("f32", b, n, d, k).kernel == F32S


@pytest.mark.parametrize("b,n,d,k", [(128, 10000, 768, 10), (256, 5000, 768, 10), (49, 16384, 384, 5), (256, 2401, 64, 32),
                                     (257, 1000, 768, 5), (16, 16385, 768, 5), (16, 1000, 768, 33), (16, 1000, 100, 5)])
def test_other_float32_caches_are_tiled(b, n, d, k):
    assert KERNEL[plan("f32", b, n, d, k).kernel] == "k_tile"


@pytest.mark.parametrize("k", range(1, 17))
@pytest.mark.parametrize("b,n", [(1, 300000), (32, 57558), (97, 15170), (200, 50000), (2000, 3000)])
def test_few_splits_meet_in_a_bucket(b, n, k):
    """256 splits on one address per query held up the kernel (k = 1 to 3)."""
    p = plan("f16", b, n, 640, k)
    assert p.kernel == TILE and p.splits <= 16 * k * p.parts and (p.parts == 1 or p.splits > 8 * k * p.parts)
    assert k * p.parts <= 64                              # a wavefront reads them
