"""Which kernel a match is given to, and its tiles (host only: no GPU call)."""
import math
import random

import pytest

from tests.match_plan import F32S, KERNEL, SIZE, TILE, merge_by_heads, plan, workspace


@pytest.mark.parametrize("b,n,d,k", [(49, 1000, 1536, 5), (100, 1000, 768, 10), (256, 2000, 768, 10), (96, 5000, 384, 10),
                                     (48, 16384, 256, 10), (64, 300, 64, 32), (256, 2400, 64, 32)])
def test_small_float32_caches_have_their_kernel(b, n, d, k):
    """The tiled kernel takes 1.1 to 4 times as long there."""
    assert plan("f32", b, n, d, k).kernel == F32S


@pytest.mark.parametrize("b,n,d,k", [(128, 10000, 768, 10), (256, 5000, 768, 10), (49, 16384, 384, 5), (256, 2401, 64, 32),
                                     (257, 1000, 768, 5), (16, 16385, 768, 5), (16, 1000, 768, 33), (16, 1000, 100, 5)])
def test_other_float32_caches_are_tiled(b, n, d, k):
    assert KERNEL[plan("f32", b, n, d, k).kernel] == "k_tile"


@pytest.mark.parametrize("kernel,dtype,b,n,d,k", [
    # the tiled kernel took 1.1 to 1.5 times as long here
    ("k_qs8", "e4m3", 4250, 434517, 512, 1), ("k_qs8", "bf16", 7894, 182636, 384, 2), ("k_qs8", "f16", 1401, 640566, 384, 2),
    ("k_qs8", "e4m3", 15116, 6805, 768, 1), ("k_qs8", "e4m3", 14323, 5904, 768, 32), ("k_qs8", "f16", 13929, 3410, 384, 20),
    ("k_qs8", "e4m3", 10991, 92492, 512, 16),
    ("k_qs", "e4m3", 80, 145030, 1536, 2), ("k_qs", "f16", 54, 15577, 768, 1), ("k_qs", "f16", 237, 18384, 768, 2), ("k_qs", "bf16", 13, 88611, 768, 1), ("k_qs", "f16", 54, 15577, 768, 3),
    ("k_qs", "f16", 446, 136863, 768, 10), ("k_qs", "f16", 50, 197590, 768, 2), ("k_qs", "e4m3", 5065, 6702, 1536, 1), ("k_qs", "bf16", 300, 32000, 768, 10),
    # and these it took as long or less
    ("k_tile", "f16", 12, 130000, 768, 10), ("k_tile", "f16", 600, 500000, 768, 10), ("k_tile", "e4m3", 2048, 260000, 1536, 2), ("k_tile", "e4m3", 600, 9000, 768, 1),
    ("k_tile", "f16", 6000, 100000, 512, 10), ("k_tile", "bf16", 3000, 6000, 512, 32), ("k_tile", "e4m3", 411, 312831, 1536, 8), ("k_tile", "bf16", 2, 40048, 768, 2),
])
def test_kernel_of_a_shape(kernel, dtype, b, n, d, k):
    assert KERNEL[plan(dtype, b, n, d, k).kernel] == kernel


@pytest.mark.parametrize("k", range(1, 17))
@pytest.mark.parametrize("b,n", [(1, 300000), (32, 57558), (97, 15170), (200, 50000), (2000, 3000)])
def test_few_splits_meet_in_a_bucket(b, n, k):
    """256 splits on one address per query held up the kernel (k = 1 to 3)."""
    p = plan("f16", b, n, 640, k)
    assert p.kernel == TILE and p.splits <= 16 * k * p.parts and (p.parts == 1 or p.splits > 8 * k * p.parts)
    assert k * p.parts <= 64                              # a wavefront reads them


@pytest.mark.parametrize("dtype,b,n,d,k,most", [("f32", 5916, 1318, 1536, 1, 2), ("f32", 2000, 300, 1536, 5, 1), ("f32", 600, 1000, 3072, 5, 1),
                                                ("f32", 4000, 1000, 1024, 10, 1), ("f16", 16384, 1000, 1024, 10, 3), ("e4m3", 16384, 300, 256, 64, 1)])
def test_few_rows_take_many_queries_per_pass(dtype, b, n, d, k, most):
    """Passes of few queries over few rows leave most of the chip idle."""
    p = plan(dtype, b, n, d, k)
    assert p.kernel == TILE and p.passes <= most and p.qtiles * p.splits >= 64


@pytest.mark.parametrize("dtype,b,n,d,k,far", [("e4m3", 166, 2500191, 256, 1, True), ("e4m3", 190, 1896002, 384, 20, True), ("f16", 151, 9461309, 384, 10, True),
                                               ("bf16", 180, 400000, 640, 10, True), ("f16", 151, 200000, 384, 10, False), ("f16", 60, 9461309, 384, 10, False)])
def test_tile_over_caches_beyond_the_mall(dtype, b, n, d, k, far):
    """Three or more tiles of 64 queries wait for their rows there."""
    p = plan(dtype, b, n, d, k)
    assert p.kernel == TILE and (p.bq > 64 if far else p.bq == 64), p


@pytest.mark.parametrize("dtype,b,n,d,k,passes", [("bf16", 6196, 4000, 1536, 11, 4), ("f16", 4167, 5141, 1536, 2, 3)])
def test_passes_that_fill_the_chip_stay_small(dtype, b, n, d, k, passes):
    assert plan(dtype, b, n, d, k).passes == passes


@pytest.mark.parametrize("dtype", ["f32", "f16", "e4m3"])
def test_tiled_workspace_fits_the_static_array(dtype):
    """Whatever the shape, unless 32 queries are longer than 5.8 MB or the lists of
    the shape (b x k pairs and more) already pass it."""
    rng = random.Random(4)
    for _ in range(4000):
        log = lambda lo, hi: int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
        d, b, n = log(1, 2500) * 16, log(1, 200000), log(1, 20000000)
        k = min(n, rng.randint(1, 64))
        p = plan(dtype, b, n, d, k)
        if p.kernel == TILE and 32 * d * SIZE[dtype] < 5 << 20:
            assert p.off_end <= 32 << 20, (dtype, b, n, d, k, p)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "e4m3"])
def test_workspace_never_falls_as_the_batch_grows(dtype):
    """A workspace for the largest batch serves the smaller ones, and what a batch
    is asked covers its plan, and is at most 36 MiB or twice what it or a
    smaller one uses."""
    rng = random.Random(6)
    log = lambda lo, hi: int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    for _ in range(1500):
        d = rng.choice([256, 384, 512, 768, 1024, 1536, log(1, 2500) * 16])
        n = log(1, 20000000)
        k = min(n, rng.choice([1, 3, 10, 16, 17, 32, 33, 64]))
        last, used = 0, 0
        for b in sorted({log(1, 50000) for _ in range(24)} | {16, 17, 48, 49, 64, 65, 127, 128, 256, 257, 512, 513, 1023, 1024}):
            ask, need = workspace(dtype, b, n, d, k), plan(dtype, b, n, d, k).bytes
            used = max(used, need)
            assert ask >= last and ask >= need, (dtype, b, n, d, k, last, ask, need)
            last = ask
        assert last <= max(36 << 20, 2 * used), (dtype, n, d, k, last, used)


def test_workspace_of_the_shapes_that_fell():
    """127 queries were asked 8.6 times what 128 were, and so on."""
    for dtype, d, n, k, small, large in (("f16", 768, 300000, 5, 127, 128), ("f16", 256, 300000, 10, 2000, 8192), ("f32", 1024, 200000, 5, 256, 257)):
        assert workspace(dtype, small, n, d, k) <= workspace(dtype, large, n, d, k)


@pytest.mark.parametrize("g,kin,k", [(64, 10, 10), (64, 48, 48), (64, 1, 1), (2, 1, 1), (64, 16, 3), (8, 64, 1), (64, 24, 24)])
def test_few_of_many_shards_entries_by_heads(g, kin, k):
    """The registers' merge takes 1.2 to 7 times as long there."""
    assert merge_by_heads(g, kin, k)


@pytest.mark.parametrize("g,kin,k", [(2, 10, 10), (16, 10, 10), (64, 8, 8), (64, 16, 16), (32, 24, 24), (8, 32, 32),
                                     (16, 64, 64), (8, 10, 64), (2, 64, 10)])
def test_other_shard_lists_in_registers(g, kin, k):
    assert not merge_by_heads(g, kin, k)
