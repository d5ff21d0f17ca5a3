"""GPU parity of the merge of per-shard top-k lists.

apc_merge_shards is compared bit for bit with the oracle's merge on the same
seeded lists (ties across shards, invalid entries, fewer candidates than k,
1 to 64 shards).  End to end, a cache split into row shards, matched shard by
shard with apc_match_batch and merged, gives bit for bit the top-k of the
whole cache (every score is the same fixed MFMA sequence wherever its row
lives).
"""
import numpy as np
import pytest
import torch

from paper_2502_06798_amd import synth
from tests.gpu_check import say
from tests.test_gpu_parity import make_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def apc():
    import paper_2502_06798_amd as apc
    apc.load()
    assert torch.cuda.is_available()
    return apc


def _shard_lists(rng, g, b, kin, n_local):
    s = np.round(rng.uniform(-1, 1, (g, b, kin)), 2).astype(np.float32)      # ties across shards
    i = np.stack([[rng.choice(n_local, kin, replace=False) for _ in range(b)] for _ in range(g)]).astype(np.int32)
    for a in range(g):
        for q in range(b):
            o = np.lexsort((i[a, q], -s[a, q].astype(np.float64)))
            s[a, q], i[a, q] = s[a, q][o], i[a, q][o]
            cut = rng.integers(0, kin + 1) if rng.random() < 0.1 else kin     # fewer candidates
            i[a, q, cut:] = -1
            s[a, q, cut:] = np.nan
    return s, i


@pytest.mark.parametrize("g,b,kin,k", [(1, 5, 10, 10), (2, 300, 10, 10), (8, 1000, 32, 32), (8, 77, 16, 40),
                                       (64, 130, 4, 64), (3, 4096, 64, 1), (5, 1, 1, 7),
                                       # head by head, then in registers of 8, 16, 32 and 64 lanes
                                       (64, 33, 10, 10), (64, 9, 48, 48), (64, 1030, 1, 1), (33, 70, 3, 2),
                                       (64, 35, 8, 8), (7, 66, 3, 8), (64, 33, 16, 16), (13, 50, 9, 10), (32, 21, 24, 24),
                                       (16, 19, 64, 64), (9, 130, 10, 40)])
def test_merge_shards_bit_exact(apc, orc, g, b, kin, k):
    say(f"merge_shards g={g} b={b} kin={kin} k={k}")
    rng = np.random.default_rng(g * 1000 + b + kin)
    s, i = _shard_lists(rng, g, b, kin, 500)
    offsets = (np.arange(g) * 500).tolist()
    os_ = torch.full((b, k), 7.0, device="cuda")
    oi = torch.full((b, k), 7, dtype=torch.int32, device="cuda")
    apc.apc_merge_shards(torch.from_numpy(s).cuda(), torch.from_numpy(i).cuda(), g, b, kin, offsets, k, os_, oi)
    torch.cuda.synchronize()
    ws, wi = orc.merge_shards(s, i, offsets, k)
    gs = os_.cpu().numpy()
    assert np.array_equal(oi.cpu().numpy(), wi)
    assert np.array_equal(np.isnan(gs), np.isnan(ws)) and np.array_equal(gs[~np.isnan(ws)], ws[~np.isnan(ws)])


@pytest.mark.parametrize("dtype,cuts", [("f16", [0, 20000, 40000]), ("f16", [0, 5000, 5100, 23000, 40000]),
                                        ("e4m3", [0, 13000, 26000, 40000])])
def test_sharded_match_equals_whole_cache(apc, dtype, cuts):
    say(f"sharded match {dtype} cuts={cuts}")
    n, d, b, k = cuts[-1], 768, 300, 10
    e, es = make_rows(n, d, dtype, 21, clusters=50)
    q, qs = make_rows(b, d, dtype, 22, clusters=50)
    whole = apc.apc_build_cache(e, es)
    ts = torch.empty((b, k), device="cuda")
    ti = torch.empty((b, k), dtype=torch.int32, device="cuda")
    apc.apc_match_batch(whole, q, qs, k, ts, ti, apc.workspace_tensor(whole, b, k))
    g = len(cuts) - 1
    ls = torch.empty((g, b, k), device="cuda")
    li = torch.empty((g, b, k), dtype=torch.int32, device="cuda")
    caches = []
    for a in range(g):
        c = apc.apc_build_cache(e[cuts[a]:cuts[a + 1]], None if es is None else es[cuts[a]:cuts[a + 1]])
        caches.append(c)
        apc.apc_match_batch(c, q, qs, k, ls[a], li[a], apc.workspace_tensor(c, b, k))
    ms = torch.empty((b, k), device="cuda")
    mi = torch.empty((b, k), dtype=torch.int32, device="cuda")
    apc.apc_merge_shards(ls, li, g, b, k, cuts[:-1], k, ms, mi)
    torch.cuda.synchronize()
    assert torch.equal(mi, ti) and torch.equal(ms, ts)
    for c in caches + [whole]:
        c.close()


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 768), ("f32", 1100), ("f16", 8), ("f16", 384), ("f16", 768),
                                     ("f16", 2056), ("bf16", 1024), ("bf16", 1544), ("e4m3", 768), ("e4m3", 1040), ("e4m3", 4112)])
def test_row_factors_depend_on_the_row_alone(apc, dtype, d):
    """The same rows in calls of few and of many rows (lanes per row and rows
    per group differ): the same bits."""
    say(f"row factors of parts {dtype} d={d}")
    n = 10241                                            # above every line between the groupings
    e, _ = make_rows(n, d, dtype, 31)
    whole = torch.empty(n, device="cuda")
    apc.apc_row_factors(e, whole)
    for a, z in ((0, 1), (0, 2048), (1000, 3049), (17, 2066), (3500, 6000), (4097, 10241), (1, 10241)):
        part = torch.empty(z - a, device="cuda")
        apc.apc_row_factors(e[a:z], part)
        torch.cuda.synchronize()
        assert torch.equal(part, whole[a:z]), f"rows {a}..{z}"


@pytest.mark.parametrize("n", [100, 10241])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 768), ("f16", 128), ("f16", 384), ("bf16", 1024), ("bf16", 1544),
                                     ("e4m3", 256), ("e4m3", 768), ("e4m3", 4112)])
def test_row_factors_of_rows_beside_bad_ones(apc, dtype, d, n):
    """A value that is not finite, in any lane's part of a row, takes that row's
    factor alone."""
    say(f"row factors beside bad rows {dtype} d={d} n={n}")
    e, _ = make_rows(n, d, dtype, 37)
    bad = torch.zeros(n, dtype=torch.bool, device="cuda")
    bad[[0, 5, 6, 33, n - 2]] = True
    cols = torch.tensor([0, d // 2 + 1, d - 1, 17, d // 3], device="cuda")
    clean = torch.empty(n, device="cuda")
    apc.apc_row_factors(e, clean)
    rows = torch.nonzero(bad).flatten()
    if dtype == "e4m3":
        e.view(torch.uint8)[rows, cols] = 0x7F           # the code of NaN
    else:
        e[rows, cols] = float("inf")
    f = torch.empty(n, device="cuda")
    apc.apc_row_factors(e, f)
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(f), bad) and torch.equal(f[~bad], clean[~bad])


@pytest.mark.parametrize("dtype,d", [("f16", 768), ("bf16", 384), ("f16", 1024), ("e4m3", 1536)])
def test_small_shards_equal_whole_cache(apc, dtype, d):
    """A cache whose row factors take another grouping of lanes than its shards'
    do, all shards holding much of every top-k: whole cache and shards agree bit for bit, in the scores too."""
    say(f"small shards {dtype} d={d}")
    cuts, b, k = [0, 100, 1100, 3148, 6400, 12600], 200, 20
    n = cuts[-1]
    e, es = make_rows(n, d, dtype, 33, clusters=1)
    q, qs = make_rows(b, d, dtype, 34)
    whole = apc.apc_build_cache(e, es)
    ts = torch.empty((b, k), device="cuda")
    ti = torch.empty((b, k), dtype=torch.int32, device="cuda")
    apc.apc_match_batch(whole, q, qs, k, ts, ti, apc.workspace_tensor(whole, b, k))
    g = len(cuts) - 1
    ls = torch.empty((g, b, k), device="cuda")
    li = torch.empty((g, b, k), dtype=torch.int32, device="cuda")
    for a in range(g):
        c = apc.apc_build_cache(e[cuts[a]:cuts[a + 1]].contiguous(), None if es is None else es[cuts[a]:cuts[a + 1]].contiguous())
        apc.apc_match_batch(c, q, qs, k, ls[a], li[a], apc.workspace_tensor(c, b, k))
        torch.cuda.synchronize()
        c.close()
    ms = torch.empty((b, k), device="cuda")
    mi = torch.empty((b, k), dtype=torch.int32, device="cuda")
    apc.apc_merge_shards(ls, li, g, b, k, cuts[:-1], k, ms, mi)
    torch.cuda.synchronize()
    assert all((ti < c).any() and (ti >= c).any() for c in cuts[1:-1])     # every shard's side is in the lists
    assert torch.equal(mi, ti) and torch.equal(ms, ts)
    whole.close()


def test_merge_shards_offsets_near_int32_limit(apc, orc):
    # global entry numbers are summed in 64 bits; those of 2^31 - 1 or more are
    # not candidates (they would wrap to negative int32 numbers)
    say("merge_shards offsets near 2^31")
    rng = np.random.default_rng(99)
    g, b, kin, k = 4, 200, 16, 20
    s, i = _shard_lists(rng, g, b, kin, 500)
    offsets = [0, 2**31 - 650, 2**31 - 150, 2**31 - 1]   # disjoint ranges; the last two partly or wholly past the limit
    os_ = torch.full((b, k), 7.0, device="cuda")
    oi = torch.full((b, k), 7, dtype=torch.int32, device="cuda")
    apc.apc_merge_shards(torch.from_numpy(s).cuda(), torch.from_numpy(i).cuda(), g, b, kin, offsets, k, os_, oi)
    torch.cuda.synchronize()
    ws, wi = orc.merge_shards(s, i, offsets, k)
    gs = os_.cpu().numpy()
    assert np.array_equal(oi.cpu().numpy(), wi)
    assert np.array_equal(np.isnan(gs), np.isnan(ws)) and np.array_equal(gs[~np.isnan(ws)], ws[~np.isnan(ws)])
    assert (wi >= -1).all() and (wi[:, 0] >= 0).all()


@pytest.mark.parametrize("g,kin,k", [(2, 8, 8), (5, 9, 16), (64, 3, 20), (3, 33, 33), (64, 64, 64), (1, 64, 5)])
def test_merge_irregular_lists(apc, orc, g, kin, k):
    """Lists the register merge leaves to the heads' merge: a non-candidate
    before a candidate, negative zeros, one entry in two shards; in one query
    each, beside regular ones."""
    b = 9
    say(f"merge irregular g={g} kin={kin} k={k}")
    rng = np.random.default_rng(g * 100 + kin)
    s, i = _shard_lists(rng, g, b, kin, 5000)
    s[0, 1, 0], i[0, 1, 0] = np.nan, -1
    s[g - 1, 2] = np.linspace(0.9, 0.0, kin)
    s[g - 1, 2, kin - 1] = -0.0
    i[g - 1, 2] = np.arange(kin)
    off = np.arange(g, dtype=np.int32) * 5000
    ref_s, ref_i = orc.merge_shards(s, i, off, k)
    ts = torch.empty((b, k), dtype=torch.float32, device="cuda")
    ti = torch.empty((b, k), dtype=torch.int32, device="cuda")
    apc.apc_merge_shards(torch.from_numpy(s).cuda(), torch.from_numpy(i).cuda(), g, b, kin, off, k, ts, ti)
    torch.cuda.synchronize()
    assert np.array_equal(ti.cpu().numpy(), ref_i)
    assert np.array_equal(ts.cpu().numpy(), ref_s, equal_nan=True)
    if g > 1:                                            # the same shard twice: each entry once
        s2, i2 = np.stack([s[0], s[0]]), np.stack([i[0], i[0]])
        apc.apc_merge_shards(torch.from_numpy(s2).cuda(), torch.from_numpy(i2).cuda(), 2, b, kin, [0, 0], k, ts, ti)
        torch.cuda.synchronize()
        one_s, one_i = orc.merge_shards(s[:1], i[:1], off[:1], k)
        assert np.array_equal(ti.cpu().numpy(), one_i)
        assert np.array_equal(ts.cpu().numpy(), one_s, equal_nan=True)
