"""The tiled similarity kernel at the sizes where it can go wrong: every query
tile (32, 64, 128, 256 queries) of every type over splits of several tiles, rows
that end inside a stage of 64 bytes or a slot of 128, splits whose last tile is
partial or a single row, k at the edges of its bounds and logs, batches of
several passes, logs that overflow.  Then the lines between the kernels, and the
kernels with lists at the shapes they have.  A test that is about one kernel or
tile asserts that the plan gives its shape to it."""
import pytest
import torch

from tests.gpu_check import say
from tests.match_plan import KERNEL, SIZE, TILE, plan

pytestmark = pytest.mark.gpu

DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "e4m3": torch.float8_e4m3fn}


@pytest.fixture(scope="module")
def apc():
    import paper_2502_06798_amd as apc
    apc.load()
    assert torch.cuda.is_available()
    return apc


def rows(n, d, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn((n, d), device="cuda", generator=g)
    x /= torch.linalg.vector_norm(x, dim=1, keepdim=True)
    if dtype == "e4m3":
        return (x * 300.0).clamp(-448.0, 448.0).to(DT[dtype]), torch.full((n,), 1 / 300.0, device="cuda")
    return x.to(DT[dtype]), None


def match(apc, e, es, q, qs, k):
    c = apc.apc_build_cache(e, es)
    b = q.shape[0]
    ts = torch.empty((b, k), dtype=torch.float32, device="cuda")
    ti = torch.empty((b, k), dtype=torch.int32, device="cuda")
    ws = apc.workspace_tensor(c, b, k)
    apc.apc_match_batch(c, q, qs, k, ts, ti, ws)
    torch.cuda.synchronize()
    s1, i1 = ts.clone(), ti.clone()
    ws.random_(0, 256)                                   # nothing may depend on what the workspace held
    apc.apc_match_batch(c, q, qs, k, ts, ti, ws)
    torch.cuda.synchronize()
    assert torch.equal(ts.view(torch.int32), s1.view(torch.int32)) and torch.equal(ti, i1), "a second pass differs"
    c.close()
    return ts.double(), ti.long()


def check(e, q, k, ts, ti, tol):
    """Scores of the returned entries and of the exact ranking, in float64;
    entries equal wherever the exact scores are further apart than float32 sums
    can be off (d products of magnitude at most 1: under 1e-5 here; e4m3 MFMAs
    align 64 products before they add them: 1e-4)."""
    q64 = q.double() / torch.linalg.vector_norm(q.double(), dim=1, keepdim=True)
    e64 = e.double() / torch.linalg.vector_norm(e.double(), dim=1, keepdim=True)
    s = q64 @ e64.T
    best, idx = torch.sort(s, dim=1, descending=True, stable=True)
    assert (ti >= 0).all() and all(len(set(r.tolist())) == k for r in ti)
    assert (torch.gather(s, 1, ti) - ts).abs().max() <= tol and (best[:, :k] - ts).abs().max() <= tol
    lone = torch.ones_like(ti, dtype=torch.bool)
    gap = (best[:, :-1] - best[:, 1:]) > tol
    lone[:, 1:] &= gap[:, : k - 1]
    m = min(k, gap.shape[1])
    lone[:, :m] &= gap[:, :m]
    assert torch.equal(ti[lone], idx[:, :k][lone])


@pytest.mark.parametrize("dtype,b,n,d,k", [
    ("f16", 32, 257, 8, 1), ("f16", 33, 513, 40, 10), ("bf16", 64, 2048, 1024, 16), ("f16", 65, 4100, 640, 17),
    ("bf16", 128, 3000, 200, 32), ("f16", 129, 2900, 1544, 33), ("f16", 700, 3333, 640, 10), ("f16", 2000, 9000, 72, 13),
    ("f32", 1, 20000, 4, 1), ("f32", 300, 2500, 100, 10), ("f32", 31, 20001, 768, 48), ("f32", 513, 1000, 260, 64),
    ("e4m3", 1, 300, 16, 5), ("e4m3", 100, 2000, 384, 10), ("e4m3", 257, 5000, 640, 20), ("e4m3", 600, 1025, 240, 40),
    ("e4m3", 1500, 4000, 256, 9),
])
def test_tile_edges(apc, dtype, b, n, d, k):
    say(f"tile {dtype} b={b} n={n} d={d} k={k}")
    e, es = rows(n, d, dtype, n + d)
    q, qs = rows(b, d, dtype, b + 7)
    ts, ti = match(apc, e, es, q, qs, k)
    check(e, q, k, ts, ti, {"f32": 1e-5, "e4m3": 1e-4}.get(dtype, 1e-5))


@pytest.mark.parametrize("k", [1, 2, 3, 5, 9, 15])
@pytest.mark.parametrize("dtype,b,n,d", [("f16", 40, 140001, 256), ("e4m3", 130, 70000, 640)])
def test_tile_buckets_of_several_parts(apc, dtype, b, n, d, k):
    """256 and 85 splits of several tiles: buckets of 16 parts to one."""
    say(f"tile parts {dtype} b={b} n={n} d={d} k={k}")
    p = plan(dtype, b, n, d, k)
    assert p.kernel == TILE and p.tiles >= 3 and p.splits in (256, 85)
    assert p.parts == ({1: 16, 2: 8, 3: 8, 5: 4, 9: 2, 15: 2} if p.splits == 256 else {1: 8, 2: 4, 3: 2, 5: 2, 9: 1, 15: 1})[k]
    e, es = rows(n, d, dtype, n + k)
    q, qs = rows(b, d, dtype, b + k)
    ts, ti = match(apc, e, es, q, qs, k)
    check(e, q, k, ts, ti, {"e4m3": 1e-4}.get(dtype, 1e-5))


@pytest.mark.parametrize("dtype,b,n,d,k", [
    ("f16", 16, 500000, 768, 10), ("f16", 17, 66000, 768, 10), ("bf16", 127, 65536, 768, 9), ("bf16", 128, 65536, 768, 10),
    ("f16", 256, 65537, 768, 1), ("f16", 256, 65537, 768, 11), ("f16", 257, 65537, 768, 10),      # 1536-byte rows
    ("f32", 48, 2000, 256, 5), ("f32", 49, 2000, 256, 5), ("f32", 48, 16384, 256, 5), ("f32", 49, 16384, 256, 5),   # small float32 or tiled
    ("f32", 256, 2400, 64, 32), ("f32", 256, 2401, 64, 32), ("f32", 257, 2000, 128, 9), ("f32", 60, 9600, 192, 1), ("f32", 65, 9600, 192, 1),
    ("e4m3", 12288, 20001, 512, 7), ("e4m3", 12288, 20000, 512, 7), ("f16", 4097, 20001, 256, 17),
])
def test_routes_meet(apc, dtype, b, n, d, k):
    """Around lines between the kernels, those of the small float32 kernel among
    them (the other lines: test_kernels_agree_where_they_meet)."""
    say(f"route {dtype} b={b} n={n} d={d} k={k}")
    e, es = rows(n, d, dtype, n + k)
    q, qs = rows(b, d, dtype, b)
    ts, ti = match(apc, e, es, q, qs, k)
    r = torch.arange(0, b, max(1, b // 97), device="cuda")
    check(e, q[r], k, ts[r], ti[r], {"f32": 1e-5, "e4m3": 1e-4}.get(dtype, 1e-5))


@pytest.mark.parametrize("dtype,d,k,first,second", [
    # (b, n) whose kernel holds lists, and beside it (b, n) of the tiled one
    ("e4m3", 512, 1, (5000, 50000), (5000, 49999)), ("f16", 384, 3, (1024, 488282), (1023, 488282)),
    ("bf16", 256, 7, (12288, 2000), (12287, 2000)), ("f16", 384, 20, (8192, 6000), (8191, 6000)), ("e4m3", 1024, 16, (4096, 244141), (4095, 244141)),
    ("e4m3", 1536, 3, (64, 16000), (64, 16001)), ("f16", 768, 5, (20, 8000), (20, 7999)), ("bf16", 768, 5, (65, 4000), (64, 4000)), ("f16", 768, 7, (129, 12000), (128, 12000)),
    ("e4m3", 1536, 10, (257, 16000), (256, 16000)), ("f16", 768, 10, (128, 65536), (127, 65536)), ("f16", 768, 2, (513, 131072), (513, 131073)),
    ("e4m3", 1536, 8, (600, 60000), (600, 60001)), ("bf16", 768, 10, (2560, 4000), (2559, 4000)), ("bf16", 768, 4, (513, 2000), (513, 1999)),
])
def test_kernels_agree_where_they_meet(apc, dtype, d, k, first, second):
    """Both sides of a line between the kernels: right, and where they have the
    same rows, bit for bit the same lists."""
    say(f"lines {dtype} d={d} k={k} {first} {second}")
    assert [KERNEL[plan(dtype, b, n, d, k).kernel] for b, n in (first, second)] == ["k_qs" if d * SIZE[dtype] == 1536 else "k_qs8", "k_tile"]
    e, es = rows(max(first[1], second[1]), d, dtype, d + k)
    q, qs = rows(max(first[0], second[0]), d, dtype, d + k + 1)
    got = []
    for b, n in (first, second):
        ts, ti = match(apc, e[:n].contiguous(), None if es is None else es[:n].contiguous(), q[:b].contiguous(), None if qs is None else qs[:b].contiguous(), k)
        r = torch.arange(0, b, max(1, b // 97), device="cuda")
        check(e[:n], q[r], k, ts[r], ti[r], {"e4m3": 1e-4}.get(dtype, 1e-5))
        got.append((ts, ti))
    b = min(first[0], second[0])
    if first[1] == second[1]:
        assert torch.equal(got[0][0][:b], got[1][0][:b]) and torch.equal(got[0][1][:b], got[1][1][:b])


@pytest.mark.parametrize("b", [60, 150])
def test_tile_batches_of_several_passes(apc, b):
    """Rows so wide that the copy of the queries takes several passes."""
    d, n, k = 40000, 300, 5
    say(f"tile passes b={b} d={d}")
    e, _ = rows(n, d, "f32", 3)
    q, _ = rows(b, d, "f32", 4)
    ts, ti = match(apc, e, None, q, None, k)
    check(e, q, k, ts, ti, 1e-5)


# (dtype, queries per tile, b, n, d): splits of 3 to 10 tiles, the last one partial
TILES = [("f32", 64, 257, 30001, 208), ("f32", 128, 1500, 12001, 208), ("f32", 256, 1500, 30001, 640),
         ("f16", 64, 129, 50001, 208), ("f16", 128, 2049, 9001, 208), ("f16", 256, 2049, 20001, 640),
         ("bf16", 64, 129, 50001, 640), ("bf16", 128, 2049, 9001, 640), ("bf16", 256, 3000, 50001, 208),
         ("e4m3", 64, 257, 30001, 208), ("e4m3", 128, 3000, 9001, 208), ("e4m3", 256, 3000, 30001, 640)]


def special(e, es, q, qs):
    """The last 40 entries are copies of the first, the first 40 queries too; query
    41 is zero, 50 holds a NaN, the last an infinity (e4m3, which has none: a NaN)."""
    n = e.shape[0]
    raw = lambda t: t.view(torch.uint8) if t.dtype == torch.float8_e4m3fn else t
    raw(e)[n - 40:] = raw(e)[:40]
    raw(q)[:40] = raw(e)[:40]
    bad = [41, 50, q.shape[0] - 1]
    if q.dtype == torch.float8_e4m3fn:
        raw(q)[41], raw(q)[50, 3], raw(q)[-1, -1] = 0, 0x7F, 0xFF
    else:
        q[41], q[50, 3], q[-1, -1] = 0, float("nan"), float("inf")
    if es is not None:
        es[n - 40:], qs[:40] = es[:40], es[:40]
    return bad


def check_special(e, q, k, ts, ti, bad, tol, every=97):
    n, b = e.shape[0], q.shape[0]
    assert (ti[bad] == -1).all() and torch.isnan(ts[bad]).all()
    first = torch.arange(40, device="cuda")
    if k >= 2:                                            # equal scores: the lower entry first
        assert torch.equal(ti[:40, 0], first) and torch.equal(ti[:40, 1], first + n - 40) and torch.equal(ts[:40, 0], ts[:40, 1])
    else:
        assert torch.equal(ti[:40, 0], first)
    r = torch.tensor(sorted((set(range(0, b, max(1, b // every))) | {b - 2, b // 2}) - set(bad)), device="cuda")
    check(e, q[r], k, ts[r], ti[r], tol)


@pytest.mark.parametrize("dtype,bq,b,n,d", TILES)
def test_every_tile(apc, dtype, bq, b, n, d):
    for k in (1, 10, 16) if bq == 256 else (7, 40):
        say(f"tile of {bq} {dtype} b={b} n={n} d={d} k={k}")
        p = plan(dtype, b, n, d, k)
        assert p.kernel == TILE and p.bq == bq and p.tiles >= 3 and p.rows % 256
        e, es = rows(n, d, dtype, n + d)
        q, qs = rows(b, d, dtype, b + 7)
        bad = special(e, es, q, qs)
        ts, ti = match(apc, e, es, q, qs, k)
        check_special(e, q, k, ts, ti, bad, {"e4m3": 1e-4}.get(dtype, 1e-5))


@pytest.mark.parametrize("dtype,bq,b,n,d", TILES)
def test_every_tile_logs_overflow(apc, dtype, bq, b, n, d):
    """In every split each row is nearer than those before it, so every pair of
    every tile after the first passes the bounds: 256 pairs per query, split and
    tile for logs of 48 or 96, cut again and again between the tiles."""
    for k in (5, 16) if bq == 256 else (16, 48):
        say(f"overflow, tile of {bq} {dtype} b={b} n={n} d={d} k={k}")
        p = plan(dtype, b, n, d, k)
        assert p.kernel == TILE and p.bq == bq and p.tiles >= 3
        a, _ = rows(1, d, "f32", 5)
        z, _ = rows(1, d, "f32", 6)
        blocks = (n + 31) // 32
        starts = torch.tensor([blocks * s // p.splits * 32 for s in range(p.splits)], device="cuda")
        row = torch.arange(n, device="cuda")
        pos = row - starts[torch.searchsorted(starts, row, right=True) - 1]
        t = (1.5 - 1.49 * (pos + row / n) / (p.rows + 1))[:, None]
        e = a + t * z
        e /= torch.linalg.vector_norm(e, dim=1, keepdim=True)
        q = a.repeat(b, 1)
        sc = [None, None]
        if dtype == "e4m3":
            e, q, sc = e * 300, q * 300, [torch.ones(n, device="cuda"), torch.ones(b, device="cuda")]
        e, q = e.to(DT[dtype]).contiguous(), q.to(DT[dtype]).contiguous()
        ts, ti = match(apc, e, sc[0], q, sc[1], k)
        assert torch.equal(ti, ti[:1].expand_as(ti)) and torch.equal(ts, ts[:1].expand_as(ts)), "equal queries differ"
        check(e, q[:2], k, ts[:2], ti[:2], {"e4m3": 1e-4}.get(dtype, 1e-5))


@pytest.mark.parametrize("dtype,bq,b,n,d", [("f32", 128, 3001, 6001, 640), ("f32", 256, 3001, 20001, 640), ("f16", 128, 5001, 6001, 640),
                                            ("bf16", 256, 3001, 20001, 1040), ("e4m3", 128, 9001, 3001, 640), ("e4m3", 256, 9001, 20001, 640)])
def test_every_tile_in_several_passes(apc, dtype, bq, b, n, d):
    """The last pass is not full; both sides of every line between passes."""
    k = 7
    say(f"passes, tile of {bq} {dtype} b={b} n={n} d={d}")
    p = plan(dtype, b, n, d, k)
    assert p.kernel == TILE and p.bq == bq and p.passes >= 2
    e, es = rows(n, d, dtype, n + d)
    q, qs = rows(b, d, dtype, b + 7)
    bad = special(e, es, q, qs)
    ts, ti = match(apc, e, es, q, qs, k)
    check_special(e, q, k, ts, ti, bad, {"e4m3": 1e-4}.get(dtype, 1e-5))
    few = q[-300:].contiguous()                           # one pass: the same lists, bit for bit
    assert plan(dtype, 300, n, d, k).passes == 1
    ts1, ti1 = match(apc, e, es, few, None if qs is None else qs[-300:].contiguous(), k)
    assert torch.equal(ts1[:-1], ts[-300:-1]) and torch.equal(ti1, ti[-300:])


@pytest.mark.parametrize("dtype,b,n,k", [("f16", 40, 6000, 10), ("f16", 300, 3000, 32), ("f32", 300, 5000, 64), ("e4m3", 130, 4000, 16)])
def test_tile_logs_overflow(apc, dtype, b, n, k):
    """Every row is nearer than all before it, so every pair passes the bounds:
    the logs fill and are cut again and again."""
    d = 640
    say(f"tile overflow {dtype} b={b} n={n} k={k}")
    a, _ = rows(1, d, "f32", 5)
    z, _ = rows(1, d, "f32", 6)
    t = torch.linspace(1.5, 0.01, n, device="cuda")[:, None]
    e = a + t * z
    e /= torch.linalg.vector_norm(e, dim=1, keepdim=True)
    q = a.repeat(b, 1)
    sc = [None, None]
    if dtype == "e4m3":
        e, q, sc = e * 300, q * 300, [torch.ones(n, device="cuda"), torch.ones(b, device="cuda")]
    e, q = e.to(DT[dtype]).contiguous(), q.to(DT[dtype]).contiguous()
    ts, ti = match(apc, e, sc[0], q, sc[1], k)
    check(e, q, k, ts, ti, {"f32": 1e-5, "e4m3": 1e-4}.get(dtype, 1e-5))
    assert torch.equal(ti, ti[:1].expand_as(ti)), "equal queries differ"


def test_tile_equal_rows_take_lower_index(apc):
    for n, k in ((5000, 16), (3000, 64)):
        say(f"tile ties n={n} k={k}")
        row, _ = rows(1, 640, "f16", 8)
        q, _ = rows(70, 640, "f16", 9)
        _, ti = match(apc, row.repeat(n, 1).contiguous(), None, q, None, k)
        assert torch.equal(ti, torch.arange(k, device="cuda").expand(70, k))


def test_tile_invalid_queries(apc):
    e, _ = rows(3000, 640, "f16", 10)
    q, _ = rows(140, 640, "f16", 11)
    q[3] = 0
    q[77, 5] = float("nan")
    q[139, 639] = float("inf")
    c = apc.apc_build_cache(e)
    ts = torch.empty((140, 9), dtype=torch.float32, device="cuda")
    ti = torch.empty((140, 9), dtype=torch.int32, device="cuda")
    apc.apc_match_batch(c, q, None, 9, ts, ti, apc.workspace_tensor(c, 140, 9))
    torch.cuda.synchronize()
    bad = [3, 77, 139]
    good = [i for i in range(140) if i not in bad]
    assert (ti[bad] == -1).all() and torch.isnan(ts[bad]).all()
    check(e, q[good], 9, ts[good].double(), ti[good].long(), 1e-5)
    c.close()


@pytest.mark.parametrize("dtype,b,n,d,k", [("f16", 200, 70000, 768, 10), ("bf16", 70, 20000, 768, 5),
                                            ("e4m3", 12288, 20001, 768, 32), ("f16", 4096, 600000, 256, 3)])
def test_scores_do_not_depend_on_the_kernel(apc, dtype, b, n, d, k):
    """Lists of a batch that another kernel serves, bit for bit those of the
    tiled kernel on some of its queries: the sums run over d in one order."""
    say(f"one order {dtype} b={b} n={n} d={d} k={k}")
    few = min(b // 2, 100)
    assert plan(dtype, b, n, d, k).kernel != TILE and plan(dtype, few, n, d, k).kernel == TILE
    e, es = rows(n, d, dtype, 31)
    q, qs = rows(b, d, dtype, 32)
    ts, ti = match(apc, e, es, q, qs, k)
    ts2, ti2 = match(apc, e, es, q[:few].contiguous(), None if qs is None else qs[:few].contiguous(), k)
    assert torch.equal(ts[:few], ts2) and torch.equal(ti[:few], ti2)


@pytest.mark.parametrize("k", [1, 16, 17, 32])
@pytest.mark.parametrize("rb", [512, 768, 1024])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "e4m3"])
def test_two_wavefront_kernel(apc, dtype, rb, k):
    """Every shape that is built, a partial last group of rows and a batch just
    past a tile of 256 queries."""
    b, n, d = 12289, 2111, rb // SIZE[dtype]
    say(f"k_qs8 {dtype} b={b} n={n} d={d} k={k}")
    assert KERNEL[plan(dtype, b, n, d, k).kernel] == "k_qs8"
    e, es = rows(n, d, dtype, n + d)
    q, qs = rows(b, d, dtype, b + 7)
    bad = special(e, es, q, qs)
    ts, ti = match(apc, e, es, q, qs, k)
    check_special(e, q, k, ts, ti, bad, {"e4m3": 1e-4}.get(dtype, 1e-5), every=200)


@pytest.mark.parametrize("b,n,k", [(70, 3001, 1), (70, 3001, 3), (300, 17011, 10), (60, 130, 2)])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "e4m3"])
def test_query_stationary_kernel(apc, dtype, b, n, k):
    d = 1536 // SIZE[dtype]
    say(f"k_qs {dtype} b={b} n={n} d={d} k={k}")
    assert KERNEL[plan(dtype, b, n, d, k).kernel] == "k_qs"
    e, es = rows(n, d, dtype, n + d)
    q, qs = rows(b, d, dtype, b + 7)
    bad = special(e, es, q, qs)
    ts, ti = match(apc, e, es, q, qs, k)
    check_special(e, q, k, ts, ti, bad, {"e4m3": 1e-4}.get(dtype, 1e-5))
