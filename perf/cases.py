"""The work whose speed is measured: what a user of the library has it do, through its public entry points.

Five kinds of case:

* ``step``   one batch through the whole path (match, top-k, optional resident fallback, level, placement, latent
             gather) on a ``MatchStep``, as a dispatcher calls it for every batch of prompts;
* ``match``  the nearest cached prompts alone (``apc_match_batch``), as a caller with its own placement uses it;
* ``ingest`` float32 embeddings into a cache: storage type, row checks, cache build, row factors;
* ``place``  what follows a match whose lists are in hand: resident fallback, level histogram, load-aware placement,
             gather of the latents at the assigned levels;
* ``merge``  the merge of the row shards' top-k lists.

Embeddings follow the repository's synthetic recipe: Gaussian clusters, entries normalise(c + 0.3 z), queries
normalise(c + sigma z), stored in float32, float16, bfloat16 or e4m3fn codes with a float32 scale per row.
"""
import math

import numpy as np
import torch

import paper_2502_06798_amd as apc
from paper_2502_06798_amd import synth

DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "e4m3": torch.float8_e4m3fn}
SIZE = {"f32": 4, "f16": 2, "bf16": 2, "e4m3": 1}
WIDTHS = (256, 384, 512, 640, 768, 1024, 1536)


def _step(name, b, n, d, dtype, k, clusters, lo, hi, levels, inst, cap, latent, slots, route="rounds", fallback=False):
    return {"name": name, "kind": "step", "b": b, "n": n, "d": d, "dtype": dtype, "k": k, "clusters": clusters,
            "sigma_lo": lo, "sigma_hi": hi, "levels": levels, "inst": inst, "cap": cap, "latent": latent,
            "slots": slots, "route": route, "fallback": fallback}


def _match(name, b, n, d, dtype, k, clusters, lo=0.4, hi=0.4):
    return {"name": name, "kind": "match", "b": b, "n": n, "d": d, "dtype": dtype, "k": k, "clusters": clusters,
            "sigma_lo": lo, "sigma_hi": hi}


def listed():
    return [
        # a small deployment: 16 prompts against 10,000 cached ones, every latent (4 x 64 x 64 halves) resident
        _step("step_b16_n10k_d768_f32", 16, 10_000, 768, "f32", 5, 100, 0.4, 0.4, 5, 2, 8, 32768, 10_000),
        # an ordinary batch and cache
        _step("step_b256_n100k_d768_f16", 256, 100_000, 768, "f16", 10, 1_000, 0.4, 0.4, 5, 4, 64, 32768, 100_000),
        # a large cache of which some entries' latents are resident, placement by Route-Plan
        _step("step_b1024_n1m_d768_bf16", 1_024, 1_000_000, 768, "bf16", 10, 10_000, 0.4, 0.4, 5, 8, 128, 32768, 65_536,
              "planned", True),
        # large batch: match and placement only
        _step("step_b4096_n4m_d512_f16", 4_096, 4_000_000, 512, "f16", 16, 20_000, 0.2, 0.8, 10, 16, 256, 0, 0),
        # the largest: 16,384 prompts against 10 million, a small hot set of resident 128 KB latents
        _step("step_b16384_n10m_d768_e4m3", 16_384, 10_000_000, 768, "e4m3", 32, 50_000, 0.2, 0.8, 10, 32, 512, 131072, 512),
        # low load: a few prompts stream a cache larger than the last-level cache
        _match("match_b4_n1m_d768_bf16", 4, 1_000_000, 768, "bf16", 10, 10_000),
        # nothing a round number: queries, rows and k off every tile
        _match("match_b77_n300007_d384_f16", 77, 300_007, 384, "f16", 7, 3_000),
        # wide half-precision rows, a mid-sized batch
        _match("match_b512_n250k_d1024_f16", 512, 250_000, 1_024, "f16", 10, 2_500),
        # float32 embeddings kept as they come, more rows than the small-cache kernel takes
        _match("match_b64_n200k_d768_f32", 64, 200_000, 768, "f32", 10, 2_000),
        # a million float32 embeddings stored as e4m3 codes and built into a cache
        {"name": "ingest_n1m_d768_e4m3", "kind": "ingest", "n": 1_000_000, "d": 768, "dtype": "e4m3"},
        # a full batch placed under capacity over ten levels, latents kept per level
        {"name": "place_b16384_k32", "kind": "place", "b": 16_384, "k": 32, "n": 10_000_000, "levels": 10, "inst": 32,
         "cap": 512, "latent": 32768, "slots": 4_096, "greedy": True},
        # eight row shards' lists of a full batch
        {"name": "merge_g8_b16384_k32", "kind": "merge", "g": 8, "b": 16_384, "k": 32},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _shape(rng):
    """Batch, rows, width, type and neighbours of a match that reads at most 8 GB and costs less than the largest listed."""
    dtype = rng.choice(("f32", "f16", "f16", "bf16", "bf16", "e4m3", "e4m3"))
    d = rng.choice(WIDTHS)
    b, k = _log(rng, 1, 16_384), _log(rng, 1, 48)
    most = min(8e9 / (d * SIZE[dtype]), (2e12 if dtype == "f32" else 8e12) / (2 * b * d), 10e6)
    return dtype, d, b, k, _log(rng, 1_000, max(2_000, int(most)))


def _sigma(rng):
    return (0.4, 0.4) if rng.random() < 0.5 else (0.2, 0.8)


def draw(rng):
    kind = rng.choice(("step", "step", "step", "match", "match", "match", "match", "ingest", "place", "merge"))
    if kind in ("step", "match"):
        dtype, d, b, k, n = _shape(rng)
        lo, hi = _sigma(rng)
        clusters = max(1, n // rng.randint(60, 240))
        if kind == "match":
            c = _match("", b, n, d, dtype, k, clusters, lo, hi)
        else:
            inst = rng.randint(1, 48)
            cap = max(1, int(b * rng.uniform(0.7, 1.5) / inst))
            latent = rng.choice((0, 32768, 131072))
            slots = 0 if latent == 0 else min(n, 16_384, _log(rng, 256, 65_536))
            c = _step("", b, n, d, dtype, k, clusters, lo, hi, rng.choice((5, 10)), inst, cap, latent, slots,
                      rng.choice(("rounds", "planned")), latent > 0 and rng.random() < 0.5)
    elif kind == "ingest":
        d = rng.choice(WIDTHS)
        c = {"kind": "ingest", "n": _log(rng, 1_000, 1_500_000 * 768 // d), "d": d, "dtype": rng.choice(("f16", "bf16", "e4m3"))}
    elif kind == "place":
        b, inst = _log(rng, 1, 16_384), rng.randint(1, 64)
        c = {"kind": "place", "b": b, "k": _log(rng, 1, 48), "n": _log(rng, 10_000, 10_000_000), "levels": rng.choice((5, 10)),
             "inst": inst, "cap": max(1, int(b * rng.uniform(0.7, 1.5) / inst)), "latent": rng.choice((32768, 131072)),
             "slots": _log(rng, 256, 4_096), "greedy": rng.random() < 0.7}
    else:
        c = {"kind": "merge", "g": rng.randint(2, 64), "b": _log(rng, 1, 16_384), "k": _log(rng, 1, 48)}
    c.pop("name", None)
    return c


# ---- inputs ------------------------------------------------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1_000_003 + stream * 7_919 + 12_345) & ((1 << 62) - 1))
    return g


def _store(x, dtype):
    """float32 rows rounded to the storage type, and the row scales (e4m3fn only)."""
    if dtype != "e4m3":
        return x.to(DTYPE[dtype]), None
    scale = (x.abs().amax(dim=1).to(torch.float64) / 448.0).to(torch.float32)   # the correctly rounded quotient
    return (x / scale[:, None]).clamp_(-448.0, 448.0).to(DTYPE[dtype]), scale


def _rows(centres, n, d, dtype, lo, hi, g):
    out = torch.empty((n, d), dtype=DTYPE[dtype], device="cuda")
    scale = torch.empty(n, dtype=torch.float32, device="cuda") if dtype == "e4m3" else None
    step = max(1, (1 << 29) // d)
    for r0 in range(0, n, step):
        r1 = min(n, r0 + step)
        x = torch.randn((r1 - r0, d), device="cuda", generator=g)
        x *= lo if lo == hi else lo + (hi - lo) * torch.rand((r1 - r0, 1), device="cuda", generator=g)
        x += centres[torch.randint(0, centres.shape[0], (r1 - r0,), device="cuda", generator=g)]
        x /= torch.linalg.vector_norm(x, dim=1, keepdim=True)
        y, s = _store(x, dtype)
        out[r0:r1] = y
        if scale is not None:
            scale[r0:r1] = s
    return out, scale


def _embeddings(case, seed):
    """(entries, their scales, queries, their scales)"""
    g = _gen(seed, 1)
    centres = torch.randn((case["clusters"], case["d"]), device="cuda", generator=g)
    e, es = _rows(centres, case["n"], case["d"], case["dtype"], 0.3, 0.3, g)
    q, qs = _rows(centres, case["b"], case["d"], case["dtype"], case["sigma_lo"], case["sigma_hi"], g)
    return e, es, q, qs


def _pool(case, seed, rows):
    """Latent pool of `rows` latents (halves drawn from uniform(-1, 1), as bytes)."""
    out = torch.empty((rows, case["latent"] // 2), dtype=torch.float16, device="cuda")
    out.uniform_(-1.0, 1.0, generator=_gen(seed, 2))
    return out.view(torch.uint8)


def _slot_map(n, slots, seed):
    """Entry -> latent slot (-1: not resident) for a random sample of `slots` entries; None when all are resident."""
    if slots == n:
        return None
    m = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    hot = torch.randperm(n, device="cuda", generator=_gen(seed, 3))[:slots]
    m[hot] = torch.arange(slots, dtype=torch.int32, device="cuda")
    return m


def _tables(case, seed):
    """Thresholds, skip counts and the instance table (host): instance i at level i mod (L + 1)."""
    L = case["levels"]
    theta = np.array(synth.THETA5 if L == 5 else synth.THETA10, dtype=np.float32)
    K = np.array(synth.K5 if L == 5 else synth.K10, dtype=np.int32)
    rng = np.random.default_rng(seed)
    lvl = np.arange(case["inst"], dtype=np.int32) % (L + 1)
    cap = np.full(case["inst"], case["cap"], dtype=np.int32)
    queue = rng.integers(0, case["cap"] + 1, size=case["inst"]).astype(np.int32)
    rand = rng.integers(0, 1 << 32, size=case["inst"], dtype=np.uint64).astype(np.uint32)
    return theta, K, lvl, cap, queue, rand


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "match"):
        e, es, q, qs = _embeddings(case, seed)
        if kind == "match":
            b, k = case["b"], case["k"]
            cache = apc.apc_build_cache(e, es)
            return {"case": case, "cache": cache, "q": q, "qs": qs, "ws": apc.workspace_tensor(cache, b, k),
                    "top_score": torch.empty((b, k), dtype=torch.float32, device="cuda"),
                    "top_idx": torch.empty((b, k), dtype=torch.int32, device="cuda")}
        theta, K, lvl, cap, queue, _ = _tables(case, seed)
        pool = _pool(case, seed, case["slots"]) if case["latent"] else None
        smap = _slot_map(case["n"], case["slots"], seed) if case["latent"] else None
        cache = apc.apc_build_cache(e, es, pool, smap)
        step = apc.MatchStep(cache, case["b"], case["k"], theta, K, lvl, cap, queue, latent_bytes=case["latent"],
                             route=case["route"], resident_fallback=case["fallback"])
        if step.batch is not None:
            step.batch.zero_()      # places that no latent goes to are not written
        return {"case": case, "step": step, "q": q, "qs": qs}
    g = _gen(seed, 4)
    if kind == "ingest":
        n, d, dtype = case["n"], case["d"], case["dtype"]
        x = torch.randn((n, d), device="cuda", generator=g)
        x /= torch.linalg.vector_norm(x, dim=1, keepdim=True)
        return {"case": case, "x": x, "rows": torch.empty((n, d), dtype=DTYPE[dtype], device="cuda"),
                "scale": torch.empty(n, dtype=torch.float32, device="cuda") if dtype == "e4m3" else None,
                "bad": torch.empty(n, dtype=torch.uint8, device="cuda"),
                "factors": torch.empty(n, dtype=torch.float32, device="cuda"), "cache": None}
    if kind == "place":
        b, k, n, L = case["b"], case["k"], case["n"], case["levels"]
        slots = case["slots"]
        # lists as a match leaves them: scores falling from the best one, entries of which some are resident
        best = torch.rand((b, 1), device="cuda", generator=g) * 0.38 + 0.6
        top_score = (best - torch.rand((b, k), device="cuda", generator=g).cumsum(1) * (0.1 / k)).contiguous()
        smap = _slot_map(n, slots, seed)
        hot = torch.nonzero(smap >= 0).flatten()
        idx = torch.randint(0, n, (b, k), device="cuda", generator=g)
        near = hot[torch.randint(0, hot.numel(), (b, k), device="cuda", generator=g)]
        top_idx = torch.where(torch.rand((b, k), device="cuda", generator=g) < 1.0 / k, near, idx).to(torch.int32).contiguous()
        emb = torch.ones((n, 16), dtype=torch.float8_e4m3fn, device="cuda")
        pool = _pool(case, seed, slots * L)
        cache = apc.apc_build_cache(emb, torch.ones(n, device="cuda"), pool, smap)
        i32 = dict(dtype=torch.int32, device="cuda")
        out = {"res_score": torch.empty(b, dtype=torch.float32, device="cuda"), "res_idx": torch.empty(b, **i32),
               "opt_level": torch.empty(b, **i32), "out_level": torch.empty(b, **i32), "out_inst": torch.empty(b, **i32),
               "out_slot": torch.empty(b, **i32), "fill": torch.empty(case["inst"], **i32), "hist": torch.empty(L + 1, **i32),
               "hit": torch.empty(b, **i32),
               "batch": torch.zeros((case["inst"] * case["cap"], case["latent"]), dtype=torch.uint8, device="cuda")}
        return {"case": case, "cache": cache, "top_score": top_score, "top_idx": top_idx, "tables": _tables(case, seed), "out": out}
    gs, b, k = case["g"], case["b"], case["k"]
    scores = torch.sort(torch.rand((gs, b, k), device="cuda", generator=g) * 0.4 + 0.55, dim=2, descending=True).values.contiguous()
    rows = 1_000_000
    idx = torch.randint(0, rows, (gs, b, k), device="cuda", generator=g).to(torch.int32)
    return {"case": case, "scores": scores, "idx": idx, "offsets": [rows * s for s in range(gs)],
            "top_score": torch.empty((b, k), dtype=torch.float32, device="cuda"),
            "top_idx": torch.empty((b, k), dtype=torch.int32, device="cuda")}


# ---- one pass ----------------------------------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        s = state["step"]
        s.run(state["q"], state["qs"])
        out = {"top_score": s.top_score, "top_idx": s.top_idx, "opt_level": s.opt_level, "out_level": s.out_level,
               "out_inst": s.out_inst, "out_slot": s.out_slot, "inst_fill": s.inst_fill}
        if case["fallback"]:
            out["res_score"], out["res_idx"] = s.res_score, s.res_idx
        if s.plan is not None:
            out["plan"] = s.plan
        if s.batch is not None:
            out["hit"], out["batch"] = s.hit, s.batch
        return out
    if kind == "match":
        apc.apc_match_batch(state["cache"], state["q"], state["qs"], case["k"], state["top_score"], state["top_idx"], state["ws"])
        return {"top_score": state["top_score"], "top_idx": state["top_idx"]}
    if kind == "ingest":
        apc.apc_quantize_rows(state["x"], state["rows"], state["scale"])
        n_bad, first_bad = apc.apc_validate_rows(state["rows"], state["scale"], state["bad"])
        state["cache"] = apc.apc_build_cache(state["rows"], state["scale"])
        apc.apc_cache_row_factors(state["cache"], state["factors"])
        out = {"rows": state["rows"].view(torch.uint8), "bad": state["bad"], "factors": state["factors"], "n_bad": n_bad,
               "first_bad": first_bad}
        if state["scale"] is not None:
            out["scale"] = state["scale"]
        return out
    if kind == "place":
        o, b, k, L = state["out"], case["b"], case["k"], case["levels"]
        theta, K, lvl, cap, queue, rand = state["tables"]
        apc.apc_resident_best(state["cache"], state["top_score"], state["top_idx"], k, k, b, o["res_score"], o["res_idx"])
        apc.apc_assign_load_aware(o["res_score"], 1, b, theta, K, lvl, cap, queue, rand, b if case["greedy"] else 0, 1,
                                  o["opt_level"], o["out_level"], o["out_inst"], o["out_slot"], o["fill"])
        apc.apc_level_histogram(o["opt_level"], b, L, o["hist"])
        apc.apc_gather_latents_at_level(state["cache"], o["res_idx"], 1, b, o["out_level"], o["out_inst"], o["out_slot"],
                                        case["inst"], case["cap"], L, o["batch"], o["hit"])
        return dict(o)
    apc.apc_merge_shards(state["scores"], state["idx"], case["g"], case["b"], case["k"], state["offsets"], case["k"],
                         state["top_score"], state["top_idx"])
    return {"top_score": state["top_score"], "top_idx": state["top_idx"]}


# ---- what a pass cannot do without, and how far another correct one may be off -----------------------------------

def work(case):
    kind = case["kind"]
    if kind in ("step", "match"):
        b, n, d, k, es = case["b"], case["n"], case["d"], case["k"], SIZE[case["dtype"]]
        nbytes = (n + b) * d * es + 8 * b * k
        if kind == "step":
            nbytes += 16 * b
            if case["latent"]:
                share = 1.0 - (1.0 - case["slots"] / n) ** (k if case["fallback"] else 1)
                placed = min(b, case["inst"] * case["cap"])
                above = sum(1 for i in range(case["inst"]) if i % (case["levels"] + 1)) / case["inst"]
                nbytes += int(2 * case["latent"] * placed * share * above)
        return {"bytes": nbytes, "flops": 2.0 * b * n * d}
    if kind == "ingest":
        n, d, es = case["n"], case["d"], SIZE[case["dtype"]]
        return {"bytes": n * d * (4 + es) + 9 * n, "flops": 4.0 * n * d}
    if kind == "place":
        placed = min(case["b"], case["inst"] * (case["cap"] if case["greedy"] else 1))
        above = sum(1 for i in range(case["inst"]) if i % (case["levels"] + 1)) / case["inst"]
        return {"bytes": 8 * case["b"] * case["k"] + 28 * case["b"] + int(2 * case["latent"] * placed * above * 0.63),
                "flops": case["b"] * (case["k"] + case["levels"])}
    return {"bytes": 8 * case["b"] * case["k"] * (case["g"] + 1), "flops": case["b"] * case["k"] * case["g"]}


def tolerance(case):
    # Scores are float32 sums of d products, then two factors.  Measured against 64 bits they are off (2-norm, relative)
    # by 1.1e-7 to 4e-7 for float32, float16 and bfloat16, and by 1.6e-6 to 2e-6 for e4m3fn, whose matrix instructions
    # align 64 products before they add them.  Neighbours whose scores are nearer than that may change places in a list.
    # Row factors and scales are single float32 results.  Placement, gather and merge move whole numbers, bytes and
    # given scores.
    kind = case["kind"]
    if kind in ("step", "match"):
        if case["dtype"] == "e4m3":
            return {"rel": 8e-6, "max": 4e-5, "differ": 0.01}
        return {"rel": 1.6e-6, "max": 8e-6, "differ": 0.002}
    if kind == "ingest":
        return {"rel": 5e-7, "max": 2e-6}
    return "exact"


# ---- the same in 64 bits -----------------------------------------------------------------------------------------

def _exact_topk(e, q, k):
    """Best k cosines of every query in 64 bits, and their entries (rows taken a chunk at a time)."""
    q64 = q.to(torch.float64)
    q64 = q64 / torch.linalg.vector_norm(q64, dim=1, keepdim=True)
    best = idx = None
    step = max(k, (1 << 28) // max(1, max(q.shape[0], e.shape[1])))
    for r0 in range(0, e.shape[0], step):
        x = e[r0:r0 + step].to(torch.float64)
        s = q64 @ (x / torch.linalg.vector_norm(x, dim=1, keepdim=True)).T
        v, i = torch.topk(s, min(k, s.shape[1]), dim=1)
        i = i + r0
        if best is not None:
            v, i = torch.cat((best, v), 1), torch.cat((idx, i), 1)
            v, o = torch.topk(v, min(k, v.shape[1]), dim=1)
            i = torch.gather(i, 1, o)
        best, idx = v, i
    return best.clamp(-1.0, 1.0), idx.to(torch.int32)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "match"):
        if 1.0 * case["b"] * case["n"] > 3e10:
            return None                                     # over 20 seconds
        e, _, q, _ = _embeddings(case, seed)                # e4m3fn: the row scales cancel in the cosine
        s, i = _exact_topk(e, q, case["k"])
        out = {"top_score": s, "top_idx": i}
        if kind == "step":                                  # whole numbers and bytes that follow from the lists
            out.update({p: None for p in ("opt_level", "out_level", "out_inst", "out_slot", "inst_fill", "res_score", "res_idx",
                                          "plan", "hit", "batch")})
        return out
    if kind == "ingest":
        n, d = case["n"], case["d"]
        x = torch.randn((n, d), device="cuda", generator=_gen(seed, 4))
        x /= torch.linalg.vector_norm(x, dim=1, keepdim=True)
        y, _ = _store(x, case["dtype"])
        step = 1 << 17
        f = torch.cat([1.0 / torch.linalg.vector_norm(y[r:r + step].to(torch.float64), dim=1) for r in range(0, n, step)])
        out = {"rows": y.view(torch.uint8), "bad": None, "factors": f, "n_bad": 0, "first_bad": -1}
        if case["dtype"] == "e4m3":
            out["scale"] = x.abs().amax(dim=1).to(torch.float64) / 448.0
        return out
    if kind == "merge":
        s = prepare(case, seed)
        g, b, k = case["g"], case["b"], case["k"]
        v = s["scores"].permute(1, 0, 2).reshape(b, g * k).to(torch.float64)
        top = torch.topk(v, k, dim=1).values
        return {"top_score": top, "top_idx": None}
    return None
