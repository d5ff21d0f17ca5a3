"""The plan that the library makes for a match (host only): which kernel, its
query tile, splits, passes.  Not part of the C ABI: the structure mirrors
MatchPlan in csrc/apc_internal.h, and plan() checks that the two agree."""
import collections
import ctypes

import paper_2502_06798_amd as apc

TILE, QS, QS8, F32S = range(4)
DT = {"f32": 0, "f16": 1, "bf16": 2, "e4m3": 3}
SIZE = {"f32": 4, "f16": 2, "bf16": 2, "e4m3": 1}
KERNEL = {TILE: "k_tile", QS: "k_qs", QS8: "k_qs8", F32S: "k_f32s"}


class _Plan(ctypes.Structure):
    _fields_ = ([(f, ctypes.c_int) for f in ("kernel", "bq", "qtiles", "splits")] + [("b_pad", ctypes.c_int64)] +
                [(f, ctypes.c_int) for f in ("chunk", "buckets")] +
                [(f, ctypes.c_size_t) for f in ("off_fq", "off_gt", "off_g2", "off_ps", "off_pi", "off_qp", "bytes")])


Plan = collections.namedtuple("Plan", "kernel bq qtiles splits passes rows tiles bytes parts off_end")


def plan(dtype, b, n, d, k):
    """kernel, queries per tile, tiles, splits, passes over the batch, rows of the
    largest split, tiles of 256 rows in it (k_tile), workspace bytes, parts of a
    shared bucket (k_tile; 0: no buckets), the end of what the kernel uses of the
    workspace."""
    f = apc.load()._ZN3apc10plan_matchEiliii
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32]
    f.restype = _Plan
    p = f(DT[dtype], n, d, b, k)
    assert p.kernel in KERNEL and p.b_pad == p.bq * p.qtiles and p.off_fq == 0 and p.off_fq < p.off_gt <= p.bytes
    passes = (b + p.chunk - 1) // p.chunk if p.kernel == TILE else 1
    assert p.b_pad >= (min(b, p.chunk) if p.kernel == TILE else b)
    blocks = (n + 31) // 32
    rows = -(-blocks // p.splits) * 32
    parts = (p.off_g2 - p.off_gt) // (4 * p.b_pad * k) if p.kernel == TILE and p.buckets else 0
    stages = max(4, -(-d * SIZE[dtype] // 128) * 2)
    return Plan(p.kernel, p.bq, p.qtiles, p.splits, passes, rows, -(-rows // 256), p.bytes, parts,
                p.off_qp + p.b_pad * stages * 64 if p.kernel == TILE else p.bytes)


def workspace(dtype, b, n, d, k):
    """What apc_match_workspace asks for a batch of b."""
    f = apc.load()._ZN3apc15match_workspaceEiliii
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32]
    f.restype = ctypes.c_size_t
    return f(DT[dtype], n, d, b, k)


def merge_by_heads(g, kin, k):
    """Whether shard lists are merged head by head (csrc/shards.hip)."""
    f = apc.load()._ZN3apc14merge_by_headsEiii
    f.argtypes = [ctypes.c_int32] * 3
    f.restype = ctypes.c_bool
    return f(g, kin, k)
