// Nearest cached prompts: cosine similarity of every query against every
// cache entry, fused with an exact per-query top-k.
//
// The plan of a match (which kernel, its tiles and splits, the workspace), the
// launches, and k_topk_merge: one wavefront per query merges the partial lists
// of all splits (each sorted, ranges disjoint) by repeated wave argmax.
//
// Every score is produced by the same fixed sequence of MFMAs whatever the
// tiling, and the final list is the unique top-k of those scores under a
// total order, so results are deterministic.
#include "apc_internal.h"
#include "tile.h"

namespace apc {
namespace {

constexpr int IDX_NONE = 0x7fffffff;

__device__ inline float neg_inf() { return -__builtin_huge_valf(); }

// (sa, ia) comes before (sb, ib) in the order score desc, index asc
__device__ inline bool before(float sa, int ia, float sb, int ib)
{
    return sa > sb || (sa == sb && ia < ib);
}

// ---- merge of the per-split partial lists ----------------------------------
// (score, index) as one key ordered like (score desc, index asc): the score's
// bits mapped to an order-preserving unsigned integer, then the complement of
// the index.  Adding +0 turns -0 into +0, which compare equal as scores.
__device__ inline uint64_t merge_key(float s, int i)
{
    const uint32_t u = __float_as_uint(s + 0.0f);
    const uint32_t o = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((uint64_t)o << 32) | (uint32_t)~(uint32_t)i;
}
__device__ inline float merge_key_score(uint64_t key)
{
    const uint32_t o = (uint32_t)(key >> 32);
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}
// one step of a wavefront maximum: the key of the lane that the DPP control
// names (own key where it names none, or the row is masked off)
template <int CTRL, int ROWS>
__device__ inline uint64_t dpp_max_step(uint64_t v)
{
    const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
    const uint32_t olo = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
    const uint32_t ohi = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
    const uint64_t o = ((uint64_t)ohi << 32) | olo;
    return o > v ? o : v;
}
// largest key of the wavefront, in every lane: quads (xor 1, xor 2), half
// rows (mirror), rows (mirror), then rows 1 and 3 take row 0's and row 2's
// maximum (broadcast of lane 15) and rows 2 and 3 row 1's (lane 31): lane 63
// ends with the maximum of all 64 lanes
__device__ inline uint64_t wave_max_key(uint64_t v)
{
    v = dpp_max_step<0xB1, 0xf>(v);      // quad_perm [1, 0, 3, 2]
    v = dpp_max_step<0x4E, 0xf>(v);      // quad_perm [2, 3, 0, 1]
    v = dpp_max_step<0x141, 0xf>(v);     // row_half_mirror
    v = dpp_max_step<0x140, 0xf>(v);     // row_mirror
    v = dpp_max_step<0x142, 0xa>(v);     // row_bcast:15
    v = dpp_max_step<0x143, 0xc>(v);     // row_bcast:31
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

template <int MAXOWN>
__global__ __launch_bounds__(256) void k_topk_merge(const float* __restrict__ part_s,
                                                     const int* __restrict__ part_i, int splits,
                                                     int64_t b_pad, int32_t k, int32_t b,
                                                     const float* __restrict__ fq,
                                                     float* __restrict__ top_s, int32_t* __restrict__ top_i)
{
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (q >= b) return;
    const float f = fq[q];
    if (!(f == f)) {                      // invalid query row
        for (int p = lane; p < k; p += 64) {
            top_s[q * k + p] = __int_as_float(0x7fc00000);
            top_i[q * k + p] = -1;
        }
        return;
    }
    const int ne = splits * k;                                     // this query's entries
    const float* gs = part_s + (int64_t)q * ne;
    const int* gi = part_i + (int64_t)q * ne;
    // a lane's list heads advance by loads from this query's block, which the
    // first loads bring into the vector cache
    auto fetch = [&](int l, int hd, float& sc, int& ix) {
        sc = gs[l * k + hd];
        ix = gi[l * k + hd];
    };
    int head[MAXOWN];
    float cs[MAXOWN];
    int ci[MAXOWN];
#pragma unroll
    for (int j = 0; j < MAXOWN; ++j) {
        const int l = lane + 64 * j;
        head[j] = 0;
        if (l < splits) {
            fetch(l, 0, cs[j], ci[j]);
        } else {
            cs[j] = neg_inf();
            ci[j] = IDX_NONE;
        }
    }
    for (int p = 0; p < k; ++p) {
        float bs = cs[0];
        int bi = ci[0], bj = 0;
#pragma unroll
        for (int j = 1; j < MAXOWN; ++j)
            if (before(cs[j], ci[j], bs, bi)) { bs = cs[j]; bi = ci[j]; bj = j; }
        const uint64_t wk = wave_max_key(merge_key(bs, bi));
        const float ws = merge_key_score(wk);
        const int wi = (int)~(uint32_t)wk;
        if (lane == 0) {
            top_s[q * k + p] = ws;
            top_i[q * k + p] = wi == IDX_NONE ? -1 : wi;
        }
        if (wi != IDX_NONE && bi == wi) {          // entry indices are unique: one owner
#pragma unroll
            for (int j = 0; j < MAXOWN; ++j)
                if (j == bj) {
                    ++head[j];
                    const int l = lane + 64 * j;
                    if (head[j] < k) {
                        fetch(l, head[j], cs[j], ci[j]);
                    } else {
                        cs[j] = neg_inf();
                        ci[j] = IDX_NONE;
                    }
                }
        }
    }
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

namespace {

// The workspace of a plan with one list of k pairs for every (query, split),
// by shape.  It covers k_qs, k_qs8 and k_f32s, and every plan asks at least this
// much, so that apc_match_batch_static refuses the same batches whichever
// kernel serves them: those whose lists (or, for rows that k_qs or k_qs8 is
// built for, lists and queries) pass the static array.  (No plan of the tiled
// kernel passes it by itself unless 32 of its queries are longer than 5.8 MB.)
// most: the largest for a batch of b or fewer.
size_t list_bytes(int dt, int64_t n, int64_t rb, int64_t b, int32_t k, bool most)
{
    const bool stationary = dt != APC_F32 && k <= 32 && (rb == 512 || rb == 768 || rb == 1024 || rb == 1536);
    const bool eight = stationary && rb != 1536 && b > 256;
    const bool small = dt == APC_F32 && rb % 256 == 0 && k <= 32 && n <= 16384 && b <= 256;
    const bool wide = stationary && (eight || (rb != 1536 && k <= 16));
    const int64_t bq = small ? 16 : wide ? 256 : 128;
    const int64_t rows = small ? 32 : eight || (stationary && (wide || (rb == 1536 && k > 16))) ? 64 : 128;
    const int64_t qt = (b + bq - 1) / bq, parts = (n + rows - 1) / rows;
    const int64_t target = stationary || k > 16 ? 256 : 512;
    int64_t splits = small ? parts : stationary ? (qt >= target ? 1 : target / qt) : (target + qt - 1) / qt;
    if (splits > parts) splits = parts;
    int64_t pairs = qt * splits;                                   // (query tile, split)
    if (most && !small) {
        // fewer tiles may have more splits each, up to the target between them all
        // (one short of a tile more where splits are rounded up)
        const int64_t bound = (target > qt ? target : qt) + (stationary ? 0 : qt - 1);
        pairs = bound < qt * parts ? bound : qt * parts;
    }
    const size_t bp = (size_t)(qt * bq), lists = (size_t)(pairs * bq);
    const size_t bytes = 2 * align256(4 * bp) + align256(eight ? 4 * lists : 0) + 2 * align256(4 * lists * k) +
                         align256(stationary ? bp * (size_t)rb : 0);
    const size_t below = most && b > 256 ? list_bytes(dt, n, rb, 256, k, true) : 0;   // (another shape up to 256 queries)
    return bytes > below ? bytes : below;
}

// Most queries of a pass of the tiled kernel: the logs stay below 26 MB, the copy
// of the queries below 5.8 MB unless 32 queries are longer.
int64_t tile_pass(int64_t rb)
{
    const int64_t copy = tile_stages(rb) * 64, pass = (11 << 19) / copy / 256 * 256;
    return pass >= 256 ? pass : (11 << 19) / copy >= 128 ? 128 : (11 << 19) / copy >= 64 ? 64 : 32;
}

// The same over a cache of few tiles, whose logs are few (a split has a tile at
// least): logs and copy below 30 MB together.  0: no more than tile_pass.
int64_t tile_pass_few(int64_t n, int64_t rb, int32_t k)
{
    const int64_t copy = tile_stages(rb) * 64, tiles = (n + 255) / 256;
    const int64_t few = 30000000 / (copy + tiles * (8 * tile_log_cap(k) + 8) + 4 * k + 8) / 256 * 256;
    return few > tile_pass(rb) && few * tiles <= (k <= 16 ? 65536 : 32768) ? few : 0;
}

// passes of equal size (a pass takes as long for a part of its queries)
int64_t tile_even(int64_t b, int64_t pass)
{
    const int64_t passes = (b + pass - 1) / pass, unit = pass < 256 ? pass : 256;
    return ((b + passes - 1) / passes + unit - 1) / unit * unit;
}

// tiles of 256 queries have no room for the longer logs of k > 16 (tile_log_cap)
bool tile_takes(int bq, int64_t pass, int32_t k) { return (bq <= 128 || k <= 16) && bq <= pass; }

// The most that a plan of the tiled kernel asks for a batch of b or fewer.  A
// tile of bq queries is never the best for bq / 2 queries or fewer, and the
// splits of all query tiles are 256 in all, or one each.
size_t tile_bytes_most(int64_t n, int64_t rb, int64_t b, int32_t k)
{
    const int64_t few = tile_pass_few(n, rb, k), pass = few ? few : tile_pass(rb);
    const int64_t copy = tile_stages(rb) * 64, tiles = (n + 255) / 256;
    const int64_t bc = b < pass ? b : pass;
    size_t bytes = 0;
    for (int bq = 32; bq <= 256; bq *= 2) {
        if (!tile_takes(bq, pass, k) || (bq > 32 && b <= bq / 2)) continue;
        const int64_t qt = (bc + bq - 1) / bq, bound = qt > 256 ? qt : 256, pairs = bound < qt * tiles ? bound : qt * tiles;
        const size_t bp = (size_t)(qt * bq), lists = (size_t)(pairs * bq);
        // (parts of a bucket: k parts below an eighth of the splits, see tile_ways)
        const size_t buckets = bp * k > lists / 8 ? bp * k : lists / 8;
        const size_t t = align256(4 * bp) + align256(4 * buckets) + align256(4 * lists) + align256(8 * lists * tile_log_cap(k)) +
                         align256(bp * copy);
        if (t > bytes) bytes = t;
    }
    return bytes;
}

MatchPlan plan_tile(int dt, int64_t n, int64_t rb, int32_t b, int32_t k)
{
    MatchPlan p{};
    p.kernel = KERNEL_TILE;
    const int64_t copy = tile_stages(rb) * 64, tiles = (n + 255) / 256;
    int64_t pass = tile_pass(rb), chunk = tile_even(b, pass);
    // Where such passes leave a quarter of the chip idle (128 queries and one tile
    // to a workgroup) and larger ones fit: float32 5,916 x 1,318 x 1,536 in seven
    // passes 611 us, in two 374; 2,000 x 300 x 1,536 228 and 79; 600 x 1,000 x 3,072
    // 409 and 138; f16 16,384 x 1,000 x 1,024 210 and 142; e4m3 16,384 x 1,000 x 768
    // 122 and 96.  Elsewhere they are as fast or faster (6,196 x 4,000 x 1,536 bf16:
    // 182 us in four passes, 224 in two).
    if (const int64_t few = tile_pass_few(n, rb, k); few && b > chunk && chunk / 128 * tiles < 192) {
        pass = few;
        chunk = tile_even(b, pass);
    }
    const int64_t bc = b < chunk ? b : chunk;
    p.chunk = (int)chunk;
    // The tile that takes the least time by this model: a workgroup goes
    // through its tiles one after the other (one workgroup per CU), each
    // stage of 64 bytes taking s us (float32, which its MFMAs bound: s32), each
    // tile e us besides, and the first one f us, as measured.  256 queries pay
    // where the batch fills them (512 x 250,000 x 1,024 f16: 307 us against 329
    // with 128; 1,024 x 1,000,000 x 640: 1,346 against 1,477); for other batches
    // the padding and the uneven last round decide (600 x 100,000 x 640 f16:
    // 146 us with 256, 124 with 128; 256 x 100,000 x 768: 92 and 85; 300 x
    // 20,000 x 384 float32: 127 us with 256, 72 with 64).  800 random shapes, time
    // over the fastest tile's in the mean: float32 1.011, 16-bit 1.012, e4m3 1.014,
    // so 16-bit and e4m3 rows share the stage's time.
    static const struct { int bq; float s, s32, e, f; } kinds[4] = {{256, 1.10f, 4.00f, 4.0f, 12.f},
                                                                    {128, 0.60f, 2.05f, 2.0f, 6.f},
                                                                    {64, 0.36f, 1.05f, 1.2f, 3.f},
                                                                    {32, 0.30f, 0.57f, 1.0f, 2.f}};
    const int64_t stages = tile_stages(rb);
    float best = 0.f;
    for (const auto& kd : kinds) {
        if (!tile_takes(kd.bq, pass, k)) continue;
        const int64_t qt = (bc + kd.bq - 1) / kd.bq;
        int64_t sp = qt >= 256 ? 1 : 256 / qt;
        if (sp > tiles) sp = tiles;                                // fewer rows than a tile's gain nothing
        const int64_t passes = (qt * sp + 255) / 256;
        const float rounds = dt == APC_F32 ? (float)tiles / sp : (float)((tiles + sp - 1) / sp);
        // (three or more tiles of 64 queries over a cache beyond the MALL wait for
        // their rows.  246 random shapes there, time over the fastest tile's, mean and
        // shapes more than 20% off: 1.064 and 47 without this term, 1.010 and 4 with
        // half of it, 1.005 and none: 151 x 9,461,309 x 384 f16 2,731 us without,
        // 2,045; 166 x 2,500,191 x 256 e4m3, k = 1, 373 with half, 252)
        const float far = kd.bq == 64 && qt > 2 && n * rb > (256ll << 20) && dt != APC_F32 ? 0.12f : 0.f;
        const float t = passes * (rounds * (stages * ((dt == APC_F32 ? kd.s32 : kd.s) + far) + kd.e) + kd.f);
        if (best > 0.f && t >= best) continue;
        best = t;
        p.bq = kd.bq;
        p.qtiles = (int)qt;
        p.splits = (int)sp;
    }
    p.b_pad = (int64_t)p.qtiles * p.bq;
    const size_t lists = (size_t)p.splits * p.b_pad;
    p.off_fq = 0;
    p.off_gt = align256(sizeof(float) * (size_t)p.b_pad);          // buckets
    // (the buckets are used where every one of the k gets rows: see tile_kernel.h)
    p.buckets = TL_CLASSES * p.splits >= k;
    p.off_g2 = align256(p.off_gt + (p.buckets ? sizeof(int) * (size_t)p.b_pad * k * tile_ways(k, p.splits) : 0));   // log lengths
    p.off_ps = align256(p.off_g2 + sizeof(int) * lists);           // logs
    p.off_qp = align256(p.off_ps + sizeof(uint64_t) * lists * tile_log_cap(k));
    p.bytes = align256(p.off_qp + (size_t)(p.b_pad * copy));
    return p;
}

// Where the kernel of two wavefronts per SIMD with the queries in registers (no
// query loads at all; rows of 512, 768 or 1024 bytes, k <= 32) is ahead of the
// tiled one.  It reads the cache once per 256 queries from the L2, while the
// tiled kernel also streams the queries; but its lists are slow to fill, so it
// needs rows to pay for them, more of them the longer the lists, until the tiled
// kernel's logs of 96 places cost as much (k > 16).  This kernel's time over the
// tiled one's, geometric means over 900 random shapes, by query-row pairs b n:
//   k = 1     1.1 at 1e8, 0.98 at 2.5e8, 0.88 at 1e9     k <= 3  1.0 at 5e8, 0.91 at 1e9
//   k <= 6    1.1 at 5e8, 0.98 at 1.2e9                  k <= 11 1.08 at 1e9, 0.98 at 2.4e9
//   k <= 16   1.1 at 6e8, 0.96 at 1e9                    k > 16  1.1 at 2e8, 0.93 at 5e8
// for 8,192 queries and more with k >= 14 0.9 (0.74 to 1.1) from 6,000 rows on, and
// for 12,288 queries and more 0.69 to 0.96 from 2,000 rows on.
bool qs8_ahead(int64_t n, int64_t b, int32_t k)
{
    if (b >= 12288) return n >= 2000;
    if (b >= 8192 && k >= 14 && n >= 6000) return true;
    const int64_t pairs = k == 1 ? 250000000 : k <= 3 ? 500000000 : k <= 6 ? 1200000000ll : k <= 11 ? 2400000000ll
                        : k <= 16 ? 1000000000ll : 400000000;
    return b * n >= pairs && b >= (k <= 6 ? 1024 : 4096);
}

// Where the kernel with the queries of a wavefront in registers (rows of 1536
// bytes, k <= 10) is ahead of the tiled one.  Its lists are in registers: an
// insertion costs a pass over the wavefront, so it is ahead for small k, where
// few pairs are inserted, and for middling caches, over which the tiled kernel's
// tiles of 256 rows divide unevenly (its 128-row groups lose less) or its prep
// and merge weigh.  This kernel's time over the tiled one's, geometric means
// over 1,500 random shapes (f16, bf16, e4m3), at rows n:
//   b <= 64            k = 1, 2 0.80 to 1.0; k = 3 0.95 to 16,000, 1.0 to 1.15 beyond; k = 5 1.0 to 1.16 but
//                      0.91 to 0.97 at 8,000 to 16,000; k = 10 1.0 to 1.28
//   b 65 to 512        k <= 3 0.74 to 1.0 (b > 128: 1.0 to 1.1 from 1,000,000); k = 5 1.05 below 4,000, 0.78 to 0.95, 1.03 from 500,000;
//                      k = 7 1.1 below 8,000, 0.84 to 0.97; k = 10 1.2 below 8,000, 0.82 to 1.0 from
//                      65,000 (b > 256: 16,000), 1.0 to 1.1 from 500,000 (e4m3: with b > 350 too)
//   b > 512            k = 1 0.63 to 0.95; k = 5 0.81 to 0.95 from 2,000; k = 10 1.15 at 1,000, 0.88 to 1.04
//                      from 8,000 (b > 2,560: 4,000), 1.05 to 1.1 from 130,000 (e4m3: 60,000)
bool qs_ahead(int dt, int64_t n, int64_t b, int32_t k)
{
    if (b > 512) {
        const int64_t least = k <= 3 ? 0 : k <= 5 ? 2000 : k <= 7 ? 6000 : b >= 2560 ? 4000 : 8192;
        return n >= least && n <= (dt == APC_E4M3 ? 60000 : 131072);
    }
    if (k >= 8 && dt == APC_E4M3 && b > 350) return false;
    if (k >= 8) return n < 500000 && (b > 256 ? n >= 16000 : b >= 128 && n >= 65536);
    if (k >= 6) return n < 500000 && b > 128 && n >= 12000;
    if (k >= 4) return b > 64 ? n >= 4000 && n < 500000 : n >= 8000 && n <= 16000;
    if (k == 3 && b <= 64) return n <= 16000;
    if (b <= 8 && n > 32768 && n <= 50000) return false;           // two groups in the longest of 256 splits, one tile
    return b <= 128 || n < 1000000;
}

MatchPlan plan_kernel(int dt, int64_t n, int32_t d, int32_t b, int32_t k)
{
    MatchPlan p{};
    const int64_t rb = (int64_t)d * elem_bytes(dt);
    const int q2b = qs_queries(dt, rb, k);
    const int q8b = qs8_queries(dt, rb, k);
    if (q8b > 0 && qs8_ahead(n, b, k)) {
        p.kernel = KERNEL_QS8;
        p.bq = q8b;
        p.qtiles = (b + p.bq - 1) / p.bq;
        const int64_t ngr = (n + qs8_group_rows() - 1) / qs8_group_rows();
        int64_t splits = p.qtiles >= 256 ? 1 : 256 / p.qtiles;
        if (splits > ngr) splits = ngr;
        if (splits < 1) splits = 1;
        p.splits = (int)splits;
    } else if (q2b > 0 && qs_ahead(dt, n, b, k)) {
        // queries in VGPRs, cache rows through LDS, one workgroup per CU; the query
        // tiles of a split share an XCD
        p.kernel = KERNEL_QS;
        p.bq = q2b;
        p.qtiles = (b + p.bq - 1) / p.bq;
        if (p.qtiles < 1) p.qtiles = 1;
        const int64_t gr = qs_group_rows();
        const int64_t ngr = (n + gr - 1) / gr;
        int64_t splits = p.qtiles >= 256 ? 1 : 256 / p.qtiles;
        if (splits > ngr) splits = ngr;
        if (splits < 1) splits = 1;
        p.splits = (int)splits;
    } else if (f32s_fits(dt, n, d, b, k)) {
        // small float32 caches and few queries: a workgroup per 32-row block, d
        // over its wavefronts
        p.kernel = KERNEL_F32S;
        p.bq = f32s_queries();
        p.qtiles = (b + p.bq - 1) / p.bq;
        p.splits = (int)((n + f32s_rows() - 1) / f32s_rows());
    } else {
        return plan_tile(dt, n, rb, b, k);
    }
    p.b_pad = (int64_t)p.qtiles * p.bq;
    p.off_fq = 0;
    p.off_gt = align256(p.off_fq + sizeof(float) * (size_t)p.b_pad);
    // the two-wavefront kernel's per-split quantile scores (splits x b_pad)
    p.off_g2 = align256(p.off_gt + sizeof(int) * (size_t)p.b_pad);
    const size_t g2_bytes = p.kernel == KERNEL_QS8 ? sizeof(int) * (size_t)p.splits * p.b_pad : 0;
    p.off_ps = align256(p.off_g2 + g2_bytes);
    p.off_pi = align256(p.off_ps + sizeof(float) * (size_t)p.splits * p.b_pad * k);
    p.off_qp = align256(p.off_pi + sizeof(int) * (size_t)p.splits * p.b_pad * k);
    const size_t qp_bytes =
        p.kernel == KERNEL_QS || p.kernel == KERNEL_QS8 ? (size_t)p.b_pad * (size_t)d * elem_bytes(dt) : 0;
    p.bytes = align256(p.off_qp + qp_bytes);
    return p;
}

}  // namespace

MatchPlan plan_match(int dt, int64_t n, int32_t d, int32_t b, int32_t k)
{
    MatchPlan p = plan_kernel(dt, n, d, b, k);
    const size_t least = list_bytes(dt, n, (int64_t)d * elem_bytes(dt), b, k, false);
    if (p.bytes < least) p.bytes = least;
    return p;
}

size_t match_workspace(int dt, int64_t n, int32_t d, int32_t b, int32_t k)
{
    const int64_t rb = (int64_t)d * elem_bytes(dt);
    const size_t lists = list_bytes(dt, n, rb, b, k, true);
    if (f32s_fits(dt, n, d, b, k)) return lists;                   // and so does every smaller batch
    const size_t tile = tile_bytes_most(n, rb, b, k);
    return tile > lists ? tile : lists;
}

hipError_t launch_match(const MatchPlan& p, int dt, int64_t n, int32_t d, const void* emb,
                        const float* fe, const void* q, const float* q_scale, int32_t b, int32_t k,
                        float* top_score, int32_t* top_idx, void* ws, hipStream_t s,
                        hipEvent_t ev_start, hipEvent_t ev_stop)
{
    uint8_t* w = static_cast<uint8_t*>(ws);
    float* fq = reinterpret_cast<float*>(w + p.off_fq);
    float* ps = reinterpret_cast<float*>(w + p.off_ps);
    int* pi = reinterpret_cast<int*>(w + p.off_pi);
    const int64_t row_bytes = (int64_t)d * elem_bytes(dt);

    hipError_t e;
    if (p.kernel == KERNEL_TILE) {
        TileArgs a{};
        a.emb = static_cast<const uint8_t*>(emb);
        a.fe = fe;
        a.n = n;
        a.fe_len = factor_pad(n);
        a.fq = fq;
        a.bucket = reinterpret_cast<int*>(w + p.off_gt);
        a.cnt = reinterpret_cast<int32_t*>(w + p.off_g2);
        a.log = reinterpret_cast<uint64_t*>(w + p.off_ps);
        a.b_pad = p.b_pad;
        a.rb = (int32_t)row_bytes;
        a.k = k;
        a.nst = (int32_t)tile_stages(row_bytes);
        a.qcopy = w + p.off_qp;
        a.splits = p.splits;
        a.qtiles = p.qtiles;
        a.cap = tile_log_cap(k);
        a.buckets = p.buckets;
        a.ways = tile_ways(k, p.splits);
        // query tiles that share an L2 (4 MB): about half of it
        const int64_t fit = (2 << 20) / ((int64_t)a.nst * 64 * p.bq);
        a.group = fit < 2 ? 2 : fit > 32 ? 32 : (int32_t)fit;
        if (a.group > p.qtiles) a.group = p.qtiles;
        const int32_t chunk = p.chunk;
        for (int32_t q0 = 0; q0 < b; q0 += chunk) {
            a.b = b - q0 < chunk ? b - q0 : chunk;
            if ((e = launch_tile_prep(dt, static_cast<const uint8_t*>(q) + (int64_t)q0 * row_bytes,
                                      q_scale ? q_scale + q0 : nullptr, a.b, row_bytes, p.bq, a, fq, w + p.off_qp, s)) !=
                hipSuccess)
                return e;
            if (ev_start && q0 == 0 && (e = hipEventRecord(ev_start, s)) != hipSuccess) return e;
            if ((e = launch_tile(dt, p.bq, a, s)) != hipSuccess) return e;
            if (ev_stop && q0 + chunk >= b && (e = hipEventRecord(ev_stop, s)) != hipSuccess) return e;
            if ((e = launch_tile_merge(a, top_score + (int64_t)q0 * k, top_idx + (int64_t)q0 * k, s)) != hipSuccess) return e;
        }
        return hipSuccess;
    } else if (p.kernel == KERNEL_F32S) {
        if (ev_start && (e = hipEventRecord(ev_start, s)) != hipSuccess) return e;
        e = launch_f32s(p, n, d, emb, fe, q, fq, b, k, ps, pi, s);
    } else if (p.kernel == KERNEL_QS) {
        int* gt = reinterpret_cast<int*>(w + p.off_gt);
        uint8_t* qp = w + p.off_qp;
        if ((e = launch_qprep(dt, q, q_scale, b, p.b_pad, row_bytes, fq, gt, qp, p.bq, 4, nullptr, 0, s)) != hipSuccess)
            return e;
        if (ev_start && (e = hipEventRecord(ev_start, s)) != hipSuccess) return e;
        e = launch_qs(p, dt, n, d, emb, fe, qp, fq, gt, b, k, ps, pi, s);
    } else if (p.kernel == KERNEL_QS8) {
        int* gt = reinterpret_cast<int*>(w + p.off_gt);
        uint8_t* qp = w + p.off_qp;
        int* g2 = reinterpret_cast<int*>(w + p.off_g2);
        if ((e = launch_qprep(dt, q, q_scale, b, p.b_pad, row_bytes, fq, gt, qp, p.bq, 8, g2, p.splits, s)) != hipSuccess)
            return e;
        if (ev_start && (e = hipEventRecord(ev_start, s)) != hipSuccess) return e;
        e = launch_qs8(p, dt, n, d, emb, fe, qp, fq, gt, g2, b, k, ps, pi, s);
    } else {
        return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    if (ev_stop && (e = hipEventRecord(ev_stop, s)) != hipSuccess) return e;
    const dim3 grid((unsigned)((b + 3) / 4)), block(256);
    if (p.splits <= 64)
        k_topk_merge<1><<<grid, block, 0, s>>>(ps, pi, p.splits, p.b_pad, k, b, fq, top_score, top_idx);
    else if (p.splits <= 128)
        k_topk_merge<2><<<grid, block, 0, s>>>(ps, pi, p.splits, p.b_pad, k, b, fq, top_score, top_idx);
    else if (p.splits <= 256)
        k_topk_merge<4><<<grid, block, 0, s>>>(ps, pi, p.splits, p.b_pad, k, b, fq, top_score, top_idx);
    else
        k_topk_merge<8><<<grid, block, 0, s>>>(ps, pi, p.splits, p.b_pad, k, b, fq, top_score, top_idx);
    return hipGetLastError();
}

}  // namespace apc
