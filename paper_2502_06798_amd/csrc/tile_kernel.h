// Tiled similarity + exact top-k for any row width and k up to 64.
//
// Grid: splits x query tiles.  A workgroup of eight wavefronts (two per
// SIMD, so that one's vector work runs beside the other's MFMAs) owns BQ
// queries and a range of cache rows (its split), which it goes through in
// tiles of 256 rows: wavefront (we, wq) holds the scores of ME x MQ blocks of
// 32 rows x 32 queries in registers, and both operands stream through LDS
// rings, loaded straight from global memory and counted by hand (see
// q2_dma16).  Rows come 128 bytes at a time (whole cache lines: 64-byte pieces
// reach 78 GB/s per CU, 128-byte ones 140), queries 64 bytes at a time from a
// copy that the preparation writes in the order of these loads (1 KB each), so
// that the rings are deep enough: rows are loaded at least 2 NE - 3 stages of
// 64 bytes early, queries NQ - 1.  The 16-byte units of a row are swizzled by
// row so that the operand reads are free of bank conflicts.  Neither operand
// has to fit in registers, so any width runs here; 256 x 256 scores read
// 0.75 KB of LDS per 32x32 MFMA, where a wavefront of 32 queries held in
// registers reads 1 KB.  Past a row's end the copy of the queries holds zeros
// (and rows repeat their last unit).  Every score is the float32 sum over all
// of d, in the same order whatever the split or tile.
//
// Top-k.  A workgroup keeps no sorted lists.  It filters every tile against a
// lower bound F of each query's k-th best score, and the pairs that reach F
// go to the (query, split) log in global memory: an LDS counter hands out the
// places, the stores wait for nothing.  F comes from three places:
//  * a split's first tile: its rows fall into 32 or 64 disjoint groups per
//    query, and a value that k groups' maxima reach has k pairs at or above it;
//  * all splits together: the lanes' running maxima (of disjoint rows, 16
//    classes per workgroup) go into k buckets per query by atomic max, after
//    tiles 1, 2, 4, 8, ..; the smallest bucket has k pairs at or above it.
//    A bucket is the largest of its parts (tile_ways), which keep the splits'
//    atomics apart.  It is read during the next tile.  After the first tiles this is close to the
//    k-th best of everything seen by all splits, so almost nothing passes;
//  * a log that is full is cut to its k best, whose smallest is a bound too.
// Any of them may lag: F then only lets more pairs through.  k_tile_merge takes
// the k best of a query's logs.
//
// Measured (whole match, against the tiled and streaming kernels before it,
// which kept sorted lists in LDS and staged both operands through registers):
// 512 x 250,000 x 1,024 f16 1,369 -> 318 us (0.83 PFLOP/s), 64 x 200,000 x 768
// float32 329 -> 225 us, 300 x 5,000 x 640 bf16 218 -> 22 us, 1,024 x 1,000,000
// x 640 e4m3 1.7 PFLOP/s.  What bounds it at 1,024 x 1,000,000 x 640 f16 (1.39
// ms): its MFMAs alone with the barriers take 0.83 ms, the filter adds 0.15,
// the operand reads 0.08, the loads 0.30 (the loads alone take 0.89), logging
// 0.04; neither deeper rings, loads two stages earlier into the L2, loads
// spread between the MFMAs nor wave priorities moved that sum.
#pragma once

#include "qs_kernel.h"
#include "tile.h"

namespace apc {
namespace {

constexpr int TL_NW = 8;                    // wavefronts per workgroup
constexpr int TL_NT = TL_NW * 64;
constexpr int TL_BE = 256;                  // cache rows per tile
constexpr int TL_SB = 64;                   // bytes of d per stage
constexpr int TL_ROWB = 2 * TL_SB;          // bytes of a cache row per load: two stages
constexpr int TL_ESLOT = TL_BE * TL_ROWB;   // bytes of a slot of the rows' ring
constexpr int TL_FR = 4;                    // tiles whose entry factors are in LDS at once

template <int DT> struct TlOp { typedef uint4 Frag; static constexpr int STEPS = 2; };
template <> struct TlOp<APC_E4M3> { typedef i32x8 Frag; static constexpr int STEPS = 1; };

template <int ME, int MQ, int WE, int WQ, int NE_, int NQ_>
struct TlCfg {
    static_assert(WE * WQ == TL_NW && WE * ME * 32 == TL_BE, "eight wavefronts, 256 rows");
    static constexpr int BQ = WQ * MQ * 32;
    static constexpr int NE = NE_, NQ = NQ_;                  // slots of the rings
    static constexpr int QSLOT = BQ * TL_SB;
    static constexpr int ELD = TL_ESLOT / 1024 / TL_NW / 2;   // row loads per wavefront and stage (half a slot's)
    static constexpr int QWB = QSLOT / TL_NW;                 // bytes of queries a wavefront loads per stage
    static constexpr int QLD = QWB >= 1024 ? QWB / 1024 : 1;  // in loads of 1 KB (or one of fewer lanes)
    static constexpr int OPS = ELD + QLD;
    struct Smem {
        uint8_t e[NE * TL_ESLOT];
        uint8_t q[NQ * QSLOT];
        float fe[TL_FR][TL_BE];
        float fq[BQ];
        float f[BQ];                                          // bounds
        int cnt[BQ];                                          // log lengths
        int ovf;                                              // a pair found its log full
        float seed[64 * 33];
    };
    static_assert(sizeof(Smem) <= 160 * 1024, "LDS of a CU");
    static_assert(2 * NE - 2 >= NQ && NQ >= 2, "rows are loaded earlier than queries");
    static_assert(2 * (TL_FR - 2) >= NE - 1, "a tile's factors are loaded with its first rows; tiles have two slots or more");
};

// one unit of d (16 bytes per lane and operand; 32 for e4m3): c += a b
template <int DT>
__device__ inline void tl_mma(f32x16& c, const typename TlOp<DT>::Frag a, const typename TlOp<DT>::Frag b, bool first)
{
    if constexpr (DT == APC_F32) {
        const f32x16 cin = first ? f32x16{} : c;
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), cin, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    } else {
        q2_mma<DT>(c, a, b, first);
    }
}

// value j of a block's sixteen, through a tree of bit selects
__device__ inline float tl_pick(const f32x16& v, int j)
{
    const uint32_t m0 = q2_opaque(0u - (uint32_t)(j & 1)), m1 = q2_opaque(0u - (uint32_t)((j >> 1) & 1));
    const uint32_t m2 = q2_opaque(0u - (uint32_t)((j >> 2) & 1)), m3 = q2_opaque(0u - (uint32_t)((j >> 3) & 1));
    float l8[8], l4[4];
#pragma unroll
    for (int i = 0; i < 8; ++i) l8[i] = q2_bsel(m0, v[2 * i + 1], v[2 * i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) l4[i] = q2_bsel(m1, l8[2 * i + 1], l8[2 * i]);
    return q2_bsel(m3, q2_bsel(m2, l4[3], l4[2]), q2_bsel(m2, l4[1], l4[0]));
}

// sum over the aligned group of TPQ (4 or 8) lanes, in every lane of it
template <int TPQ>
__device__ inline int tl_group_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);                    // lane ^ 1
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);                    // lane ^ 2
    if constexpr (TPQ == 8) v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true);   // mirrored half row
    return v;
}
template <int TPQ>
__device__ inline float tl_group_max(float v)
{
    auto step = [&](auto ctrl) __attribute__((always_inline)) {
        const float o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true));
        v = __builtin_fmaxf(v, o);
    };
    step(std::integral_constant<int, 0xB1>{});
    step(std::integral_constant<int, 0x4E>{});
    if constexpr (TPQ == 8) step(std::integral_constant<int, 0x141>{});
    return v;
}

// q2_dma16 from a wave-uniform base and a per-lane offset.  The base may come
// out of a vector instruction (v_readfirstlane), after which a vector-memory
// instruction must not read the scalar register for five wait states; the
// compiler does not see the load inside the asm, so the asm waits itself.
__device__ inline void tl_dma16(const uint8_t* base, uint32_t off, uint32_t lds)
{
    const uint64_t p = reinterpret_cast<uint64_t>(base);           // into scalar registers, wherever it was computed
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p), hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
    base = reinterpret_cast<const uint8_t*>(((uint64_t)hi << 32) | lo);
    asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "{m0}"(lds) : "memory");
}

template <int DT, int ME, int MQ, int WE, int WQ, int NE, int NQ>
__global__ __launch_bounds__(TL_NT) void k_tile(const TileArgs A)
{
    typedef TlCfg<ME, MQ, WE, WQ, NE, NQ> C;
    typedef typename TlOp<DT>::Frag Frag;
    constexpr int BQ = C::BQ, QSLOT = C::QSLOT;
    __shared__ typename C::Smem sm;
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, r32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), we = wave / WQ, wq = wave % WQ;
    const int64_t n = A.n;
    const int rb = A.rb, k = A.k, splits = A.splits, nst = A.nst, cap = A.cap;

    // workgroup id -> (split, query tile).  Workgroups are dealt round-robin
    // over the 8 XCDs; consecutive ids lin share one, and with it an L2.  They
    // run over the query tiles of a group first, which read the same rows, then
    // over the splits, which read the same queries, then over the groups: a
    // group's queries (A.group tiles) stay in the L2.
    const int grid = (int)gridDim.x, work = splits * A.qtiles;
    const int lin = (grid & 7) == 0 ? (int)(blockIdx.x & 7) * (grid >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    if (lin >= work) return;                                       // whole workgroup: uniform
    const int gi = lin / (A.group * splits), gl = lin - gi * A.group * splits;
    const int gsize = A.qtiles - gi * A.group < A.group ? A.qtiles - gi * A.group : A.group;
    const int split = gl / gsize, qtile = gi * A.group + gl % gsize;
    const int64_t q0 = (int64_t)qtile * BQ;

    // the split's rows: whole blocks of 32, so that splits differ by one block
    const int64_t nblk = (n + 31) / 32;
    const int64_t r0 = nblk * split / splits * 32;
    const int64_t r1 = nblk * (split + 1) / splits * 32 < n ? nblk * (split + 1) / splits * 32 : n;
    const int ntile = (int)((r1 - r0 + TL_BE - 1) / TL_BE);

    // ---- loads of a stage: half a slot of rows, all of the queries' slot.  A
    // row load brings 8 rows x 128 bytes, lane l the unit stored at place
    // l % 8 of row l / 8; rows past the split repeat its last. ----
    const uint32_t lds_e = (uint32_t)(size_t)(lds_void*)sm.e;
    const uint32_t lds_q = (uint32_t)(size_t)(lds_void*)sm.q;
    const uint32_t lds_fe = (uint32_t)(size_t)(lds_void*)&sm.fe[0][0];
    static_assert(C::ELD == 2, "a wavefront's rows: 16 per stage's loads, 32 per slot");
    const int er = wave * 32 + (lane >> 3);                        // this lane's first row; the others are 8 apart
    const int eu = ((lane & 7) ^ ((lane >> 4) & 3)) * 16;          // its byte of the 128 (rows 8 on: ^ 64)
    const uint8_t* ep[4];                                          // its rows of the tile being loaded
    int ct = 0, ej = 0, eslot = 0;                                 // that tile, its slot of d, the ring slot
    const int nd = nst / 2;                                        // slots of rows per tile
    // load i (0 .. 3) of the slot's rows; past the split they repeat its last row
    auto load_rows = [&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        if (i == 0 && ej == 0) {
            const int64_t e0 = r0 + (int64_t)ct * TL_BE;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int64_t row = e0 + er + 8 * x;
                ep[x] = A.emb + (row < r1 ? row : r1 - 1) * rb;
            }
            // the tile's entry factors, 32 per wavefront (one load more than
            // the stage waits count, which only makes them wait longer)
            int64_t f0 = e0 + wave * 32 + lane * 4;
            f0 = f0 < A.fe_len - 4 ? f0 : A.fe_len - 4;
            if (lane < 8) q2_dma16(A.fe + f0, lds_fe + (uint32_t)(((ct & (TL_FR - 1)) * TL_BE + wave * 32) * 4));
        }
        const int k0 = ej * TL_ROWB + (i & 1 ? eu ^ 64 : eu);
        q2_dma16(ep[i] + (k0 < rb - 16 ? k0 : rb - 16), lds_e + (uint32_t)(eslot * TL_ESLOT + (wave * 4 + i) * 1024));
        if (i == 3) {
            if (++ej == nd) { ej = 0; ++ct; }
            if (++eslot == NE) eslot = 0;
        }
    };
    const uint8_t* const qfirst = A.qcopy + (int64_t)qtile * nst * QSLOT + wave * C::QWB;
    const uint8_t* qnext = qfirst;
    int qj = 0, qslot = 0;
    const bool qlane = C::QWB >= 1024 || lane < C::QWB / 16;
    auto load_queries = [&](auto ic) __attribute__((always_inline)) {   // load i (below QLD) of the queries' slot
        constexpr int i = decltype(ic)::value;
        if (qlane) tl_dma16(qnext + i * 1024, lane * 16, lds_q + (uint32_t)(qslot * QSLOT + wave * C::QWB + i * 1024));
        if (i == C::QLD - 1) {
            qnext += QSLOT;
            if (++qj == nst) { qj = 0; qnext = qfirst; }
            if (++qslot == NQ) qslot = 0;
        }
    };
    // Stage v's own loads, issued after stage v is entered: half of the rows'
    // slot v / 2 + NE - 1, the queries' stage v + NQ - 1 (both refill what
    // stage v - 1 and the slot before v / 2 held, which every wavefront has
    // read).  Before stage v is read, its queries, loaded with stage
    // v - NQ + 1, have landed, and with them its older rows.  The loads go on
    // past the split's end (into slots that nothing reads), so that every
    // count is the same.
    auto enter = [&](int v) __attribute__((always_inline)) {
        if (v > 0) __builtin_amdgcn_s_waitcnt(q2_vmcnt((NQ - 2) * C::OPS));
        else __builtin_amdgcn_s_waitcnt(q2_vmcnt(0));
        __syncthreads();
    };
    for (int i = 0; i < NE - 1; ++i) static_for<4>([&](auto ic) __attribute__((always_inline)) { load_rows(ic); });
    for (int i = 0; i < NQ - 1; ++i) static_for<C::QLD>([&](auto ic) __attribute__((always_inline)) { load_queries(ic); });

    // ---- state per query ----
    for (int i = tid; i < BQ; i += TL_NT) {
        sm.fq[i] = q0 + i < A.b ? A.fq[q0 + i] : qnan();
        sm.f[i] = neg_inf();
        sm.cnt[i] = 0;
    }
    if (tid == 0) sm.ovf = 0;
    float rm[MQ][ME];                                              // largest product so far of this lane's rows per block
#pragma unroll
    for (int mq = 0; mq < MQ; ++mq)
#pragma unroll
        for (int mb = 0; mb < ME; ++mb) rm[mq][mb] = neg_inf();
    // Lane numbers for the work after a tile's MFMAs.  They go through an empty
    // asm there, so that what follows from them is computed there and not kept in
    // registers through the MFMAs.  (Tiles of 256 queries still spill a few, 12
    // bytes per lane for e4m3 and 24 for 16-bit rows; the build checks that it
    // stays there.)
    int hl = h, cl = r32;
    auto qloc = [&](int mq) __attribute__((always_inline)) { return wq * (MQ * 32) + mq * 32 + cl; };
    auto log_of = [&](int ql) __attribute__((always_inline)) { return A.log + ((q0 + ql) * splits + split) * cap; };

    // ---- operand reads: lane (h, r32) supplies row r32 of a block; step s of
    // half j of a slot multiplies units 4 h + 2 j + s of its 128 bytes (e4m3:
    // that and the next), which is the order of the other kernels' sums too;
    // a stage of the queries' copy holds unit 4 h + 2 j + s at place 2 h + s ----
    const uint32_t aoff = (uint32_t)((we * ME * 32 + r32) * TL_ROWB + (((4 * h) ^ ((r32 >> 1) & 7)) * 16));
    const uint32_t boff = (uint32_t)((wq * MQ * 32 + r32) * TL_SB + (((2 * h) ^ ((r32 >> 2) & 3)) * 16));
    auto rd16 = [&](const uint8_t* p) __attribute__((always_inline)) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // (a load that is known to be aligned)
        return *reinterpret_cast<const u32x4*>(__builtin_assume_aligned(p, 16));
    };
    auto rd = [&](const uint8_t* ring, uint32_t at) __attribute__((always_inline)) -> Frag {
        if constexpr (DT == APC_E4M3) {
            const auto x0 = rd16(ring + at), x1 = rd16(ring + (at ^ 16u));
            return Frag{(int)x0.x, (int)x0.y, (int)x0.z, (int)x0.w, (int)x1.x, (int)x1.y, (int)x1.z, (int)x1.w};
        } else {
            const auto x = rd16(ring + at);
            return Frag{x.x, x.y, x.z, x.w};
        }
    };

    f32x16 acc[ME][MQ];
    uint32_t mk[MQ][ME];                                           // pairs of a block that are to be logged
    int64_t e0 = r0;                                               // first row of the tile

    // the pairs of this lane marked in mk go to the logs as far as there is
    // room; the others stay marked
    auto append = [&]() __attribute__((always_inline)) {
        bool pend = false;
#pragma unroll
        for (int mq = 0; mq < MQ; ++mq) {
            int total = 0;
#pragma unroll
            for (int mb = 0; mb < ME; ++mb) total += __builtin_popcount(mk[mq][mb]);
            if (!__builtin_amdgcn_ballot_w64(total != 0)) continue;
            const int ql = qloc(mq);
            const float fq = sm.fq[ql];
            const int base = total ? atomicAdd(&sm.cnt[ql], total) : 0;
            int left = base < cap ? cap - base : 0;
            left = left < total ? left : total;
            pend |= left < total;
            uint64_t* p = log_of(ql) + base;
#pragma unroll
            for (int mb = 0; mb < ME; ++mb) {
                while (__builtin_amdgcn_ballot_w64(left > 0 && mk[mq][mb] != 0)) {
                    const bool act = left > 0 && mk[mq][mb] != 0;
                    const int j = act ? __builtin_ctz(mk[mq][mb]) : 0;
                    const float sc = clamp1(tl_pick(acc[mb][mq], j) * fq) + 0.0f;      // -0 becomes +0: equal scores
                    const int e = (int)(e0 + (we * ME + mb) * 32 + 8 * (j >> 2) + 4 * hl + (j & 3));
                    if (act) {
                        *p++ = q2_pack(sc, e);
                        mk[mq][mb] &= mk[mq][mb] - 1;
                        --left;
                    }
                }
            }
        }
        if (pend) sm.ovf = 1;
    };
    // marks (keep: only among the marked) the pairs whose score reaches the
    // query's bound: clamp1(y) >= F exactly when y >= F for -1 < F <= 1; with
    // F <= -1 every row passes (rows past the split hold -inf or NaN)
    auto mark = [&](int mq, int mb, bool pass, float fq, float F, bool keep) __attribute__((always_inline)) {
        const float Fy = F <= -1.f ? -3.402823466e+38f : F;
        uint32_t b = 0;
#pragma unroll
        for (int j = 15; j >= 0; --j) b = q2_shift_in(b, acc[mb][mq][j] * fq >= Fy);
        b = pass ? b : 0u;
        mk[mq][mb] = keep ? mk[mq][mb] & b : b;
    };

    // Logs that were full: every wavefront cuts its share of the long ones to
    // their k best (whose last is a bound), then what is still marked and
    // reaches the new bound is logged; again until everything found a place
    // (each pass makes room for cap - k pairs).  Entered by the whole
    // workgroup after a barrier.
    auto resolve = [&]() __attribute__((always_inline)) {
        while (*(volatile int*)&sm.ovf) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wavefront's log stores
            __syncthreads();
            if (tid == 0) sm.ovf = 0;
            // four logs at a time: their loads go out together
            constexpr int CQ = BQ / TL_NW < 4 ? BQ / TL_NW : 4;
#pragma unroll 1
            for (int q4 = wave * CQ; q4 < BQ; q4 += TL_NW * CQ) {
                uint64_t x0[CQ], x1[CQ];
                int c[CQ];
#pragma unroll
                for (int i = 0; i < CQ; ++i) {
                    const int v = __builtin_amdgcn_readfirstlane(*(volatile int*)&sm.cnt[q4 + i]);
                    c[i] = v <= cap - cap / 4 ? 0 : v < cap ? v : cap;   // at least k of them, or the log stays
                    const uint64_t* lg = log_of(q4 + i);
                    x0[i] = lane < c[i] ? __hip_atomic_load(lg + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
                    x1[i] = lane + 64 < c[i] ? __hip_atomic_load(lg + lane + 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
                }
#pragma unroll
                for (int i = 0; i < CQ; ++i) {
                    if (c[i] == 0) continue;                       // uniform
                    // every pair's rank, by counting the larger keys (keys are unique)
                    int r0 = 0, r1 = 0;
                    auto count = [&](uint64_t x, int m) __attribute__((always_inline)) {
                        for (int j = 0; j < m; ++j) {
                            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, j);
                            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), j);
                            const uint64_t t = ((uint64_t)hi << 32) | lo;
                            r0 += t > x0[i];
                            r1 += t > x1[i];
                        }
                    };
                    count(x0[i], c[i] < 64 ? c[i] : 64);
                    count(x1[i], c[i] - 64);
                    uint64_t* lg = log_of(q4 + i);
                    const bool in0 = lane < c[i] && r0 < k, in1 = lane + 64 < c[i] && r1 < k;
                    if (in0) lg[r0] = x0[i];
                    if (in1) lg[r1] = x1[i];
                    if ((in0 && r0 == k - 1) || (in1 && r1 == k - 1)) {
                        const float F = q2_key_score(in0 && r0 == k - 1 ? x0[i] : x1[i]);
                        sm.cnt[q4 + i] = k;
                        sm.f[q4 + i] = __builtin_fmaxf(sm.f[q4 + i], F);
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int mq = 0; mq < MQ; ++mq) {
                const int ql = qloc(mq);
                const float F = *(volatile float*)&sm.f[ql], fq = sm.fq[ql];
#pragma unroll
                for (int mb = 0; mb < ME; ++mb)
                    if (__builtin_amdgcn_ballot_w64(mk[mq][mb] != 0)) mark(mq, mb, true, fq, F, true);
            }
            append();
            __syncthreads();
        }
    };

    // ---- the tiles ----
#pragma unroll
    for (int mq = 0; mq < MQ; ++mq)
#pragma unroll
        for (int mb = 0; mb < ME; ++mb) mk[mq][mb] = 0;
    int u = 0, aslot = 0, bslot = 0;                               // stage being computed and its slots
    for (int it = 0; it < ntile; ++it) {
        enter(u);
        load_rows(std::integral_constant<int, 0>{});
        load_rows(std::integral_constant<int, 1>{});
        if (it > 0) resolve();                                     // uniform: the flag was set before the barrier
        e0 = r0 + (int64_t)it * TL_BE;

        constexpr int ST = TlOp<DT>::STEPS;                        // steps of a stage
        Frag a0[ME], b0[MQ], a1[ME], b1[MQ];
        auto read_b = [&](int sl, int s, Frag (&b)[MQ]) __attribute__((always_inline)) {
            const uint32_t base = (uint32_t)sl * QSLOT + (boff ^ (uint32_t)(s * 16));
#pragma unroll
            for (int mq = 0; mq < MQ; ++mq) b[mq] = rd(sm.q, base + mq * 32 * TL_SB);
        };
        // half: the even or odd stage of the slot
        auto a_at = [&](int sl, int half, int s) __attribute__((always_inline)) {
            return (uint32_t)sl * TL_ESLOT + (aoff ^ (uint32_t)(half * 32 + s * 16));
        };
        auto read_a = [&](int sl, int half, int s, Frag (&a)[ME]) __attribute__((always_inline)) {
            const uint32_t base = a_at(sl, half, s);
#pragma unroll
            for (int mb = 0; mb < ME; ++mb) a[mb] = rd(sm.e, base + mb * 32 * TL_ROWB);
        };
        // blocks with rows of the split in this tile.  A split's last tile is
        // rarely whole; float32 MFMAs bound their kernel, so those of empty
        // blocks are left out (their scores are masked below): 64 queries x
        // 200,000 rows of 768 are 3.05 tiles per split instead of 4
        const int blocks = (int)(r1 - e0 < TL_BE ? r1 - e0 : TL_BE) - we * ME * 32 + 31;
        auto mma_row = [&](int mb, const Frag& a, const Frag (&b)[MQ], bool first) __attribute__((always_inline)) {
            if (DT == APC_F32 && blocks < 32 * (mb + 1)) return;   // uniform
#pragma unroll
            for (int mq = 0; mq < MQ; ++mq) tl_mma<DT>(acc[mb][mq], a, b[mq], first);
        };
        // a step's MFMAs, with a load after some of its rows of blocks: all of
        // a workgroup's loads in one burst would hold up every wavefront's
        // MFMAs.  LOADS: 0 the stage's queries, 1 + half its rows, -1 none
        auto mma_step = [&](auto lc, const Frag (&a)[ME], const Frag (&b)[MQ], bool first) __attribute__((always_inline)) {
            constexpr int LOADS = decltype(lc)::value, NL = LOADS < 0 ? 0 : LOADS == 0 ? C::QLD : 2;
            static_for<ME>([&](auto mc) __attribute__((always_inline)) {
                constexpr int mb = decltype(mc)::value;
                mma_row(mb, a[mb], b, first);
                static_for<NL>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (i * ME / NL == mb) {
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (LOADS == 0) load_queries(ic);
                        else load_rows(std::integral_constant<int, (LOADS - 1) * 2 + i>{});
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
            });
        };
        // One stage (half hc of its slot): the operands of its step 0 are in
        // a0, b0.  The next stage is entered (ahead) before this one's last
        // MFMAs, which cover the reads of its first operands; its row loads go
        // out between them, its query loads between its own first MFMAs.
        auto stage = [&](auto hc, auto fc, auto ac) __attribute__((always_inline)) {
            constexpr int half = decltype(hc)::value;
            constexpr bool first = decltype(fc)::value, ahead = decltype(ac)::value;
            const int nb = bslot + 1 == NQ ? 0 : bslot + 1;
            const int na = half == 0 ? aslot : aslot + 1 == NE ? 0 : aslot + 1;
            using QL = std::integral_constant<int, 0>;
            using RL = std::integral_constant<int, ahead ? 1 + (half ^ 1) : -1>;
            if constexpr (ST == 2) {
                read_b(bslot, 1, b1);
                read_a(aslot, half, 1, a1);
                mma_step(QL{}, a0, b0, first);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (ahead) {
                    enter(u + 1);
                    read_b(nb, 0, b0);
                    read_a(na, half ^ 1, 0, a0);
                }
                mma_step(RL{}, a1, b1, false);
                __builtin_amdgcn_sched_barrier(0);
            } else {
                // e4m3 operands are twice as wide: a block's next rows replace
                // its current ones as soon as its MFMAs have gone out
                static_for<C::QLD>([&](auto ic) __attribute__((always_inline)) { load_queries(ic); });
                if constexpr (ahead) {
                    enter(u + 1);
                    read_b(nb, 0, b1);
                }
                static_for<ME>([&](auto mc) __attribute__((always_inline)) {
                    constexpr int mb = decltype(mc)::value;
                    mma_row(mb, a0[mb], b0, first);
                    if constexpr (ahead) {
                        a0[mb] = rd(sm.e, a_at(na, half ^ 1, 0) + mb * 32 * TL_ROWB);
                        if constexpr (mb * 2 % ME == 0 && ME >= 2) load_rows(std::integral_constant<int, (half ^ 1) * 2 + mb * 2 / ME>{});
                        if constexpr (ME == 1) {
                            load_rows(std::integral_constant<int, (half ^ 1) * 2>{});
                            load_rows(std::integral_constant<int, (half ^ 1) * 2 + 1>{});
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (ahead) {
#pragma unroll
                    for (int mq = 0; mq < MQ; ++mq) b0[mq] = b1[mq];
                }
            }
            ++u;
            bslot = nb;
            aslot = na;
        };
        using Y = std::true_type;
        using N = std::false_type;
        // the shared buckets are read one tile after the lanes' maxima went
        // there, half way through (the maxima have arrived by then; the
        // barriers that follow make the bounds visible before the filter)
        const bool fresh = A.buckets && it > 0 && (it & (it - 1)) == 0;
        auto refresh = [&]() __attribute__((always_inline)) {
            constexpr int RU = BQ == 256 ? 4 : 8;                  // loads that go out together
            const int parts = k * A.ways;
            for (int ql = tid; ql < BQ; ql += TL_NT) {
                int mn = 0x7fffffff, mx = (int)0x80000000;
                for (int j0 = 0; j0 < parts; j0 += RU) {
                    int v[RU];
#pragma unroll
                    for (int i = 0; i < RU; ++i)
                        v[i] = __hip_atomic_load(A.bucket + (int64_t)(j0 + i < parts ? j0 + i : parts - 1) * A.b_pad + q0 + ql,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int i = 0; i < RU; ++i) {
                        mx = v[i] > mx ? v[i] : mx;
                        if (((j0 + i + 1) & (A.ways - 1)) == 0) {  // uniform: a bucket's last part
                            if (j0 + i < parts) mn = mx < mn ? mx : mn;
                            mx = (int)0x80000000;
                        }
                    }
                }
                const float F = q2_unkey(mn);
                if (F > sm.f[ql]) sm.f[ql] = F;
            }
        };
        using E = std::integral_constant<int, 0>;                  // even and odd stages
        using O = std::integral_constant<int, 1>;
        read_b(bslot, 0, b0);
        read_a(aslot, 0, 0, a0);
        stage(E{}, Y{}, Y{});                                      // nd >= 2
        stage(O{}, N{}, Y{});
#pragma unroll 1
        for (int j = 1; j < nd - 1; ++j) {
            if (fresh && j == nd / 2) refresh();
            stage(E{}, N{}, Y{});
            stage(O{}, N{}, Y{});
        }
        if (fresh && nd == 2) refresh();
        stage(E{}, N{}, Y{});
        stage(O{}, N{}, N{});

        // ---- filter: products times entry factors, the blocks' maxima ----
        // lane (h, c) holds, of block (mb, mq), query c and rows 8 g + 4 h + i (g, i < 4)
        asm volatile("" : "+v"(hl), "+v"(cl));
        const float* fr = sm.fe[it & (TL_FR - 1)] + we * ME * 32 + 4 * hl;
        float m[MQ][ME];
        const int lim = (int)(r1 - e0 < TL_BE ? r1 - e0 : TL_BE) - we * ME * 32 - 4 * hl;   // rows below it are the split's
        const bool part = r1 - e0 < TL_BE;
#pragma unroll
        for (int mb = 0; mb < ME; ++mb) {
            float4 f4[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) f4[g] = *reinterpret_cast<const float4*>(fr + mb * 32 + 8 * g);
#pragma unroll
            for (int mq = 0; mq < MQ; ++mq) {
                float x = neg_inf();
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const float4 f = f4[j >> 2];
                    const float v = acc[mb][mq][j] * ((j & 3) == 0 ? f.x : (j & 3) == 1 ? f.y : (j & 3) == 2 ? f.z : f.w);
                    acc[mb][mq][j] = v;
                }
                if (part) {                                        // uniform
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if (mb * 32 + 8 * (j >> 2) + (j & 3) >= lim) acc[mb][mq][j] = neg_inf();
                }
#pragma unroll
                for (int j = 0; j < 16; ++j) x = __builtin_fmaxf(x, acc[mb][mq][j]);
                m[mq][mb] = x;
                rm[mq][mb] = __builtin_fmaxf(rm[mq][mb], x);
            }
        }

        // ---- the first tile's bound: the rows of a query in NG groups ----
        if (it == 0 && k <= 48) {                                  // uniform
            auto seed = [&](auto ngc) __attribute__((always_inline)) {
                constexpr int NG = decltype(ngc)::value;           // 32: half-quads pairs of four rows; 64: four rows
                constexpr int GPB = NG / 16;                       // groups per lane and block
                constexpr int QR = 2048 / NG < BQ ? 2048 / NG : BQ;   // queries per round
                constexpr int TPQ = NG / 8;                        // threads per query, eight groups each
                constexpr int LD = QR + 1;
#pragma unroll 1
                for (int q1 = 0; q1 < BQ; q1 += QR) {
#pragma unroll
                    for (int mq = 0; mq < MQ; ++mq) {
                        const int ql = qloc(mq) - q1;
                        if (ql >= 0 && ql < QR) {
#pragma unroll
                            for (int mb = 0; mb < ME; ++mb)
#pragma unroll
                                for (int g = 0; g < GPB; ++g) {
                                    float x = neg_inf();
#pragma unroll
                                    for (int j = 0; j < 16 / GPB; ++j) x = __builtin_fmaxf(x, acc[mb][mq][g * (16 / GPB) + j]);
                                    sm.seed[(((we * ME + mb) * 2 + hl) * GPB + g) * LD + ql] = x;
                                }
                        }
                    }
                    __syncthreads();
                    if (tid < QR * TPQ) {
                        const int ql = tid / TPQ, p = tid % TPQ;
                        float v[8], hi = neg_inf(), lo = neg_inf();   // lo: minus the smallest finite value
                        int real = 0;
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            v[i] = sm.seed[(p * 8 + i) * LD + ql];
                            hi = __builtin_fmaxf(hi, v[i]);
                            if (v[i] > neg_inf()) {
                                ++real;
                                lo = __builtin_fmaxf(lo, -v[i]);
                            }
                        }
                        hi = tl_group_max<TPQ>(hi);
                        lo = -tl_group_max<TPQ>(lo);
                        if (tl_group_sum<TPQ>(real) >= k) {
                            // at least k groups reach lo, always
#pragma unroll 1
                            for (int s = 0; s < 12; ++s) {
                                const float mid = 0.5f * (lo + hi);
                                int c = 0;
#pragma unroll
                                for (int i = 0; i < 8; ++i) c += v[i] >= mid;
                                if (tl_group_sum<TPQ>(c) >= k) lo = mid;
                                else hi = mid;
                            }
                            const float F = clamp1(lo * sm.fq[q1 + ql]);
                            if (p == 0 && F > neg_inf()) sm.f[q1 + ql] = F;      // NaN factor: no bound
                        }
                    }
                    __syncthreads();
                }
            };
            if (k <= 16) seed(std::integral_constant<int, 32>{});
            else seed(std::integral_constant<int, 64>{});
        }

        // ---- the pairs that reach the bound ----
        bool any = false;
#pragma unroll
        for (int mq = 0; mq < MQ; ++mq) {
            const int ql = qloc(mq);
            const float F = *(volatile float*)&sm.f[ql], fq = sm.fq[ql];
#pragma unroll
            for (int mb = 0; mb < ME; ++mb) {
                const bool pass = fq == fq && m[mq][mb] > neg_inf() && clamp1(m[mq][mb] * fq) >= F;
                mk[mq][mb] = 0;
                if (__builtin_amdgcn_ballot_w64(pass)) {
                    mark(mq, mb, pass, fq, F, false);
                    any = true;
                }
            }
        }
        if (any) append();

        // ---- the bound shared by all splits ----
        // (a maximum that is not above this workgroup's bound cannot raise the
        // smallest bucket above it; without this, 256 splits x 16 maxima of a query
        // met in one bucket for k = 1: 64 x 28,549 x 1,024 f16 took 109 us,
        // 39 now)
        if (A.buckets && (it & (it + 1)) == 0) {                   // after tiles 1, 2, 4, 8, ..
#pragma unroll
            for (int mq = 0; mq < MQ; ++mq) {
                const int ql = qloc(mq);
                const float F = *(volatile float*)&sm.f[ql], fq = sm.fq[ql];
#pragma unroll
                for (int mb = 0; mb < ME; ++mb) {
                    // (a query with a NaN factor logs nothing, whatever its bound)
                    if (rm[mq][mb] > neg_inf() && clamp1(rm[mq][mb] * fq) > F) {
                        const int c = split * TL_CLASSES + (we * ME + mb) * 2 + hl, g = c / k;
                        const int part = (c - g * k) * A.ways + (g & (A.ways - 1));
                        __hip_atomic_fetch_max(A.bucket + (int64_t)part * A.b_pad + q0 + ql, q2_key(clamp1(rm[mq][mb] * fq)),
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // the loads past the split
    __syncthreads();
    resolve();
    for (int i = tid; i < BQ; i += TL_NT) A.cnt[(q0 + i) * splits + split] = sm.cnt[i];
}

template <int DT, int ME, int MQ, int WE, int WQ, int NE, int NQ>
hipError_t run_tile(const TileArgs& a, hipStream_t s)
{
    const int work = a.splits * a.qtiles;
    const int grid = work >= 8 ? (work + 7) / 8 * 8 : work;
    k_tile<DT, ME, MQ, WE, WQ, NE, NQ><<<grid, TL_NT, 0, s>>>(a);
    return hipGetLastError();
}

// query tiles of 256, 128, 64 or 32
template <int DT>
hipError_t tile_dispatch(int bq, const TileArgs& a, hipStream_t s)
{
    switch (bq) {
    case 256: return run_tile<DT, 4, 2, 2, 4, 3, 3>(a, s);
    case 128: return run_tile<DT, 2, 2, 4, 2, 3, 4>(a, s);
    case 64: return run_tile<DT, 1, 2, 8, 1, 4, 4>(a, s);
    case 32: return run_tile<DT, 1, 1, 8, 1, 4, 4>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace apc
