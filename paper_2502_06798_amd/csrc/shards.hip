// Merge of the top-k lists of row shards of a cache (the step after the
// exchange of partial lists when the cache is split over devices): one
// wavefront per query.
//
// The lists sit in registers, 64 / P of them side by side (P lanes each, P the
// power of two that holds a list and k), and are merged register by register:
// the larger of a[i] and b[P - 1 - i] are the P largest of two sorted lists, a
// bitonic sequence that log2 P compare-exchanges sort; at the end the lists of
// a register are merged the same way.  All loads of a query go out at once and
// the chain is (g P / 64 + log2(64 / P)) log2 2P exchanges, where taking the
// largest head k times over made k dependent rounds (16,384 queries, 8 shards,
// k = 32: 61 us before, 29 now, the latency of the chain: its LDS permutes, two
// per exchange, take about 7 us of the LDS's time and its vector instructions 9
// of the SIMDs').  Where a list is not strictly falling (a
// non-candidate before a candidate, the same entry twice), a score is -0, or
// two shards hold the same entry, the wavefront takes the heads one by one:
// lane s owns the head of shard s's list, each round takes the wavefront
// maximum of the heads' keys, (score desc, global entry asc) packed into 64
// bits, and the owning lane advances.  Few entries out of many registers take
// fewer rounds than exchanges: they go to the heads at once (merge_by_heads).
#include "apc_internal.h"

namespace apc {
namespace {

constexpr int MS_WAVES = 4;

// order-preserving key; 0 is below every candidate (an empty head)
__device__ inline uint64_t shard_key(float s, int32_t e)
{
    const uint32_t u = __float_as_uint(s + 0.0f);            // -0 -> +0: equal scores
    const uint32_t o = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((uint64_t)o << 32) | (uint32_t)~(uint32_t)e;
}

// max with the key of the lane a DPP control names (own key where it names
// none or the row is masked off)
template <int CTRL, int ROWS>
__device__ inline uint64_t dpp_max(uint64_t v)
{
    const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
    const uint64_t o = ((uint64_t)(uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false) << 32) |
                       (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
    return o > v ? o : v;
}

// largest key of the wavefront: within quads, half rows and rows by
// permutes and mirrors, then across rows by the broadcasts of lanes 15 and
// 31; lane 63 ends with the maximum, read back as a scalar
__device__ inline uint64_t wave_max_u64(uint64_t v)
{
    v = dpp_max<0xB1, 0xf>(v);       // quad_perm [1, 0, 3, 2]
    v = dpp_max<0x4E, 0xf>(v);       // quad_perm [2, 3, 0, 1]
    v = dpp_max<0x141, 0xf>(v);      // row_half_mirror
    v = dpp_max<0x140, 0xf>(v);      // row_mirror
    v = dpp_max<0x142, 0xa>(v);      // row_bcast:15 into rows 1 and 3
    v = dpp_max<0x143, 0xc>(v);      // row_bcast:31 into rows 2 and 3
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

// query q's heads, one by one
__device__ void merge_heads(const float* __restrict__ sc, const int32_t* __restrict__ ix, int32_t g, int32_t b,
                            int32_t kin, const ShardOffsets& off, int32_t k, int64_t q, int lane,
                            float* __restrict__ out_s, int32_t* __restrict__ out_i)
{
    const int64_t base = ((int64_t)lane * b + q) * kin;       // shard `lane`'s list of query q
    const int32_t o = lane < g ? off.v[lane] : 0;
    int head = 0;
    float hs = 0.f;
    int32_t he = 0;
    uint64_t key = 0;
    auto load = [&]() {
        key = 0;
        while (lane < g && head < kin) {                      // skip non-candidates
            hs = sc[base + head];
            const int32_t e = ix[base + head];
            // the global entry number, in 64 bits: one that does not fit below
            // 2^31 - 1 (the largest cache a handle takes) is not a candidate
            const int64_t ge = (int64_t)e + o;
            if (e >= 0 && hs == hs && ge < INT32_MAX) {
                he = (int32_t)ge;
                key = shard_key(hs, he);
                break;
            }
            ++head;
        }
    };
    load();
    for (int p = 0; p < k; ++p) {
        const uint64_t m = wave_max_u64(key);
        const bool mine = m != 0 && key == m;
        const uint64_t who = __ballot(mine);
        const int wl = who ? __builtin_ctzll(who) : 0;
        const float ws = __shfl(hs, wl);
        const int32_t we = __shfl(he, wl);
        if (lane == 0) {
            out_s[q * k + p] = who ? ws : __builtin_nanf("");
            out_i[q * k + p] = who ? we : -1;
        }
        if (mine) {
            ++head;
            load();
        }
    }
}

__device__ inline uint64_t xor_lane(uint64_t v, int m)
{
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, m, 64);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), m, 64);
    return ((uint64_t)hi << 32) | lo;
}

// the key of the lane before (lane 0: its own)
__device__ inline uint64_t lane_before(uint64_t v, int lane)
{
    const int from = lane > 0 ? lane - 1 : 0;
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, from, 64);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), from, 64);
    return ((uint64_t)hi << 32) | lo;
}
__device__ inline uint64_t max_key(uint64_t a, uint64_t b) { return a > b ? a : b; }

// a: the larger keys of a bitonic sequence per P lanes, sorted descending
template <int P>
__device__ inline uint64_t clean(uint64_t a, int lane)
{
#pragma unroll
    for (int m = P / 2; m >= 1; m >>= 1) {
        const uint64_t o = xor_lane(a, m);
        const bool low = (lane & m) != 0;                     // keeps the smaller
        a = (o > a) != low ? o : a;
    }
    return a;
}

template <int P>
__global__ __launch_bounds__(MS_WAVES * 64) void k_merge_shards(const float* __restrict__ sc,
                                                                const int32_t* __restrict__ ix, int32_t g,
                                                                int32_t b, int32_t kin, const ShardOffsets off,
                                                                int32_t k, float* __restrict__ out_s,
                                                                int32_t* __restrict__ out_i)
{
    constexpr int LPR = 64 / P, U = 4;                        // lists per register, registers loaded at once
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * MS_WAVES + (threadIdx.x >> 6);
    if (q >= b) return;                                       // uniform per wavefront
    const int pos = lane % P, seg = lane / P;
    uint64_t acc = 0;
    bool odd = false;                                         // something only the heads' merge handles
    for (int s0 = 0; s0 < g; s0 += U * LPR) {
        float s[U];
        int32_t e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int sh = s0 + u * LPR + seg;
            s[u] = 0.f;
            e[u] = -1;
            if (sh < g && pos < kin) {
                const int64_t at = ((int64_t)sh * b + q) * kin + pos;
                s[u] = sc[at];
                e[u] = ix[at];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + u * LPR >= g) break;                     // uniform
            const int sh = s0 + u * LPR + seg;
            uint64_t key = 0;
            const int64_t ge = (int64_t)e[u] + (sh < g ? off.v[sh] : 0);
            // (as in merge_heads: an entry number that does not fit is not a candidate)
            if (e[u] >= 0 && s[u] == s[u] && ge < INT32_MAX) {
                key = shard_key(s[u], (int32_t)ge);
                odd |= __float_as_uint(s[u]) == 0x80000000u;
            }
            const uint64_t up = lane_before(key, lane);
            odd |= pos > 0 && key != 0 && up <= key;
            acc = s0 + u == 0 ? key : clean<P>(max_key(acc, xor_lane(key, P - 1)), lane);
        }
    }
#pragma unroll
    for (int m = P; m < 64; m *= 2) {                         // the register's lists
        const uint64_t o = xor_lane(acc, m + P - 1);
        acc = clean<P>(max_key(acc, o), lane);
    }
    const uint64_t up = lane_before(acc, lane);
    odd |= pos > 0 && acc != 0 && up == acc;                  // one entry from two shards
    if (__ballot(odd)) {
        merge_heads(sc, ix, g, b, kin, off, k, q, lane, out_s, out_i);
        return;
    }
    if (lane < k) {
        const uint32_t o = (uint32_t)(acc >> 32);
        out_s[q * k + lane] = acc ? __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o) : __builtin_nanf("");
        out_i[q * k + lane] = acc ? (int32_t)~(uint32_t)acc : -1;
    }
}

__global__ __launch_bounds__(MS_WAVES * 64) void k_merge_heads(const float* __restrict__ sc,
                                                               const int32_t* __restrict__ ix, int32_t g,
                                                               int32_t b, int32_t kin, const ShardOffsets off,
                                                               int32_t k, float* __restrict__ out_s,
                                                               int32_t* __restrict__ out_i)
{
    const int64_t q = (int64_t)blockIdx.x * MS_WAVES + (threadIdx.x >> 6);
    if (q >= b) return;                                       // uniform per wavefront
    merge_heads(sc, ix, g, b, kin, off, k, q, threadIdx.x & 63, out_s, out_i);
}

// lanes per list in the registers' merge
int list_lanes(int32_t kin, int32_t k)
{
    const int most = kin > k ? kin : k;
    return most <= 8 ? 8 : most <= 16 ? 16 : most <= 32 ? 32 : 64;
}

}  // namespace

// A round of the heads' merge takes as long as about six exchanges (four where a
// list fills the wavefront: its registers also load the most lanes that hold
// nothing).  Heads and registers in us: 64 shards of 1,024 queries, k = 10, 7.2
// and 9.7; 16,384 queries, k = 1, 64 shards 13.4 and 24.2, two 4.8 and 7.4; 64
// shards of 1,024, k = 48, 26 and 56; on the other side of the line 32 shards of
// 1,024, k = 24, 14.2 and 10.2; 16,384 queries, two shards, k = 10, 21.4 and 6.5.
bool merge_by_heads(int32_t g, int32_t kin, int32_t k)
{
    const int P = list_lanes(kin, k), regs = (g * P + 63) / 64;
    const int log = __builtin_ctz(P);
    const int exchanges = (regs - 1 + 6 - log) * (log + 1);
    return exchanges + 6 > (P == 64 ? 4 : 6) * k;
}

hipError_t launch_merge_shards(const float* scores, const int32_t* idx, int32_t g, int32_t b, int32_t kin,
                               const ShardOffsets& off, int32_t k, float* out_s, int32_t* out_i, hipStream_t s)
{
    if (b <= 0) return hipSuccess;
    const unsigned grid = (unsigned)((b + MS_WAVES - 1) / MS_WAVES);
#define APC_MS(KERNEL) KERNEL<<<grid, MS_WAVES * 64, 0, s>>>(scores, idx, g, b, kin, off, k, out_s, out_i)
    if (merge_by_heads(g, kin, k)) APC_MS(k_merge_heads);
    else
        switch (list_lanes(kin, k)) {
        case 8: APC_MS(k_merge_shards<8>); break;
        case 16: APC_MS(k_merge_shards<16>); break;
        case 32: APC_MS(k_merge_shards<32>); break;
        default: APC_MS(k_merge_shards<64>);
        }
#undef APC_MS
    return hipGetLastError();
}

}  // namespace apc
