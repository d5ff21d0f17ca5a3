// Resident-aware fallback and the per-batch level histogram.
//
// k_resident_best: one wavefront per query; lane j looks up the residency of
// neighbour j (j < k) and a ballot picks the first resident one, i.e. the
// best, since the lists are ordered best first.  k_level_histogram: one block;
// the lanes of a wavefront with the same level find each other by a ballot per
// bit of it, and the first adds their count in LDS; of one or two levels each
// wavefront counts its queries with a ballot per level.
#include "apc_internal.h"

namespace apc {
namespace {

constexpr int RB_WAVES = 4;

__global__ __launch_bounds__(RB_WAVES * 64) void k_resident_best(const int32_t* __restrict__ slot_of_entry,
                                                                 int64_t n_entries, int64_t n_slots,
                                                                 const float* __restrict__ top_score,
                                                                 const int32_t* __restrict__ top_idx, int32_t ld,
                                                                 int32_t k, int32_t b, float* __restrict__ out_score,
                                                                 int32_t* __restrict__ out_idx)
{
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * RB_WAVES + (threadIdx.x >> 6);
    if (q >= b) return;                                   // uniform per wavefront
    bool res = false;
    int32_t e = -1;
    float s = 0.f;
    if (lane < k) {
        e = top_idx[q * ld + lane];
        s = top_score[q * ld + lane];
        if (e >= 0 && e < n_entries) {
            const int64_t slot = slot_of_entry ? (int64_t)slot_of_entry[e] : (int64_t)e;
            res = slot >= 0 && slot < n_slots;
        }
    }
    const uint64_t m = __ballot(res);
    const int j = m ? __builtin_ctzll(m) : 0;
    const int32_t ej = __shfl(e, j);
    const float sj = __shfl(s, j);
    if (lane == 0) {
        out_idx[q] = m ? ej : -1;
        out_score[q] = m ? sj : __builtin_nanf("");
    }
}

// values loaded at once by every thread (with one at a time, and a ballot per
// level in place of one per bit of it, 16,384 queries over 11 levels took 15 us,
// and the placement with it 217 us: 210 now).  Where a value has no more levels
// than bits, a ballot per level is less work: 300,000 queries of one level 40 us,
// 61 with one per bit and an atomic for every 64, of two 40 and 78.
constexpr int LH_NT = 1024, LH_U = 8;

__global__ __launch_bounds__(LH_NT) void k_level_histogram(const int32_t* __restrict__ level, int32_t b, int32_t L,
                                                           int32_t* __restrict__ hist)
{
    __shared__ int h[APC_MAX_LEVELS + 1];
    const int tid = threadIdx.x, lane = tid & 63, n = L + 1;
    if (tid <= L) h[tid] = 0;
    __syncthreads();
    const int bits = 32 - __builtin_clz(n);               // of values 0..n - 1, and n: not counted
    const bool few = n <= 2;
    int mine = 0;                                         // few: lane l's count of level l
    for (int base = 0; base < b; base += LH_U * LH_NT) {
        int v[LH_U];
#pragma unroll
        for (int u = 0; u < LH_U; ++u) {
            const int q = base + u * LH_NT + tid;
            v[u] = q < b ? level[q] : n;
        }
#pragma unroll
        for (int u = 0; u < LH_U; ++u) {
            if (base + u * LH_NT >= b) break;             // uniform
            const int x = v[u] < 0 || v[u] > L ? n : v[u];
            if (few) {
                const int c0 = __popcll(__ballot(x == 0)), c1 = __popcll(__ballot(x == 1));
                mine += lane == 0 ? c0 : c1;
                continue;
            }
            uint64_t same = ~0ull;
            for (int i = 0; i < bits; ++i) {
                const uint64_t m = __ballot((x >> i) & 1);
                same &= (x >> i) & 1 ? m : ~m;
            }
            if (x < n && lane == __builtin_ctzll(same)) atomicAdd(&h[x], __popcll(same));
        }
    }
    if (few && lane < n && mine) atomicAdd(&h[lane], mine);
    __syncthreads();
    if (tid <= L) hist[tid] = h[tid];
}

}  // namespace

hipError_t launch_resident_best(const int32_t* slot_of_entry, int64_t n_entries, int64_t n_slots,
                                const float* top_score, const int32_t* top_idx, int32_t ld, int32_t k, int32_t b,
                                float* out_score, int32_t* out_idx, hipStream_t s)
{
    if (b <= 0) return hipSuccess;
    const unsigned grid = (unsigned)((b + RB_WAVES - 1) / RB_WAVES);
    k_resident_best<<<grid, RB_WAVES * 64, 0, s>>>(slot_of_entry, n_entries, n_slots, top_score, top_idx, ld, k,
                                                   b, out_score, out_idx);
    return hipGetLastError();
}

hipError_t launch_level_histogram(const int32_t* level, int32_t b, int32_t L, int32_t* hist, hipStream_t s)
{
    k_level_histogram<<<1, LH_NT, 0, s>>>(level, b, L, hist);
    return hipGetLastError();
}

}  // namespace apc
