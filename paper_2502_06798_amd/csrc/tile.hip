// Around the tiled similarity kernel: the batch's preparation, the merge of
// the logs, the plan (query tiles, splits, log lengths) and the launches.
#include "tile.h"

#include "qs_common.h"

namespace apc {
namespace {

constexpr int TM_NT = 256;
constexpr int TM_BUF = 768;                 // candidates held while a query's logs are read
constexpr int TM_UNROLL = 8;

__device__ inline int tm_key(float f)
{
    const int i = __float_as_int(f);
    return i >= 0 ? i : i ^ 0x7fffffff;
}

// Query factors f = 1/|q| (NaN for rows that cannot be matched: non-finite,
// zero norm, bad e4m3 scale, padding) and the copy of the queries in the load
// order of the similarity kernel, one wavefront per padded query row; the
// shared buckets reset to -inf.
template <int DT>
__global__ __launch_bounds__(256) void k_tile_prep(const uint8_t* __restrict__ qry, const float* __restrict__ q_scale,
                                                    int32_t b, int64_t b_pad, int64_t row_bytes, int bq, int nst,
                                                    float* __restrict__ fq, uint8_t* __restrict__ qcopy,
                                                    int* __restrict__ bucket, int64_t n_bucket)
{
    const int lane = threadIdx.x & 63;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n_bucket; i += (int64_t)gridDim.x * 256)
        bucket[i] = tm_key(neg_inf());
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= b_pad) return;
    const int64_t tile = r / bq;
    const int local = (int)(r - tile * bq);
    uint8_t* to = qcopy + (tile * nst * bq + local) * 64;
    float ss = 0.f;
    bool bad = false;
    const uint8_t* row = qry + r * row_bytes;
    for (int64_t u = lane; u < (int64_t)nst * 4; u += 64) {        // 16-byte units
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (r < b && u * 16 < row_bytes) {
            v = *reinterpret_cast<const uint4*>(row + u * 16);
            sumsq16<DT>(v, ss, bad);
        }
        const int64_t stage = (u >> 3) * 2 + ((u >> 1) & 1);
        const int place = (int)(((u >> 2) & 1) * 2 + (u & 1));
        *reinterpret_cast<uint4*>(to + stage * bq * 64 + ((place ^ ((local >> 2) & 3)) * 16)) = v;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m, 64);
    bad = __any(bad);
    if (lane != 0) return;
    bool ok = r < b && !bad && __builtin_isfinite(ss) && ss > 0.f;
    if (ok && q_scale) {
        const float sc = q_scale[r];
        ok = __builtin_isfinite(sc) && sc > 0.f;
    }
    fq[r] = ok ? 1.0f / __builtin_sqrtf(ss) : qnan();
}

// The k best of a query's logs, one workgroup per query: the pairs that reach
// the shared bound collect in LDS; when they are many, and at the end, every
// pair finds its rank by counting the larger keys (keys are unique), the k
// best keep their places and their last becomes the bound.
__global__ __launch_bounds__(TM_NT) void k_tile_merge(const uint64_t* __restrict__ log, const int32_t* __restrict__ cnt,
                                                      const int* __restrict__ bucket, int ways, int64_t b_pad,
                                                      int splits, int cap, int32_t k, const float* __restrict__ fq,
                                                      float* __restrict__ top_s, int32_t* __restrict__ top_i)
{
    __shared__ uint64_t buf[2][TM_BUF];
    __shared__ int m;                                     // pairs in the current buffer
    __shared__ int bound, most;
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t q = blockIdx.x;
    if (!(fq[q] == fq[q])) {                              // invalid query row
        for (int p = tid; p < k; p += TM_NT) {
            top_s[q * k + p] = qnan();
            top_i[q * k + p] = -1;
        }
        return;
    }
    if (tid == 0) {
        m = 0;
        bound = 0x7fffffff;
    }
    __syncthreads();
    uint64_t least = 1;                                   // smallest key of interest
    if (ways) {                                           // 0: no buckets
        if (tid < 64) {                                   // k ways <= 64: a bucket's parts in neighbouring lanes
            int v = tid < k * ways ? bucket[(int64_t)tid * b_pad + q] : 0x7fffffff;
            for (int w = 1; w < ways; w *= 2) {
                const int o = __shfl_xor(v, w, 64);
                v = o > v ? o : v;
            }
            if (tid < k * ways) atomicMin(&bound, v);
        }
        __syncthreads();
        const int i = bound;
        const uint32_t u = (uint32_t)(i >= 0 ? i : i ^ 0x7fffffff);
        const uint32_t o = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
        least = (uint64_t)o << 32;
    }
    int cur = 0;
    auto cut = [&]() {                                    // after a barrier: the k best of buf[cur] into the other
        const int c = m;
        for (int t = tid; t < c; t += TM_NT) {
            const uint64_t x = buf[cur][t];
            int rank = 0;
            for (int j = 0; j < c; ++j) rank += buf[cur][j] > x;
            if (rank < k) buf[cur ^ 1][rank] = x;
        }
        __syncthreads();
        cur ^= 1;
        if (c >= k) least = buf[cur][k - 1] > least ? buf[cur][k - 1] : least;
        if (tid == 0) m = c < k ? c : k;
        __syncthreads();
    };
    // (at most a thread per log.)  Thread t reads the places t / splits,
    // t / splits + per, .. of log t % splits (a log's entries are few: each thread's
    // loads go out together)
    const int per = TM_NT / splits, sp = tid % splits, sub = tid / splits;
    const bool mine = sub < per;
    const int c = mine ? cnt[q * splits + sp] : 0;
    const uint64_t* lg = log + (q * splits + sp) * cap;
    if (tid == 0) most = 0;
    __syncthreads();
    if (mine && sub == 0) atomicMax(&most, c);
    __syncthreads();
    const int end = most;
    for (int p0 = 0; p0 < end; p0 += TM_UNROLL * per) {
        uint64_t v[TM_UNROLL];
#pragma unroll
        for (int i = 0; i < TM_UNROLL; ++i) {
            const int at = p0 + i * per + sub;
            v[i] = at < c ? lg[at] : 0;
        }
#pragma unroll
        for (int i = 0; i < TM_UNROLL; ++i) {
            const bool in = v[i] >= least;
            const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
            if (mask) {
                int at = 0;
                if (lane == 0) at = atomicAdd(&m, __builtin_popcountll(mask));
                at = __builtin_amdgcn_readfirstlane(at);
                if (in) buf[cur][at + __builtin_popcountll(mask & ((1ull << lane) - 1ull))] = v[i];
            }
            if (i % 2 == 1) {                             // room for two more batches after every cut
                __syncthreads();
                const bool full = m > TM_BUF - 2 * TM_NT;
                __syncthreads();
                if (full) cut();
            }
        }
    }
    __syncthreads();
    cut();
    for (int p = tid; p < k; p += TM_NT) {
        const uint64_t x = p < m ? buf[cur][p] : 0;
        const uint32_t o = (uint32_t)(x >> 32);
        top_s[q * k + p] = x ? __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o) : neg_inf();
        top_i[q * k + p] = x ? (int)~(uint32_t)x : -1;
    }
}

}  // namespace

// A split's first tile logs about 12 pairs for k = 10, 21 for 16, 41 for 32
// and 75 for 48; a log that fills costs its workgroup a pass over all its logs
// (tens of us).  256 workgroups of 256 queries with logs of 48, or of 128 with
// 96, take 25 MB.
int tile_log_cap(int32_t k) { return k <= 16 ? 48 : 96; }

hipError_t launch_tile_prep(int dt, const void* q, const float* q_scale, int32_t b, int64_t row_bytes, int bq,
                            const TileArgs& a, float* fq, uint8_t* qcopy, hipStream_t s)
{
    const dim3 grid((unsigned)((a.b_pad + 3) / 4)), block(256);
    const uint8_t* qp = static_cast<const uint8_t*>(q);
    const int64_t nb = a.buckets ? a.b_pad * a.k * a.ways : 0;
#define APC_PREP(DT) k_tile_prep<DT><<<grid, block, 0, s>>>(qp, q_scale, b, a.b_pad, row_bytes, bq, a.nst, fq, qcopy, a.bucket, nb)
    switch (dt) {
    case APC_F32: APC_PREP(APC_F32); break;
    case APC_F16: APC_PREP(APC_F16); break;
    case APC_BF16: APC_PREP(APC_BF16); break;
    default: APC_PREP(APC_E4M3); break;
    }
#undef APC_PREP
    return hipGetLastError();
}

hipError_t launch_tile(int dt, int bq, const TileArgs& a, hipStream_t s)
{
    switch (dt) {
    case APC_F32: return launch_tile_f32(bq, a, s);
    case APC_F16: return launch_tile_f16(bq, a, s);
    case APC_BF16: return launch_tile_bf16(bq, a, s);
    default: return launch_tile_e4m3(bq, a, s);
    }
}

hipError_t launch_tile_merge(const TileArgs& a, float* top_s, int32_t* top_i, hipStream_t s)
{
    if (a.splits > TM_NT) return hipErrorInvalidValue;             // (plans have at most 256)
    k_tile_merge<<<(unsigned)a.b, TM_NT, 0, s>>>(a.log, a.cnt, a.bucket, a.buckets ? a.ways : 0, a.b_pad, a.splits, a.cap, a.k, a.fq,
                                                 top_s, top_i);
    return hipGetLastError();
}

}  // namespace apc
