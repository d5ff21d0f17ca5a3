// Row factors f = 1/|x| for cache entries (build) and queries (each batch).
//
// A group of lanes strides over a row in 16-byte chunks (coalesced), decodes to
// float32, sums squares, then reduces in a fixed order, the same for every
// grouping, so the result is deterministic.  For e4m3fn rows the norm is that
// of the codes: the positive row scale cancels in the cosine.
#include "apc_internal.h"

namespace apc {
namespace {

__device__ inline float dec_bf16(uint32_t h) { return __uint_as_float(h << 16); }

__device__ inline float dec_f16(uint32_t h)
{
    _Float16 x;
    uint16_t b = (uint16_t)h;
    __builtin_memcpy(&x, &b, 2);
    return (float)x;
}

template <int DT>
__device__ inline void accum_chunk(const uint4 v, float& ss, bool& bad)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if constexpr (DT == APC_F32) {
            float x = __uint_as_float(w[j]);
            bad |= !__builtin_isfinite(x);
            ss = fmaf(x, x, ss);
        } else if constexpr (DT == APC_F16 || DT == APC_BF16) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t c = (w[j] >> (16 * h)) & 0xffffu;
                float x = DT == APC_F16 ? dec_f16(c) : dec_bf16(c);
                bad |= !__builtin_isfinite(x);
                ss = fmaf(x, x, ss);
            }
        } else {
            // the hardware's conversion of e4m3fn codes (exact; NaN codes give NaN)
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[j], false);
            const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[j], true);
            const float x[4] = {lo.x, lo.y, hi.x, hi.y};
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                bad |= !__builtin_isfinite(x[h]);
                ss = fmaf(x[h], x[h], ss);
            }
        }
    }
}

// A group of G lanes per row (16, 32 or 64: the smallest with at most eight
// units per lane), RPG rows per group at once, so that every wavefront has
// several rows' loads in flight whatever the row size.  A wavefront per row of
// 768 bytes had one load of 48 lanes in flight (1,000,000 e4m3 rows: 470 us, 1.6
// TB/s); now 125 us, 6.2 TB/s, what plain reads reach.
//
// A row's sum does not depend on G, so the same row has the same factor bits in
// a call of any size: unit u of 16 bytes always belongs to partial sum u % 64,
// of which a lane keeps 64 / G, and the 64 are added in one order.  Rows of at
// most A G units leave all but a lane's first A partial sums 0: those take no
// registers (1,000,000 e4m3 rows of 256: 62 us, 69 with all four).
template <int DT, int G, int RPG, int A = 64 / G>
__global__ __launch_bounds__(256) void k_row_factors(const uint8_t* __restrict__ rows, int64_t n,
                                                      int64_t row_bytes, const float* __restrict__ scale,
                                                      const int32_t* __restrict__ slot_of_entry,
                                                      int64_t n_slots, float* __restrict__ f,
                                                      BuildStatus* __restrict__ st, uint8_t* __restrict__ rowflags)
{
    constexpr int GPB = 256 / G;                          // groups per block
    static_assert(A <= 64 / G, "a lane has 64 / G partial sums");
    const int gl = threadIdx.x % G;
    const int64_t r0 = ((int64_t)blockIdx.x * GPB + threadIdx.x / G) * RPG;
    float ss[RPG][A];
    bool bad[RPG];
#pragma unroll
    for (int i = 0; i < RPG; ++i) {
#pragma unroll
        for (int a = 0; a < A; ++a) ss[i][a] = 0.f;
        bad[i] = false;
    }
    for (int64_t off = (int64_t)gl * 16; off < row_bytes; off += 64 * 16) {
        uint4 v[A][RPG];
#pragma unroll
        for (int a = 0; a < A; ++a)
            if (off + a * G * 16 < row_bytes)
#pragma unroll
                for (int i = 0; i < RPG; ++i) {
                    const int64_t r = r0 + i < n ? r0 + i : n - 1;
                    v[a][i] = *reinterpret_cast<const uint4*>(rows + r * row_bytes + off + a * G * 16);
                }
#pragma unroll
        for (int a = 0; a < A; ++a)
            if (off + a * G * 16 < row_bytes)
#pragma unroll
                for (int i = 0; i < RPG; ++i) accum_chunk<DT>(v[a][i], ss[i][a], bad[i]);
    }
#pragma unroll
    for (int i = 0; i < RPG; ++i) {
        // partial sum p plus p ^ 32, then ^ 16, .. ^ 1: within a lane as far as
        // it holds both, then by lane distance
#pragma unroll
        for (int m = 32 / G; m >= 1; m >>= 1)
#pragma unroll
            for (int a = 0; a < m && a + m < A; ++a) ss[i][a] += ss[i][a + m];
#pragma unroll
        for (int m = G / 2; m >= 1; m >>= 1) ss[i][0] += __shfl_xor(ss[i][0], m, 64);
        // any lane of the group
        const uint64_t who = __ballot(bad[i]);
        bad[i] = (who >> (threadIdx.x % 64 / G * G) & (~0ull >> (64 - G))) != 0;
    }
    if (gl != 0) return;
#pragma unroll
    for (int i = 0; i < RPG; ++i) {
        const int64_t r = r0 + i;
        if (r >= n) return;
        const float sum = ss[i][0];
        uint32_t flags = 0;
        if (bad[i] || !__builtin_isfinite(sum)) flags |= ST_NONFINITE;
        else if (!(sum > 0.f)) flags |= ST_ZERO;
        if (scale) {
            float s = scale[r];
            if (!(__builtin_isfinite(s) && s > 0.f)) flags |= ST_SCALE;
        }
        if (f) f[r] = flags ? __int_as_float(0x7fc00000) : 1.0f / __builtin_sqrtf(sum);
        if (slot_of_entry) {
            int32_t v = slot_of_entry[r];
            if (v < -1 || (int64_t)v >= n_slots) flags |= ST_SLOT;
        }
        if (rowflags) rowflags[r] = (uint8_t)flags;
        if (st && flags) {
            atomicOr(&st->flags, flags);
            atomicMin(&st->first_bad, (unsigned long long)r);
            atomicAdd(&st->n_bad, 1ull);
        }
    }
}

template <int DT>
void run_row_factors(int64_t n, int64_t row_bytes, const uint8_t* r, const float* scale, const int32_t* slots,
                     int64_t n_slots, float* f, BuildStatus* st, uint8_t* rowflags, hipStream_t s)
{
    auto grid = [n](int64_t per) { return dim3((unsigned)((n + per - 1) / per)); };
#define APC_RF(G, RPG, ...) \
    k_row_factors<DT, G, RPG, ##__VA_ARGS__><<<grid(256 / G * RPG), 256, 0, s>>>(r, n, row_bytes, scale, slots, n_slots, f, st, rowflags)
    // A wavefront per row, every row's loads at once, up to the number of rows where
    // that is no longer faster: 4,000 rows of 768 f16 3.4 us, 4.5 with two rows per
    // 16 lanes, 20,000 8.2 and 7.0; 10,000 of 2,048 e4m3 4.6 and 8.1; 8,000 of 256
    // f16 3.6 and 3.5.  Wide rows that take little decoding have loads enough in
    // flight so at any number (200,000 rows of 1,024 floats: 127 us, 138 with two
    // rows per 32 lanes; 300,000 of 2,048 bf16 192 and 206), e4m3 rows do not
    // (1,000,000 of 768: 470 us, 125 with two per 16 lanes)
    const bool wide = DT != APC_E4M3 && row_bytes > (DT == APC_F32 ? 2048 : 3072);
    if (n <= (row_bytes <= 512 ? 6144 : 10240) || wide) APC_RF(64, 1);
    else if (row_bytes <= 16 * 16) APC_RF(16, 2, 1);
    else if (row_bytes <= 2 * 16 * 16) APC_RF(16, 2, 2);
    else if (row_bytes <= 8 * 16 * 16) APC_RF(16, 2);
    else if (row_bytes <= 8 * 32 * 16) APC_RF(32, 2);
    else APC_RF(64, 2);
#undef APC_RF
}

}  // namespace

hipError_t launch_row_factors(int dt, int64_t n, int32_t d, const void* rows, const float* scale,
                              const int32_t* slot_of_entry, int64_t n_slots, float* f,
                              BuildStatus* st, hipStream_t s, uint8_t* rowflags)
{
    if (n <= 0) return hipSuccess;
    const int64_t row_bytes = (int64_t)d * elem_bytes(dt);
    const uint8_t* r = static_cast<const uint8_t*>(rows);
    switch (dt) {
    case APC_F32: run_row_factors<APC_F32>(n, row_bytes, r, scale, slot_of_entry, n_slots, f, st, rowflags, s); break;
    case APC_F16: run_row_factors<APC_F16>(n, row_bytes, r, scale, slot_of_entry, n_slots, f, st, rowflags, s); break;
    case APC_BF16: run_row_factors<APC_BF16>(n, row_bytes, r, scale, slot_of_entry, n_slots, f, st, rowflags, s); break;
    default: run_row_factors<APC_E4M3>(n, row_bytes, r, scale, slot_of_entry, n_slots, f, st, rowflags, s); break;
    }
    return hipGetLastError();
}

}  // namespace apc
