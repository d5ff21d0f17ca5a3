// Vector types, score helpers and decoding shared by the similarity kernels.
#pragma once

#include "apc_internal.h"

namespace apc {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int IDX_NONE = 0x7fffffff;

__device__ inline float neg_inf() { return -__builtin_huge_valf(); }
__device__ inline float qnan() { return __int_as_float(0x7fc00000); }

__device__ inline float clamp1(float s) { return __builtin_fminf(__builtin_fmaxf(s, -1.f), 1.f); }

// ---- decoding (row norms) ----------------------------------------------------
__device__ inline float dec_e4m3(uint32_t c)
{
    // selects only (no branches): this runs on hundreds of codes per lane
    const uint32_t e = (c >> 3) & 15u, m = c & 7u;
    const float sub = (float)m * 0.001953125f;                             // m/8 * 2^-6
    const float nrm = __uint_as_float(((e + 120u) << 23) | (m << 20));     // (1 + m/8) * 2^(e - 7)
    float v = e == 0u ? sub : nrm;
    v = (c & 0x80u) ? -v : v;
    return (c & 0x7fu) == 0x7fu ? qnan() : v;
}

__device__ inline float dec_bf16(uint32_t h) { return __uint_as_float(h << 16); }

__device__ inline float dec_f16(uint32_t h)
{
    _Float16 x;
    uint16_t b = (uint16_t)h;
    __builtin_memcpy(&x, &b, 2);
    return (float)x;
}

// sum of squares of the elements packed in 16 bytes; bad |= any non-finite
template <int DT>
__device__ inline void sumsq16(const uint4 v, float& ss, bool& bad)
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
            for (int hh = 0; hh < 2; ++hh) {
                uint32_t c = (w[j] >> (16 * hh)) & 0xffffu;
                float x = DT == APC_F16 ? dec_f16(c) : dec_bf16(c);
                bad |= !__builtin_isfinite(x);
                ss = fmaf(x, x, ss);
            }
        } else {
#pragma unroll
            for (int hh = 0; hh < 4; ++hh) {
                float x = dec_e4m3((w[j] >> (8 * hh)) & 0xffu);
                bad |= !__builtin_isfinite(x);
                ss = fmaf(x, x, ss);
            }
        }
    }
}

}  // namespace apc
