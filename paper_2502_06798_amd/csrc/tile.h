// Arguments and launches of the tiled similarity kernel (tile_kernel.h).
#pragma once

#include "apc_internal.h"

namespace apc {

struct TileArgs {
    const uint8_t* emb;
    const float* fe;
    int64_t n;
    int64_t fe_len;         // entry factors allocated (zeros past n)
    const uint8_t* qcopy;   // the queries in the kernel's load order (tile_copy_bytes)
    const float* fq;        // query factors (NaN: cannot be matched), b_pad
    int* bucket;            // [k][b_pad] order-preserving keys of the shared maxima
    uint64_t* log;          // [b_pad][splits][cap] keys
    int32_t* cnt;           // [b_pad][splits]
    int64_t b_pad;
    int32_t b, rb, k, nst, splits, qtiles, cap, buckets, group;
};

hipError_t launch_tile_f32(int bq, const TileArgs& a, hipStream_t s);
hipError_t launch_tile_f16(int bq, const TileArgs& a, hipStream_t s);
hipError_t launch_tile_bf16(int bq, const TileArgs& a, hipStream_t s);
hipError_t launch_tile_e4m3(int bq, const TileArgs& a, hipStream_t s);

// query factors, reset buckets, and the copy of the queries: stage 2 c + j
// (half j of the 128 bytes c of d) of query tile t is the BQ x 64 bytes at
// (t nst + 2 c + j) BQ 64; unit 4 h + 2 j + s (h, j, s < 2) of row r's 128 bytes
// is in its stage at place (2 h + s) ^ (r / 4 % 4); zeros past d and past b
hipError_t launch_tile_prep(int dt, const void* q, const float* q_scale, int32_t b, int64_t row_bytes, int bq,
                            const TileArgs& a, float* fq, uint8_t* qcopy, hipStream_t s);
hipError_t launch_tile(int dt, int bq, const TileArgs& a, hipStream_t s);
hipError_t launch_tile_merge(const TileArgs& a, float* top_s, int32_t* top_i, hipStream_t s);
// stages of 64 bytes per row: an even number, at least four
inline int64_t tile_stages(int64_t row_bytes) { return row_bytes > 256 ? (row_bytes + 127) / 128 * 2 : 4; }
// classes of disjoint rows per split whose running maxima go into the buckets:
// the two lane halves of each of a tile's eight 32-row blocks
constexpr int TL_CLASSES = 16;
// places of a (query, split) log
int tile_log_cap(int32_t k);

}  // namespace apc
