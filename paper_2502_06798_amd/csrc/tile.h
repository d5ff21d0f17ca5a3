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
    int* bucket;            // [k][ways][b_pad] order-preserving keys of the shared maxima
    uint64_t* log;          // [b_pad][splits][cap] keys
    int32_t* cnt;           // [b_pad][splits]
    int64_t b_pad;
    int32_t b, rb, k, nst, splits, qtiles, cap, buckets, ways, group;
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
// Parts of a bucket (its value is the largest of them), a power of two: the
// classes of at most 16 splits meet in one part.  With one part, the atomics of
// 256 splits on one to three addresses per query held up the kernel (32 x 57,558
// x 1,024 f16: k = 1 46.8 us, 33.6 now; k = 2 58.5 and 34.8; k = 5 44.5 and 36.3;
// 200 x 50,000 x 512, k = 2: 55.9 and 41.8; 64 x 200,000 x 512 bf16, k = 10: 65.0
// and 61.0).  More parts take longer to read (1 x 300,000 x 768 e4m3, k = 3:
// 51.1 us, 55.6 with 8 splits per part; 77 x 300,007 x 384 f16, k = 7: 69.1 and
// 73.2), and parts where few splits meet are only prepared and read for nothing
// (2,187 x 1,862 x 256 e4m3, k = 2, 7 splits: 26 us, 33 with eight parts).
inline int tile_ways(int32_t k, int splits)
{
    int w = 1;
    while (k * w * 16 < splits) w *= 2;
    return w;
}
// places of a (query, split) log
int tile_log_cap(int32_t k);

}  // namespace apc
