// Instantiations of the query-stationary similarity + top-k kernel for e4m3 rows.
#include "qs_kernel.h"

namespace apc {

hipError_t launch_qs_e4m3(const MatchPlan& p, int64_t n, int64_t rb, const void* emb, const float* fe, const void* q,
                        const float* fq, int* gthr, int32_t b, int32_t k, float* ps, int* pi, hipStream_t s)
{
    return q2_dispatch<APC_E4M3>(p, n, rb, emb, fe, q, fq, gthr, b, k, ps, pi, s);
}

}  // namespace apc
