// Instantiations of the query kernel with an FP8 MLP.
#include "lsnif_query.hpp"

namespace lsnif {

hipError_t launch_query_fp8(const QueryArgs &A, int feat_dtype, int F, int max_L, bool pairs, uint32_t grid,
                         hipStream_t s)
{
    return launch_query<fp8e4m3>(A, feat_dtype, F, max_L, pairs, grid, s);
}

}  // namespace lsnif
