// Instantiations of the query kernel with a float32 MLP.
#include "lsnif_query.hpp"

namespace lsnif {

hipError_t launch_query_f32(const QueryArgs &A, int feat_dtype, int F, int max_L, bool pairs, uint32_t grid,
                         hipStream_t s)
{
    return launch_query<float>(A, feat_dtype, F, max_L, pairs, grid, s);
}

}  // namespace lsnif
