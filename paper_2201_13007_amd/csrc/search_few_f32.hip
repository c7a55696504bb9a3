// The single-worker search kernels for few queries (search_single.h) for float32 vector storage.
#include "search_single.h"

namespace sa {

int launch_search_few_f32(const search_detail::KArgs &A, int64_t nq, hipStream_t s, bool *taken)
{
    return single_detail::launch_few_dt<SA_F32>(A, nq, s, taken);
}

}  // namespace sa
