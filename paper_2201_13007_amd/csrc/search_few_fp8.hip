// The single-worker search kernels for few queries (search_single.h) for fp8 e4m3 vector storage.
#include "search_single.h"

namespace sa {

int launch_search_few_fp8(const search_detail::KArgs &A, int64_t nq, hipStream_t s, bool *taken)
{
    return single_detail::launch_few_dt<SA_FP8E4M3>(A, nq, s, taken);
}

}  // namespace sa
