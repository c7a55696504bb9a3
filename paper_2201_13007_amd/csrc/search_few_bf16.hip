// The single-worker search kernels for few queries (search_single.h) for bfloat16 vector storage.
#include "search_single.h"

namespace sa {

int launch_search_few_bf16(const search_detail::KArgs &A, int64_t nq, hipStream_t s, bool *taken)
{
    return single_detail::launch_few_dt<SA_BF16>(A, nq, s, taken);
}

}  // namespace sa
