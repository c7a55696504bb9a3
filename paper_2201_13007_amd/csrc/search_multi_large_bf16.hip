// The general search kernels (search_multi.h) for bfloat16 vector storage, L > 256.
#include "search_multi.h"

namespace sa {

int launch_search_multi_large_bf16(const search_detail::KArgs &A, int64_t nq, hipStream_t s)
{
    return search_detail::launch_multi_dt<SA_BF16, true>(A, nq, s);
}

}  // namespace sa
