// The general search kernels (search_multi.h) for fp8 e4m3 vector storage.
#include "search_multi.h"

namespace sa {

int launch_search_multi_fp8(const search_detail::KArgs &A, int64_t nq, hipStream_t s)
{
    return search_detail::launch_multi_dt<SA_FP8E4M3, false>(A, nq, s);
}

}  // namespace sa
