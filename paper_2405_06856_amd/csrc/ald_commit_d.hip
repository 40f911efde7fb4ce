// Commit launches that check constraint (d) against the residents' decode history.
#include "ald_commit.h"

namespace ald {

hipError_t launch_commit_d(const State& st, int32_t blocks, hipStream_t stream)
{
    const dim3 g(blocks);
    if (st.out_diag != nullptr) {
        hipLaunchKernelGGL((k_commit<true, true>), g, dim3(COMMIT_THREADS * commit_waves(true)), 0, stream, st);
    } else {
        hipLaunchKernelGGL((k_commit<false, true>), g, dim3(COMMIT_THREADS * commit_waves(false)), 0, stream, st);
    }
    return hipGetLastError();
}

}  // namespace ald
