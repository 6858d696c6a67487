// walk_kernel for second-order PageRank: uniform and h-proportional proposals.
#include "fw_trial.h"

namespace fw {

hipError_t launch_trial_secondpr(const WalkArgs &a, bool weighted, bool batch, int ev, int grid, hipStream_t s)
{
    if (!weighted) launch_trial_p<kSecondPR, false, 0>(a, batch, ev, grid, s);
    else if (a.proposal == 0) launch_trial_p<kSecondPR, true, 0>(a, batch, ev, grid, s);
    else launch_trial_p<kSecondPR, true, 1>(a, batch, ev, grid, s);
    return hipGetLastError();
}

int trial_blocks_secondpr(bool weighted, bool batch, int proposal, int ev, int lds_cap)
{
    if (!weighted) return trial_blocks_p<kSecondPR, false, 0>(batch, ev, lds_cap);
    return proposal == 0 ? trial_blocks_p<kSecondPR, true, 0>(batch, ev, lds_cap)
                         : trial_blocks_p<kSecondPR, true, 1>(batch, ev, lds_cap);
}

}  // namespace fw
