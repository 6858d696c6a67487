// walk_kernel for Node2Vec: uniform and h-proportional proposals.
#include "fw_trial.h"

namespace fw {

hipError_t launch_trial_node2vec(const WalkArgs &a, bool weighted, bool batch, int ev, int grid, hipStream_t s)
{
    if (!weighted) launch_trial_p<kNode2Vec, false, 0>(a, batch, ev, grid, s);
    else if (a.proposal == 0) launch_trial_p<kNode2Vec, true, 0>(a, batch, ev, grid, s);
    else launch_trial_p<kNode2Vec, true, 1>(a, batch, ev, grid, s);
    return hipGetLastError();
}

int trial_blocks_node2vec(bool weighted, bool batch, int proposal, int ev, int lds_cap)
{
    if (!weighted) return trial_blocks_p<kNode2Vec, false, 0>(batch, ev, lds_cap);
    return proposal == 0 ? trial_blocks_p<kNode2Vec, true, 0>(batch, ev, lds_cap)
                         : trial_blocks_p<kNode2Vec, true, 1>(batch, ev, lds_cap);
}

}  // namespace fw
