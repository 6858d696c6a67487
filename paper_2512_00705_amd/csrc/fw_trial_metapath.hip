// walk_kernel for MetaPath: uniform, h-proportional and label-conditioned proposals.
#include "fw_trial.h"

namespace fw {

hipError_t launch_trial_metapath(const WalkArgs &a, bool weighted, bool batch, int ev, int grid, hipStream_t s)
{
    if (a.proposal == 2) {
        if (weighted) launch_trial_p<kMetaPath, true, 2>(a, batch, ev, grid, s);
        else launch_trial_p<kMetaPath, false, 2>(a, batch, ev, grid, s);
    } else if (weighted && a.proposal == 1) {
        launch_trial_p<kMetaPath, true, 1>(a, batch, ev, grid, s);
    } else {
        if (weighted) launch_trial_p<kMetaPath, true, 0>(a, batch, ev, grid, s);
        else launch_trial_p<kMetaPath, false, 0>(a, batch, ev, grid, s);
    }
    return hipGetLastError();
}

int trial_blocks_metapath(bool weighted, bool batch, int proposal, int ev, int lds_cap)
{
    if (proposal == 2)
        return weighted ? trial_blocks_p<kMetaPath, true, 2>(batch, ev, lds_cap)
                        : trial_blocks_p<kMetaPath, false, 2>(batch, ev, lds_cap);
    if (!weighted) return trial_blocks_p<kMetaPath, false, 0>(batch, ev, lds_cap);
    return proposal == 1 ? trial_blocks_p<kMetaPath, true, 1>(batch, ev, lds_cap)
                         : trial_blocks_p<kMetaPath, true, 0>(batch, ev, lds_cap);
}

}  // namespace fw
