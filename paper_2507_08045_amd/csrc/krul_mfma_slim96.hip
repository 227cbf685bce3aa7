// Instantiations of the similarity kernel: the slim tile shape for heads above 64, up to 96: in the
// 128-wide rows of LDS, but with six MFMAs a block in the place of eight (one translation unit per
// group of shapes, so that they compile side by side).  Tile shapes must match make_plan().
#include "krul_mfma_kernel.h"

namespace krul {

hipError_t launch_sim_mfma_slim128(const SimParams &p, int n_workgroups, hipStream_t st);

hipError_t launch_sim_mfma_slim96(const SimParams &p, int n_workgroups, hipStream_t st)
{
    // (the 32 x 512 form, which a plan takes at these sizes from some 38 GB of keys on, runs as for 128)
    if (p.lay.variant != kMfmaSlimShort) return launch_sim_mfma_slim128(p, n_workgroups, st);
    //                 D  WR WK KBW NC KS
    return launch_cfg<Cfg<128, 1, 4, 1, 2, 6>>(p, n_workgroups, st);   //  32 x 256, 4 waves, ring 2 x 128 keys: two workgroups per CU
}

}  // namespace krul
