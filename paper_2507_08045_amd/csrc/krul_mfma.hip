// Dispatch of the 16-bit matrix-core similarity kernel (krul_mfma_kernel.h) over its tile shapes; the
// shapes are instantiated in krul_mfma_<shape><head_dim>.hip.
#include "krul_common.h"

namespace krul {

hipError_t launch_sim_mfma_wide128(const SimParams &p, int n_workgroups, hipStream_t st);
hipError_t launch_sim_mfma_wide96(const SimParams &p, int n_workgroups, hipStream_t st);
hipError_t launch_sim_mfma_wide64(const SimParams &p, int n_workgroups, hipStream_t st);
hipError_t launch_sim_mfma_mid128(const SimParams &p, int n_workgroups, hipStream_t st);
hipError_t launch_sim_mfma_mid96(const SimParams &p, int n_workgroups, hipStream_t st);
hipError_t launch_sim_mfma_mid64(const SimParams &p, int n_workgroups, hipStream_t st);
hipError_t launch_sim_mfma_slim128(const SimParams &p, int n_workgroups, hipStream_t st);
hipError_t launch_sim_mfma_slim96(const SimParams &p, int n_workgroups, hipStream_t st);
hipError_t launch_sim_mfma_slim64(const SimParams &p, int n_workgroups, hipStream_t st);

hipError_t launch_sim_mfma(const SimParams &p, int n_workgroups, hipStream_t st)
{
    // Head sizes below the kernel's ride in zero-padded LDS rows.  Heads above 64, up to 96, have kernels of six MFMAs a block
    // (the same bits as eight): 2 x 77 tokens over 5003 keys with heads of 96 404 -> 378 us, 700 over 4096 with heads of 80
    // 738 -> 700, 16 over 20000 188 -> 181; a decode step, bound by its keys, is as fast.
    switch (p.lay.variant) {
    case kMfmaBig:
        return launch_sim_mfma_big(p, n_workgroups, st);
    case kMfmaWide:
    case kMfmaWideShort:
    case kMfmaWideDeep:
        return p.d > 96 ? launch_sim_mfma_wide128(p, n_workgroups, st) : p.d > 64 ? launch_sim_mfma_wide96(p, n_workgroups, st)
                                                                          : launch_sim_mfma_wide64(p, n_workgroups, st);
    case kMfmaMid:
    case kMfmaMidShort:
        return p.d > 96 ? launch_sim_mfma_mid128(p, n_workgroups, st) : p.d > 64 ? launch_sim_mfma_mid96(p, n_workgroups, st)
                                                                          : launch_sim_mfma_mid64(p, n_workgroups, st);
    case kMfmaSlimDeep:
    case kMfmaSlimShort:
        return p.d > 96 ? launch_sim_mfma_slim128(p, n_workgroups, st) : p.d > 64 ? launch_sim_mfma_slim96(p, n_workgroups, st)
                                                                          : launch_sim_mfma_slim64(p, n_workgroups, st);
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace krul
