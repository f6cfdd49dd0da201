// Iteration / evaluation launches of a batch's main loop, squared objective:
// each block first applies its registration's pending update (the fused
// prologue), so the loop needs no separate solve launches.
#include "ups_icp_kernels.hpp"

namespace ups {

ups_status launch_icp_batch_fused(int K, int prec, int mode, const Inst *insts, const int *tile_start, int n,
                                  const StepArgs &a, int blocks, hipStream_t s) {
    UPS_DISPATCH_P(prec, UPS_DISPATCH_K(K, (launch_fused<KK, PP, false>(mode, insts, tile_start, n, a, blocks, s))))
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

}  // namespace ups
