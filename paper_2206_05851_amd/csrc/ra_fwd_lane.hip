// ra_fwd_lane.hip — FP32 forward kernels with 1-4 beads per lane, noise maps 0 and 1.
#include "ra_forward.hpp"

namespace ra {

void launch_forward_lane(const FwdArgs& a, int nmap, dim3 grid, dim3 block, hipStream_t st) {
    if (nmap == 1) launch_fwd_tsf<float, 4, 1, 1>(a, grid, block, st);
    else launch_fwd_tsf<float, 4, 1, 0>(a, grid, block, st);
}

void launch_forward_dual_lane(const FwdArgs& a, const FwdArgs& b, int blocks_a, int nmap, dim3 grid, dim3 block,
                                 hipStream_t st) {
    if (nmap == 1) launch_fwd_two<float, 4, 1, 1>(a, b, blocks_a, grid, block, st);
    else launch_fwd_two<float, 4, 1, 0>(a, b, blocks_a, grid, block, st);
}

}  // namespace ra
