// ra_fwd_wide.hip — FP32 forward kernels with 6-16 beads per lane, noise maps 0 and 2.
#include "ra_forward.hpp"

namespace ra {

void launch_forward_wide(const FwdArgs& a, int nmap, dim3 grid, dim3 block, hipStream_t st) {
    if (nmap == 2) launch_fwd_tsf<float, 16, 2, 2>(a, grid, block, st);
    else launch_fwd_tsf<float, 16, 2, 0>(a, grid, block, st);
}

void launch_forward_dual_wide(const FwdArgs& a, const FwdArgs& b, int blocks_a, int nmap, dim3 grid, dim3 block,
                                 hipStream_t st) {
    if (nmap == 2) launch_fwd_two<float, 16, 2, 2>(a, b, blocks_a, grid, block, st);
    else launch_fwd_two<float, 16, 2, 0>(a, b, blocks_a, grid, block, st);
}

}  // namespace ra
