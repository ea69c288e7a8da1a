// ra_fwd_f64.hip — FP64 forward kernels (1-4 beads per lane), noise maps 0 and 1.
#include "ra_forward.hpp"

namespace ra {

void launch_forward_f64(const FwdArgs& a, int nmap, dim3 grid, dim3 block, hipStream_t st) {
    if (nmap == 1) launch_fwd_tsf<double, 4, 1, 1>(a, grid, block, st);
    else launch_fwd_tsf<double, 4, 1, 0>(a, grid, block, st);
}

void launch_forward_dual_f64(const FwdArgs& a, const FwdArgs& b, int blocks_a, int nmap, dim3 grid, dim3 block,
                                hipStream_t st) {
    if (nmap == 1) launch_fwd_two<double, 4, 1, 1>(a, b, blocks_a, grid, block, st);
    else launch_fwd_two<double, 4, 1, 0>(a, b, blocks_a, grid, block, st);
}

}  // namespace ra
