// ra_fwd_split.hip — split forward kernels.
#include "ra_split.hpp"

namespace ra {

template <typename T, int NMAP, int TSFK, int MAX_M>
__global__ __launch_bounds__((split_threads<T, MAX_M>())) void fwd_split_kernel(FwdArgs a) {
    extern __shared__ __align__(16) unsigned char split_lds[];
    split_item<T, NMAP, TSFK, MAX_M>(a, (int)blockIdx.x, (T*)split_lds);
}

template <typename T, int NMAP, int MAX_M> static void launch_split_m(const FwdArgs& a, hipStream_t st) {
    constexpr int lds = split_lds_bytes<T, NMAP, MAX_M>();
    const dim3 grid((unsigned)a.n_items), block((split_threads<T, MAX_M>()));
    if (a.tsf) {
        hipLaunchKernelGGL((fwd_split_kernel<T, NMAP, 1, MAX_M>), grid, block, lds, st, a);
        return;
    }
    if constexpr (sizeof(T) == 4) {
        if (a.K == 1) {
            hipLaunchKernelGGL((fwd_split_kernel<T, NMAP, 3, MAX_M>), grid, block, lds, st, a);
            return;
        }
    }
    hipLaunchKernelGGL((fwd_split_kernel<T, NMAP, 0, MAX_M>), grid, block, lds, st, a);
}

template <typename T, int NMAP> static void launch_split(const FwdArgs& a, int max_m, hipStream_t st) {
    if (max_m == 1) launch_split_m<T, NMAP, 1>(a, st);
    else if (max_m == 2) launch_split_m<T, NMAP, 2>(a, st);
    else launch_split_m<T, NMAP, 4>(a, st);
}

void launch_forward_split(const FwdArgs& a, int precision, int max_m, int nmap, hipStream_t st) {
    if (precision == 64) {
        if (nmap == 1) launch_split<double, 1>(a, max_m, st);
        else launch_split<double, 0>(a, max_m, st);
    } else {
        if (nmap == 1) launch_split<float, 1>(a, max_m, st);
        else launch_split<float, 0>(a, max_m, st);
    }
}

}  // namespace ra
