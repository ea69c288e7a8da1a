// ra_fwd_split_dual.hip — split forward kernels of two contexts in one launch (see fwd_dual_kernel).
#include "ra_split.hpp"

namespace ra {

template <typename T, int NMAP, int MAX_M>
__global__ __launch_bounds__((split_threads<T, MAX_M>())) void fwd_split_dual_kernel(FwdArgs a, FwdArgs b) {
    extern __shared__ __align__(16) unsigned char split_lds[];
    const int item = (int)blockIdx.x;
    if (item < a.n_items) split_item<T, NMAP, 2, MAX_M>(a, item, (T*)split_lds);
    else split_item<T, NMAP, 2, MAX_M>(b, item - a.n_items, (T*)split_lds);
}

template <typename T, int NMAP, int MAX_M>
static void launch_split_m(const FwdArgs& a, const FwdArgs& b, hipStream_t st) {
    hipLaunchKernelGGL((fwd_split_dual_kernel<T, NMAP, MAX_M>), dim3((unsigned)(a.n_items + b.n_items)),
                       dim3((split_threads<T, MAX_M>())), (split_lds_bytes<T, NMAP, MAX_M>()), st, a, b);
}

template <typename T, int NMAP> static void launch_split(const FwdArgs& a, const FwdArgs& b, int max_m, hipStream_t st) {
    if (max_m == 1) launch_split_m<T, NMAP, 1>(a, b, st);
    else if (max_m == 2) launch_split_m<T, NMAP, 2>(a, b, st);
    else launch_split_m<T, NMAP, 4>(a, b, st);
}

void launch_forward_split_dual(const FwdArgs& a, const FwdArgs& b, int precision, int max_m, int nmap, hipStream_t st) {
    if (precision == 64) {
        if (nmap == 1) launch_split<double, 1>(a, b, max_m, st);
        else launch_split<double, 0>(a, b, max_m, st);
    } else {
        if (nmap == 1) launch_split<float, 1>(a, b, max_m, st);
        else launch_split<float, 0>(a, b, max_m, st);
    }
}

}  // namespace ra
