// FP32C scan and serving kernels.
#include "gf_scan.h"

namespace gf {
namespace {

// Six waves per SIMD (measured; the few spills sit outside the inner loop).
template <int L, bool TAYLOR, bool SPLIT, bool POLES>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6)))
scan_kernel_fp32c(ScanArgs a)
{
    scan_body<kFp32c, L, TAYLOR, SPLIT, POLES>(a);
}

template <bool SPLIT, bool POLES>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6)))
serve_kernel_fp32c(const ScanArgs *__restrict__ reqs, const WorkItem *__restrict__ items, int n_items,
        unsigned *counter)
{
    serve_loop<kFp32c, SPLIT, POLES>(reqs, items, n_items, counter);
}

struct Kernels {
    template <int L, bool TAYLOR, bool SPLIT, bool POLES>
    static ScanKernel scan()
    {
        return &scan_kernel_fp32c<L, TAYLOR, SPLIT, POLES>;
    }
    template <bool SPLIT, bool POLES>
    static ServeKernel serve()
    {
        return &serve_kernel_fp32c<SPLIT, POLES>;
    }
};

}  // namespace

ScanKernel scan_kernel_fp32c(int lanes, bool taylor, bool split, bool poles)
{
    return pick_scan<Kernels>(lanes, taylor, split, poles);
}

ServeKernel serve_kernel_fp32c(bool split, bool poles)
{
    return pick_serve<Kernels>(split, poles);
}

}  // namespace gf
