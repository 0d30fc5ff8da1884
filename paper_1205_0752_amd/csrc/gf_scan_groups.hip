// FP64 scan and serving kernels with the grouped angular sum.
#include "gf_scan.h"

namespace gf {
namespace {

// Waves per SIMD the registers are budgeted for.  The split rule's boundaries
// take the nodes' loop past 128 VGPRs: three waves without its spills (1024^2,
// 256 x 128 nodes: 4.02 ms at three, 4.09 at four).
template <bool SPLIT>
constexpr int kWaves = SPLIT ? 3 : 4;

template <int L, bool TAYLOR, bool SPLIT, bool POLES>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves<SPLIT>)))
scan_kernel_fp64(ScanArgs a)
{
    scan_body<kGroups, L, TAYLOR, SPLIT, POLES>(a);
}

template <bool SPLIT, bool POLES>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kWaves<SPLIT>)))
serve_kernel_fp64(const ScanArgs *__restrict__ reqs, const WorkItem *__restrict__ items, int n_items,
        unsigned *counter)
{
    serve_loop<kGroups, SPLIT, POLES>(reqs, items, n_items, counter);
}

struct Kernels {
    template <int L, bool TAYLOR, bool SPLIT, bool POLES>
    static ScanKernel scan()
    {
        return &scan_kernel_fp64<L, TAYLOR, SPLIT, POLES>;
    }
    template <bool SPLIT, bool POLES>
    static ServeKernel serve()
    {
        return &serve_kernel_fp64<SPLIT, POLES>;
    }
};

}  // namespace

ScanKernel scan_kernel_groups(int lanes, bool taylor, bool split, bool poles)
{
    return pick_scan<Kernels>(lanes, taylor, split, poles);
}

ServeKernel serve_kernel_groups(bool split, bool poles)
{
    return pick_serve<Kernels>(split, poles);
}

}  // namespace gf
