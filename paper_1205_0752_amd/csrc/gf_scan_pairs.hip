// FP64 scan and serving kernels with the angular sum over pairs: rules without
// groups (few or crowded nodes) and numerators in p.k.
#include "gf_scan.h"

namespace gf {
namespace {

// Waves per SIMD the registers are budgeted for: four (109 VGPRs, nothing spilled;
// five spill and are 2 % slower).  Pole sums spill at four; three are better at
// four and more lanes per point (100 x 90 points at 64 x 32 nodes 34.3 -> 28.9 us,
// with a numerator 512^2 at 256 x 128 3.46 -> 3.36 ms), not at one (1024^2: 12.70 ms
// at four, 12.88 at three).
template <int L, bool POLES>
constexpr int kWaves = POLES && L >= 4 ? 3 : 4;

template <int L, bool TAYLOR, bool SPLIT, bool POLES>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves<L, POLES>)))
scan_kernel_fp64_pairs(ScanArgs a)
{
    scan_body<kPairs, L, TAYLOR, SPLIT, POLES>(a);
}

template <bool SPLIT, bool POLES>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
serve_kernel_fp64_pairs(const ScanArgs *__restrict__ reqs, const WorkItem *__restrict__ items, int n_items,
        unsigned *counter)
{
    serve_loop<kPairs, SPLIT, POLES>(reqs, items, n_items, counter);
}

struct Kernels {
    template <int L, bool TAYLOR, bool SPLIT, bool POLES>
    static ScanKernel scan()
    {
        return &scan_kernel_fp64_pairs<L, TAYLOR, SPLIT, POLES>;
    }
    template <bool SPLIT, bool POLES>
    static ServeKernel serve()
    {
        return &serve_kernel_fp64_pairs<SPLIT, POLES>;
    }
};

}  // namespace

ScanKernel scan_kernel_pairs(int lanes, bool taylor, bool split, bool poles)
{
    return pick_scan<Kernels>(lanes, taylor, split, poles);
}

ServeKernel serve_kernel_pairs(bool split, bool poles)
{
    return pick_serve<Kernels>(split, poles);
}

}  // namespace gf
