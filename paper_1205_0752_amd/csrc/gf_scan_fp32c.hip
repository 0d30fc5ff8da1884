// FP32C scan and serving kernels.
#include "gf_scan.h"

namespace gf {
namespace {

// Waves per SIMD the registers are budgeted for: at up to eight lanes of a plain scan
// five, a compromise.  Long node loops want six, which hide the inner loop's latency
// better, short ones four, which spill less around it (ms at six, five, four: 1024^2 at
// 512 x 256 nodes, two lanes, 10.54, 10.70, 11.12; 600 x 400 at 400 x 400, eight lanes, 3.27,
// 3.24, 3.43; 512^2 at 64 x 32 0.208, 0.172, 0.148); six everywhere was slower than five
// on short rules by more than it gained on long ones.  The forms with more per node
// take four (512^2 at 256 x 128: pole sums 2.67 ms at six, 2.09 at four, with a numerator
// 5.10, 2.96; 1024^2 split rule 5.45, 4.37), and so do many lanes per point, where a wave
// is mostly set-up (200 x 150 at 64 x 64: 50.6, 43.3 us).
template <int L, bool SPLIT, bool POLES>
constexpr int kWaves = POLES || SPLIT || L >= 16 ? 4 : 5;

template <int L, bool TAYLOR, bool SPLIT, bool POLES>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves<L, SPLIT, POLES>)))
scan_kernel_fp32c(ScanArgs a)
{
    scan_body<kFp32c, L, TAYLOR, SPLIT, POLES, (L <= 8)>(a);
}

// Six waves, the nodes through scalar registers: best where a wave is mostly inner loop
// and has no LDS table (many lanes per point, or more pairs than the table holds) and
// several rounds of waves are there (ms at four or five waves, and at six): 256^2 at 128 x 1000,
// 16 lanes, 1.190 and 1.143; 400^2 at 64 x 2000, 16 lanes, 3.74 and 3.50; 700^2 at 64 x 1100, four
// lanes, 3.96 and 3.87; 200 x 150 at 512 x 2000, 64 lanes, 4.03 and 3.81.  Within one round
// the others are: 128^2 at 64 x 2000, 16 lanes, 0.514, where six would take 32 lanes to
// fill the chip, 0.518.
template <int L, bool TAYLOR>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6)))
scan_kernel_fp32c_w6(ScanArgs a)
{
    scan_body<kFp32c, L, TAYLOR, false, false>(a);
}

template <bool SPLIT, bool POLES>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kWaves<1, SPLIT, POLES>)))
serve_kernel_fp32c(const ScanArgs *__restrict__ reqs, const WorkItem *__restrict__ items, int n_items,
        unsigned *counter)
{
    serve_loop<kFp32c, SPLIT, POLES, true>(reqs, items, n_items, counter);
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6)))
serve_kernel_fp32c_w6(const ScanArgs *__restrict__ reqs, const WorkItem *__restrict__ items, int n_items,
                 unsigned *counter)
{
    serve_loop<kFp32c, false, false>(reqs, items, n_items, counter);
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

struct SixKernels {
    template <int L, bool TAYLOR, bool, bool>
    static ScanKernel scan()
    {
        return &scan_kernel_fp32c_w6<L, TAYLOR>;
    }
};

}  // namespace

ScanKernel scan_kernel_fp32c_six(int lanes, bool taylor)
{
    return pick_scan<SixKernels>(lanes, taylor, false, false);
}

ServeKernel serve_kernel_fp32c_six() { return &serve_kernel_fp32c_w6; }

ScanKernel scan_kernel_fp32c(int lanes, bool taylor, bool split, bool poles)
{
    return pick_scan<Kernels>(lanes, taylor, split, poles);
}

ServeKernel serve_kernel_fp32c(bool split, bool poles)
{
    return pick_serve<Kernels>(split, poles);
}

}  // namespace gf
