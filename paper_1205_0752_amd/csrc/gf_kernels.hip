// Subtraction-sum kernels, and the choice and launch of the scan and serving
// kernels (their bodies are in gf_scan.h).
#include <atomic>

#include "gf_device.h"

namespace gf {
namespace {

// Subtraction sum at the real point mu^2 on the real axis, by one wavefront.
// Higher Taylor coefficients of one folded angular sum about x = mu^2 on the
// real axis (y = r real): with delta = x - mu^2, each symmetric pair
// contributes A(delta) / D(delta) with D = U^2 - 4 x y z^2 = D0 + D1 delta +
// delta^2 (U = U0 + delta), whose power series q_i follows from D q = A term
// by term.  Without a numerator A = 2w U.  With one (N: its polynomials N_j(y)
// in p.k, the same for every pole), the pair carries
//   2w U N0 + 2w z^2 (V^2/2) N1 + 2w z^2 (V^2 U/4) N2,   V^2 = 4 (mu^2 + delta) y,
// a quadratic A = a0 + a1 delta + a2 delta^2 in delta.  The middle node
// (z = 0) w_mid N0 / (U0 + delta) has q_i = w_mid N0 (-1)^i / U0^(i+1).
// acc[i] += omega q_i for i = 1..n.
template <class Args>
__device__ void taylor_node(const Args &a, cd U0, double y, cd omega, int n, cd *acc,
                            const cd *N = nullptr)
{
    const double *tab = a.ang;
    const double mu2 = a.mu2;
    for (int j = 0; j < a.n_a / 2; ++j) {
        const double z2 = ro(tab)[3 * j], w2 = ro(tab)[3 * j + 1];
        const cd D0 = mk(U0.r * U0.r - U0.i * U0.i - 4.0 * mu2 * y * z2, 2.0 * U0.r * U0.i);
        const cd D1 = mk(2.0 * U0.r - 4.0 * y * z2, 2.0 * U0.i);
        cd a0 = cscale(U0, w2), a1 = mk(w2, 0.0), a2 = mk(0.0, 0.0);
        if (N) {
            // a0 = 2w N0 U0 + 2w z^2 y mu^2 (2 N1 + U0 N2)
            // a1 = 2w N0 + 2w z^2 y (2 N1 + (mu^2 + U0) N2)
            // a2 = 2w z^2 y N2
            const double wy = w2 * z2 * y;
            const cd n2u = cmul(N[2], U0);
            a0 = cadd(cmul(a0, N[0]), cscale(cadd(cscale(N[1], 2.0), n2u), wy * mu2));
            a1 = cadd(cscale(N[0], w2),
                      cscale(cadd(cadd(cscale(N[1], 2.0), cscale(N[2], mu2)), n2u), wy));
            a2 = cscale(N[2], wy);
        }
        const cd rD = cdiv(mk(1.0, 0.0), D0);
        cd qm2 = mk(0.0, 0.0);
        cd qm1 = cmul(a0, rD);  // q_0
        for (int i = 1; i <= n; ++i) {
            cd rhs = mk(-(D1.r * qm1.r - D1.i * qm1.i) - qm2.r, -(D1.r * qm1.i + D1.i * qm1.r) - qm2.i);
            if (i == 1) rhs = cadd(rhs, a1);
            if (i == 2) rhs = cadd(rhs, a2);
            const cd q = cmul(rhs, rD);
            acc[i] = cadd(acc[i], cmul(omega, q));
            qm2 = qm1;
            qm1 = q;
        }
    }
    if (a.wmid != 0.0) {
        const cd rU = cdiv(mk(1.0, 0.0), U0);
        cd p = cscale(rU, a.wmid);
        if (N) p = cmul(p, N[0]);
        for (int i = 1; i <= n; ++i) {
            p = cscale(cmul(p, rU), -1.0);
            acc[i] = cadd(acc[i], cmul(omega, p));
        }
    }
}

// <1/(U - V z)> pair by pair from the direct denominators (where V^2 = 0 leaves the
// groups no sigma, i.e. mu^2 = 0).
template <class Args>
__device__ cd pairs_one_by_one(const Args &a, cd U, cd V2)
{
    const auto *t = ro(a.ang);
    const cd U2 = cmul(U, U);
    cd A = mk(0.0, 0.0);
    for (int j = 0; j < a.n_a / 2; ++j)
        A = cadd(A, cscale(cinv(mk(fma(-V2.r, t[3 * j], U2.r), fma(-V2.i, t[3 * j], U2.i))),
                           t[3 * j + 1]));
    A = cmul(A, U);
    if (a.wmid != 0.0) A = cadd(A, cscale(cinv(U), a.wmid));
    return A;
}

// Subtraction coefficients at the real point mu^2 on the real axis, by one
// wavefront: K_0 = the subtraction sum of eq. 14 (the order-0 operator t^0),
// and for t^n with n >= 1 the Taylor coefficients K_i = (1/i!) d^i/dx^i of the
// same sum (eq. 13 about x = mu^2).
//
// Where the scan's sums run in groups (GROUPED) so do these, and like there every
// reciprocal takes a cubic step: S and J are about ten times their difference
// G, so a bias of either alone would show (the pair form's Newton steps bias
// both alike).
template <bool SPLIT, bool POLES, bool GROUPED, class Args>
__device__ __forceinline__ void jmu_wave_impl(const Args &a, double mu2, double *dst, int lane)
{
    const PointCtx pc = point_setup<SPLIT, POLES>(a, mu2, 0.0, mu2, 0.0, kR, 0, 0);
    double sr = 0.0, si = 0.0;
    cd acc[GF_MAX_TAYLOR + 1];
    for (int i = 0; i <= GF_MAX_TAYLOR; ++i) acc[i] = mk(0.0, 0.0);
    for (int k = lane; k < pc.nodes; k += 64) {
        cd U, V2, w;
        node_coeffs<SPLIT, POLES>(a, pc, k, U, V2, w);
        cd N[3];
        const bool num = POLES && a.num;
        if (num) numerator_at(a, U, pc.x1, N);
        cd A;
        if constexpr (GROUPED) {
            double r, g, rinv;
            radial_node<SPLIT>(a, pc, k, r, g, &rinv);
            const cd iv = mk(rinv * rcp64c(4.0 * mu2), 0.0);
            auto e0 = [&] { return mk((mu2 - r) * (mu2 - r) * iv.r, 0.0); };
            A = angular_sum_grouped_p<POLES, false>(a, mk(mu2 + r, 0.0), iv, e0,
                                             [&](cd Ua) { return pairs_one_by_one(a, Ua, V2); });
            if (!POLES) w = cscale(cinv(mk(r + a.m2_re, a.m2_im)), g);
        } else {
            A = angular_sum_p<0, POLES>(a, U, V2, ~0, num ? N : nullptr);
        }
        cd t = cmul(w, A);
        sr += t.r;
        si += t.i;
        if (a.n_taylor > 0) {
            double r, g;
            radial_node<SPLIT>(a, pc, k, r, g);
            if (!POLES) {
                taylor_node(a, U, r, w, a.n_taylor, acc);
            } else {
                for (int p = 0; p < a.n1; ++p) {  // pole a of P1: U_a, weight c1_a omega
                    const auto *q = &a.p1[4 * p];
                    const cd Ua = mk(U.r + (q[0] - a.m1_re), U.i + (q[1] - a.m1_im));
                    taylor_node(a, Ua, r, cmul(w, mk(q[2], q[3])), a.n_taylor, acc,
                                num ? N : nullptr);
                }
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        sr += __shfl_xor(sr, off);
        si += __shfl_xor(si, off);
    }
    for (int i = 1; i <= a.n_taylor; ++i) {
        double ar = acc[i].r, ai = acc[i].i;
        for (int off = 32; off > 0; off >>= 1) {
            ar += __shfl_xor(ar, off);
            ai += __shfl_xor(ai, off);
        }
        if (lane == 0) {
            dst[2 * i] = ar;
            dst[2 * i + 1] = ai;
        }
    }
    if (lane == 0) {
        // t^-1 (no subtraction) leaves K_0 = 0
        dst[0] = a.n_taylor < 0 ? 0.0 : sr;
        dst[1] = a.n_taylor < 0 ? 0.0 : si;
    }
}

template <bool GROUPED, class Args>
__device__ __forceinline__ void jmu_wave_form(const Args &a, double mu2, double *dst, int lane)
{
    if (a.poles)
        jmu_wave_impl<false, true, GROUPED>(a, mu2, dst, lane);  // split needs single poles
    else if (a.split)
        jmu_wave_impl<true, false, GROUPED>(a, mu2, dst, lane);
    else
        jmu_wave_impl<false, false, GROUPED>(a, mu2, dst, lane);
}

template <class Args>
__device__ __forceinline__ void jmu_wave(const Args &a, double mu2, double *dst, int lane)
{
    if (a.n_grp > 0 && !a.num)
        jmu_wave_form<true>(a, mu2, dst, lane);
    else
        jmu_wave_form<false>(a, mu2, dst, lane);
}

__global__ void __launch_bounds__(64) jmu_kernel(ScanArgs a, double mu2, double *dst)
{
    jmu_wave(a, mu2, dst, threadIdx.x);
}

// One wave per request: installs request i's argument record (staged[i]) in
// its slot of the request table, and writes J_mu (and the Taylor
// coefficients) of that request into the record's jmu slot.
__global__ void __launch_bounds__(64) jmu_batch_kernel(ScanArgs *__restrict__ reqs,
                                                       const ScanArgs *__restrict__ staged,
                                                       const int *__restrict__ slots,
                                                       const double *__restrict__ mu2, int n)
{
    static_assert(sizeof(ScanArgs) % sizeof(unsigned long long) == 0, "record size");
    const int i = blockIdx.x;
    if (i >= n) return;
    const int slot = __builtin_amdgcn_readfirstlane(slots[i]);
    constexpr int words = sizeof(ScanArgs) / sizeof(unsigned long long);
    const auto *src = reinterpret_cast<const unsigned long long *>(staged + i);
    auto *dst = reinterpret_cast<unsigned long long *>(reqs + slot);
    for (int k = threadIdx.x; k < words; k += 64) dst[k] = src[k];
    const auto &a = ro(staged)[i];
    jmu_wave(a, mu2[i], const_cast<double *>(a.jmu), threadIdx.x);
}

}  // namespace

int scan_form(const ScanArgs &a, int precision)
{
    if (precision == GF_PREC_FP32C) return kFp32c;
    return a.n_grp > 0 && !a.num ? kGroups : kPairs;
}

namespace {

ScanKernel scan_kernel(int form, int lanes, bool taylor, bool split, bool poles)
{
    return form == kGroups  ? scan_kernel_groups(lanes, taylor, split, poles)
           : form == kPairs ? scan_kernel_pairs(lanes, taylor, split, poles)
           : form == kFp32c ? scan_kernel_fp32c(lanes, taylor, split, poles)
                            : nullptr;
}

ServeKernel serve_kernel(int form, bool split, bool poles)
{
    return form == kGroups  ? serve_kernel_groups(split, poles)
           : form == kPairs ? serve_kernel_pairs(split, poles)
           : form == kFp32c ? serve_kernel_fp32c(split, poles)
                            : nullptr;
}

}  // namespace

hipError_t launch_scan(const ScanArgs &a, int precision, int lanes, hipStream_t s)
{
    if (a.n_tiles <= 0) return hipSuccess;
    const ScanKernel k =
        scan_kernel(scan_form(a, precision), lanes, a.n_taylor > 0, a.split != 0, a.poles != 0);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(a.n_tiles), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_jmu(const ScanArgs &a, double mu2, double *dst, hipStream_t s)
{
    hipLaunchKernelGGL(jmu_kernel, dim3(1), dim3(64), 0, s, a, mu2, dst);
    return hipGetLastError();
}

hipError_t launch_jmu_batch(ScanArgs *reqs, const ScanArgs *staged, const int *slots,
                            const double *mu2, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(jmu_batch_kernel, dim3(n), dim3(64), 0, s, reqs, staged, slots, mu2, n);
    return hipGetLastError();
}

int scan_resident_waves(int form, int lanes, bool taylor, bool split, bool poles)
{
    // cached per device and kernel form: [device][form][log2 lanes][taylor][split][poles]
    constexpr int kDevices = 16;
    static std::atomic<int> cache[kDevices][3][7][2][2][2];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 4096;
    int lg = 0;
    while (lg < 7 && (1 << lg) != lanes) ++lg;
    if (lg == 7 || form < 0 || form > 2) return 4096;
    std::atomic<int> *slot = dev >= 0 && dev < kDevices
                                 ? &cache[dev][form][lg][taylor][split][poles]
                                 : nullptr;
    if (slot) {
        const int v = slot->load(std::memory_order_relaxed);
        if (v > 0) return v;
    }
    const void *f =
        reinterpret_cast<const void *>(scan_kernel(form, lanes, taylor, split, poles));
    int cus = 0, blocks = 0;
    if (!f || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, f, 64, 0) != hipSuccess ||
        cus <= 0 || blocks <= 0)
        return 4096;
    const int waves = cus * blocks;  // one wave per workgroup
    if (slot) slot->store(waves, std::memory_order_relaxed);
    return waves;
}

int serve_resident_waves(int form, bool split, bool poles)
{
    const void *f = reinterpret_cast<const void *>(serve_kernel(form, split, poles));
    int dev = 0, cus = 0, blocks = 0;
    if (!f || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, f, 256, 0) != hipSuccess ||
        cus <= 0 || blocks <= 0)
        return 4096;
    return cus * blocks * 4;
}

hipError_t launch_serve(const ScanArgs *reqs, const WorkItem *items, int n_items,
                        unsigned *counter, int form, bool split, bool poles, int waves,
                        hipStream_t s)
{
    if (n_items <= 0) return hipSuccess;
    const ServeKernel k = serve_kernel(form, split, poles);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3((waves + 3) / 4), dim3(256), 0, s, reqs, items, n_items, counter);
    return hipGetLastError();
}

}  // namespace gf
