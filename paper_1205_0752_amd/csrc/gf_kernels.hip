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
// acc[i] += omega q_i for i = 1..n, over the pairs j0, j0 + step, .. (the middle node
// with j0 = 0).
template <class Args>
__device__ void taylor_node(const Args &a, cd U0, double y, cd omega, int n, cd *acc,
                            const cd *N = nullptr, int j0 = 0, int step = 1)
{
    const double *tab = a.ang;
    const double mu2 = a.mu2;
    for (int j = j0; j < a.n_a / 2; j += step) {
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
    if (j0 == 0 && a.wmid != 0.0) {
        const cd rU = cdiv(mk(1.0, 0.0), U0);
        cd p = cscale(rU, a.wmid);
        if (N) p = cmul(p, N[0]);
        for (int i = 1; i <= n; ++i) {
            p = cscale(cmul(p, rU), -1.0);
            acc[i] = cadd(acc[i], cmul(omega, p));
        }
    }
}

// <1/(U - V z)> pair by pair from the direct denominators, each reciprocal with a
// cubic step; over the pairs j0, j0 + step, .. (the middle node with j0 = 0).
template <class Args>
__device__ cd pairs_one_by_one(const Args &a, cd U, cd V2, int j0 = 0, int step = 1)
{
    const auto *t = ro(a.ang);
    const cd U2 = cmul(U, U);
    cd A = mk(0.0, 0.0);
    for (int j = j0; j < a.n_a / 2; j += step)
        A = cadd(A, cscale(cinv(mk(fma(-V2.r, t[3 * j], U2.r), fma(-V2.i, t[3 * j], U2.i))),
                           t[3 * j + 1]));
    A = cmul(A, U);
    if (j0 == 0 && a.wmid != 0.0) A = cadd(A, cscale(cinv(U), a.wmid));
    return A;
}

// Subtraction coefficients at the real point mu^2 on the real axis, by one
// block: K_0 = the subtraction sum of eq. 14 (the order-0 operator t^0),
// and for t^n with n >= 1 the Taylor coefficients K_i = (1/i!) d^i/dx^i of the
// same sum (eq. 13 about x = mu^2).
//
// Where the scan's sums run in groups (GROUPED) so do these, and like there every
// reciprocal takes a cubic step: S and J are about ten times their difference
// G, so a bias of either alone would show (the pair form's Newton steps bias
// both alike).  TABLES is false where the group tables are still being written
// (jmu_groups_kernel): the sums then go pair by pair.
//
// A plan's sum is a few hundred nodes, bound by the latency of one node's chain.
// THREADS = 64: one wave per request finds room between the blocks of scans that are
// running (blocks of four waves waited 5 ms for it, 0.2 ms by one wave, behind
// two serve kernels), and a plan computes J once.  THREADS = 256 where it is
// computed on every call; without TABLES up to 256 nodes each of the four waves takes
// every fourth pair of all nodes, a node a lane, and beyond that a thread takes whole
// nodes (the allocation-free call, 16^2 points, whole nodes and dealt pairs: 64 x 3000
// nodes 305 and 193 us, 64 x 96 25.3 and 20.8, 256 x 96 33.0 and 31.4, 1024 x 128 82.6 and 84.6,
// 2000 x 64 111 and 120).
template <bool SPLIT, bool POLES, bool GROUPED, bool TABLES, int THREADS, class Args>
__device__ __forceinline__ void jmu_block_impl(const Args &a, double mu2, double *dst)
{
    constexpr int kWaves = THREADS / 64;
    __shared__ double part[kWaves][2 * (GF_MAX_TAYLOR + 1)];
    const int tid = threadIdx.x;
    const PointCtx pc = point_setup<SPLIT, POLES>(a, mu2, 0.0, mu2, 0.0, kR, 0, 0);
    double sr = 0.0, si = 0.0;
    cd acc[GF_MAX_TAYLOR + 1];
    for (int i = 0; i <= GF_MAX_TAYLOR; ++i) acc[i] = mk(0.0, 0.0);
    const bool by_wave = GROUPED && !TABLES && pc.nodes <= THREADS;  // pairs dealt to the waves
    const int j0 = by_wave ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0, step = by_wave ? kWaves : 1;
    for (int k = by_wave ? tid & 63 : tid; k < pc.nodes; k += by_wave ? 64 : THREADS) {
        cd U, V2, w;
        node_coeffs<SPLIT, POLES>(a, pc, k, U, V2, w);
        cd N[3];
        const bool num = POLES && a.num;
        if (num) numerator_at(a, U, pc.x1, N);
        cd A;
        if constexpr (GROUPED) {
            double r, g, rinv;
            radial_node<SPLIT>(a, pc, k, r, g, &rinv);
            if constexpr (TABLES) {
                const cd iv = mk(rinv * rcp64c(4.0 * mu2), 0.0);
                auto e0 = [&] { return mk((mu2 - r) * (mu2 - r) * iv.r, 0.0); };
                A = angular_sum_grouped_p<POLES, false>(
                    a, mk(mu2 + r, 0.0), iv, e0, [&](cd Ua) { return pairs_one_by_one(a, Ua, V2); });
            } else {
                static_assert(TABLES || !POLES, "scans on device tables have single poles");
                A = pairs_one_by_one(a, U, V2, j0, step);
            }
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
                taylor_node(a, U, r, w, a.n_taylor, acc, nullptr, j0, step);
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
    // each wave's sums, then the waves' in order (t^-1, no subtraction, leaves K_0 = 0)
    acc[0] = a.n_taylor < 0 ? mk(0.0, 0.0) : mk(sr, si);
    const int n = max(a.n_taylor, 0);
    for (int i = 0; i <= n; ++i) {
        double ar = acc[i].r, ai = acc[i].i;
        for (int off = 32; off > 0; off >>= 1) {
            ar += __shfl_xor(ar, off);
            ai += __shfl_xor(ai, off);
        }
        if ((tid & 63) == 0) {
            part[tid >> 6][2 * i] = ar;
            part[tid >> 6][2 * i + 1] = ai;
        }
    }
    __syncthreads();
    if (tid < 2 * (n + 1)) {
        double v = 0.0;
        for (int w = 0; w < kWaves; ++w) v += part[w][tid];
        dst[tid] = v;
    }
}

template <bool GROUPED, class Args>
__device__ __forceinline__ void jmu_wave_form(const Args &a, double mu2, double *dst)
{
    if (a.poles)
        jmu_block_impl<false, true, GROUPED, true, 64>(a, mu2, dst);  // split needs single poles
    else if (a.split)
        jmu_block_impl<true, false, GROUPED, true, 64>(a, mu2, dst);
    else
        jmu_block_impl<false, false, GROUPED, true, 64>(a, mu2, dst);
}

template <class Args>
__device__ __forceinline__ void jmu_wave(const Args &a, double mu2, double *dst)
{
    if (a.n_grp > 0 && !a.num)
        jmu_wave_form<true>(a, mu2, dst);
    else
        jmu_wave_form<false>(a, mu2, dst);
}

__global__ void __launch_bounds__(64) jmu_kernel(ScanArgs a, double mu2, double *dst)
{
    jmu_wave(a, mu2, dst);
}

// Folded node (s, 2w) of the angular rule, an odd rule's middle node last.
__device__ __forceinline__ void folded_node(const ScanArgs &a, int j, double &s, double &w)
{
    const int np = a.n_a / 2;
    s = j < np ? a.ang[3 * j] : 0.0;
    w = j < np ? a.ang[3 * j + 1] : (j < np + a.n_a % 2 ? a.wmid : 0.0);
}

constexpr int kJmuThreads = 256;

// For tables generated on the device (single poles, no numerator): block 0 the
// subtraction coefficients, the others the group tables as group_table writes them
// on the host (see there), one thread a group.  The products run in pairs of doubles, so
// that the coefficients are rounded once as there (in single doubles they are up to 210
// eps off for 512 nodes, and a sum about the middle up to 77 eps for 127, 31 in pairs); they
// take no time, the block beside them being longer (64 x 8192 nodes 499 us either way).
template <bool SPLIT, bool GROUPED>
__global__ void __launch_bounds__(kJmuThreads)
jmu_groups_kernel(ScanArgs a, double mu2, double *dst, double *grp)
{
    if (blockIdx.x == 0) {
        jmu_block_impl<SPLIT, false, GROUPED, false, kJmuThreads>(a, mu2, dst);
        return;
    }
    const int b = (blockIdx.x - 1) * kJmuThreads + threadIdx.x;
    const int tables = a.grp_mid ? 2 : 1, nodes = a.n_a / 2 + a.n_a % 2;
    if (b >= tables * a.n_grp) return;
    const double centre = b < a.n_grp ? 1.0 : 0.5;
    // coefficients as pairs of doubles
    struct two {
        double h, l;
    };
    // c + x y
    auto add_mul = [](two c, two x, two y) {
        const double p = x.h * y.h;
        const double pl = fma(x.h, y.l, fma(x.l, y.h, fma(x.h, y.h, -p)));
        const double t = c.h + p, z = t - c.h;
        const double tl = (c.h - (t - z)) + (p - z);
        return two{t, c.l + (tl + pl)};
    };
    two P[kGroupNodes + 1], N[kGroupNodes + 1];
#pragma unroll
    for (int i = 0; i <= kGroupNodes; ++i) P[i] = N[i] = two{0.0, 0.0};
    P[0].h = 1.0;
#pragma unroll
    for (int k = 0; k < kGroupNodes; ++k) {
        const int j = b % a.n_grp + k * a.n_grp;
        double s, w;
        folded_node(a, j, s, w);
        // missing nodes: s = 0 in the first table, the centre in the second
        two t{0.0, 0.0};  // centre - s
        if (j < nodes || b < a.n_grp) {
            t.h = centre - s;
            const double z = t.h - centre;
            t.l = (centre - (t.h - z)) - (s + z);
        }
#pragma unroll
        for (int i = kGroupNodes; i >= 0; --i) {
            if (i > k + 1) continue;
            N[i] = add_mul(add_mul(i > 0 ? N[i - 1] : two{0.0, 0.0}, t, N[i]), two{w, 0.0}, P[i]);
        }
#pragma unroll
        for (int i = kGroupNodes; i >= 0; --i) {
            if (i > k + 1) continue;
            P[i] = add_mul(i > 0 ? P[i - 1] : two{0.0, 0.0}, t, P[i]);
        }
    }
    double *o = grp + (size_t)kGroupDoubles * b;
    const two W = N[kGroupNodes - 1];
    const double Wh = W.h + W.l, iW = 1.0 / Wh;
    const double Wl = W.h - Wh + W.l;  // |W.h| >= |W.l|
#pragma unroll
    for (int i = 0; i < kGroupNodes; ++i) o[i] = P[i].h + P[i].l;
#pragma unroll
    for (int i = 0; i < kGroupNodes - 1; ++i) {
        const double q = (N[i].h + N[i].l) * iW;  // one step from the quotient in the pair
        o[kGroupNodes + i] = fma(fma(-q, Wh, N[i].h) + fma(-q, Wl, N[i].l), iW, q);
    }
    o[kGroupDoubles - 1] = Wh;
}

// One wave per request: installs request i's argument record (staged[i]) in
// its slot of the request table, and writes J_mu (and the Taylor
// coefficients) of that request into the record's jmu slot.
__global__ void __launch_bounds__(64)
jmu_batch_kernel(ScanArgs *__restrict__ reqs, const ScanArgs *__restrict__ staged,
                 const int *__restrict__ slots, const double *__restrict__ mu2, int n)
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
    jmu_wave(a, mu2[i], const_cast<double *>(a.jmu));
}

}  // namespace

int scan_form(const ScanArgs &a, int precision)
{
    if (precision == GF_PREC_FP32C) return kFp32c;
    return a.n_grp > 0 && !a.num ? kGroups : kPairs;
}

int serve_form(const ScanArgs &a, int precision)
{
    const int form = scan_form(a, precision);
    return form == kFp32c && !a.poles && !a.split && a.n_a / 2 > kLdsPairs ? kFp32cSix : form;
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
           : form == kFp32cSix ? serve_kernel_fp32c_six()
                               : nullptr;
}

// FP32C plain scans without the LDS table (more pairs than it holds, or many lanes per
// point) whose waves are mostly inner loop run best at six waves per SIMD (see
// scan_kernel_fp32c_six): from 2048 pairs a lane on, where more tiles than one round of
// the other kernel's waves are there to fill them.
bool fp32c_six(const ScanArgs &a, int lanes)
{
    if (a.poles || a.split) return false;
    const long long np = a.n_a / 2, nodes = ((long long)a.n_r + a.n_arc + lanes) / lanes;
    return (lanes >= 16 || np > kLdsPairs) && np * nodes >= 2048 &&
           a.n_tiles > scan_resident_waves(kFp32c, lanes, a.n_taylor > 0, false, false);
}

}  // namespace

hipError_t launch_scan(const ScanArgs &a, int precision, int lanes, hipStream_t s)
{
    if (a.n_tiles <= 0) return hipSuccess;
    const int form = scan_form(a, precision);
    const ScanKernel k = form == kFp32c && fp32c_six(a, lanes)
                             ? scan_kernel_fp32c_six(lanes, a.n_taylor > 0)
                             : scan_kernel(form, lanes, a.n_taylor > 0, a.split != 0, a.poles != 0);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(a.n_tiles), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_jmu(const ScanArgs &a, double mu2, double *dst, hipStream_t s)
{
    hipLaunchKernelGGL(jmu_kernel, dim3(1), dim3(64), 0, s, a, mu2, dst);
    return hipGetLastError();
}

hipError_t launch_jmu_groups(const ScanArgs &a, double mu2, double *dst, double *grp, hipStream_t s)
{
    const int groups = (a.grp_mid ? 2 : 1) * a.n_grp;
    const auto kernel = a.split ? (a.n_grp > 0 ? jmu_groups_kernel<true, true> : jmu_groups_kernel<true, false>)
                                : (a.n_grp > 0 ? jmu_groups_kernel<false, true> : jmu_groups_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3(1 + (groups + kJmuThreads - 1) / kJmuThreads), dim3(kJmuThreads), 0, s,
                       a, mu2, dst, grp);
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
