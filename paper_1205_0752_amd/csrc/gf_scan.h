// The complex-plane scan on gfx950 (STEP 4 + STEP 5 fused): the body shared by
// the kernels of every form of the angular sum (gf_scan_groups.hip,
// gf_scan_pairs.hip, gf_scan_fp32c.hip).
//
// One 64-wide wavefront owns a tile of grid points; each point is handled by
// L lanes (L = 1 for large grids).  Per point, in FP64: the grid coordinate,
// sqrt(x), arg x and the contour class (STEP 3), then per contour node the
// hoisted coefficients (U, V, omega) of
//
//     omega * sum_j w_j / (U - V z_j),   U = x + y + m1^2,  V = 2 sqrt(x) sqrt(y),
//     omega = dy-weight * y / (y + m2^2),
//
// i.e. eq. 11's angular integral of the first propagator times the y-only
// factor of eq. 19.  The angular nodes are wave-uniform, so their table is
// read through the scalar cache into SGPR operands; each lane keeps its point's
// (U, V) in registers.  Partial sums of the L lanes of a point are combined
// with cross-lane shuffles, the real-axis subtraction sum at mu^2 (eq. 14) is
// removed, the result scaled, conjugated for mirror points, and written once.
#pragma once
#include <type_traits>

#include "gf_device.h"

namespace gf {
namespace {

// One wave's tile of grid points: STEP 4 (the point) and STEP 5 (eq. 15 on
// the point's contour), shared by the one-grid scan and the serving kernel so a
// point's result at L lanes does not depend on which launch computes it (other L sum
// in another order, and L > 4 leaves the groups' second table out).
// TAYLOR = false compiles out the t^n (n >= 1) epilogue, so the order-0 scan
// carries no extra live values; both forms compute order 0 identically.
// Tiles are numbered row-major over the rows from row0 on, tiles_a per row.
// PREC is the form of the angular sums (kPairs, kFp32c, kGroups).
template <int PREC, int L, bool TAYLOR, bool SPLIT, bool POLES, class Args>
__device__ __forceinline__ void process_tile(const Args &a, int tile, int lane, int row0,
                                             int tiles_a, const float *lds = nullptr)
{
    constexpr int P = 64 / L;
    constexpr int TW = P < 8 ? P : 8;
    constexpr int TH = P / TW;
    const int p = lane / L;
    const int s = lane % L;
    const int ia = (tile % tiles_a) * TW + p % TW;
    const int ib = row0 + (tile / tiles_a) * TH + p / TW;
    const bool valid = ia < a.n_re && ib < a.n_im;

    double xr = fma((double)ia + 0.5, a.d_re, a.re_lo);
    double xi = fma((double)ib + 0.5, a.d_im, a.im_lo);
    int sign = 0, info = 0;
    const PointArg pa = point_arg(xr, xi);
    double phi = pa.phi;
    int cls = valid ? classify<POLES>(a, pa.v, phi, &sign, &info) : kSingular;
    int ecls = cls;
    if (cls == kMirror) {
        // evaluate at conj x and conjugate the result; if conj x has no
        // contour of its own, the real axis where it is valid at x, else the
        // long way round at x (info holds its sets)
        int sign_b = 0, info_b = 0;
        ecls = classify<POLES>(a, pa.v, -phi, &sign_b, &info_b);
        if (ecls == kMirror || ecls == kSingular || ecls == kLong) {
            cls = ecls = (info & kInfoRValid) ? kR : kLong;
            if (cls == kR) sign = info = 0;
        } else {
            xi = -xi;
            phi = -phi;
            sign = sign_b;
            info = info_b;
        }
    }
    const PointCtx pc = point_setup<SPLIT, POLES, PREC == kFp32c>(a, xr, xi, pa.r, phi, ecls, sign, info);

    // The straight part's nodes, then the arc and residue nodes, in one
    // sequence k = s, s + L, ... per lane: two loops so that the arc's sine
    // and cosine constants are live only in the second.
    double sr = 0.0, si = 0.0;
    int k = s;
    constexpr bool grouped = PREC == kGroups;
    constexpr bool kMiddle = L <= 4;
    const int n_straight = min(pc.nodes, a.n_r);
    if (!POLES) {
        // On the straight part y = e^{i phi} r the node weight is
        //   dirD g / (e^{i phi} r + m2^2) = F g / (r + c),  c = m2^2 e^{-i phi},
        // F = dirD e^{-i phi}: F comes out of the sum, and 1/(r + c) takes one
        // real reciprocal of (r + Re c)^2 + (Im c)^2.  U = x + m1^2 + e^{i phi} r
        // and V^2 = (4x e^{i phi}) r are one FMA or product per component.
        // The FP64 sums skip their rescaling when the launch allows it
        // (wave-uniform): the loop is compiled once with and once without.
        const double cr = fma(a.m2_re, pc.dir.r, a.m2_im * pc.dir.i);
        const double ci = fma(a.m2_im, pc.dir.r, -(a.m2_re * pc.dir.i));
        const cd x4d = cmul(mk(4.0 * (pc.x1.r - a.m1_re), 4.0 * (pc.x1.i - a.m1_im)), pc.dir);
        auto straight = [&](auto scale) {
            constexpr int SC = decltype(scale)::value;
            for (; k < n_straight; k += L) {
                double r, g;
                radial_node<SPLIT>(a, pc, k, r, g);
                const cd U = mk(fma(pc.dir.r, r, pc.x1.r), fma(pc.dir.i, r, pc.x1.i));
                const cd A = angular_sum<PREC, SC>(a, U, mk(x4d.r * r, x4d.i * r), lds);
                const double br = r + cr;
                const double gq = g * rcp64(fma(br, br, ci * ci));
                const double wr = gq * br, wi = -(gq * ci);  // g / (r + c)
                sr = fma(wr, A.r, fma(-wi, A.i, sr));
                si = fma(wr, A.i, fma(wi, A.r, si));
            }
        };
        if constexpr (grouped) {
            // e and h = U / V^2 of angular_sum_grouped with the mass terms put
            // into the point's constants, 1/r from the table
            const cd m = mk(a.m1_re, a.m1_im), x = mk(xr, xi);
            const StraightCtx st = straight_ctx(a, pc, x, pa.r, ecls == kR);
            const cd h0 = cmul(pc.dir, st.kappa), h1 = cmul(pc.x1, st.kappa);
            const cd c0 = cadd(st.c0, cscale(cmul(m, h0), 2.0));
            const cd b0 = cadd(st.b0, cmul(m, cmul(cadd(x, pc.x1), st.kappa)));
            for (; k < n_straight; k += L) {
                double r, g, rinv;
                radial_node<SPLIT>(a, pc, k, r, g, &rinv);
                const double d = r - st.a, q = d * d * rinv;
                const cd e = mk(fma(st.k2.r, q, fma(b0.r, rinv, c0.r)),
                                fma(st.k2.i, q, fma(b0.i, rinv, c0.i)));
                const cd h = mk(fma(h1.r, rinv, h0.r), fma(h1.i, rinv, h0.i));
                const cd A = angular_sum_grouped<kMiddle>(a, e, h, [&] {
                    const cd U = mk(fma(pc.dir.r, r, pc.x1.r), fma(pc.dir.i, r, pc.x1.i));
                    return angular_sum64<-1, true>(a.ang, a.n_a / 2, a.wmid, U,
                                             mk(x4d.r * r, x4d.i * r), !a.unscaled);
                });
                const double br = r + cr;
                const double gq = g * rcp64c(fma(br, br, ci * ci));
                const double wr = gq * br, wi = -(gq * ci);  // g / (r + c)
                sr = fma(wr, A.r, fma(-wi, A.i, sr));
                si = fma(wr, A.i, fma(wi, A.r, si));
            }
        } else if (PREC == kPairs && a.unscaled) {
            straight(std::integral_constant<int, 0>{});
        } else {
            straight(std::integral_constant<int, 1>{});
        }
        const cd F = cmul(pc.dirD, mk(pc.dir.r, -pc.dir.i));
        const double tr = sr;
        sr = fma(F.r, tr, -(F.i * si));
        si = fma(F.r, si, F.i * tr);
    } else {
        // D = 3 with both rotations: the long group's terms see the opposite
        // sign of sqrt(y) on the shared ray (a long group alone has it in dirD)
        const int grp_long = pc.info >> kInfoGrpLong & 0xFF;
        const int ray_neg =
            a.dim == 3 && ecls == kLong && short_group<POLES>(a, pc.info) ? grp_long : 0;
        if constexpr (grouped) {
            const cd m = mk(a.m1_re, a.m1_im), x = mk(pc.x1.r - m.r, pc.x1.i - m.i);
            const cd x4 = cscale(x, 4.0), kappa = cinv(cmul(x4, pc.dir));
            for (; k < n_straight; k += L) {
                double r, g, rinv;
                radial_node<SPLIT>(a, pc, k, r, g, &rinv);
                const cd y = cscale(pc.dir, r), xy = cadd(x, y), iv = cscale(kappa, rinv);
                auto e0 = [&] {
                    const cd d = mk(x.r - pc.dir.r * r, x.i - pc.dir.i * r);
                    return cmul(cmul(d, d), iv);
                };
                const cd A = angular_sum_grouped_p<POLES, kMiddle>(
                    a, xy, iv, e0,
                    [&](cd U) {
                        return angular_sum64<-1, true>(a.ang, a.n_a / 2, a.wmid, U,
                                                 cmul(x4, cscale(pc.dir, r)), !a.unscaled);
                    },
                    ~0, ray_neg);
                const cd t = cmul(cmul(cscale(pc.dirD, g), prop2(a, cscale(pc.dir, r))), A);
                sr += t.r;
                si += t.i;
            }
        } else {
            for (; k < n_straight; k += L) {
                cd U, V2, w;
                radial_coeffs<SPLIT, POLES>(a, pc, k, U, V2, w);
                cd N[3];
                if (a.num) numerator_at(a, U, pc.x1, N);
                cd A = angular_sum_p<PREC, POLES>(a, U, V2, ~0, a.num ? N : nullptr, ray_neg, lds);
                cd t = cmul(w, A);
                sr += t.r;
                si += t.i;
            }
        }
    }
    for (; k < pc.nodes; k += L) {
        cd U, V2, w;
        int set;
        // a residue node carries a whole 2 pi i Res with no quadrature weight
        // to shrink it, and its k-leg pole can sit near the angular cut: its
        // angular sum is taken in FP64 in every precision
        const bool res = outer_coeffs<POLES, PREC == kFp32c>(a, pc, k, U, V2, w, set);
        cd A;
        if constexpr (grouped) {
            // x - y = 2x - (x + y)
            const cd m = mk(a.m1_re, a.m1_im), xy = mk(U.r - m.r, U.i - m.i), iv = cinv(V2);
            auto e0 = [&] {
                const cd d = mk(2.0 * (pc.x1.r - m.r) - xy.r, 2.0 * (pc.x1.i - m.i) - xy.i);
                return cmul(cmul(d, d), iv);
            };
            A = angular_sum_grouped_p<POLES, kMiddle>(
                a, xy, iv, e0,
                [&](cd Ua) {
                    return angular_sum64<-1, true>(a.ang, a.n_a / 2, a.wmid, Ua, V2, !a.unscaled);
                },
                set);
        } else {
            cd N[3];
            const bool num = POLES && a.num;
            if (num) numerator_at(a, U, pc.x1, N);
            A = PREC == kFp32c && res ? angular_sum_p<0, POLES>(a, U, V2, set, num ? N : nullptr)
                                      : angular_sum_p<PREC, POLES>(a, U, V2, set, num ? N : nullptr, 0, lds);
        }
        cd t = cmul(w, A);
        sr += t.r;
        si += t.i;
    }
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1) {
        sr += __shfl_xor(sr, off);
        si += __shfl_xor(si, off);
    }
    if (valid && s == 0) {
        double gr, gi;
        if (cls == kSingular) {
            gr = __builtin_nan("");
            gi = __builtin_nan("");
        } else {
            double kr = a.jmu[0], ki = a.jmu[1];
            if (TAYLOR && a.n_taylor > 0) {
                // t^n: subtract sum_i (x - mu^2)^i K_i at the evaluated point
                // (conj x for a mirror point), by Horner's rule
                const double er = fma((double)ia + 0.5, a.d_re, a.re_lo) - a.mu2;
                const double yi = fma((double)ib + 0.5, a.d_im, a.im_lo);
                const cd d = mk(er, cls == kMirror ? -yi : yi);
                cd sub = mk(a.jmu[2 * a.n_taylor], a.jmu[2 * a.n_taylor + 1]);
                for (int i = a.n_taylor - 1; i >= 0; --i)
                    sub = cadd(cmul(sub, d), mk(a.jmu[2 * i], a.jmu[2 * i + 1]));
                kr = sub.r;
                ki = sub.i;
            }
            gr = a.scale * (sr - kr);
            gi = a.scale * (si - ki);
            if (cls == kMirror) gi = -gi;
        }
        const size_t idx = (size_t)ib * (size_t)a.n_re + (size_t)ia;
        reinterpret_cast<double2 *>(a.out)[idx] = make_double2(gr, gi);
        if (a.cls) a.cls[idx] = (int8_t)cls;
    }
}

// One wave (one tile)
// per workgroup: a tile's cost depends on its points' classes (a tile of
// points without a contour ends at once), and a one-wave workgroup frees its
// slot for the next tile by itself, where a four-wave workgroup would hold
// the slots of its finished waves until the last one ends.
//
// The tail of a large scan at one lane per point (FP32C: one or two), in every
// kernel form: its last rows run as tiles of 64 / 16 points at 16 lanes per
// point, a sixteenth of a one-lane wave's work each, dispatched after every
// other tile.  They fill the slots that the last round of long waves leaves as
// it drains (waves sharing a SIMD progress oldest first, so a SIMD's last
// waves end one by one), where otherwise SIMDs would run one or two waves that
// cannot hide the reciprocal's latency.
//
// LDS (FP32C): the nodes from LDS, not at many lanes per point, where a wave's few
// nodes do not repay the copy.
template <int PREC, int L, bool TAYLOR, bool SPLIT, bool POLES, bool LDS = false>
__device__ __forceinline__ void scan_body(const ScanArgs &a)
{
    const int wave = blockIdx.x;
    if (wave >= a.n_tiles) return;  // uniform per wave
    // (written as one if-else: an early return gave the tail's pair loop
    // scalar-register spills)
    constexpr bool tail = L == 1 || (PREC == kFp32c && L == 2);
    const float *lds = nullptr;
    if constexpr (LDS) {
        __shared__ __align__(16) float squares[kLdsPairs];  // read as float4
        load_squares(a, squares, threadIdx.x & 63);
        lds = squares;
    }
    if (tail && a.tail_tiles > 0 && wave >= a.n_tiles - a.tail_tiles)
        process_tile<PREC, kTailLanes, TAYLOR, SPLIT, POLES>(
            a, wave - (a.n_tiles - a.tail_tiles), threadIdx.x & 63, a.tail_row0, a.tail_tiles_a, lds);
    else
        process_tile<PREC, L, TAYLOR, SPLIT, POLES>(a, wave, threadIdx.x & 63, 0, a.tiles_a, lds);
}

// Serving: a persistent launch over a packed list of (request, tile) items of
// many requests.  Each wave takes the next item from a device counter (one
// lane's atomic, broadcast) until the list is exhausted, so every wave exits.
template <int PREC, bool SPLIT, bool POLES, bool LDS = false>
__device__ __forceinline__ void serve_loop(const ScanArgs *reqs, const WorkItem *items, int n_items,
                                           unsigned *counter)
{
    const int lane = threadIdx.x & 63;
    const float *lds = nullptr;
    float *squares = nullptr;
    if constexpr (LDS) {
        __shared__ __align__(16) float waves[4][kLdsPairs];  // a slice for each wave of the block
        lds = squares = waves[threadIdx.x >> 6];
    }
    for (;;) {
        unsigned w = 0;
        if (lane == 0) w = atomicAdd(counter, 1u);
        w = __builtin_amdgcn_readlane(w, 0);  // wave-uniform item index
        if (w >= (unsigned)n_items) break;
        const int req = ro(items)[w].req;
        const int tile = ro(items)[w].tile;
        const auto &r = ro(reqs)[req];  // keeps the constant address space
        if constexpr (LDS) load_squares(r, squares, lane);
        process_tile<PREC, 1, true, SPLIT, POLES>(r, tile, lane, 0, r.tiles_a, lds);
    }
}

// The scan kernel of a form for these flags: K names the form's kernels.  Pole
// sums run one kernel form (t^n epilogue compiled in; the split rule needs
// single poles); single poles pick the form without unused parts.
template <class K, int L>
ScanKernel pick_scan_l(bool taylor, bool split, bool poles)
{
    return poles             ? K::template scan<L, true, false, true>()
           : taylor && split ? K::template scan<L, true, true, false>()
           : taylor          ? K::template scan<L, true, false, false>()
           : split           ? K::template scan<L, false, true, false>()
                             : K::template scan<L, false, false, false>();
}

template <class K>
ScanKernel pick_scan(int lanes, bool taylor, bool split, bool poles)
{
    switch (lanes) {
    case 1: return pick_scan_l<K, 1>(taylor, split, poles);
    case 2: return pick_scan_l<K, 2>(taylor, split, poles);
    case 4: return pick_scan_l<K, 4>(taylor, split, poles);
    case 8: return pick_scan_l<K, 8>(taylor, split, poles);
    case 16: return pick_scan_l<K, 16>(taylor, split, poles);
    case 32: return pick_scan_l<K, 32>(taylor, split, poles);
    case 64: return pick_scan_l<K, 64>(taylor, split, poles);
    default: return nullptr;
    }
}

template <class K>
ServeKernel pick_serve(bool split, bool poles)
{
    return poles ? K::template serve<false, true>()
           : split ? K::template serve<true, false>() : K::template serve<false, false>();
}

}  // namespace
}  // namespace gf
