// gfx950 diagnostic kernels: the y-plane scan at fixed x (the paper's Fig. 1)
// and the obstruction map of the original contour (Fig. 2).  Both reuse the
// device building blocks of the scan kernels.
#include "gf_device.h"

namespace gf {
namespace {

// <1/D1> or <P1((p-k)^2)> at x and y.
template <bool POLES, bool GROUPED>
__device__ __forceinline__ cd y_average(const ScanArgs &a, cd x, cd y)
{
    const cd xy = cadd(x, y), m1 = mk(a.m1_re, a.m1_im), V2 = cmul(cscale(x, 4.0), y);
    if constexpr (GROUPED) {
        const cd iv = cinv(V2);
        auto e0 = [&] {
            const cd d = mk(x.r - y.r, x.i - y.i);
            return cmul(cmul(d, d), iv);
        };
        // the pairs always rescaled: a y grid may meet U = V = 0 (x = 0, y = -m1^2), where
        // products of eight |D|^2 underflow however small the box
        return angular_sum_grouped_p<POLES, true>(a, xy, iv, e0, [&](cd U) {
            return angular_sum64<1, true>(a.ang, a.n_a / 2, a.wmid, U, V2);
        });
    } else if constexpr (POLES) {
        return angular_sum_p<0, true>(a, cadd(xy, m1), V2);
    } else {
        return angular_sum64(a.ang, a.n_a / 2, a.wmid, cadd(xy, m1), V2);
    }
}

// y-plane diagnostic (the paper's Fig. 1): at fixed x, the angular average
// <1/D1>(x, y) over a cell-centred grid of complex y (what = 0), or the
// order-0 subtracted y-integrand y^{(D-2)/2}/(y + m2^2) (<1/D1>(x, y) -
// <1/D1>(mu^2, y)) of eq. 14 (what = 1); with pole sums, <P1> and P2(y) in
// place of <1/D1> and 1/(y + m2^2).  One lane per y point, 8 x 8 tiles, FP64.
//
// Bound by FP64 VALU issue in the angular sums, so they run in groups where the
// plan has them (GROUPED), the reciprocals of both sums of the integrand with cubic
// steps: 1024^2 points, 128 nodes (the integrand) 42.8 -> 35.9 us.
template <bool POLES, bool GROUPED>
__global__ void __launch_bounds__(64, 4) yscan_kernel(ScanArgs a, double xr, double xi, double mu2,
                                                      int what)
{
    const int wave = blockIdx.x;
    const int lane = threadIdx.x;
    const int ia = (wave % a.tiles_a) * 8 + lane % 8;
    const int ib = (wave / a.tiles_a) * 8 + lane / 8;
    if (ia >= a.n_re || ib >= a.n_im) return;
    const cd y = mk(fma((double)ia + 0.5, a.d_re, a.re_lo), fma((double)ib + 0.5, a.d_im, a.im_lo));
    cd A = y_average<POLES, GROUPED>(a, mk(xr, xi), y);
    if (what == 1) {
        const cd Amu = y_average<POLES, GROUPED>(a, mk(mu2, 0.0), y);
        // the radial measure y^{(D-2)/2} (principal sqrt(y) for D = 3)
        const cd f = a.dim == 4 ? y : (a.dim == 3 ? csqrt_principal(y.r, y.i) : mk(1.0, 0.0));
        if (!POLES)
            A = cdiv(cmul(f, mk(A.r - Amu.r, A.i - Amu.i)), cadd(y, mk(a.m2_re, a.m2_im)));
        else
            A = cmul(cmul(f, mk(A.r - Amu.r, A.i - Amu.i)), prop2(a, y));
    }
    const size_t idx = (size_t)ib * (size_t)a.n_re + (size_t)ia;
    reinterpret_cast<double2 *>(a.out)[idx] = make_double2(A.r, A.i);
}

// Obstruction map (the paper's Fig. 2).  The first propagator
// x + y + m1^2 - 2 sqrt(x) sqrt(y) z vanishes for some z in [-1, 1] exactly when
// zeta(y) = (x + y + m1^2)^2 / (4 x y) is real and lies in [0, 1].  Each straight
// part of a contour is sampled at y = (e^t - 1) dir, the closing arc at
// y = Lambda^2 e^{i psi}; where Im zeta changes sign between two consecutive
// samples, 40 bisection steps on the part's parameter locate the zero of
// Im zeta, and the cut crosses the contour there if Re zeta lies in [0, 1].
struct CutWalk {
    cd x1, x4;  // x + m1^2, 4x
    cd dir;     // direction of a straight part
    double lam2;
    bool arc;   // current part: false = straight, true = arc
    bool hit;
};

__device__ __forceinline__ cd cut_zeta(const CutWalk &w, double u)
{
    cd y;
    if (w.arc) {
        double s, c;
        sincos(u, &s, &c);
        y = mk(w.lam2 * c, w.lam2 * s);
    } else {
        y = cscale(w.dir, expm1(u));
    }
    const cd U = cadd(w.x1, y);
    return cdiv(cmul(U, U), cmul(w.x4, y));
}

// A sign change of Im zeta between the samples at parameters lo and hi (Im
// zeta positive at lo when lo_pos): 40 bisection steps on the part's
// parameter (with zeta itself) locate its zero, and the cut crosses the
// contour there if Re zeta lies in [0, 1].
__device__ void cut_bisect(CutWalk &w, double lo, double hi, bool lo_pos)
{
    for (int it = 0; it < 40; ++it) {
        const double mid = 0.5 * (lo + hi);
        if ((cut_zeta(w, mid).i > 0.0) == lo_pos)
            lo = mid;
        else
            hi = mid;
    }
    const cd zc = cut_zeta(w, 0.5 * (lo + hi));
    if (zc.r >= 0.0 && zc.r <= 1.0) w.hit = true;
}

// Which samples a walk has to look at.  Im zeta changes sign with
//   straight part  f(e) = Im((x1 + dir e)^2 conj(4 x dir)),  a quadratic in e = e^u - 1,
//   arc            f(psi) = alpha + b_c cos psi + b_s sin psi,
// and the sign a sample computes is f's wherever |f| exceeds a bound B on all
// rounding of the sample: its position (a recurrence, re-anchored every 64
// samples, within 128 eps) and its value.  f = B and f = -B have at most four
// roots on a part, taken in closed form; between two of them f is either
// beyond B throughout, and every sample there has the same sign, or within it
// (no more than a few ulp wide at a simple zero, a whole part where f vanishes
// identically).  So a walk computes the signs of the samples next to each root,
// two to either side for the roots' own rounding, and of those between two
// roots where f is within B; the map is the one that all samples give.
//
// The map is bound by that per-point set-up (logarithms, arc cosines and the
// bisections' exponentials) instead of n samples a part.  1024^2 points, 4096
// samples a part: 3.5 ms when every sample was computed (7 to 10 VALU
// instructions each, VALU-bound), 0.09 ms now; of that step 0.17 ms came from
// the roots and the rest from settling most bisections by the roots (cut_settled).
//
// Up to kShortWalk samples a part, all of them are computed, which costs less than the
// roots (1024^2 points, real masses: at 2 samples 27 us against 66, at 6 37 and 70, at 8
// 65 and 72, at 12 100 and 76; complex masses 101 and 143, 117 and 147, 145 and 150,
// 172 and 154).
constexpr double kSampleTol = 1e-13;  // of the terms' magnitudes
constexpr int kPad = 2;
constexpr int kShortWalk = 8;

// Root positions in units of samples, ascending (unused ones beyond any sample).
struct Roots {
    double k[4];
};

constexpr double kNoRoot = 1e18;

__device__ __forceinline__ void sort_roots(Roots &r)
{
    auto order = [&](int a, int b) {
        const double lo = fmin(r.k[a], r.k[b]), hi = fmax(r.k[a], r.k[b]);
        r.k[a] = lo;
        r.k[b] = hi;
    };
    order(0, 1);
    order(2, 3);
    order(0, 2);
    order(1, 3);
    order(1, 2);
}

// Visits the samples first..n-1 that the roots leave undecided, in ascending
// order, each next to its predecessor: visit(k, fresh) computes sample k's
// sign, comparing it with sample k-1's unless fresh.  inside(t) says whether f
// lies within its bound at position t.  ends: also the part's first and last
// samples.
template <class Inside, class Visit>
__device__ __forceinline__ void visit_undecided(const Roots &r, int first, int n, bool ends,
                                                Inside inside, Visit visit)
{
    const double end = (double)(n - 1);
    int last = first - 1;  // last sample visited
    auto window = [&](int lo, int hi) {
        lo = max(lo, last + 1);
        hi = min(hi, n - 1);
        if (lo > hi) return;
        const bool fresh = last < first || lo > last + 1;
        int k = fresh ? max(lo - 1, first) : lo;
        for (bool f = fresh; k <= hi; ++k, f = false) visit(k, f);
        last = hi;
    };
#pragma unroll 1
    for (int i = 0; i <= 4; ++i) {
        double a = (double)first, b = kNoRoot;
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // r.k[i - 1], r.k[i] without indexing registers dynamically
            if (q == i - 1) a = r.k[q];
            if (q == i) b = r.k[q];
        }
        if (a > end + (kPad + 1)) break;
        int lo = i == 0 ? first : (int)fmax(a, (double)first) - kPad;
        int hi = i == 0 ? (ends ? first + kPad + 1 : first - 1) : (int)fmin(a, end) + kPad + 1;
        // two roots this close have touching windows
        const bool covered = i > 0 && b <= a + 2 * kPad && b < end;
        b = fmin(b, end);
        if (!covered && b > a && inside(0.5 * (a + b))) hi = (int)b + kPad + 1;
        window(lo, hi);
    }
    if (ends) window(n - 2 - kPad, n - 1);
}

// A sign change of a straight part between samples k-1 and k.  Where the two
// roots f = +-B about it stand alone and close together, the bisection ends
// between them: Re zeta there is known to the difference of its values at the
// two, and only a value next to 0 or 1 needs the bisection itself (forty
// exponentials and divisions).  Returns whether it was settled so.
__device__ __forceinline__ bool cut_settled(CutWalk &w, const Roots &r, double h, int k)
{
    int n = 0;
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (r.k[q] > k - 1.5 && r.k[q] < k + 0.5) {
            a = n == 0 ? r.k[q] : a;
            b = r.k[q];
            ++n;
        }
    if (n != 2 || !(a > k - 1 && b < k && b - a < 1e-6)) return false;
    const double za = cut_zeta(w, a * h).r, zb = cut_zeta(w, b * h).r;
    const double lo = fmin(za, zb), hi = fmax(za, zb);
    if (!(hi - lo < 1e-7)) return false;
    if (lo > 1e-6 && hi < 1.0 - 1e-6) {
        w.hit = true;
        return true;
    }
    return hi < -1e-6 || lo > 1.0 + 1e-6;
}

// Real roots of q2 e^2 + q1 e + q0 (cancellation-free; NaN where there is none).
__device__ __forceinline__ void quadratic_roots(double q2, double q1, double q0, double &r1,
                                                double &r2)
{
    const double d = sqrt(fma(q1, q1, -4.0 * (q2 * q0)));
    const double t = -0.5 * (q1 + copysign(d, q1));
    r1 = t / q2;
    r2 = q0 / t;
}

// Samples along the straight part, y_k = dir e_k, e_k = e^{u_k} - 1, u_k = k h,
// h = T/(n-1), k = 1..n-1: e follows e_{k+1} = e_k c + e_k + c (c = e^h - 1),
// taken afresh from expm1 every 64 samples, so each sample sits within ~64
// ulp of its exact position (far inside the oracle's tie band).  Im zeta has
// the sign of Im(U^2 conj(4 x y)) (|4 x y|^2 > 0), and with 4 x y = (4 x dir) e,
// e > 0, of Im(U^2 conj(4 x dir)) = ur (2 ui c_r - ur c_i) + ui^2 c_i, U = x1 + dir e:
// no division and no product with e.  On the real segment (REAL, dir = 1) ui is
// x1.i itself, as fma(0, e, x1.i) gives for finite e.
template <bool REAL>
__device__ void cut_walk_straight(CutWalk &w, int n, double T)
{
    if (w.hit) return;
    const double h = T / (n - 1);
    const double c = expm1(h);
    const cd c4 = cmul(w.x4, w.dir);
    const double c4r2 = 2.0 * c4.r;
    auto value_at = [&](double e) {
        const double ur = fma(w.dir.r, e, w.x1.r);
        const double ui = REAL ? w.x1.i : fma(w.dir.i, e, w.x1.i);
        return fma(ur, fma(ui, c4r2, -(ur * c4.i)), ui * (ui * c4.i));
    };
    Roots r = {{kNoRoot, kNoRoot, kNoRoot, kNoRoot}};
    int at = -1;  // the recurrence's sample
    double e = 0.0;
    bool prev = false;
    auto visit = [&](int k, bool fresh) {
        if (w.hit) return;
        const int anchor = ((k - 1) & ~63) + 1;
        if (at < anchor || at >= k) {
            at = anchor;
            e = expm1(anchor * h);
        }
        for (; at < k; ++at) e = fma(e, c, e + c);
        const bool p = value_at(e) > 0.0;
        if (!fresh && p != prev && !cut_settled(w, r, h, k))
            cut_bisect(w, fma((double)(k - 1), h, 0.0), fma((double)k, h, 0.0), prev);
        prev = p;
    };
    if (n <= kShortWalk) {
        for (int k = 1; k < n; ++k) visit(k, k == 1);
        return;
    }
    // f = q2 e^2 + q1 e + q0
    const cd cc = mk(c4.r, -c4.i), d2 = cmul(w.dir, w.dir), xd = cmul(w.x1, w.dir),
             x2 = cmul(w.x1, w.x1);
    const double q2 = cmul(d2, cc).i, q1 = 2.0 * cmul(xd, cc).i, q0 = cmul(x2, cc).i;
    if (q2 == 0.0 && q1 == 0.0 && q0 == 0.0) return;  // every sample's value is 0: no sign change
    // B: tol times the terms' magnitudes, not |f|'s scale |4x| (|x1| + e)^2: next to the
    // real axis every term carries the tiny Im x, and so does the rounding
    const double xr = fabs(w.x1.r), xi = fabs(w.x1.i), dr = fabs(w.dir.r),
                 di = REAL ? 0.0 : fabs(w.dir.i);
    const double tr = kSampleTol * fabs(c4r2), ti = kSampleTol * fabs(c4.i);
    const double b2 = fma(tr, dr * di, ti * fma(dr, dr, di * di));
    const double b1 = fma(tr, fma(xr, di, xi * dr), 2.0 * ti * fma(xr, dr, xi * di));
    const double b0 = fma(tr, xr * xi, ti * fma(xr, xr, xi * xi));
    const double ih = 1.0 / h, top = w.lam2 * 1.01;
    auto place = [&](double e) { return e > 0.0 && e < top ? log1p(e) * ih : kNoRoot; };
    // two roots next to one another share the logarithm
    auto place2 = [&](double ea, double eb, double &ka, double &kb) {
        ka = place(ea);
        const double d = (eb - ea) / (1.0 + ea);
        kb = ka < kNoRoot && fabs(d) < 1e-8 ? fma(d, ih, ka) : place(eb);
    };
    double e0, e1, e2, e3;
    quadratic_roots(q2 - b2, q1 - b1, q0 - b0, e0, e1);
    quadratic_roots(q2 + b2, q1 + b1, q0 + b0, e2, e3);
    place2(e0, e2, r.k[0], r.k[2]);
    place2(e1, e3, r.k[1], r.k[3]);
    sort_roots(r);
    auto inside = [&](double t) {
        const double e = expm1(t * h);
        return fabs(fma(fma(q2, e, q1), e, q0)) <= fma(fma(b2, e, b1), e, b0);
    };
    visit_undecided(r, 1, n, false, inside, visit);
}

// Samples along an arc from angle phi, psi_k = phi + span k/(n-1), k = 0..n-1
// (span = -phi: back to 0 the short way; the long way: to +-2 pi): the unit
// vector e = e^{i psi} rotates by e^{i span/(n-1)} per sample, taken afresh
// from sincos every 64 samples.  With y = Lambda^2 e and e conj(e) = 1,
//   U^2 conj(4 x y) = Lambda^2 conj(4x) (x1^2 conj(e) + 2 Lambda^2 x1 + Lambda^4 e),
// so Im zeta has the sign of alpha + b_c cos psi + b_s sin psi with
// A = conj(4x) x1^2, B = Lambda^4 conj(4x), alpha = Im(2 Lambda^2 conj(4x) x1),
// b_c = Im A + Im B, b_s = Re B - Re A: two FMAs a sample.  Its terms add up to
// at most ((Lambda^2 + |x1|) / (Lambda^2 - |x1|))^2 times the value's own scale,
// so the rounding stays that of the direct product.
__device__ void cut_walk_arc(CutWalk &w, int n, double phi, double span)
{
    if (w.hit) return;
    const double dpsi = span / (n - 1);
    double s, c;
    sincos(dpsi, &s, &c);
    const cd rot = mk(c, s);
    const cd cx4 = mk(w.x4.r, -w.x4.i);
    const double l2 = w.lam2, l4 = l2 * l2;
    const cd A = cmul(cx4, cmul(w.x1, w.x1));
    const cd B = cscale(cx4, l4);
    const double alpha = 2.0 * l2 * fma(cx4.r, w.x1.i, cx4.i * w.x1.r);
    const double bc = A.i + B.i, bs = B.r - A.r;
    int at = -1;
    cd e = mk(1.0, 0.0);
    bool prev = false;
    auto visit = [&](int k, bool fresh) {
        if (w.hit) return;
        const int anchor = k & ~63;
        if (at < anchor || at >= k) {
            at = anchor;
            double sn, cs;
            sincos(fma((double)anchor, dpsi, phi), &sn, &cs);
            e = mk(cs, sn);
        }
        for (; at < k; ++at) e = cmul(e, rot);
        const bool p = fma(bc, e.r, fma(bs, e.i, alpha)) > 0.0;
        if (!fresh && p != prev)
            cut_bisect(w, fma((double)(k - 1), dpsi, phi), fma((double)k, dpsi, phi), prev);
        prev = p;
    };
    if (n <= kShortWalk) {
        for (int k = 0; k < n; ++k) visit(k, k == 0);
        return;
    }
    if (alpha == 0.0 && bc == 0.0 && bs == 0.0) return;
    const double bound = kSampleTol * (fabs(alpha) + fabs(bc) + fabs(bs));
    // f = alpha + R cos(psi - psi0) = +-bound; on an arc of nearly a whole turn
    // a root next to one end may come out at the other: both are visited
    const double ir = 1.0 / hypot(bc, bs), psi0 = atan2(bs, bc), id = 1.0 / dpsi;
    const double period = 2.0 * M_PI * fabs(id);
    auto place = [&](double psi) {
        double t = (psi - phi) * id;
        t -= floor(t / period) * period;
        return t > period - 2 * kPad ? t - period : t;  // just before the arc's start
    };
    const bool ends = period < n + 4 * kPad;
    Roots r;
    const double g0 = (-bound - alpha) * ir, g1 = (bound - alpha) * ir;
    const double a0 = acos(fmin(fmax(g0, -1.0), 1.0)), a1 = acos(fmin(fmax(g1, -1.0), 1.0));
    const bool has0 = fabs(g0) <= 1.0 + 1e-12, has1 = fabs(g1) <= 1.0 + 1e-12;
    r.k[0] = has0 ? place(psi0 - a0) : kNoRoot;
    r.k[1] = has0 ? place(psi0 + a0) : kNoRoot;
    r.k[2] = has1 ? place(psi0 - a1) : kNoRoot;
    r.k[3] = has1 ? place(psi0 + a1) : kNoRoot;
    sort_roots(r);
    auto inside = [&](double t) {
        double sn, cs;
        sincos(fma(t, dpsi, phi), &sn, &cs);
        return fabs(fma(bc, cs, fma(bs, sn, alpha))) <= bound;
    };
    visit_undecided(r, 0, n, ends, inside, visit);
}

__device__ CutWalk cut_walk_begin(const ScanArgs &a, double xr, double xi)
{
    CutWalk w;
    w.x1 = mk(xr + a.m1_re, xi + a.m1_im);
    w.x4 = mk(4.0 * xr, 4.0 * xi);
    w.dir = mk(1.0, 0.0);
    w.lam2 = a.lam2;
    w.arc = false;
    w.hit = false;
    return w;
}

// Real segment: t = T k/(n-1), k = 1..n-1, T = log(1 + Lambda^2).
__device__ bool cut_hits_real_axis(const ScanArgs &a, double xr, double xi, int n, double T)
{
    CutWalk w = cut_walk_begin(a, xr, xi);
    cut_walk_straight<true>(w, n, T);
    return w.hit;
}

// Ray at phi = arg x (same t samples), then the closing arc, which starts
// where the ray ends: psi = phi (1 - k/(n-1)), k = 0..n-1, back to 0 the
// short way, or (the long way round) psi = phi + L k/(n-1),
// L = sign(phi) 2 pi - phi.
__device__ bool cut_hits_ray_arc(const ScanArgs &a, double xr, double xi, double phi, int n,
                                 double T, bool long_way)
{
    CutWalk w = cut_walk_begin(a, xr, xi);
    double s, c;
    sincos(phi, &s, &c);
    w.dir = mk(c, s);
    cut_walk_straight<false>(w, n, T);
    w.arc = true;
    cut_walk_arc(w, n, phi, long_way ? (phi > 0.0 ? 2.0 * M_PI : -2.0 * M_PI) - phi : -phi);
    return w.hit;
}

// One wave (one 8x8 tile) per workgroup: a tile walks one contour part (class
// R) or three (ray classes), so a four-wave workgroup would hold the slots of
// its finished waves until its slowest one ends.
__global__ void __launch_bounds__(64) obstruction_kernel(ScanArgs a, int n, double T, uint8_t *out)
{
    const int wave = blockIdx.x;
    if (wave >= a.n_tiles) return;
    const int lane = threadIdx.x & 63;
    const int ia = (wave % a.tiles_a) * 8 + lane % 8;
    const int ib = (wave / a.tiles_a) * 8 + lane / 8;
    if (ia >= a.n_re || ib >= a.n_im) return;
    const double xr = fma((double)ia + 0.5, a.d_re, a.re_lo);
    const double xi = fma((double)ib + 0.5, a.d_im, a.im_lo);
    const bool real_hit = cut_hits_real_axis(a, xr, xi, n, T);
    int sign = 0, info = 0;
    const PointArg pa = point_arg(xr, xi);
    int cls = classify(a, pa.v, pa.phi, &sign, &info);
    double ei = xi, phi = pa.phi;
    int ecls = cls;
    if (cls == kMirror) {  // the scan evaluates the conjugate point, if it has a contour
        ecls = classify(a, pa.v, -pa.phi, &sign);
        if (ecls == kMirror || ecls == kSingular || ecls == kLong) {
            cls = ecls = (info & kInfoRValid) ? kR : kLong;
        } else {
            ei = -xi;
            phi = -phi;
        }
    }
    int v = real_hit ? 1 : 0;
    if (cls == kSingular) {
        v |= 4;
    } else {
        const bool used_hit = ecls == kR ? (ei == xi ? real_hit : cut_hits_real_axis(a, xr, ei, n, T))
                                         : cut_hits_ray_arc(a, xr, ei, phi, n, T, ecls == kLong);
        if (used_hit) v |= 2;
    }
    out[(size_t)ib * (size_t)a.n_re + (size_t)ia] = (uint8_t)v;
}

}  // namespace

hipError_t launch_yscan(const ScanArgs &a, double xr, double xi, double mu2, int what,
                        hipStream_t s)
{
    if (a.n_tiles <= 0) return hipSuccess;
    const bool grouped = a.n_grp > 0;
    const auto kernel = a.poles ? (grouped ? yscan_kernel<true, true> : yscan_kernel<true, false>)
                                : (grouped ? yscan_kernel<false, true> : yscan_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3(a.n_tiles), dim3(64), 0, s, a, xr, xi, mu2, what);
    return hipGetLastError();
}

hipError_t launch_obstruction(const ScanArgs &a, int n, double T, uint8_t *out, hipStream_t s)
{
    if (a.n_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(obstruction_kernel, dim3(a.n_tiles), dim3(64), 0, s, a, n, T, out);
    return hipGetLastError();
}

}  // namespace gf
