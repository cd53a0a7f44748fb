// Weighted least-squares fits of the extrapolation zone (Sec. 3.2 step (ii))
// on gfx950: the fit itself, for one target shared by eight lanes (values read
// from the maps) or held by one (values read from a block's copy in LDS), with
// the same bits either way.  Included by the reference-map kernels only, and built
// without floating-point contraction like them.
#pragma once

#include <type_traits>

#include "lbrmt_internal.h"

namespace lbrmt {

__device__ __forceinline__ double det3(double a00, double a01, double a02, double a10,
                                       double a11, double a12, double a20, double a21,
                                       double a22)
{
    return a00 * (a11 * a22 - a12 * a21) - a01 * (a10 * a22 - a12 * a20) +
           a02 * (a10 * a21 - a11 * a20);
}

// a lane's partner value by a DPP move within its row (no LDS round trip;
// 64-bit values move as two halves)
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __int_as_float(dpp_move<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    return __hiloint2double(dpp_move<CTRL>(__double2hiint(v)), dpp_move<CTRL>(__double2loint(v)));
}
constexpr int DPP_XOR1 = 0xB1;         // quad_perm 1,0,3,2
constexpr int DPP_XOR2 = 0x4E;         // quad_perm 2,3,0,1
constexpr int DPP_HALF_MIRROR = 0x141; // lane 7 - i of an 8-lane group

// sum over the FIT_LANES = 8 lanes of a group (8 aligned lanes, all active
// together): lane i adds lane i ^ 1, then lane i ^ 2, then the other quad's
// sum from lane 7 - i.  Every lane ends with the same bits, since each
// addition sees the same two operands in either order.
static_assert(FIT_LANES == 8, "group_sum pairs the lanes of an 8-lane group");
template <typename V>
__device__ __forceinline__ V group_sum(V v)
{
    v += dpp_move<DPP_XOR1>(v);
    v += dpp_move<DPP_XOR2>(v);
    v += dpp_move<DPP_HALF_MIRROR>(v);
    return v;
}

// A target's fit is split over eight parts by the window node's number mod 8,
// each summed node by node, and the eight sums are added as the tree above
// adds lanes.  SPL = 1: part = lane of an 8-lane group.  SPL = 8: one lane
// holds all parts and makes the same additions in the same order.
template <int SPL, typename V>
__device__ __forceinline__ V parts_sum(const V (&p)[SPL])
{
    static_assert(SPL == 1 || SPL == 8, "eight lanes or one");
    if constexpr (SPL == 1) return group_sum(p[0]);
    else return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
}

// Sums of the normal equations in coordinates centred at the target, for scan
// windows wider than half-width 2.  The normal matrix and its well-posedness test are kept
// in double (sums of w dx dy with w a power of two, or the normal weight); the
// right-hand sides are accumulated in the storage precision C of the
// reference map.
template <typename C>
struct Fit {
    double M00, M01, M02, M11, M12, M22;
    C bX0, bX1, bX2, bY0, bY1, bY2;
    __device__ __forceinline__ void zero()
    {
        M00 = M01 = M02 = M11 = M12 = M22 = 0.0;
        bX0 = bX1 = bX2 = bY0 = bY1 = bY2 = C(0);
    }
    // one valid node at offset (a, b) from the target, weight of
    // Eq. (3_2_extrap_weight)
    __device__ __forceinline__ void add(int a, int b, bool use_n, double nxh, double nyh, C xv,
                                        C yv)
    {
        double w = ldexp(1.0, -(abs(a) + abs(b)));
        if (use_n) {
            const double ddx = -(double)a, ddy = -(double)b;  // d = x_target - x_valid
            const double dn = (ddx * nxh + ddy * nyh) / sqrt(ddx * ddx + ddy * ddy);
            w = dn * w > 0.0 ? dn * w : 0.0;
        }
        const double dx = a, dy = b;
        M00 += w * dx * dx;
        M01 += w * dx * dy;
        M02 += w * dx;
        M11 += w * dy * dy;
        M12 += w * dy;
        M22 += w;
        const C wc = C(w), cx = C(a), cy = C(b);
        bX0 += wc * cx * xv;
        bX1 += wc * cy * xv;
        bX2 += wc * xv;
        bY0 += wc * cx * yv;
        bY1 += wc * cy * yv;
        bY2 += wc * yv;
    }
    // intercept of the weighted linear fit, if well posed
    __device__ __forceinline__ bool solve(double det_rel, C& x, C& y) const
    {
        const double m00 = M00, m01 = M01, m02 = M02, m11 = M11, m12 = M12, m22 = M22;
        const double det = det3(m00, m01, m02, m01, m11, m12, m02, m12, m22);
        if (!(det > det_rel * m22 * m22 * m22)) return false;
        if (sizeof(C) == 8) {
            x = C(det3(m00, m01, bX0, m01, m11, bX1, m02, m12, bX2) / det);
            y = C(det3(m00, m01, bY0, m01, m11, bY1, m02, m12, bY2) / det);
        } else {
            // Cramer in float: the cofactors of the third column weigh the
            // right-hand sides
            const C c0 = C(m01 * m12 - m11 * m02), c1 = C(m01 * m02 - m00 * m12);
            const C c2 = C(m00 * m11 - m01 * m01), id = C(1.0 / det);
            x = (c0 * bX0 + c1 * bX1 + c2 * bX2) * id;
            y = (c0 * bY0 + c1 * bY1 + c2 * bY2) * id;
        }
        return true;
    }
};

// the eight lanes' sums reduced, then the intercept, if the window held three
// valid nodes and the fit is well posed
template <typename T>
__device__ __forceinline__ bool fit_finish(double det_rel, Fit<T>& f, int count, T& xo, T& yo)
{
    count = group_sum(count);
    if (count < 3) return false;
    f.M00 = group_sum(f.M00);
    f.M01 = group_sum(f.M01);
    f.M02 = group_sum(f.M02);
    f.M11 = group_sum(f.M11);
    f.M12 = group_sum(f.M12);
    f.M22 = group_sum(f.M22);
    f.bX0 = group_sum(f.bX0);
    f.bX1 = group_sum(f.bX1);
    f.bX2 = group_sum(f.bX2);
    f.bY0 = group_sum(f.bY0);
    f.bY1 = group_sum(f.bY1);
    f.bY2 = group_sum(f.bY2);
    return f.solve(det_rel, xo, yo);
}

// ---- the scan window of half-width 2 (side 5, 25 nodes, node q = 5 (b + 2) +
// a + 2 at offset (a, b)), where nearly every fit ends.
//
// With the power-of-two weights w = 2^-(|a|+|b|) the entries of the normal
// matrix are multiples of 1/16 that depend on nothing but which nodes are
// valid, a 25-bit mask: times 16 they are sums of small integers, counted with
// a few masks and bit counts.  Cofactors (times 256) and determinant (times
// 4096) are then exact in 24-bit products, so the well-posedness decision and
// the cofactors are those of sums in double, bit for bit.
struct Geo2 {
    int m00, m01, m02, m11, m12;  // 16 times the entries
    int det;                      // 4096 times the determinant
    bool ok;                      // at least three nodes and well posed
    // 256 times the cofactors of the third column
    __device__ __forceinline__ int c0() const { return __mul24(m01, m12) - __mul24(m11, m02); }
    __device__ __forceinline__ int c1() const { return __mul24(m01, m02) - __mul24(m00, m12); }
    __device__ __forceinline__ int c2() const { return __mul24(m00, m11) - __mul24(m01, m01); }
};

// bits of the window nodes (a, b) with the given property
template <typename F>
__host__ __device__ constexpr unsigned win2_mask(F f)
{
    unsigned m = 0;
    for (int b = -2; b <= 2; b++)
        for (int a = -2; a <= 2; a++)
            if ((a || b) && f(a, b)) m |= 1u << (5 * (b + 2) + a + 2);
    return m;
}
__host__ __device__ constexpr int iabs(int v) { return v < 0 ? -v : v; }

// mask: the valid nodes (the target's own bit 12 clear)
__device__ __forceinline__ Geo2 geo2(unsigned mask, double det_rel)
{
    // 16 w by |a| + |b| = 1 .. 4: 8, 4, 2, 1
#define NB(EXPR)                                                                       \
    [&]() {                                                                            \
        constexpr unsigned m_ = win2_mask([](int a, int b) { return EXPR; });          \
        return __popc(mask & m_);                                                      \
    }()
    const int m22 = 8 * NB(iabs(a) + iabs(b) == 1) + 4 * NB(iabs(a) + iabs(b) == 2) +
                    2 * NB(iabs(a) + iabs(b) == 3) + NB(iabs(a) + iabs(b) == 4);
    // 16 w a = +-8 2^-|b| for either |a|
    const int m02 = 8 * (NB(a > 0 && b == 0) - NB(a < 0 && b == 0)) +
                    4 * (NB(a > 0 && iabs(b) == 1) - NB(a < 0 && iabs(b) == 1)) +
                    2 * (NB(a > 0 && iabs(b) == 2) - NB(a < 0 && iabs(b) == 2));
    const int m12 = 8 * (NB(b > 0 && a == 0) - NB(b < 0 && a == 0)) +
                    4 * (NB(b > 0 && iabs(a) == 1) - NB(b < 0 && iabs(a) == 1)) +
                    2 * (NB(b > 0 && iabs(a) == 2) - NB(b < 0 && iabs(a) == 2));
    // 16 w a^2 = 8 |a| 2^-|b|
    const int m00 = 16 * NB(iabs(a) == 2 && b == 0) +
                    8 * NB((iabs(a) == 1 && b == 0) || (iabs(a) == 2 && iabs(b) == 1)) +
                    4 * NB((iabs(a) == 1 && iabs(b) == 1) || (iabs(a) == 2 && iabs(b) == 2)) +
                    2 * NB(iabs(a) == 1 && iabs(b) == 2);
    const int m11 = 16 * NB(iabs(b) == 2 && a == 0) +
                    8 * NB((iabs(b) == 1 && a == 0) || (iabs(b) == 2 && iabs(a) == 1)) +
                    4 * NB((iabs(b) == 1 && iabs(a) == 1) || (iabs(b) == 2 && iabs(a) == 2)) +
                    2 * NB(iabs(b) == 1 && iabs(a) == 2);
    // 16 w a b = +-4 for every a, b != 0
    const int m01 = 4 * (NB(a * b > 0) - NB(a * b < 0));
#undef NB
    Geo2 g;
    g.m00 = m00;
    g.m01 = m01;
    g.m02 = m02;
    g.m11 = m11;
    g.m12 = m12;
    g.det = __mul24(m02, g.c0()) + __mul24(m12, g.c1()) + __mul24(m22, g.c2());
    // (a power of two on both sides of det > det_rel (sum w)^3)
    const double dm = m22;
    g.ok = __popc(mask) >= 3 && (double)g.det > det_rel * dm * dm * dm;
    return g;
}

// the intercept by Cramer's rule in double (right-hand sides b0, b1, b2), the
// products in the order of det3
__device__ __forceinline__ double cramer(double m00, double m01, double m02, double m11,
                                         double m12, double c0, double b0, double b1, double b2,
                                         double det)
{
    return (m00 * (m11 * b2 - b1 * m12) - m01 * (m01 * b2 - b1 * m02) + b0 * c0) / det;
}

// What a lane (h: its number in the group) takes of the window.
template <typename T, int SPL>
struct Win2 {
    // slot s: part p = s % SPL of the lane, node q = 8 u + part, u = s / SPL
    // (one lane: slot = node)
    static constexpr int NS = SPL == 1 ? 4 : 25;

    __device__ __forceinline__ static constexpr int part(int s) { return s % SPL; }
    __device__ __forceinline__ static constexpr int node(int h, int s)
    {
        return SPL == 1 ? 8 * s + h : s;
    }
    __device__ __forceinline__ static constexpr int off_a(int h, int s) { return node(h, s) % 5 - 2; }
    __device__ __forceinline__ static constexpr int off_b(int h, int s) { return node(h, s) / 5 - 2; }
    // a node of the window, other than the target
    __device__ __forceinline__ static constexpr bool in(int h, int s)
    {
        return node(h, s) < 25 && node(h, s) != 12;
    }
    // 16 w = 16 2^-(|a|+|b|) of a slot (0 outside)
    __device__ __forceinline__ static constexpr int w16(int h, int s)
    {
        return in(h, s) ? 16 >> (iabs(off_a(h, s)) + iabs(off_b(h, s))) : 0;
    }

    // the group's validity mask
    __device__ __forceinline__ static unsigned mask_of(int h, const bool (&v)[NS])
    {
        int m = 0;
#pragma unroll
        for (int s = 0; s < NS; s++) m |= v[s] ? 1 << node(h, s) : 0;
        if (SPL == 1) {
            m |= dpp_move<DPP_XOR1>(m);
            m |= dpp_move<DPP_XOR2>(m);
            m |= dpp_move<DPP_HALF_MIRROR>(m);
        }
        return (unsigned)m;
    }

    // 1 / det, 1 <= det < 2^21 an integer: the hardware estimate and two
    // Newton steps, within one unit in the last place (rounded to float, every
    // such value is the rounded quotient: 4096 / det is no float and no
    // midpoint of two unless det is a power of two, where the steps are exact)
    __device__ __forceinline__ static double inverse(int det)
    {
        const double d = det;
        double r = __builtin_amdgcn_rcp(d);
        r = fma(fma(-d, r, 1.0), r, r);
        return fma(fma(-d, r, 1.0), r, r);
    }

    // Power-of-two weights: the right-hand sides and Cramer's rule, in double
    // (FP64) or float (FP32).  The weights times 8 (+-4 .. +-1/2 with a or b)
    // are exact factors, so fused adds round as separate ones do, and the
    // powers of two leave with the quotient.  xs, ys: zero at the nodes that
    // are not valid.
    __device__ __forceinline__ static void value(int h, const Geo2& g, const T (&xs)[NS],
                                                 const T (&ys)[NS], T& xo, T& yo)
    {
        T bX0[SPL], bX1[SPL], bX2[SPL], bY0[SPL], bY1[SPL], bY2[SPL];
#pragma unroll
        for (int p = 0; p < SPL; p++) {
            bX0[p] = bX1[p] = bX2[p] = bY0[p] = bY1[p] = bY2[p] = T(0);
#pragma unroll
            for (int s = p; s < NS; s += SPL) {
                if (SPL > 1 && !in(h, s)) continue;
                const int i = off_a(h, s), j = off_b(h, s);
                const T w = T(w16(h, s)) * T(0.5), wa = w * T(i), wb = w * T(j);
                if (SPL == 1 || i) bX0[p] = fma(wa, xs[s], bX0[p]);
                if (SPL == 1 || j) bX1[p] = fma(wb, xs[s], bX1[p]);
                bX2[p] = fma(w, xs[s], bX2[p]);
                if (SPL == 1 || i) bY0[p] = fma(wa, ys[s], bY0[p]);
                if (SPL == 1 || j) bY1[p] = fma(wb, ys[s], bY1[p]);
                bY2[p] = fma(w, ys[s], bY2[p]);
            }
        }
        const T X0 = parts_sum<SPL>(bX0), X1 = parts_sum<SPL>(bX1), X2 = parts_sum<SPL>(bX2);
        const T Y0 = parts_sum<SPL>(bY0), Y1 = parts_sum<SPL>(bY1), Y2 = parts_sum<SPL>(bY2);
        if constexpr (sizeof(T) == 8) {
            // numerator times 2048, determinant times 4096
            const double c0 = g.c0(), d = 0.5 * g.det;
            xo = cramer(g.m00, g.m01, g.m02, g.m11, g.m12, c0, X0, X1, X2, d);
            yo = cramer(g.m00, g.m01, g.m02, g.m11, g.m12, c0, Y0, Y1, Y2, d);
        } else {
            const T f0 = T(g.c0()) / T(256), f1 = T(g.c1()) / T(256), f2 = T(g.c2()) / T(256);
            const T id = T(512.0 * inverse(g.det));
            xo = (f0 * X0 + f1 * X1 + f2 * X2) * id;
            yo = (f0 * Y0 + f1 * Y1 + f2 * Y2) * id;
        }
    }

    // Normal weights of layers 1 and 2 (outward normal (nxh, nyh) at the
    // target): w max(0, d.n / |d|), d = -(a, b).  The products with a, b, a^2,
    // ab, b^2 (0, +-1, +-2, +-4) are exact, so fused adds round as separate
    // ones do.  NW holds what the values are weighed with.
    struct NW {
        T k[NS];
        double m00, m01, m02, m11, m12, det;
    };
    // (every lane of the group gets the same verdict)
    __device__ __forceinline__ static bool weights_n(int h, int count, const bool (&v)[NS],
                                                     double nxh, double nyh, double det_rel,
                                                     NW& w)
    {
        double m00[SPL], m01[SPL], m02[SPL], m11[SPL], m12[SPL], m22[SPL];
#pragma unroll
        for (int p = 0; p < SPL; p++) {
            m00[p] = m01[p] = m02[p] = m11[p] = m12[p] = m22[p] = 0.0;
#pragma unroll
            for (int s = p; s < NS; s += SPL) {
                w.k[s] = T(0);
                if (SPL > 1 && !in(h, s)) continue;
                const int i = off_a(h, s), j = off_b(h, s), d2 = i * i + j * j;
                const double a = i, b = j, w0 = w16(h, s) * (1.0 / 16.0);
                // d.n / RN(sqrt(d2)), RN(sqrt(d2)) = sc 2^k with sc = 1,
                // sqrt 2 or sqrt 5: the product with the rounded reciprocal of
                // sc and one exact residual (the correctly rounded quotient),
                // then 2^-k w
                const double t = -a * nxh + -b * nyh;
                double dn = t;
                if (SPL == 1 || d2 == 5 || d2 == 2 || d2 == 8) {
                    const bool r5 = d2 == 5, r2 = d2 == 2 || d2 == 8;
                    const double sc = r5 ? 2.23606797749978969641 : r2 ? 1.41421356237309504880 : 1.0;
                    const double rc = r5 ? 0.44721359549995793928 : r2 ? 0.70710678118654752440 : 1.0;
                    const double q = t * rc;
                    dn = fma(fma(-q, sc, t), rc, q);
                }
                dn *= d2 == 4 || d2 == 8 ? 0.5 * w0 : w0;
                const double wn = v[s] && dn > 0.0 ? dn : 0.0;
                w.k[s] = T(wn);
                m22[p] += wn;
                if (SPL == 1 || i) m02[p] = fma(wn, a, m02[p]);
                if (SPL == 1 || j) m12[p] = fma(wn, b, m12[p]);
                if (SPL == 1 || i) m00[p] = fma(wn, a * a, m00[p]);
                if (SPL == 1 || (i && j)) m01[p] = fma(wn, a * b, m01[p]);
                if (SPL == 1 || j) m11[p] = fma(wn, b * b, m11[p]);
            }
        }
        w.m00 = parts_sum<SPL>(m00);
        w.m01 = parts_sum<SPL>(m01);
        w.m02 = parts_sum<SPL>(m02);
        w.m11 = parts_sum<SPL>(m11);
        w.m12 = parts_sum<SPL>(m12);
        const double M22 = parts_sum<SPL>(m22);
        w.det = det3(w.m00, w.m01, w.m02, w.m01, w.m11, w.m12, w.m02, w.m12, M22);
        return count >= 3 && w.det > det_rel * M22 * M22 * M22;
    }
    // power-of-two weights in the same form
    __device__ __forceinline__ static bool weights_2(int h, unsigned mask, double det_rel, NW& w)
    {
        const Geo2 g = geo2(mask, det_rel);
#pragma unroll
        for (int s = 0; s < NS; s++) w.k[s] = T(w16(h, s)) / T(16);
        w.m00 = g.m00 / 16.0;
        w.m01 = g.m01 / 16.0;
        w.m02 = g.m02 / 16.0;
        w.m11 = g.m11 / 16.0;
        w.m12 = g.m12 / 16.0;
        w.det = g.det / 4096.0;
        return g.ok;
    }
    __device__ __forceinline__ static void value_n(int h, const NW& w, const T (&xs)[NS],
                                                   const T (&ys)[NS], T& xo, T& yo)
    {
        T bX0[SPL], bX1[SPL], bX2[SPL], bY0[SPL], bY1[SPL], bY2[SPL];
#pragma unroll
        for (int p = 0; p < SPL; p++) {
            bX0[p] = bX1[p] = bX2[p] = bY0[p] = bY1[p] = bY2[p] = T(0);
#pragma unroll
            for (int s = p; s < NS; s += SPL) {
                if (SPL > 1 && !in(h, s)) continue;
                const int i = off_a(h, s), j = off_b(h, s);
                const T a = T(i), b = T(j);
                const T wx = w.k[s] * xs[s], wy = w.k[s] * ys[s];
                if (SPL == 1 || i) bX0[p] = fma(a, wx, bX0[p]);
                if (SPL == 1 || j) bX1[p] = fma(b, wx, bX1[p]);
                bX2[p] += wx;
                if (SPL == 1 || i) bY0[p] = fma(a, wy, bY0[p]);
                if (SPL == 1 || j) bY1[p] = fma(b, wy, bY1[p]);
                bY2[p] += wy;
            }
        }
        const T X0 = parts_sum<SPL>(bX0), X1 = parts_sum<SPL>(bX1), X2 = parts_sum<SPL>(bX2);
        const T Y0 = parts_sum<SPL>(bY0), Y1 = parts_sum<SPL>(bY1), Y2 = parts_sum<SPL>(bY2);
        const double c0 = w.m01 * w.m12 - w.m11 * w.m02;
        if constexpr (sizeof(T) == 8) {
            xo = cramer(w.m00, w.m01, w.m02, w.m11, w.m12, c0, X0, X1, X2, w.det);
            yo = cramer(w.m00, w.m01, w.m02, w.m11, w.m12, c0, Y0, Y1, Y2, w.det);
        } else {
            const T f0 = T(c0), f1 = T(w.m01 * w.m02 - w.m00 * w.m12);
            const T f2 = T(w.m00 * w.m11 - w.m01 * w.m01), id = T(1.0 / w.det);
            xo = (f0 * X0 + f1 * X1 + f2 * X2) * id;
            yo = (f0 * Y0 + f1 * Y1 + f2 * Y2) * id;
        }
    }
};

}  // namespace lbrmt
