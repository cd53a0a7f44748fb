// Discrete adjoint of one coupled step (FP64, one solid): the exact reverse
// of the forward step of k_band.hip and k_lb.hip, with every discrete
// decision (solid set, layers, scan-window size, upwind side, stencil and
// singular-J fallbacks) taken as the forward step took it.  One step n of
// Alg. 1 is, in forward order: moments u^n (with half of F^{n-1}),
// advection of xi on S^n (Eq. (3_1_refmap_adv)), layer-by-layer weighted
// least-squares extrapolation (Sec. 3.2), relabel phi^{n+1} = phi0(xi^{n+1}),
// half-edge stresses and their divergence F^n (Eqs. (3_3_refmap_jacobian) to
// (3_3_div_solid_stress), (2_4_F_divs)), collision with the SFC equilibrium
// and Guo forcing (Eqs. (2_3_feq_sfc), (2_2_Fi)), streaming with bounce-back
// and the moving lid (Sec. 3.5).  The kernels below run them backwards.
//
// Adjoint fields: fbar (natural populations f_i(x), [9][ny][nx]), xbar, ybar
// and pbar (xi and phi on the padded reference-map grid), Fbar (force planes,
// [ny][nx]); scalar adjoints of G and of the lid speed accumulate in acc[0],
// acc[1].  Scatters that several threads share use double atomics.
#include <hip/hip_runtime.h>

#include "lbrmt_internal.h"
#include "fit_window.h"

namespace lbrmt {

namespace {

constexpr double AW0 = 4.0 / 9.0, AW1 = 1.0 / 9.0, AW2 = 1.0 / 36.0;
__constant__ int ACX[NQ] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__constant__ int ACY[NQ] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
__constant__ int AOPP[NQ] = {0, 3, 4, 1, 2, 7, 8, 5, 6};
__constant__ double AWQ[NQ] = {AW0, AW1, AW1, AW1, AW1, AW2, AW2, AW2, AW2};

// smoothed Heaviside of Eq. (2_3_heaviside) and its derivative
__device__ __forceinline__ double hv(double p, double eps)
{
    if (p <= -eps) return 0.0;
    if (p >= eps) return 1.0;
    return 0.5 * (1.0 + p / eps + sin(M_PI * p / eps) / M_PI);
}
__device__ __forceinline__ double dhv(double p, double eps)
{
    if (p <= -eps || p >= eps) return 0.0;
    return 0.5 / eps * (1.0 + cos(M_PI * p / eps));
}

// gradient of the reference level set phi0 at reference point (X, Y)
__device__ void grad_phi0(const BodyP& b, double X, double Y, double& gx, double& gy)
{
    const double dx = X - b.cx, dy = Y - b.cy;
    const double d = sqrt(dx * dx + dy * dy);
    gx = gy = 0.0;
    if (!(d > 0.0)) return;
    if (b.shape != 1) {
        gx = dx / d;
        gy = dy / d;
        return;
    }
    // phi0 = d (1 - 1/q), q = |(x'/a, y'/b)| in the body frame
    const double xp = b.ct * dx + b.st * dy, yp = -b.st * dx + b.ct * dy;
    const double ua = xp / (b.R * b.R), ub = yp / (b.Rb * b.Rb);
    const double q = sqrt((xp / b.R) * (xp / b.R) + (yp / b.Rb) * (yp / b.Rb));
    const double dqx = (ua * b.ct - ub * b.st) / q, dqy = (ua * b.st + ub * b.ct) / q;
    gx = dx / d * (1.0 - 1.0 / q) + d * dqx / (q * q);
    gy = dy / d * (1.0 - 1.0 / q) + d * dqy / (q * q);
}

// natural populations f_i(x) of the pull-stored lattice A (bounce-back at walls)
__device__ __forceinline__ void nat_gather(const GridP& g, const double* __restrict__ A, int i,
                                           int j, double f[NQ])
{
    const long long P = g.plane;
    const long long n = (long long)j * g.pitch + i;
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        int si = i - ACX[q], sj = j - ACY[q];
        if (g.px) si = wrap_axis(si, g.nx);
        if (g.py) sj = wrap_axis(sj, g.ny);
        const bool in = si >= 0 && si < g.nx && sj >= 0 && sj < g.ny;
        f[q] = in ? A[q * P + (long long)sj * g.pitch + si] : A[AOPP[q] * P + n];
    }
}

__device__ __forceinline__ double block_sum(double v)
{
    __shared__ double red[16];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x + 63) / 64; k++) s += red[k];
    __syncthreads();
    return s;
}

}  // namespace

// ---------------------------------------------------------------- lattice
// Streaming, lid, collision and moments backwards, one node per thread:
// fbar_out = dL/df^n (natural), Fpbar = dL/dF^{n-1} (this part), Fcbar +=
// the Guo part of dL/dF^n, pbar1 += the density-excess part of dL/dphi^{n+1}.
__global__ __launch_bounds__(256) void k_adj_lattice(GridP g, BodyP b, AdjSnap s, AdjBufs a)
{
    const long long N = (long long)g.nx * g.ny;
    const Rect wp = window_of(s.win, 0, g);
    const Rect wc = window_of(s.win, 1, g);
    const double om = g.omega, cf = g.cforce;
    double ubar_lid = 0.0;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < N;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(e % g.nx), j = (int)(e / g.nx);
        const long long n = (long long)j * g.pitch + i;
        double f[NQ];
        nat_gather(g, s.A, i, j, f);
        double rho = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            rho += f[q];
            jx += ACX[q] * f[q];
            jy += ACY[q] * f[q];
        }
        const bool inp = wp.has(i, j), inc = wc.has(i, j);
        const double Fpx = inp ? s.fpx[n] : s.fpo[0], Fpy = inp ? s.fpy[n] : s.fpo[1];
        const double Fx = inc ? s.fcx[n] : g.fext_x, Fy = inc ? s.fcy[n] : g.fext_y;
        const double ux = (jx + 0.5 * Fpx) / rho, uy = (jy + 0.5 * Fpy) / rho;
        double p1 = INFINITY;
        if (b.present && inc) p1 = s.P1[pidx(g, i, j)];
        const double drs = b.present ? b.rho_s - g.rho_f : 0.0;
        // adjoint of the post-collision values: where each one streams to
        const bool top = !g.py && j == g.ny - 1;
        double gq[NQ];
        double rhobar = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            int di = i + ACX[q], dj = j + ACY[q];
            if (g.px) di = wrap_axis(di, g.nx);
            if (g.py) dj = wrap_axis(dj, g.ny);
            const bool in = di >= 0 && di < g.nx && dj >= 0 && dj < g.ny;
            gq[q] = in ? a.fb_in[q * N + (long long)dj * g.nx + di] : a.fb_in[AOPP[q] * N + e];
            if (top && (q == 5 || q == 6)) {
                // f_opp(q)(x) = fhat_q(x) -/+ rho U / 6 through the lid (Sec. 3.5)
                const double sg = q == 5 ? -1.0 : 1.0;
                const double fo = a.fb_in[AOPP[q] * N + e];
                if (!g.lid_rho_mode) rhobar += fo * sg * g.lid_ux / 6.0;
                ubar_lid += fo * sg * (g.lid_rho_mode ? g.rho_f : rho) / 6.0;
            }
        }
        // collision: fhat_q = f_q + om (feq_q - f_q) + cf Fi_q
        const double usq = ux * ux + uy * uy, uF = ux * Fx + uy * Fy;
        double uxb = 0.0, uyb = 0.0, drb = 0.0, Fxb = 0.0, Fyb = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            const double eb = om * gq[q], Fib = cf * gq[q], w = AWQ[q];
            const double cx = ACX[q], cy = ACY[q];
            const double cu = cx * ux + cy * uy, cF = cx * Fx + cy * Fy;
            if (q == 0) {
                rhobar += eb * w * (1.0 - 1.5 * usq);
                uxb += eb * w * rho * (-3.0 * ux);
                uyb += eb * w * rho * (-3.0 * uy);
                drb += eb * (5.0 / 9.0);
                uxb += Fib * w * (-3.0 * Fx);
                uyb += Fib * w * (-3.0 * Fy);
                Fxb += Fib * w * (-3.0 * ux);
                Fyb += Fib * w * (-3.0 * uy);
            } else {
                rhobar += eb * w * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * usq);
                uxb += eb * w * rho * (3.0 * cx + 9.0 * cu * cx - 3.0 * ux);
                uyb += eb * w * rho * (3.0 * cy + 9.0 * cu * cy - 3.0 * uy);
                drb += eb * (-w);
                uxb += Fib * w * (-3.0 * Fx + 9.0 * cF * cx);
                uyb += Fib * w * (-3.0 * Fy + 9.0 * cF * cy);
                Fxb += Fib * w * (3.0 * (cx - ux) + 9.0 * cu * cx);
                Fyb += Fib * w * (3.0 * (cy - uy) + 9.0 * cu * cy);
            }
        }
        // u = (j + F^{n-1} / 2) / rho
        const double jxb = uxb / rho, jyb = uyb / rho;
        rhobar += -(uxb * ux + uyb * uy) / rho;
#pragma unroll
        for (int q = 0; q < NQ; q++)
            a.fb_out[q * N + e] = (1.0 - om) * gq[q] + rhobar + ACX[q] * jxb + ACY[q] * jyb;
        a.Fpbar_x[e] = inp ? 0.5 * jxb : 0.0;
        a.Fpbar_y[e] = inp ? 0.5 * jyb : 0.0;
        if (inc) {
            a.Fcbar_x[e] += Fxb;
            a.Fcbar_y[e] += Fyb;
            // density excess (1 - H(phi^{n+1})) (rho_s - rho_f), Eq. (2_3_drho)
            if (p1 < INFINITY) a.pbar1[pidx(g, i, j)] += drb * (-dhv(p1, g.eps)) * drs;
        }
    }
    const double t = block_sum(ubar_lid);
    if (threadIdx.x == 0 && t != 0.0) atomicAdd(&a.acc[1], t);
}

// ---------------------------------------------------------------- force
// Half-edge stresses backwards: edge e (x-edge between a = (i-1, j) and
// b = (i, j), y-edge between a = (i, j-1) and b) enters F(b) with a minus
// sign and F(a) with a plus sign.  dL/d(tau_e) -> lambda_e (phi^{n+1} at a
// and b), J_e (xi^{n+1} at the six stencil nodes) and G.  Also the buoyancy
// and fluid-force terms of F at each interior node.
__device__ void adj_edge(const GridP& g, const BodyP& b, const AdjSnap& s, const AdjBufs& a,
                         const Rect& V, const Rect& wc, int i, int j, int dir, double& Gbar)
{
    const int ia = dir == 0 ? i - 1 : i, ja = dir == 0 ? j : j - 1;
    auto fbar = [&](int x, int y, double& fx, double& fy) {
        fx = fy = 0.0;
        if (g.px) x = wrap_axis(x, g.nx);
        if (g.py) y = wrap_axis(y, g.ny);
        if (x < 0 || x >= g.nx || y < 0 || y >= g.ny || !wc.has(x, y)) return;
        fx = a.Fcbar_x[(long long)y * g.nx + x];
        fy = a.Fcbar_y[(long long)y * g.nx + x];
    };
    double fax, fay, fbx, fby;
    fbar(ia, ja, fax, fay);
    fbar(i, j, fbx, fby);
    // dL/d(tau_xx, tau_xy, tau_yy) of this edge
    double tb0, tb1, tb2;
    if (dir == 0) {
        tb0 = fax - fbx;
        tb1 = fay - fby;
        tb2 = 0.0;
    } else {
        tb0 = 0.0;
        tb1 = fax - fbx;
        tb2 = fay - fby;
    }
    if (tb0 == 0.0 && tb1 == 0.0 && tb2 == 0.0) return;
    // the six stencil nodes a, b, s1..s4 (as in the forward force pass)
    int ci[6], cj[6];
    ci[0] = ia; cj[0] = ja;
    ci[1] = i; cj[1] = j;
    if (dir == 0) {
        ci[2] = i; cj[2] = j + 1;
        ci[3] = i - 1; cj[3] = j + 1;
        ci[4] = i; cj[4] = j - 1;
        ci[5] = i - 1; cj[5] = j - 1;
    } else {
        ci[2] = i + 1; cj[2] = j;
        ci[3] = i + 1; cj[3] = j - 1;
        ci[4] = i - 1; cj[4] = j;
        ci[5] = i - 1; cj[5] = j - 1;
    }
    long long k[6];
    double X[6], Y[6], P[6];
    for (int t = 0; t < 6; t++) {
        int x = ci[t], y = cj[t];
        const bool in = canon(g, x, y) && V.has(x, y);
        k[t] = in ? pidx(g, x, y) : -1;
        P[t] = in ? s.P1[k[t]] : INFINITY;
        X[t] = in ? s.X1[k[t]] : 0.0;
        Y[t] = in ? s.Y1[k[t]] : 0.0;
    }
    if (!(P[0] < INFINITY) || !(P[1] < INFINITY)) return;
    const double pe = 0.5 * (P[0] + P[1]);
    const double lam = 1.0 - hv(pe, g.eps);
    if (!(lam > 0.0)) return;
    for (int t = 2; t < 6; t++)
        if (!(P[t] < INFINITY)) return;
    const double nX = X[1] - X[0], nY = Y[1] - Y[0];
    const double tX = (X[2] + X[3] - X[4] - X[5]) / 4.0;
    const double tY = (Y[2] + Y[3] - Y[4] - Y[5]) / 4.0;
    double J0, J1, J2, J3;
    if (dir == 0) {
        J0 = nX; J1 = tX; J2 = nY; J3 = tY;
    } else {
        J0 = tX; J1 = nX; J2 = tY; J3 = nY;
    }
    const double det = J0 * J3 - J1 * J2;
    if (!(det > g.detJ_min)) return;
    const double F00 = J3 / det, F01 = -J1 / det, F10 = -J2 / det, F11 = J0 / det;
    const double Bxx = F00 * F00 + F01 * F01, Bxy = F00 * F10 + F01 * F11;
    const double Byy = F10 * F10 + F11 * F11, tr = Bxx + Byy;
    // deviatoric parts per unit G, Eq. (3_3_solid_stress)
    const double s0 = Bxx - (tr + 1.0) / 3.0, s1 = Bxy, s2 = Byy - (tr + 1.0) / 3.0;
    const double G = b.G;
    // edge stress = lam G (s0, s1, s2)
    const double lamb = G * (tb0 * s0 + tb1 * s1 + tb2 * s2);
    Gbar += lam * (tb0 * s0 + tb1 * s1 + tb2 * s2);
    const double pb = lamb * (-dhv(pe, g.eps)) * 0.5;
    if (pb != 0.0) {
        atomicAdd(&a.pbar1[k[0]], pb);
        atomicAdd(&a.pbar1[k[1]], pb);
    }
    // B adjoint (tau_s = G (B - (tr B + 1)/3 I))
    const double t0 = lam * G * tb0, t1 = lam * G * tb1, t2 = lam * G * tb2;
    const double Bxxb = t0 * (2.0 / 3.0) - t2 / 3.0, Byyb = t2 * (2.0 / 3.0) - t0 / 3.0;
    const double Bxyb = t1;
    // F adjoint (B = F F^T)
    const double Fb00 = 2.0 * F00 * Bxxb + F10 * Bxyb, Fb01 = 2.0 * F01 * Bxxb + F11 * Bxyb;
    const double Fb10 = F00 * Bxyb + 2.0 * F10 * Byyb, Fb11 = F01 * Bxyb + 2.0 * F11 * Byyb;
    // J adjoint (F = J^{-1}): Jbar = -F^T Fbar F^T
    const double m00 = F00 * Fb00 + F10 * Fb10, m01 = F00 * Fb01 + F10 * Fb11;
    const double m10 = F01 * Fb00 + F11 * Fb10, m11 = F01 * Fb01 + F11 * Fb11;
    const double Jb0 = -(m00 * F00 + m01 * F01), Jb1 = -(m00 * F10 + m01 * F11);
    const double Jb2 = -(m10 * F00 + m11 * F01), Jb3 = -(m10 * F10 + m11 * F11);
    double nXb, tXb, nYb, tYb;
    if (dir == 0) {
        nXb = Jb0; tXb = Jb1; nYb = Jb2; tYb = Jb3;
    } else {
        tXb = Jb0; nXb = Jb1; tYb = Jb2; nYb = Jb3;
    }
    const double cX[6] = {-nXb, nXb, tXb / 4.0, tXb / 4.0, -tXb / 4.0, -tXb / 4.0};
    const double cY[6] = {-nYb, nYb, tYb / 4.0, tYb / 4.0, -tYb / 4.0, -tYb / 4.0};
    for (int t = 0; t < 6; t++) {
        if (cX[t] != 0.0) atomicAdd(&a.xbar1[k[t]], cX[t]);
        if (cY[t] != 0.0) atomicAdd(&a.ybar1[k[t]], cY[t]);
    }
}

__global__ __launch_bounds__(256) void k_adj_force(GridP g, BodyP b, AdjSnap s, AdjBufs a)
{
    const Rect wc = window_of(s.win, 1, g);
    const Rect V = wc;  // the force pass's window: where xi^{n+1}, phi^{n+1} are valid
    double Gbar = 0.0;
    const int ex = g.nx + (g.px ? 0 : 1), ey = g.ny + (g.py ? 0 : 1);
    const long long NE = (long long)ex * ey;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < NE;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(e % ex), j = (int)(e / ex);
        if (b.present) {
            if (j < g.ny) adj_edge(g, b, s, a, V, wc, i, j, 0, Gbar);
            if (i < g.nx) adj_edge(g, b, s, a, V, wc, i, j, 1, Gbar);
        }
        // buoyancy (1 - H)(rho_s - rho_f) g and fluid force H f_ext at node (i, j)
        if (b.present && i < g.nx && j < g.ny && wc.has(i, j)) {
            const long long kk = pidx(g, i, j);
            const double p = s.P1[kk];
            if (p < INFINITY) {
                const long long m = (long long)j * g.nx + i;
                const double fx = a.Fcbar_x[m], fy = a.Fcbar_y[m];
                const double dh = dhv(p, g.eps);
                const double v = (fx * g.gx + fy * g.gy) * (-dh) * (b.rho_s - g.rho_f) +
                                 (fx * g.fext_x + fy * g.fext_y) * dh;
                if (v != 0.0) atomicAdd(&a.pbar1[kk], v);
            }
        }
    }
    const double t = block_sum(Gbar);
    if (threadIdx.x == 0 && t != 0.0) atomicAdd(&a.acc[0], t);
}

// ---------------------------------------------------------------- relabel
// phi^{n+1} = phi0(xi^{n+1}) at every node holding a map: pbar1 -> xbar1,
// then pbar1 is spent (cleared).
__global__ __launch_bounds__(256) void k_adj_relabel(GridP g, BodyP b, AdjSnap s, AdjBufs a)
{
    const Rect V = window_of(s.win, 1, g);
    if (!V.ok) return;
    const int w = V.i1 - V.i0 + 1, h = V.j1 - V.j0 + 1;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < (long long)w * h;
         e += (long long)gridDim.x * blockDim.x) {
        int i = V.i0 + (int)(e % w), j = V.j0 + (int)(e / w);
        if (!canon(g, i, j)) continue;
        const long long k = pidx(g, i, j);
        const double pb = a.pbar1[k];
        if (pb == 0.0) continue;
        a.pbar1[k] = 0.0;
        if (!(s.P1[k] < INFINITY)) continue;
        double gx, gy;
        grad_phi0(b, s.X1[k], s.Y1[k], gx, gy);
        a.xbar1[k] += pb * gx;
        a.ybar1[k] += pb * gy;
    }
}

// ---------------------------------------------------------------- extrapolation
// One target of layer l backwards: the fitted intercept c = e3^T M^{-1} b with
// M = sum w a a^T, b = sum w a xi (a = (dx, dy, 1) in target-centred
// coordinates) sends dL/dc to every valid node k with weight w_k (a_k . s),
// s = M^{-1} e3; with the normal weights of layers 1 and 2 the weights
// themselves depend on phi^n at the target's four neighbours:
// dc/dw_k = (a_k . s)(xi_k - a_k . p), p = M^{-1} b.
// Scan windows of half-width 2 .. rmax (RMAX > 0: at compile time).
// node(aa, bb): the handle of the scan node at that offset, -1 if it is not
// valid (no map, or of layer l or later); val(h, x, y): xi^{n+1} there;
// add(h, vx, vy): adds to its adjoint.  own: the target's normal is this
// call's to pass on (to pbar0).
template <int RMAX, typename Node, typename Val, typename Add>
__device__ __forceinline__ void adj_fit_target(const GridP& g, const Rect& D, const AdjSnap& s,
                                               const AdjBufs& a, int l, int i, int j, double Xb,
                                               double Yb, bool own, Node node, Val val, Add add)
{
    // outward normal of phi^n at the target (layers 1, 2)
    bool use_n = false;
    double nxh = 0.0, nyh = 0.0, gx = 0.0, gy = 0.0, gn = 0.0;
    long long kn[4] = {-1, -1, -1, -1};
    if (l <= 2) {
        const int di[4] = {1, -1, 0, 0}, dj[4] = {0, 0, 1, -1};
        double pv[4];
        bool ok = true;
        for (int q = 0; q < 4; q++) {
            int x = i + di[q], y = j + dj[q];
            kn[q] = (canon(g, x, y) && D.has(x, y)) ? pidx(g, x, y) : -1;
            pv[q] = kn[q] >= 0 ? s.P0[kn[q]] : INFINITY;
            ok = ok && pv[q] < INFINITY;
        }
        if (ok) {
            gx = (pv[0] - pv[1]) / 2.0;
            gy = (pv[2] - pv[3]) / 2.0;
            gn = sqrt(gx * gx + gy * gy);
            if (gn > 0.0) {
                nxh = gx / gn;
                nyh = gy / gn;
                use_n = true;
            }
        }
    }
    auto weight = [&](int aa, int bb, double& dn, double& ddx, double& ddy, double& dl) {
        const double w0 = ldexp(1.0, -(abs(aa) + abs(bb)));
        if (!use_n) return w0;
        ddx = -(double)aa;
        ddy = -(double)bb;
        dl = sqrt(ddx * ddx + ddy * ddy);
        dn = (ddx * nxh + ddy * nyh) / dl;
        return dn * w0 > 0.0 ? dn * w0 : 0.0;
    };
    const int rmax = RMAX > 0 ? RMAX : g.r_max;
#pragma unroll 1
    for (int rr = 2; rr <= rmax; rr++) {
        const int r = RMAX == 2 ? 2 : rr;
        double M00 = 0, M01 = 0, M02 = 0, M11 = 0, M12 = 0, M22 = 0;
        double bX0 = 0, bX1 = 0, bX2 = 0, bY0 = 0, bY1 = 0, bY2 = 0;
        int count = 0;
#pragma unroll RMAX == 2 ? 5 : 1
        for (int bb = -r; bb <= r; bb++)
#pragma unroll RMAX == 2 ? 5 : 1
            for (int aa = -r; aa <= r; aa++) {
                if (aa == 0 && bb == 0) continue;  // (the target is of layer l)
                const auto k = node(aa, bb);
                if (k < 0) continue;
                count++;
                double dn = 0.0, ddx, ddy, dl;
                const double wt = weight(aa, bb, dn, ddx, ddy, dl);
                const double dx = aa, dy = bb;
                M00 += wt * dx * dx; M01 += wt * dx * dy; M02 += wt * dx;
                M11 += wt * dy * dy; M12 += wt * dy; M22 += wt;
                if (use_n && own) {
                    double xv, yv;
                    val(k, aa, bb, xv, yv);
                    bX0 += wt * dx * xv; bX1 += wt * dy * xv; bX2 += wt * xv;
                    bY0 += wt * dx * yv; bY1 += wt * dy * yv; bY2 += wt * yv;
                }
            }
        if (count < 3) continue;
        const double det = M00 * (M11 * M22 - M12 * M12) - M01 * (M01 * M22 - M12 * M02) +
                           M02 * (M01 * M12 - M11 * M02);
        if (!(det > g.det_rel * M22 * M22 * M22)) continue;
        // inverse of the symmetric normal matrix
        const double i02 = (M01 * M12 - M11 * M02) / det;
        const double i12 = (M01 * M02 - M00 * M12) / det, i22 = (M00 * M11 - M01 * M01) / det;
        // s = M^{-1} e3, plane coefficients p = M^{-1} b
        const double s0 = i02, s1 = i12, s2 = i22;
        double pX0 = 0, pX1 = 0, pX2 = 0, pY0 = 0, pY1 = 0, pY2 = 0;
        if (use_n && own) {
            const double i00 = (M11 * M22 - M12 * M12) / det, i01 = (M02 * M12 - M01 * M22) / det;
            const double i11 = (M00 * M22 - M02 * M02) / det;
            pX0 = i00 * bX0 + i01 * bX1 + i02 * bX2;
            pX1 = i01 * bX0 + i11 * bX1 + i12 * bX2;
            pX2 = i02 * bX0 + i12 * bX1 + i22 * bX2;
            pY0 = i00 * bY0 + i01 * bY1 + i02 * bY2;
            pY1 = i01 * bY0 + i11 * bY1 + i12 * bY2;
            pY2 = i02 * bY0 + i12 * bY1 + i22 * bY2;
        }
        double nbx = 0.0, nby = 0.0;  // dL/d(normal)
#pragma unroll RMAX == 2 ? 5 : 1
        for (int bb = -r; bb <= r; bb++)
#pragma unroll RMAX == 2 ? 5 : 1
            for (int aa = -r; aa <= r; aa++) {
                if (aa == 0 && bb == 0) continue;
                const auto k = node(aa, bb);
                if (k < 0) continue;
                double dn = 0.0, ddx = 0.0, ddy = 0.0, dl = 0.0;
                const double wt = weight(aa, bb, dn, ddx, ddy, dl);
                const double w0 = ldexp(1.0, -(abs(aa) + abs(bb)));
                const double as = s0 * aa + s1 * bb + s2;
                if (wt != 0.0) add(k, Xb * wt * as, Yb * wt * as);
                if (use_n && own && dn * w0 > 0.0) {
                    double xv, yv;
                    val(k, aa, bb, xv, yv);
                    const double rX = xv - (pX0 * aa + pX1 * bb + pX2);
                    const double rY = yv - (pY0 * aa + pY1 * bb + pY2);
                    const double wb = as * (Xb * rX + Yb * rY);
                    const double dnb = wb * w0;
                    nbx += dnb * ddx / dl;
                    nby += dnb * ddy / dl;
                }
            }
        if (use_n && own && (nbx != 0.0 || nby != 0.0)) {
            // n = g / |g|, g = ((phi_e - phi_w) / 2, (phi_n - phi_s) / 2)
            const double dotp = nbx * nxh + nby * nyh;
            const double gbx = (nbx - dotp * nxh) / gn, gby = (nby - dotp * nyh) / gn;
            atomicAdd(&a.pbar0[kn[0]], gbx / 2.0);
            atomicAdd(&a.pbar0[kn[1]], -gbx / 2.0);
            atomicAdd(&a.pbar0[kn[2]], gby / 2.0);
            atomicAdd(&a.pbar0[kn[3]], -gby / 2.0);
        }
        break;
    }
}

// relabel backwards at one node (see k_adj_relabel), into x and y
__device__ __forceinline__ void adj_relabel_node(const BodyP& b, const AdjSnap& s, long long k,
                                                 double pb, double& x, double& y)
{
    if (pb == 0.0 || !(s.P1[k] < INFINITY)) return;
    double gx, gy;
    grad_phi0(b, s.X1[k], s.Y1[k], gx, gy);
    x += pb * gx;
    y += pb * gy;
}

// Target (i, j) of layer l, node kt, on the adjoint fields in memory.  RELABEL:
// its relabel first (only its own thread touches a node of layer l in this
// pass).
template <bool RELABEL>
__device__ __forceinline__ void adj_fit_node(const GridP& g, const BodyP& b, const AdjSnap& s,
                                             const AdjBufs& a, const Rect& W, const Rect& D, int l,
                                             int i, int j, long long kt)
{
    // (past the caches: any block may have added to it in this launch)
    double Xb = __hip_atomic_load(&a.xbar1[kt], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    double Yb = __hip_atomic_load(&a.ybar1[kt], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (RELABEL) adj_relabel_node(b, s, kt, a.pbar1[kt], Xb, Yb);
    if (Xb == 0.0 && Yb == 0.0) return;
    adj_fit_target<0>(
        g, D, s, a, l, i, j, Xb, Yb, true,
        [&](int aa, int bb) -> long long {
            int x = i + aa, y = j + bb;
            if (!canon(g, x, y) || !W.has(x, y)) return -1;
            const long long k = pidx(g, x, y);
            const int t = s.tag[k];
            return t == TAG_SOLID || (t > 0 && t < l) ? k : -1;
        },
        [&](long long k, int, int, double& xv, double& yv) {
            xv = s.X1[k];
            yv = s.Y1[k];
        },
        [&](long long k, double vx, double vy) {
            atomicAdd(&a.xbar1[k], vx);
            atomicAdd(&a.ybar1[k], vy);
        });
}

// one launch per layer, last layer first
__global__ __launch_bounds__(256) void k_adj_fit(GridP g, BodyP b, AdjSnap s, AdjBufs a, int l)
{
    const Rect W = window_of(s.win, 1, g);
    const Rect D = window_of(s.win, 0, g);
    if (!W.ok) return;
    const int w = W.i1 - W.i0 + 1, h = W.j1 - W.j0 + 1;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < (long long)w * h;
         e += (long long)gridDim.x * blockDim.x) {
        int i = W.i0 + (int)(e % w), j = W.j0 + (int)(e / w);
        if (!canon(g, i, j)) continue;
        const long long kt = pidx(g, i, j);
        if (s.tag[kt] != l) continue;  // not this layer, or its fit failed
        adj_fit_node<false>(g, b, s, a, W, D, l, i, j, kt);
    }
}

// Every layer on the fields in memory, by all blocks of a launch, where a fit
// has a wider scan window than a tile's copy serves.  The layers' shares of the
// window (last layer first) are numbered, and a block takes the next number by
// an atomic: a share waits for those of the layer before it, whose numbers are
// smaller, so that running blocks hold them all and the wait ends however few
// blocks run at a time (a block works its numbers off in their order).  What
// one share adds and another reads goes through atomics, complete before the
// share counts as done.  a.work: 0 between launches; the numbers taken, the
// blocks that have left, each layer's shares done.  Bound by what a layer's
// targets do one after the other, ~18 us a layer.  One block alone scanned the
// window once per layer; thin solids, us per reverse step, 256^2 / 768^2: one
// block 1311 / 5953, this 271 / 448 (a launch per layer, which every other step
// would pay for, 238 / 387).
__device__ __forceinline__ void adj_fit_shared(const GridP& g, const BodyP& b, const AdjSnap& s,
                                               const AdjBufs& a, const Rect& W, const Rect& D,
                                               int L)
{
    __shared__ unsigned number[2];
    const int w = W.i1 - W.i0 + 1, nt = blockDim.x;
    const long long n = (long long)w * (W.j1 - W.j0 + 1);
    // nodes per thread of a share, 32 at most (bits of hit): a share to half the
    // blocks that run at a time, one on each of the chip's 256 units, so that
    // the others look through the next layer's meanwhile
    const int half = max(1, min((int)gridDim.x, 256) / 2);
    const int rounds = (int)min((n + half * nt - 1) / (half * nt), 32ll);
    const unsigned shares = (unsigned)((n + rounds * nt - 1) / (rounds * nt)), all = shares * L;
    unsigned *taken = a.work, *left = a.work + 1, *done = a.work + 2;
    if (threadIdx.x == 0) number[0] = atomicAdd(taken, 1u);
    __syncthreads();
    for (int turn = 0;; turn ^= 1) {
        const unsigned q = number[turn];
        if (q >= all) break;
        const int k = q / shares, l = L - k;
        const long long e0 = (long long)(q % shares) * (rounds * nt) + threadIdx.x;
        // (which of the thread's nodes are targets, and the next number: before the wait)
        unsigned hit = 0;
        for (int u0 = 0; u0 < rounds; u0 += 4) {
            int tv[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int e = (int)min(e0 + (u0 + u) * nt, n - 1);
                tv[u] = s.tag[pidx(g, W.i0 + e % w, W.j0 + e / w)];
            }
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (tv[u] == l && u0 + u < rounds && e0 + (u0 + u) * nt < n) hit |= 1u << (u0 + u);
        }
        if (threadIdx.x == 0) {
            number[turn ^ 1] = atomicAdd(taken, 1u);
            if (k > 0)
                while (__hip_atomic_load(&done[k - 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                       shares)
                    __builtin_amdgcn_s_sleep(1);
        }
        __syncthreads();
        while (hit) {
            const int e = (int)e0 + (__ffs(hit) - 1) * nt;  // (a window has fewer than 2^26 nodes)
            hit &= hit - 1;
            const int i = W.i0 + e % w, j = W.j0 + e / w;
            adj_fit_node<true>(g, b, s, a, W, D, l, i, j, pidx(g, i, j));
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) atomicAdd(&done[k], 1u);
    }
    if (threadIdx.x == 0 && atomicAdd(left, 1u) == gridDim.x - 1) {
        __threadfence();
        for (int k = 0; k < ADJ_WORK; k++) a.work[k] = 0u;
    }
}

// Relabel and every layer backwards in one launch (up to FF_LAYERS layers).
// A block takes AT x AT tiles of the window: what reaches a solid node comes
// from targets within 2 nodes of it, to which targets of later layers within
// 2 nodes of them send, so that a target of layer l is taken within 2 l nodes
// of the tile, on a copy of the tags and adjoints of the tile and a margin of
// 2 L + 2 nodes (a margin's targets are recomputed by each block that needs
// them).  Only the tile's solid nodes are written: what the zone's nodes hold
// is spent after this, and k_adj_advect clears it, so no block reads what
// another writes.  A node is a tile's own where it lies in the window without
// wrapping: the last tile of a periodic axis may run over the seam, where it
// holds nodes of the window's first tile.  Bound by a chain of L dependent layers in LDS; launches of
// their own each scanned the window's tags again (256^2, solid of radius 40:
// 12 launches, ~75 us a step -> one, 43 us).
// s.wide: some target of the step has a wider scan window (or none): then the
// blocks run the layers on the fields in memory (adj_fit_shared).
constexpr int AT = FF_TILE, AT_THREADS = 512;
constexpr int AT_R = AT + 4 * FF_LAYERS + 4;  // side of the copy at FF_LAYERS layers
// LC: the layer count (FF_LAYERS), or 0 (the grid's)
template <int LC>
__global__ __launch_bounds__(AT_THREADS) void k_adj_fits(GridP g, BodyP b, AdjSnap s, AdjBufs a)
{
    constexpr int NN = AT_R * AT_R, NIT = (NN + AT_THREADS - 1) / AT_THREADS;
    constexpr int NSET = 4, SW = AT_THREADS / NSET;  // sets of threads, targets per pass
    __shared__ double xb[NN], yb[NN];
    __shared__ unsigned char st[NN];
    __shared__ unsigned short lst[NN];
    __shared__ int cnt[FF_LAYERS + 2], at[FF_LAYERS + 2], near;
    const Rect W = window_of(s.win, 1, g);
    const Rect D = window_of(s.win, 0, g);
    if (!W.ok) return;
    const int L = LC > 0 ? LC : g.layers;
    if (*s.wide != 0) {
        adj_fit_shared(g, b, s, a, W, D, L);
        return;
    }
    const int m = 2 * L + 2, rw = LC == FF_LAYERS ? AT_R : AT + 2 * m;
    const int ntx = (W.i1 - W.i0 + AT) / AT, nty = (W.j1 - W.j0 + AT) / AT;
    for (int t = blockIdx.x; t < ntx * nty; t += gridDim.x) {
        const int x0 = W.i0 + (t % ntx) * AT - m, y0 = W.j0 + (t / ntx) * AT - m;
        // (behind an empty asm: what follows from the thread's number is
        // computed here, not held over the loop)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        // node of the copy (unwrapped; a periodic axis wraps)
        auto global_of = [&](int q) -> long long {
            int x = x0 + q % rw, y = y0 + q / rw;
            if (!canon(g, x, y) || !W.has(x, y)) return -1;
            return pidx(g, x, y);
        };
        auto dist = [&](int q) {
            const int lx = q % rw - m, ly = q / rw - m;
            return max(max(-lx, lx - (AT - 1)), max(-ly, ly - (AT - 1)));
        };
        int tvs[NIT];  // the thread's tags, all in flight together
#pragma unroll
        for (int u = 0; u < NIT; u++) {
            const int q = tid + u * AT_THREADS;
            const long long k = q < rw * rw ? global_of(q) : -1;
            const int tv = s.tag[k >= 0 ? k : 0];
            tvs[u] = k >= 0 ? tv : TAG_NONE;
        }
        if (tid <= FF_LAYERS + 1) cnt[tid] = 0;
        if (tid == 0) near = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NIT; u++) {
            const int q = tid + u * AT_THREADS, tv = tvs[u];
            if (q >= rw * rw) continue;
            st[q] = (unsigned char)tv;
            xb[q] = 0.0;
            yb[q] = 0.0;
            if (tv >= 1 && tv <= L) {
                const int d = dist(q);
                if (d <= 2 * tv) atomicAdd(&cnt[tv], 1);
                else tvs[u] = TAG_NONE;  // no target of this block
                if (d <= 2) near = 1;
            }
        }
        __syncthreads();
        if (!near) continue;  // (uniform; nothing of the tile hears from the zone)
        if (tid == 0) {
            int o = 0;
            for (int l = 1; l <= L; l++) {
                at[l] = o;
                o += cnt[l];
                cnt[l] = 0;
            }
            at[L + 1] = o;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NIT; u++) {
            const int q = tid + u * AT_THREADS, tv = tvs[u];
            if (tv < 1 || tv > L) continue;
            lst[at[tv] + atomicAdd(&cnt[tv], 1)] = (unsigned short)q;
        }
        __syncthreads();
        // the targets' adjoints, relabelled (every load in flight together)
#pragma unroll 1
        for (int e = tid; e < at[L + 1]; e += AT_THREADS) {
            const int q = lst[e];
            const long long k = global_of(q);
            double x = a.xbar1[k], y = a.ybar1[k];
            const double pb = a.pbar1[k], P = s.P1[k], X = s.X1[k], Y = s.Y1[k];
            if (pb != 0.0 && P < INFINITY) {
                double gx, gy;
                grad_phi0(b, X, Y, gx, gy);
                x += pb * gx;
                y += pb * gy;
            }
            xb[q] = x;
            yb[q] = y;
        }
        __syncthreads();
        // layers 3 and up, a set of threads to each layer in turn: a set
        // finds its targets' valid nodes and s while the others add.  The
        // matrix is counted from the mask (its entries times 16 are whole),
        // so s has the bits of sums in double.
        const int set = tid / SW, lane = tid % SW;
        int pq = -1;
        unsigned pm = 0;
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
        auto prep = [&](int l, int e, int end) {
            pq = -1;
            if (e >= end) return;
            const int q = lst[e];
            unsigned mk = 0;
#pragma unroll
            for (int n = 0; n < 25; n++)
                if (n != 12) mk |= st[q + (n / 5 - 2) * rw + n % 5 - 2] < l ? 1u << n : 0u;
            const Geo2 G = geo2(mk, g.det_rel);
            if (!G.ok) return;
            const double det = (double)G.det * 0x1p-12;
            s0 = (double)G.c0() * 0x1p-8 / det;
            s1 = (double)G.c1() * 0x1p-8 / det;
            s2 = (double)G.c2() * 0x1p-8 / det;
            pq = q;
            pm = mk;
        };
        auto send = [&]() {
            if (pq < 0) return;
            const double Xb = xb[pq], Yb = yb[pq];
            if (Xb == 0.0 && Yb == 0.0) return;
#pragma unroll
            for (int n = 0; n < 25; n++) {
                if (n == 12 || !(pm >> n & 1)) continue;
                const int aa = n % 5 - 2, bb = n / 5 - 2;
                const double wt = 1.0 / (1 << ((aa < 0 ? -aa : aa) + (bb < 0 ? -bb : bb)));
                const double as = s0 * aa + s1 * bb + s2;
                const int k = pq + bb * rw + aa;
                atomicAdd(&xb[k], Xb * wt * as);
                atomicAdd(&yb[k], Yb * wt * as);
            }
        };
        int lm = L - set;  // the set's next layer
        if (lm >= 3) prep(lm, at[lm] + lane, at[lm + 1]);
#pragma unroll 1
        for (int l = L; l >= 3; l--) {
            if (l == lm) {
                const int end = at[l + 1];
                int e = at[l] + lane;
#pragma unroll 1
                while (true) {
                    send();
                    e += SW;
                    if (e >= end) break;
                    prep(l, e, end);
                }
            }
            __syncthreads();
            if (l == lm) {
                lm -= NSET;
                if (lm >= 3) prep(lm, at[lm] + lane, at[lm + 1]);
            }
        }
        // layers 2 and 1: normal weights
#pragma unroll 1
        for (int l = min(L, 2); l >= 1; l--) {
#pragma unroll 1
            for (int e = at[l] + tid; e < at[l + 1]; e += AT_THREADS) {
                const int q = lst[e];
                const double Xb = xb[q], Yb = yb[q];
                if (Xb == 0.0 && Yb == 0.0) continue;
                const int i0 = x0 + q % rw, j0 = y0 + q / rw;
                const bool own = dist(q) <= 0 && W.has(i0, j0);
                int i = i0, j = j0;
                canon(g, i, j);
                // xi^{n+1} of the scan nodes, all in flight together
                double xs[25], ys[25];
                if (own) {
                    int kx[5], ky[5];
#pragma unroll
                    for (int n = 0; n < 5; n++) {
                        int x = i0 + n - 2, y = j0 + n - 2;
                        if (g.px) x = wrap_axis(x, g.nx);
                        if (g.py) y = wrap_axis(y, g.ny);
                        kx[n] = min(max(x, W.i0), W.i1) + PAD;
                        ky[n] = (min(max(y, W.j0), W.j1) + PAD) * g.pp;
                    }
#pragma unroll
                    for (int n = 0; n < 25; n++) {
                        xs[n] = s.X1[ky[n / 5] + kx[n % 5]];
                        ys[n] = s.Y1[ky[n / 5] + kx[n % 5]];
                    }
                }
                adj_fit_target<2>(
                    g, D, s, a, l, i, j, Xb, Yb, own,
                    [&](int aa, int bb) {
                        const int k = q + bb * rw + aa;
                        return st[k] < l ? k : -1;
                    },
                    [&](int, int aa, int bb, double& xv, double& yv) {
                        xv = xs[(bb + 2) * 5 + aa + 2];
                        yv = ys[(bb + 2) * 5 + aa + 2];
                    },
                    [&](int k, double vx, double vy) {
                        atomicAdd(&xb[k], vx);
                        atomicAdd(&yb[k], vy);
                    });
            }
            __syncthreads();
        }
        for (int e = tid; e < AT * AT; e += AT_THREADS) {
            const int q = (m + e / AT) * rw + m + e % AT;
            if (st[q] != TAG_SOLID || !W.has(x0 + q % rw, y0 + q / rw)) continue;
            const double x = xb[q], y = yb[q];
            if (x == 0.0 && y == 0.0) continue;
            const long long k = global_of(q);
            a.xbar1[k] += x;
            a.ybar1[k] += y;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- advection
// Solid nodes of S^n backwards: xi~ = xi - (u d/dx + v d/dy) xi with the
// upwind side of the forward step.  dL/dxi~ (held in xbar1 at solid nodes,
// after their relabel backwards) -> xbar0 at the node and its stencil nodes,
// and u^n -> f^n, F^{n-1}.  The adjoints of state n + 1 are spent: every node
// of their window (nothing outside it was added to) is cleared here, the next
// step's xbar0, ybar0, pbar0 to be.
__global__ __launch_bounds__(256) void k_adj_advect(GridP g, BodyP b, AdjSnap s, AdjBufs a)
{
    const Rect W = window_of(s.win, 1, g);
    const Rect D = window_of(s.win, 0, g);
    if (!W.ok) return;
    const long long N = (long long)g.nx * g.ny;
    const int w = W.i1 - W.i0 + 1, h = W.j1 - W.j0 + 1;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < (long long)w * h;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = W.i0 + (int)(e % w), j = W.j0 + (int)(e / w);
        const long long k0 = pidx(g, i, j);
        double Xb = a.xbar1[k0], Yb = a.ybar1[k0];
        const double pb = a.pbar1[k0];
        const bool solid = s.tag[k0] == TAG_SOLID;
        a.xbar1[k0] = 0.0;
        a.ybar1[k0] = 0.0;
        a.pbar1[k0] = 0.0;
        if (i < 0 || i >= g.nx || j < 0 || j >= g.ny || !solid) continue;
        adj_relabel_node(b, s, k0, pb, Xb, Yb);
        if (Xb == 0.0 && Yb == 0.0) continue;
        // u^n at the node
        double f[NQ];
        nat_gather(g, s.A, i, j, f);
        double rho = 0.0, jx = 0.0, jy = 0.0;
        for (int q = 0; q < NQ; q++) {
            rho += f[q];
            jx += ACX[q] * f[q];
            jy += ACY[q] * f[q];
        }
        const long long n = (long long)j * g.pitch + i;
        const bool inp = D.has(i, j);
        const double Fpx = inp ? s.fpx[n] : s.fpo[0], Fpy = inp ? s.fpy[n] : s.fpo[1];
        const double u = (jx + 0.5 * Fpx) / rho, v = (jy + 0.5 * Fpy) / rho;
        // stencils along x and y, as in the forward step
        auto stencil = [&](int dx, int dy, double vel, long long kk[3], double cf[3], double& dX,
                           double& dY) -> bool {
            kk[0] = k0;
            kk[1] = kk[2] = -1;
            cf[0] = cf[1] = cf[2] = 0.0;
            dX = dY = 0.0;
            if (vel == 0.0) return true;
            const int sg = vel > 0.0 ? 1 : -1;
            for (int t = 1; t <= 2; t++) {
                int x = i - sg * t * dx, y = j - sg * t * dy;
                if (!canon(g, x, y) || !D.has(x, y)) return false;
                kk[t] = pidx(g, x, y);
                if (!(s.P0[kk[t]] < INFINITY)) return false;
            }
            if (sg > 0) {
                cf[0] = 1.5; cf[1] = -2.0; cf[2] = 0.5;
            } else {
                cf[0] = -1.5; cf[1] = 2.0; cf[2] = -0.5;
            }
            for (int t = 0; t < 3; t++) {
                dX += cf[t] * s.X0[kk[t]];
                dY += cf[t] * s.Y0[kk[t]];
            }
            return true;
        };
        long long kx[3], ky[3];
        double cx[3], cy[3], dXx, dYx, dXy, dYy;
        const bool okx = stencil(1, 0, u, kx, cx, dXx, dYx);
        const bool oky = stencil(0, 1, v, ky, cy, dXy, dYy);
        if (!okx || !oky) {
            // the forward step kept xi (missing stencil node)
            atomicAdd(&a.xbar0[k0], Xb);
            atomicAdd(&a.ybar0[k0], Yb);
            continue;
        }
        atomicAdd(&a.xbar0[k0], Xb);
        atomicAdd(&a.ybar0[k0], Yb);
        for (int t = 0; t < 3; t++) {
            if (cx[t] != 0.0) {
                atomicAdd(&a.xbar0[kx[t]], -u * cx[t] * Xb);
                atomicAdd(&a.ybar0[kx[t]], -u * cx[t] * Yb);
            }
            if (cy[t] != 0.0) {
                atomicAdd(&a.xbar0[ky[t]], -v * cy[t] * Xb);
                atomicAdd(&a.ybar0[ky[t]], -v * cy[t] * Yb);
            }
        }
        const double ub = -(dXx * Xb + dYx * Yb), vb = -(dXy * Xb + dYy * Yb);
        // u = (j + F^{n-1} / 2) / rho
        const double jxb = ub / rho, jyb = vb / rho;
        const double rb = -(ub * u + vb * v) / rho;
        const long long m = (long long)j * g.nx + i;
        for (int q = 0; q < NQ; q++) a.fb_out[q * N + m] += rb + ACX[q] * jxb + ACY[q] * jyb;
        if (inp) {
            a.Fpbar_x[m] += 0.5 * jxb;
            a.Fpbar_y[m] += 0.5 * jyb;
        }
    }
}

// ---------------------------------------------------------------- loss
// L_n = (|c - c*|^2 + |d - d*|^2) / T with c = sum lambda x / sum lambda,
// d = sum lambda (x - xi) / sum lambda, lambda = 1 - H(phi): coef = {c_x, c_y,
// d_x, d_y, gc_x, gc_y, gd_x, gd_y} with gc = dL/dc / sum lambda and
// gd = dL/dd / sum lambda.  which = 0: the step's input state (xi^n, phi^n,
// adds to xbar0, pbar0); 1: its output state (xi^{n+1}, phi^{n+1}, adds to
// xbar1, pbar1).
__global__ __launch_bounds__(256) void k_adj_loss(GridP g, BodyP b, AdjSnap s, AdjBufs a,
                                                  int which, LossCoef c)
{
    const Rect V = window_of(s.win, which == 0 ? 0 : 1, g);
    if (!V.ok || !b.present) return;
    const double* X = which == 0 ? s.X0 : s.X1;
    const double* Y = which == 0 ? s.Y0 : s.Y1;
    const double* P = which == 0 ? s.P0 : s.P1;
    double* xb = which == 0 ? a.xbar0 : a.xbar1;
    double* yb = which == 0 ? a.ybar0 : a.ybar1;
    double* pb = which == 0 ? a.pbar0 : a.pbar1;
    const int i0 = max(V.i0, 0), i1 = min(V.i1, g.nx - 1);
    const int j0 = max(V.j0, 0), j1 = min(V.j1, g.ny - 1);
    const int w = i1 - i0 + 1, h = j1 - j0 + 1;
    if (w <= 0 || h <= 0) return;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < (long long)w * h;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = i0 + (int)(e % w), j = j0 + (int)(e / w);
        const long long k = pidx(g, i, j);
        const double p = P[k];
        if (!(p < INFINITY)) continue;
        double x = i + 0.5, y = j + 0.5;
        if (g.px) x = b.cx + (x - b.cx) - g.nx * floor((x - b.cx) / g.nx + 0.5);
        if (g.py) y = b.cy + (y - b.cy) - g.ny * floor((y - b.cy) / g.ny + 0.5);
        const double lam = 1.0 - hv(p, g.eps);
        const double dl = c.gc[0] * (x - c.c[0]) + c.gc[1] * (y - c.c[1]) +
                          c.gd[0] * ((x - X[k]) - c.d[0]) + c.gd[1] * ((y - Y[k]) - c.d[1]);
        pb[k] += dl * (-dhv(p, g.eps));
        xb[k] += -c.gd[0] * lam;
        yb[k] += -c.gd[1] * lam;
    }
}

// ---------------------------------------------------------------- initial state
// f^0 = f^eq(rho_0, u_0, drho_0) (natural form): dL/du_0 from dL/df^0.
__global__ __launch_bounds__(256) void k_adj_init(GridP g, BodyP b, AdjSnap s, AdjBufs a,
                                                  double* u0bar)
{
    const long long N = (long long)g.nx * g.ny;
    const Rect D = window_of(s.win, 0, g);
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < N;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(e % g.nx), j = (int)(e / g.nx);
        // rho_0 and u_0 from f^0 itself (its moments are rho_0 and rho_0 u_0)
        double f[NQ];
        nat_gather(g, s.A, i, j, f);
        double rho = 0.0, jx = 0.0, jy = 0.0;
        for (int q = 0; q < NQ; q++) {
            rho += f[q];
            jx += ACX[q] * f[q];
            jy += ACY[q] * f[q];
        }
        (void)D;
        const double ux = jx / rho, uy = jy / rho;
        double bx = 0.0, by = 0.0;
        for (int q = 0; q < NQ; q++) {
            const double cx = ACX[q], cy = ACY[q], cu = cx * ux + cy * uy, fb = a.fb_in[q * N + e];
            bx += fb * AWQ[q] * rho * (3.0 * cx + 9.0 * cu * cx - 3.0 * ux);
            by += fb * AWQ[q] * rho * (3.0 * cy + 9.0 * cu * cy - 3.0 * uy);
        }
        u0bar[e] = bx;
        u0bar[N + e] = by;
    }
}

// ---------------------------------------------------------------- launchers

hipError_t launch_adjoint_step(const GridP& g, const BodyP& b, const AdjSnap& s,
                               const AdjBufs& a, bool fused, hipStream_t st)
{
    const long long N = (long long)g.nx * g.ny;
    const int blocks = (int)((N + 255) / 256 < 4096 ? (N + 255) / 256 : 4096);
    k_adj_lattice<<<blocks, 256, 0, st>>>(g, b, s, a);
    k_adj_force<<<blocks, 256, 0, st>>>(g, b, s, a);
    if (b.present) {
        if (fused) {
            const long long tiles = fused_tiles(g.nx, g.ny);
            const int nb = (int)(tiles < 1024 ? tiles : 1024);
            if (g.layers == FF_LAYERS) k_adj_fits<FF_LAYERS><<<nb, AT_THREADS, 0, st>>>(g, b, s, a);
            else k_adj_fits<0><<<nb, AT_THREADS, 0, st>>>(g, b, s, a);
        } else {
            k_adj_relabel<<<blocks, 256, 0, st>>>(g, b, s, a);
            for (int l = g.layers; l >= 1; l--) k_adj_fit<<<blocks, 256, 0, st>>>(g, b, s, a, l);
        }
        k_adj_advect<<<blocks, 256, 0, st>>>(g, b, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_adjoint_loss(const GridP& g, const BodyP& b, const AdjSnap& s,
                               const AdjBufs& a, int which, const LossCoef& c, hipStream_t st)
{
    const long long N = (long long)g.nx * g.ny;
    const int blocks = (int)((N + 255) / 256 < 4096 ? (N + 255) / 256 : 4096);
    k_adj_loss<<<blocks, 256, 0, st>>>(g, b, s, a, which, c);
    return hipGetLastError();
}

hipError_t launch_adjoint_init(const GridP& g, const BodyP& b, const AdjSnap& s,
                               const AdjBufs& a, double* u0bar, hipStream_t st)
{
    const long long N = (long long)g.nx * g.ny;
    const int blocks = (int)((N + 255) / 256 < 4096 ? (N + 255) / 256 : 4096);
    k_adj_init<<<blocks, 256, 0, st>>>(g, b, s, a, u0bar);
    return hipGetLastError();
}

// ---------------------------------------------------------------- snapshot

// Every piece of a snapshot in one launch (block row y copies piece y, 8 bytes
// a thread and access; twelve copies and a fill of their own, each a few us,
// took longer than the step), with the two windows, the uniform force
// F^{n-1} and the wide-window flag of the step's extrapolation
__global__ __launch_bounds__(256) void k_snapshot(SnapCopy c)
{
    const SnapPiece p = c.piece[blockIdx.y];
    const unsigned long long* src = (const unsigned long long*)p.src;
    unsigned long long* dst = (unsigned long long*)p.dst;
    const long long n = p.bytes / 8, st = (long long)gridDim.x * blockDim.x;
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    constexpr int U = 4;
    for (long long e = t; e < n; e += U * st) {
        unsigned long long v[U];
#pragma unroll
        for (int u = 0; u < U; u++) v[u] = src[e + u * st < n ? e + u * st : e];
#pragma unroll
        for (int u = 0; u < U; u++)
            if (e + u * st < n) dst[e + u * st] = v[u];
    }
    if (blockIdx.x == 0 && (long long)threadIdx.x < p.bytes % 8)
        ((char*)p.dst)[n * 8 + threadIdx.x] = ((const char*)p.src)[n * 8 + threadIdx.x];
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        c.win[0] = *c.wprev;
        c.win[1] = *c.wcur;
        c.fpo[0] = c.fpo_x;
        c.fpo[1] = c.fpo_y;
        *c.wide = c.wide_src ? *c.wide_src : 1;
    }
}

hipError_t launch_snapshot(const SnapCopy& c, int pieces, hipStream_t st)
{
    long long most = 0;
    for (int k = 0; k < pieces; k++) most = most < c.piece[k].bytes ? c.piece[k].bytes : most;
    const long long want = (most / 8 + 1023) / 1024;  // four accesses per thread
    const dim3 grid((unsigned)(want < 1 ? 1 : want < 1024 ? want : 1024), pieces);
    k_snapshot<<<grid, 256, 0, st>>>(c);
    return hipGetLastError();
}

}  // namespace lbrmt
