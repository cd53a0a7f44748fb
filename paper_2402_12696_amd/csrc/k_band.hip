// Reference-map ("band") kernels of the LBRMT step on gfx950: advection of xi
// (Sec. 3.1), the extrapolation zone and its layer-by-layer least-squares
// extrapolation (Sec. 3.2), relabel phi = phi0(xi), and the divergence of the
// blended half-edge solid stress fed back as the LB force density (Sec. 3.3,
// Eq. (2_4_F_divs)).
//
// Every kernel works inside one rectangular window per body: the box of the
// interior solid nodes dilated by the number of extrapolation layers, kept in
// a device ring of three boxes (previous, current, next step) so no host round
// trip is needed.  A node outside a window holds no reference map.
//
// One step runs: advect (tags: solid / none, exact Manhattan layer numbers of
// the zone, its tiles or one node list per layer) -> fits of every layer in one
// launch, or one per layer -> force (relabel with per-block boxes, LDS-tiled
// half edges, the lattice update of the window's nodes; the last block reduces
// the boxes).
//
// These kernels take every discrete decision of the method (solid set, layers,
// window growth of the fit, singular Jacobians); this file is compiled without
// floating-point contraction so they are taken in plain IEEE arithmetic.
//
// Storage type T of the reference map: double (FP64 mode) holds xi itself;
// float (FP32 mode) holds the displacement d = xi - x, x the node coordinate,
// so values stay small and stencils add the exact lattice offsets (the upwind
// and central differences of x itself are exactly 1).  The FP32 mode runs the
// stencil arithmetic in float and keeps FP64 for the level set phi0(x + d)
// (it decides the solid set), the normal matrix of the fit and its
// well-posedness test (exact sums of powers of two on a few nodes), and the
// inversion of grad xi where det < kappa_J.
#include <type_traits>

#include "lb_node.h"
#include "fit_window.h"
#include "mb_recentre.h"

namespace lbrmt {

constexpr double PI_D = 3.14159265358979323846;

template <typename C>
__device__ __forceinline__ C heaviside(C phi, C eps)
{
    // Eq. (2_3_heaviside)
    const C pi = C(PI_D);
    if (phi <= -eps) return C(0);
    if (phi >= eps) return C(1);
    return C(0.5) * (C(1) + phi / eps + sin(pi * phi / eps) / pi);
}

// reference shape level set phi0(X) (Sec. 3.1): the disc's signed distance
// |X - c| - R; for an ellipse the radial form |X - c| (1 - 1/q), with q the
// normalised radius sqrt((x'/R)^2 + (y'/Rb)^2) in the body frame, zero on the
// boundary and negative inside (at the centre: minus the smaller semi-axis).
// Built without contraction: the sign taken at initialisation and relabel
// decides node sets, so the arithmetic is the plain sequence of rounded ops.
__device__ __forceinline__ double shape_phi(const BodyP& b, double X, double Y)
{
    const double dx = X - b.cx, dy = Y - b.cy;
    const double d = sqrt(dx * dx + dy * dy);
    if (b.shape != 1) return d - b.R;
    if (d == 0.0) return -(b.R < b.Rb ? b.R : b.Rb);
    const double xp = b.ct * dx + b.st * dy, yp = -b.st * dx + b.ct * dy;
    const double q = sqrt((xp / b.R) * (xp / b.R) + (yp / b.Rb) * (yp / b.Rb));
    return d * (1.0 - 1.0 / q);
}

// coordinate of node index i on an axis; on a periodic axis the image nearest
// to the body centre keeps the reference map continuous
__device__ __forceinline__ double node_coord(int i, int periodic, int n, double c)
{
    double x = i + 0.5;
    if (periodic) {
        const double L = n;
        double d = x - c;
        d -= L * floor(d / L + 0.5);
        x = c + d;
    }
    return x;
}

// position of reference-map node (i, j) of grid g, seen by body b (a solid's
// sub-window starts at lattice column ox; its positions are unwrapped)
__device__ __forceinline__ double pos_x(const GridP& g, const BodyP& b, int i)
{
    return node_coord(i + g.ox, g.px, g.nx, b.cx);
}
__device__ __forceinline__ double pos_y(const GridP& g, const BodyP& b, int j)
{
    return node_coord(j + g.oy, g.py, g.ny, b.cy);
}

// lattice column / row of reference-map node i / j
__device__ __forceinline__ int lat_col(const GridP& g, int i)
{
    return g.wx ? wrap_axis(i + g.ox, g.lnx) : i;
}
__device__ __forceinline__ int lat_row(const GridP& g, int j)
{
    return g.wy ? wrap_axis(j + g.oy, g.lny) : j;
}

// a level-set value computed in double, stored as T with its sign kept (a
// negative value too small for float is stored as the smallest negative float)
template <typename T>
__device__ __forceinline__ T store_phi(double p)
{
    T v = T(p);
    if (p < 0.0 && !(v < T(0))) v = -T(1.401298464324817e-45);
    return v;
}

// clears the layer counters of a step (block 0 of the kernel before the
// distance transform)
__device__ __forceinline__ void clear_lcount(int* lcount)
{
    if (blockIdx.x == 0 && threadIdx.x < (MAX_LAYERS + 1) * NSUB)
        lcount[threadIdx.x * LCOUNT_PAD] = 0;
}

// tags: TAG_NONE, TAG_SOLID, layer l (1..layers), or layer | TAG_FAIL
__device__ __forceinline__ bool tag_valid_before(int t, int l)
{
    // solid, or set by an earlier layer
    return t == TAG_SOLID || (t > 0 && t < l);
}

__device__ __forceinline__ bool tag_set(int t)
{
    return t == TAG_SOLID || (t > 0 && t < TAG_FAIL);
}

// ---------------------------------------------------------------- block helpers

// true in exactly one block: the last to arrive (all blocks must call it)
__device__ bool last_block(unsigned* ticket)
{
    __shared__ bool last;
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        last = atomicAdd(ticket, 1u) == gridDim.x - 1;
    }
    __syncthreads();
    if (last) __threadfence();
    return last;
}

// The same among n blocks in the passes of a step, without the fences: a
// release writes back all that an XCD's L2 holds dirty, which beside a
// lattice update of 2048^2 nodes costs more than the launch it saves (force
// pass 64 -> 141 us, FP64).  What the last block reads of the others goes
// through that cache by itself (through()), and every thread waits for its
// stores before its block arrives; the last block reads it by seen() or after
// a fence.  It leaves the ticket 0.
template <typename V>
__device__ __forceinline__ void through(V* p, V v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V>
__device__ __forceinline__ V seen(const V* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool last_arrival(unsigned* ticket, int n)
{
    __shared__ bool last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        last = atomicAdd(ticket, 1u) == (unsigned)n - 1u;
        if (last) *ticket = 0u;
    }
    __syncthreads();
    return last;
}

// box of the block's flagged nodes, stored as one partial per block
__device__ void block_box(int i0, int i1, int j0, int j1, int* out4)
{
    __shared__ int sb[4][16];
    i0 = wave_min(i0);
    i1 = wave_max(i1);
    j0 = wave_min(j0);
    j1 = wave_max(j1);
    const int wid = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int nw = (blockDim.x + 63) / 64;
    if (lane == 0) {
        sb[0][wid] = i0;
        sb[1][wid] = i1;
        sb[2][wid] = j0;
        sb[3][wid] = j1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < nw; w++) {
            i0 = min(i0, sb[0][w]);
            i1 = max(i1, sb[1][w]);
            j0 = min(j0, sb[2][w]);
            j1 = max(j1, sb[3][w]);
        }
        // (through the cache: the last block of a pass may read them)
        through(&out4[0], i0);
        through(&out4[1], i1);
        through(&out4[2], j0);
        through(&out4[3], j1);
    }
    __syncthreads();
}

// ---------------------------------------------------------------- window ring

__global__ void k_win_reset(Win* win, int slot)
{
    if (threadIdx.x == 0) {
        win[slot].i0 = 0x3fffffff;
        win[slot].i1 = -0x3fffffff;
        win[slot].j0 = 0x3fffffff;
        win[slot].j1 = -0x3fffffff;
    }
}

hipError_t launch_win_reset(Win* win, int slot, hipStream_t st)
{
    k_win_reset<<<1, 64, 0, st>>>(win, slot);
    return hipGetLastError();
}

// ---------------------------------------------------------------- initialisation

__device__ __forceinline__ bool init_solid(const GridP& g, const BodyP& b, int i, int j)
{
    if (i < 0 || i >= g.nx || j < 0 || j >= g.ny) return false;
    const double x = pos_x(g, b, i);
    const double y = pos_y(g, b, j);
    return shape_phi(b, x, y) < 0.0;
}

// box of the initial solid set {interior nodes: phi0(x) < 0}
__global__ __launch_bounds__(256) void k_init_solid_box(GridP g, BodyP b, int* boxpart,
                                                        unsigned* ticket, Win* win, int s0, int s1)
{
    const long long N = (long long)g.nx * g.ny;
    int i0 = 0x3fffffff, i1 = -0x3fffffff, j0 = 0x3fffffff, j1 = -0x3fffffff;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < N; e += stride) {
        const int i = (int)(e % g.nx), j = (int)(e / g.nx);
        if (init_solid(g, b, i, j)) {
            i0 = min(i0, i);
            i1 = max(i1, i);
            j0 = min(j0, j);
            j1 = max(j1, j);
        }
    }
    block_box(i0, i1, j0, j1, boxpart + 4 * blockIdx.x);
    if (last_block(ticket)) {
        reduce_boxes<true>(boxpart, gridDim.x, &win[s0], &win[s1]);
        if (threadIdx.x == 0) *ticket = 0u;
    }
}

hipError_t launch_init_solid_box(const GridP& g, const BodyP& b, const BandBufs& bb, int slot0,
                                 int slot1, hipStream_t st)
{
    k_init_solid_box<<<BOX_BLOCKS, 256, 0, st>>>(g, b, bb.boxpart, bb.ticket, bb.win, slot0,
                                                 slot1);
    return hipGetLastError();
}

// initial tags over the window (solid / none)
__global__ __launch_bounds__(256) void k_init_tags(GridP g, BodyP b, int8_t* tag, const Win* win,
                                                   int wslot, int* lcount)
{
    clear_lcount(lcount);
    const Rect W = window_of(win, wslot, g);
    if (!W.ok) return;
    const int w = W.i1 - W.i0 + 1, h = W.j1 - W.j0 + 1;
    const long long total = (long long)w * h;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = W.i0 + (int)(e % w), j = W.j0 + (int)(e / w);
        tag[pidx(g, i, j)] = init_solid(g, b, i, j) ? TAG_SOLID : TAG_NONE;
    }
}

hipError_t launch_init_tags(const GridP& g, const BodyP& b, const BandBufs& bb, int wslot,
                            hipStream_t st)
{
    k_init_tags<<<2048, 256, 0, st>>>(g, b, bb.tag, bb.win, wslot, bb.lcount);
    return hipGetLastError();
}

// xi_0 = x on the solid and its extrapolation zone, phi = phi0(x) (Alg. 1 init)
template <typename T>
__global__ void k_init_fill(GridP g, BodyP b, const int8_t* tag, const Win* win, int wslot,
                            T* X, T* Y, T* phi, int* lcount)
{
    constexpr bool DISP = sizeof(T) == 4;
    clear_lcount(lcount);  // for the first step's distance transform
    const Rect W = window_of(win, wslot, g);
    if (!W.ok) return;
    const int w = W.i1 - W.i0 + 1, h = W.j1 - W.j0 + 1;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < (long long)w * h;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = W.i0 + (int)(e % w), j = W.j0 + (int)(e / w);
        const long long k = pidx(g, i, j);
        if (tag[k] != TAG_NONE) {
            const double x = pos_x(g, b, i);
            const double y = pos_y(g, b, j);
            X[k] = DISP ? T(0) : T(x);
            Y[k] = DISP ? T(0) : T(y);
            phi[k] = store_phi<T>(shape_phi(b, x, y));
        } else {
            X[k] = T(NAN);
            Y[k] = T(NAN);
            phi[k] = T(INFINITY);
        }
    }
}

hipError_t launch_init_fill(const GridP& g, const BodyP& b, const BandBufs& bb, int wslot,
                            hipStream_t st)
{
    if (g.rm32)
        k_init_fill<float><<<2048, 256, 0, st>>>(g, b, bb.tag, bb.win, wslot, (float*)bb.X[0],
                                                 (float*)bb.Y[0], (float*)bb.phi[0], bb.lcount);
    else
        k_init_fill<double><<<2048, 256, 0, st>>>(g, b, bb.tag, bb.win, wslot, (double*)bb.X[0],
                                                  (double*)bb.Y[0], (double*)bb.phi[0],
                                                  bb.lcount);
    return hipGetLastError();
}

// ---------------------------------------------------------------- advection

// reference-map node (i, j) of step n: canonical index, or -1 if it holds no
// value (outside the domain or outside the window D where xi^n was written)
__device__ __forceinline__ long long ref_index(const GridP& g, const Rect& D, int i, int j)
{
    if (!canon(g, i, j) || !D.has(i, j)) return -1;
    return pidx(g, i, j);
}

// one-sided second-order upwind derivative of Eq. (3_1_eno) from preloaded
// stencil values (m1, m2: one and two nodes behind; p1, p2: ahead).  For
// displacement storage the derivative of the node coordinate itself, exactly
// 1 along the axis, is added by the caller.
template <typename C>
__device__ __forceinline__ bool upwind_d(C vel, C X0, C Y0, bool okm1, bool okm2, C Xm1, C Ym1,
                                         C Xm2, C Ym2, bool okp1, bool okp2, C Xp1, C Yp1, C Xp2,
                                         C Yp2, C& dX, C& dY)
{
    dX = dY = C(0);
    if (vel == C(0)) return true;
    if (vel > C(0)) {
        if (!okm1 || !okm2) return false;
        dX = (C(3) * X0 - C(4) * Xm1 + Xm2) / C(2);
        dY = (C(3) * Y0 - C(4) * Ym1 + Ym2) / C(2);
    } else {
        if (!okp1 || !okp2) return false;
        dX = (C(-3) * X0 + C(4) * Xp1 - Xp2) / C(2);
        dY = (C(-3) * Y0 + C(4) * Yp1 - Yp2) / C(2);
    }
    return true;
}

// Eq. (3_1_refmap_adv) at one solid node (i, j) of S^n = {interior,
// phi^n < 0}.  Every load (the eight upwind stencil nodes with their level
// sets, the nine populations and the previous force) is issued before any is
// used; addresses of absent nodes are clamped to the node itself.  S is both
// the population and the reference-map storage type (FP64: xi; FP32:
// population deviations and displacement).  LATCHK: every lattice node the
// pull gather reads must lie in D (with the chain beside the bulk update,
// the nodes of D are the ones the previous step's force pass updated); a
// solid node on D's rim is counted as an advection miss and keeps its value.
// INNER: every stencil node lies in D, and the lattice node off the lattice's
// border, so that all addresses are fixed offsets from the node's (the same
// loads and arithmetic, without the tests: about a third fewer instructions,
// which bound the pass where a solid is large; MI355X, 2048^2 cavity FP64 22 ->
// 18 us, 96 batch members FP32 94 -> 80).
template <typename S, bool LATCHK, bool INNER>
__device__ __forceinline__ void advect_at(const GridP& g, const S* __restrict__ A,
                                            const double* __restrict__ fpx,
                                            const double* __restrict__ fpy,
                                            const S* __restrict__ X, const S* __restrict__ Y,
                                            const S* __restrict__ phi, S* X1, S* Y1,
                                            const Rect& D, int i, int j, unsigned* health)
{
    using C = S;
    constexpr bool DISP = sizeof(S) == 4;
    const long long P = g.plane;
    const int k = (int)pidx(g, i, j);  // (a map has fewer than 2^26 nodes)
    // stencil nodes: x-1, x-2, x+1, x+2, y-1, y-2, y+1, y+2
    const int di[8] = {-1, -2, 1, 2, 0, 0, 0, 0};
    const int dj[8] = {0, 0, 0, 0, -1, -2, 1, 2};
    int ks[8];
#pragma unroll
    for (int q = 0; q < 8; q++)
        ks[q] = INNER ? k + dj[q] * g.pp + di[q] : (int)ref_index(g, D, i + di[q], j + dj[q]);
    // populations of the pull gather (the node is interior), at the node's
    // lattice position (a solid's window may be a sub-range of the lattice)
    const int li = lat_col(g, i), lj = lat_row(g, j);
    const bool bw = !INNER && !g.lpx && li == 0, be = !INNER && !g.lpx && li == g.lnx - 1;
    const bool bs = !INNER && !g.lpy && lj == 0, bn = !INNER && !g.lpy && lj == g.lny - 1;
    int im = li - 1, ip = li + 1, jm = lj - 1, jp = lj + 1;
    if (!INNER) {
        im = im < 0 ? (g.lpx ? g.lnx - 1 : 0) : im;
        ip = ip >= g.lnx ? (g.lpx ? 0 : g.lnx - 1) : ip;
        jm = jm < 0 ? (g.lpy ? g.lny - 1 : 0) : jm;
        jp = jp >= g.lny ? (g.lpy ? 0 : g.lny - 1) : jp;
    }
    bool lat_ok = true;
    if (LATCHK && !INNER) {
        // D is a rectangle holding (i, j): the four axis neighbours decide
        int iw = i - 1, ie = i + 1, js = j - 1, jn = j + 1;
        if (g.px) {
            iw = wrap_axis(iw, g.nx);
            ie = wrap_axis(ie, g.nx);
        }
        if (g.py) {
            js = wrap_axis(js, g.ny);
            jn = wrap_axis(jn, g.ny);
        }
        lat_ok = (bw || D.has(iw, j)) && (be || D.has(ie, j)) && (bs || D.has(i, js)) &&
                 (bn || D.has(i, jn));
        if (!lat_ok) {
            im = ip = li;
            jm = jp = lj;
        }
    }
    const int r0 = lj * g.pitch, rm = jm * g.pitch, rp = jp * g.pitch, n = r0 + li;
    // ---- all loads
    const C X0 = X[k], Y0 = Y[k];
    C ps[8], xs[8], ys[8];
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const int kq = INNER || ks[q] >= 0 ? ks[q] : k;
        ps[q] = phi[kq];
        xs[q] = X[kq];
        ys[q] = Y[kq];
    }
    C f[NQ];
    f[0] = A[n];
    f[1] = bw ? (A + 3 * P)[n] : (A + 1 * P)[r0 + im];
    f[2] = bs ? (A + 4 * P)[n] : (A + 2 * P)[rm + li];
    f[3] = be ? (A + 1 * P)[n] : (A + 3 * P)[r0 + ip];
    f[4] = bn ? (A + 2 * P)[n] : (A + 4 * P)[rp + li];
    f[5] = (bw || bs) ? (A + 7 * P)[n] : (A + 5 * P)[rm + im];
    f[6] = (be || bs) ? (A + 8 * P)[n] : (A + 6 * P)[rm + ip];
    f[7] = (be || bn) ? (A + 5 * P)[n] : (A + 7 * P)[rp + ip];
    f[8] = (bw || bn) ? (A + 6 * P)[n] : (A + 8 * P)[rp + im];
    const C Fx = C(fpx[n]), Fy = C(fpy[n]);
    // ---- arithmetic: half-force velocity of Eq. (2_2_lbm_moments_force); the
    // FP32 mode stores f_i - w_i rho_f (sum w_i = 1, sum w_i c_i = 0)
    const C s9 = f[0] + f[1] + f[2] + f[3] + f[4] + f[5] + f[6] + f[7] + f[8];
    const C rho = DISP ? C(g.rho_f) + s9 : s9;
    const C u = (f[1] + f[5] + f[8] - f[3] - f[6] - f[7]) / rho + Fx / (C(2) * rho);
    const C v = (f[2] + f[5] + f[6] - f[4] - f[7] - f[8]) / rho + Fy / (C(2) * rho);
    bool okq[8];
#pragma unroll
    for (int q = 0; q < 8; q++) okq[q] = (INNER || ks[q] >= 0) && ps[q] < C(INFINITY);
    C dXx, dYx, dXy, dYy;
    const bool okx = upwind_d<C>(u, X0, Y0, okq[0], okq[1], xs[0], ys[0], xs[1], ys[1], okq[2],
                                 okq[3], xs[2], ys[2], xs[3], ys[3], dXx, dYx);
    const bool oky = upwind_d<C>(v, X0, Y0, okq[4], okq[5], xs[4], ys[4], xs[5], ys[5], okq[6],
                                 okq[7], xs[6], ys[6], xs[7], ys[7], dXy, dYy);
    if (!okx || !oky || !lat_ok) {
        atomicAdd(&health[0], 1u);
        X1[k] = X0;
        Y1[k] = Y0;
    } else if (DISP) {
        // xi = x + d: d(X)/dx = 1 + dXx, d(Y)/dy = 1 + dYy
        X1[k] = X0 - (u * (C(1) + dXx) + v * dXy);
        Y1[k] = Y0 - (u * dYx + v * (C(1) + dYy));
    } else {
        X1[k] = X0 - (u * dXx + v * dXy);
        Y1[k] = Y0 - (u * dYx + v * dYy);
    }
}

template <typename S, bool LATCHK = false>
__device__ __forceinline__ void advect_node(const GridP& g, const S* __restrict__ A,
                                            const double* __restrict__ fpx,
                                            const double* __restrict__ fpy,
                                            const S* __restrict__ X, const S* __restrict__ Y,
                                            const S* __restrict__ phi, S* X1, S* Y1,
                                            const Rect& D, int i, int j, unsigned* health)
{
    const int li = lat_col(g, i), lj = lat_row(g, j);
    const bool inner = i - 2 >= D.i0 && i + 2 <= D.i1 && j - 2 >= D.j0 && j + 2 <= D.j1 &&
                       li > 0 && li < g.lnx - 1 && lj > 0 && lj < g.lny - 1;
    if (__all(inner))
        advect_at<S, LATCHK, true>(g, A, fpx, fpy, X, Y, phi, X1, Y1, D, i, j, health);
    else
        advect_at<S, LATCHK, false>(g, A, fpx, fpy, X, Y, phi, X1, Y1, D, i, j, health);
}

// ---------------------------------------------------------------- layers

// Layers of Sec. 3.2: layer 1 = non-solid nodes 4-adjacent to the solid,
// layer l = unmarked nodes 4-adjacent to layer l-1.  Inside a rectangle this
// is the Manhattan distance to the solid set, computed here exactly on tiles
// of DTX x TH nodes with a halo of `layers` nodes.
//
// Up to DT_MASK_LAYERS layers (LC = 11, the count as a compile-time constant,
// or LC = 0) a row of the region is one 64-bit word of solid flags: a wave
// reads a row with one node per lane, coalesced, and ballots the signs; then
// lane r holds row r, and a layer is one dilation of the region, d | d << 1 |
// d >> 1 | the rows above and below (a lane to either side), whose new bits are
// added to the planes of a bit-sliced layer number.  Every wave runs all of
// it (14 instructions a layer), which spares the barriers between layers.
// Bound by its chain of loads (window, level set) and, for a large solid, by
// the advection's loads in flight (MI355X, pass over the solid of a 64^2
// cavity 12.4 -> 8.9 us against scans of 38 x 54 flags in LDS with 16-row
// tiles; 96 members of 96^2 .. 768^2, FP32, 107 -> 96 us).
// More layers (LC = -1, the region wider than a word): two separable passes
// over flags in LDS, per column the distance to the nearest solid node of the
// column (capped at layers + 1), per row the minimum over |e| of |e| + that.
//
// Then the tile's tags are written and its zone nodes listed: for the
// extrapolation in one launch the tile alone (ff_list), else the nodes of
// each layer (lists, split into NSUB sub-lists by block so that few blocks
// share a counter; the order inside a list does not matter since targets of
// one layer are independent).  The counters were cleared by the kernels
// before.
constexpr int DTX = 32, DTY = 16;
// rows of a tile when no layer lists are made: fewer halo rows read per node,
// and a tile is listed by its own block
constexpr int DTY_FF = FF_TILE;
static_assert(DTX == FF_TILE, "a fused-fit tile");
constexpr int DT_MASK_LAYERS = 16;
static_assert(DTX + 2 * DT_MASK_LAYERS <= 64 && DTY_FF + 2 * DT_MASK_LAYERS <= 64,
              "a region's row is one word, its rows one wave's lanes");
static_assert(FF_LAYERS <= DT_MASK_LAYERS, "DTY_FF tiles use the words");
constexpr int DRW = DTX + 2 * MAX_LAYERS, DRH = DTY + 2 * MAX_LAYERS;

// the word of the lane below (r - 1) or above (r + 1), 0 beyond the wave
template <int CTRL>
__device__ __forceinline__ unsigned long long row_shift(unsigned long long v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, true);
    return (unsigned long long)(unsigned)hi << 32 | (unsigned)lo;
}
constexpr int DPP_WAVE_SHL1 = 0x130, DPP_WAVE_SHR1 = 0x138;

// ADV = false (initialisation): the solid set is read from the tags.  ADV =
// true (a step): the solid set S^n = {interior, phi^n < 0, inside the
// previous window} is read from the level set, the tile's solid nodes are
// tagged and advected (Sec. 3.1) in the same pass, and the tags of the window
// are all written here.
template <int LC, int TH, bool ADV, typename S, bool LATCHK = false>
__device__ __forceinline__ void dt_tile_body(GridP g, const Win* __restrict__ win, int wslot,
                                             int wprev, int8_t* tag, int* lists, int* lcount,
                                             unsigned* health, const S* __restrict__ A,
                                             const double* __restrict__ fpx,
                                             const double* __restrict__ fpy,
                                             const S* __restrict__ X, const S* __restrict__ Y,
                                             const S* __restrict__ phi, S* X1, S* Y1,
                                             int* ff_list = nullptr, int* ff_n = nullptr)
{
    constexpr bool MASK = LC >= 0;
    static_assert(MASK || TH == DTY, "the scans' region");
    const Rect W = window_of(win, wslot, g);
    if (!W.ok) return;
    const Rect D = window_of(win, wprev, g);
    const int L = LC > 0 ? LC : g.layers;
    const int w = W.i1 - W.i0 + 1, h = W.j1 - W.j0 + 1;
    const int ntx = (w + DTX - 1) / DTX, nty = (h + TH - 1) / TH;
    // When the grid has enough blocks beyond the tiles (ADV_MIN_WORKERS, or
    // one thread for each node of the solid set's box), block t < ntile takes
    // tile t without its advection, and the blocks beyond advect the solid
    // nodes of that box, 256 nodes of it (row-major) at a time, one per
    // thread: interior tiles no longer advect their nodes in turn while
    // boundary tiles idle.  The solid set is the same (interior, phi^n < 0,
    // inside D), and each node's advection is the same arithmetic, so the
    // bits are too.
    const int ntile = ntx * nty;
    bool adv_here = ADV;
    if (ADV) {
        const Win B = win[wslot];  // (a box of interior nodes)
        const int bw = B.i1 - B.i0 + 1;
        const long long nn = (long long)bw * (B.j1 - B.j0 + 1);
        const int nwork = (int)gridDim.x - ntile;
        if (nwork >= ADV_MIN_WORKERS || (nwork > 0 && nwork * 256ll >= nn)) {
            adv_here = false;
            if ((int)blockIdx.x >= ntile) {
                for (long long e = (long long)(blockIdx.x - ntile) * blockDim.x + threadIdx.x;
                     e < nn; e += (long long)nwork * blockDim.x) {
                    const int x = B.i0 + (int)(e % bw), y = B.j0 + (int)(e / bw);
                    if (D.has(x, y) && phi[pidx(g, x, y)] < S(0))
                        advect_node<S, LATCHK>(g, A, fpx, fpy, X, Y, phi, X1, Y1, D, x, y,
                                               health);
                }
                return;
            }
        }
    }
    __shared__ int cnt[MAX_LAYERS + 1];
    __shared__ int base[MAX_LAYERS + 1];
    const long long cap = g.lcap;
    const int sub = blockIdx.x % NSUB;
    const int rw = DTX + 2 * L, rh = TH + 2 * L;  // region in use
    const int lane = __lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    constexpr int NPT = DTX * TH / 256;  // nodes per thread, row-major in waves
    // the nodes whose flag is read: the rest holds no solid
    Rect Z = W;
    if (ADV) {
        Z.i0 = max(max(W.i0, D.i0), 0);
        Z.i1 = min(min(W.i1, D.i1), g.nx - 1);
        Z.j0 = max(max(W.j0, D.j0), 0);
        Z.j1 = min(min(W.j1, D.j1), g.ny - 1);
        Z.ok = D.ok && Z.i0 <= Z.i1 && Z.j0 <= Z.j1;
    }
    for (int t = blockIdx.x; t < ntile; t += gridDim.x) {
        const int x0 = W.i0 + (t % ntx) * DTX, y0 = W.j0 + (t / ntx) * TH;
        // (behind an empty asm: what follows from the thread's number is
        // computed here, not held over the loop)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        int lay[NPT];       // layer number, 0: none
        unsigned solid = 0; // bit u: node u is solid
        bool zone = false;  // the zone reaches the tile
        if constexpr (MASK) {
            constexpr int NP = LC == 11 ? 4 : 5;  // planes of a layer number
            __shared__ unsigned long long rows[64];
            const int x = x0 - L + lane;
            const bool xin = lane < rw && x >= Z.i0 && x <= Z.i1;
            const int xc = xin ? x + PAD : W.i0 + PAD;
            auto flag = [&](int r) {
                const int y = y0 - L + r;
                const bool in = Z.ok && r < rh && y >= Z.j0 && y <= Z.j1;  // (wave-uniform)
                const int k = (in ? y + PAD : W.j0 + PAD) * g.pp + xc;
                if (ADV) {
                    const S p = phi[k];
                    return in && xin && p < S(0);
                }
                return in && xin && tag[k] == TAG_SOLID;
            };
            if constexpr (LC > 0) {
                // all of a wave's rows in flight together
                constexpr int NR = (TH + 2 * LC + 3) / 4;
                bool f[NR];
#pragma unroll
                for (int u = 0; u < NR; u++) f[u] = flag(wv + 4 * u);
                __syncthreads();  // the previous tile's words are no longer read
#pragma unroll
                for (int u = 0; u < NR; u++) {
                    const unsigned long long b = __ballot(f[u]);
                    if (lane == u) rows[wv + 4 * u] = b;
                }
            } else {
                __syncthreads();
                for (int r = wv; r < rh; r += 4) {
                    const unsigned long long b = __ballot(flag(r));
                    if (lane == 0) rows[r] = b;
                }
            }
            if (tid <= MAX_LAYERS) cnt[tid] = 0;
            __syncthreads();
            unsigned long long d = lane < rh ? rows[lane] : 0ull;
            const unsigned ps = (unsigned)(d >> L);
            unsigned pl[NP] = {}, any = 0;
#pragma unroll LC > 0 ? LC : 1
            for (int l = 1; l <= L; l++) {
                const unsigned long long n = d | d << 1 | d >> 1 | row_shift<DPP_WAVE_SHL1>(d) |
                                             row_shift<DPP_WAVE_SHR1>(d);
                const unsigned fresh = (unsigned)((n & ~d) >> L);
                any |= fresh;
#pragma unroll
                for (int b = 0; b < NP; b++)
                    if (l >> b & 1) pl[b] |= fresh;
                d = n;
            }
            const unsigned cols = W.i1 - x0 >= 31 ? ~0u : (2u << (W.i1 - x0)) - 1u;
            zone = __ballot(lane >= L && lane < L + TH && y0 + lane - L <= W.j1 &&
                            (any & cols) != 0) != 0ull;
#pragma unroll
            for (int u = 0; u < NPT; u++) {
                const int e = u * 256 + tid, cx = e % DTX, src = L + e / DTX;
                int l = 0;
#pragma unroll
                for (int b = 0; b < NP; b++) l |= ((unsigned)__shfl((int)pl[b], src) >> cx & 1u) << b;
                lay[u] = l;
                solid |= ((unsigned)__shfl((int)ps, src) >> cx & 1u) << u;
            }
        } else {
            __shared__ int8_t sol[DRH * DRW];  // solid flags of the tile and its halo
            __shared__ int8_t gc[DTY * DRW];   // column distances of the tile rows
            __syncthreads();
            if (tid <= MAX_LAYERS) cnt[tid] = 0;
            for (int e = tid; e < rw * rh; e += blockDim.x) {
                const int x = x0 - L + e % rw, y = y0 - L + e / rw;
                const bool in = Z.ok && x >= Z.i0 && x <= Z.i1 && y >= Z.j0 && y <= Z.j1;
                const long long k = in ? pidx(g, x, y) : pidx(g, W.i0, W.j0);
                bool s;
                if (ADV) s = in && phi[k] < S(0);
                else s = in && tag[k] == TAG_SOLID;
                sol[(e / rw) * DRW + e % rw] = s ? 1 : 0;
            }
            __syncthreads();
            // column pass over the tile rows, the whole region width
            for (int e = tid; e < rw * DTY; e += blockDim.x) {
                const int cx = e % rw, cy = e / rw;
                int best = L + 1;
                for (int d = -L; d <= L; d++)
                    if (sol[(cy + L + d) * DRW + cx]) best = min(best, abs(d));
                gc[cy * DRW + cx] = (int8_t)best;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NPT; u++) {
                const int e = u * 256 + tid;
                const int cx = e % DTX, cy = e / DTX;
                if (sol[(cy + L) * DRW + cx + L]) solid |= 1u << u;
                int best = 2 * L + 2;
                for (int d = -L; d <= L; d++) best = min(best, abs(d) + gc[cy * DRW + cx + L + d]);
                lay[u] = best <= L && !(solid >> u & 1) ? best : 0;
            }
        }
        // tags (a wave covers two rows of the tile)
#pragma unroll
        for (int u = 0; u < NPT; u++) {
            const int e = u * 256 + tid;
            const int x = x0 + e % DTX, y = y0 + e / DTX;
            const bool in = x <= W.i1 && y <= W.j1, s = solid >> u & 1;
            if (!in) {
                lay[u] = 0;
                solid &= ~(1u << u);
            } else if (ADV || !s) {
                tag[pidx(g, x, y)] = s ? TAG_SOLID : lay[u] > 0 ? (int8_t)lay[u] : TAG_NONE;
            }
        }
        if (ff_list) {
            // the tile is the fused extrapolation's (TH = FF_TILE)
            if (zone && tid == 0) ff_list[atomicAdd(ff_n, 1)] = t;
        } else {
            // each node's slot in the block's share of its layer list comes
            // from one LDS atomic per wave and layer present
            int slot[NPT];
#pragma unroll
            for (int u = 0; u < NPT; u++) {
                slot[u] = 0;
                for (int l = 1; l <= L; l++) {
                    const unsigned long long mask = __ballot(lay[u] == l);
                    if (mask == 0ull) continue;
                    const int leader = __ffsll((long long)mask) - 1;
                    int wb = 0;
                    if (lane == leader) wb = atomicAdd(&cnt[l], __popcll(mask));
                    wb = __shfl(wb, leader);
                    if (lay[u] == l) slot[u] = wb + __popcll(mask & ((1ull << lane) - 1ull));
                }
            }
            __syncthreads();
            // one reservation per layer present in the tile
            if (tid >= 1 && tid <= L && cnt[tid] > 0)
                base[tid] =
                    atomicAdd(&lcount[(tid * NSUB + sub) * LCOUNT_PAD], cnt[tid]);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NPT; u++) {
                if (lay[u] > 0) {
                    const int e = u * 256 + tid;
                    const long long at = (long long)base[lay[u]] + slot[u];
                    if (at < cap)
                        lists[(lay[u] * NSUB + sub) * cap + at] =
                            (int)pidx(g, x0 + e % DTX, y0 + e / DTX);
                    else atomicAdd(&health[7], 1u);  // beyond the sub-list capacity
                }
            }
        }
        if (adv_here) {
            // advection of the tile's solid nodes
#pragma unroll 1
            for (int u = 0; u < NPT; u++) {
                const int e = u * 256 + tid;
                if (solid >> u & 1)
                    advect_node<S, LATCHK>(g, A, fpx, fpy, X, Y, phi, X1, Y1, D, x0 + e % DTX,
                                           y0 + e / DTX, health);
            }
        }
    }
}

// initialisation: layers of the initial solid set (from the tags)
template <int LC>
__global__ __launch_bounds__(256) void k_dt_tile(GridP g, const Win* __restrict__ win, int wslot,
                                                 int8_t* tag, int* lists, int* lcount,
                                                 unsigned* health)
{
    dt_tile_body<LC, DTY, false, double>(g, win, wslot, 0, tag, lists, lcount, health, nullptr,
                                         nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                                         nullptr);
}

// a step: advection of xi plus the layers of the extrapolation zone
// FP64: five waves per SIMD (96 registers) run the 2048 blocks in fewer
// rounds (2048^2 step 0.1626 -> 0.1614 ms); FP32 needs 73 and runs six
template <int LC, int TH, typename S>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(sizeof(S) == 8 ? 5 : 1, 8))) void k_advect_dt(
    GridP g, const S* __restrict__ A,
                                                   const double* __restrict__ fpx,
                                                   const double* __restrict__ fpy,
                                                   const S* __restrict__ X,
                                                   const S* __restrict__ Y,
                                                   const S* __restrict__ phi, S* X1, S* Y1,
                                                   int8_t* tag, const Win* __restrict__ win,
                                                   int wprev, int wcur, int* lists, int* lcount,
                                                   unsigned* health, int* ff_list, int* ff_n)
{
    // beside a bulk lattice update the chain's waves take the issue slots of
    // a SIMD first (2048^2 step FP64 155 -> 151 us, FP32 103 -> 93, with the
    // whole bulk update behind this pass)
    __builtin_amdgcn_s_setprio(3);
    dt_tile_body<LC, TH, true, S, true>(g, win, wcur, wprev, tag, lists, lcount, health, A,
                                              fpx, fpy, X, Y, phi, X1, Y1, ff_list, ff_n);
}

// five waves per SIMD: the suspension's 6400 blocks (400 solids) run in
// fewer rounds (FP32 step 0.634 -> 0.619 ms; FP64 0.998 -> 0.994)
template <int LC, int TH, typename S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) void kb_advect_dt(
    const AdvectArgs* __restrict__ args, const int* __restrict__ ord,
    const long long* __restrict__ dstep, long long* dcur)
{
    const AdvectArgs& a = args[ord ? ord[blockIdx.y] : blockIdx.y];
    // several solids: this step's number for the passes that follow (the
    // counter itself moves on before the step ends)
    if (dcur && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *dcur = *dstep;
    dt_tile_body<LC, TH, true, S>(a.g, a.win, a.wcur, a.wprev, a.tag, a.lists, a.lcount, a.health,
                                  (const S*)a.A, a.fpx, a.fpy, (const S*)a.X, (const S*)a.Y,
                                  (const S*)a.phi, (S*)a.X1, (S*)a.Y1, a.ff_list, a.ff_n);
}

// the kernel of a layer count and of the tile rows: KERN(LC, TH)
#define DT_DISPATCH(LAYERS, FUSED, KERN)            \
    do {                                            \
        if (FUSED) {                                \
            if ((LAYERS) == 11) KERN(11, DTY_FF);   \
            else KERN(0, DTY_FF);                   \
        } else if ((LAYERS) == 11) {                \
            KERN(11, DTY);                          \
        } else if ((LAYERS) <= DT_MASK_LAYERS) {    \
            KERN(0, DTY);                           \
        } else {                                    \
            KERN(-1, DTY);                          \
        }                                           \
    } while (0)

hipError_t launch_advect_layers(const GridP& g, int precision, const BandBufs& bb,
                                const StepSlots& s, const void* A, const double* fpx,
                                const double* fpy, hipStream_t st, bool fused)
{
    int* ffs = fused ? bb.ff_list : nullptr;
    int* ffn = fused ? bb.ff_n : nullptr;
    // blocks beyond the tiles of the largest window and one advection thread
    // per node of it find nothing to do
    const long long ths = fused ? DTY_FF : DTY;
    const long long tiles = ((g.nx + 2 * PAD + DTX - 1) / DTX) * ((g.ny + 2 * PAD + ths - 1) / ths);
    const long long nodes = ((long long)g.nx * g.ny + 255) / 256;
    const long long want = tiles + std::max<long long>(nodes, ADV_MIN_WORKERS);
    const int blocks = (int)std::min<long long>(DT_BLOCKS, want);
#define ADT(S, LC, TH)                                                                            \
    k_advect_dt<LC, TH, S><<<blocks, 256, 0, st>>>(                                             \
        g, (const S*)A, fpx, fpy, (const S*)bb.X[s.cur], (const S*)bb.Y[s.cur],                   \
        (const S*)bb.phi[s.cur], (S*)bb.X[s.nxt], (S*)bb.Y[s.nxt], bb.tag, bb.win, s.wprev,      \
        s.wcur, bb.lists, bb.lcount, bb.health, ffs, ffn)
#define ADT_D(LC, TH) ADT(double, LC, TH)
#define ADT_F(LC, TH) ADT(float, LC, TH)
    if (precision == 0) DT_DISPATCH(g.layers, fused, ADT_D);
    else DT_DISPATCH(g.layers, fused, ADT_F);
#undef ADT_F
#undef ADT_D
#undef ADT
    return hipGetLastError();
}

hipError_t launch_layers(const GridP& g, const BandBufs& bb, int wslot, hipStream_t st)
{
#define KDT(LC, TH)                                                                              \
    k_dt_tile<LC><<<DT_BLOCKS, 256, 0, st>>>(g, bb.win, wslot, bb.tag, bb.lists, bb.lcount,      \
                                             bb.health)
    DT_DISPATCH(g.layers, false, KDT);
#undef KDT
    return hipGetLastError();
}

// ---------------------------------------------------------------- extrapolation

// outward normal of phi^n at a target from its four neighbours (e, w, n, s),
// used by the weights of layers 1 and 2
__device__ __forceinline__ bool normal_from(double pe, double pw, double pn, double ps,
                                            double& nxh, double& nyh)
{
    if (!(pe < INFINITY && pw < INFINITY && pn < INFINITY && ps < INFINITY)) return false;
    const double gx = (pe - pw) / 2.0;
    const double gy = (pn - ps) / 2.0;
    const double gn = sqrt(gx * gx + gy * gy);
    if (!(gn > 0.0)) return false;
    nxh = gx / gn;
    nyh = gy / gn;
    return true;
}

// Sums of the normal equations over the nodes of the scan window of
// half-width r (side 2r + 1, nodes q = 0 .. side^2 - 1 row by row) that fall
// to this lane: node q goes to lane q mod FIT_LANES; each lane issues the
// loads of PER nodes before adding them.  The offsets (a, b) of node q are
// stepped along instead of divided out.
template <typename T>
__device__ __forceinline__ void fit_window(const GridP& g, const Rect& W, int l, int i, int j,
                                           int kt, int r, int sub, bool use_n, double nxh,
                                           double nyh, const int8_t* tag, const T* X1,
                                           const T* Y1, Fit<T>& f, int& count)
{
    constexpr int PER = 4;
    const int side = 2 * r + 1, nq = side * side;
    // offsets of this lane's first node
    int a = sub % side - r, b = sub / side - r;
    for (int q0 = sub; q0 < nq; q0 += PER * FIT_LANES) {
        long long kk[PER];
        int tk[PER], aa[PER], bb[PER];
        T xv[PER], yv[PER];
#pragma unroll
        for (int u = 0; u < PER; u++) {
            aa[u] = a;
            bb[u] = b;
            int ci = i + a, cj = j + b;
            kk[u] = (q0 + u * FIT_LANES < nq && canon(g, ci, cj) && W.has(ci, cj))
                        ? pidx(g, ci, cj) : -1;
            // advance by FIT_LANES nodes along the rows
            a += FIT_LANES;
            while (a > r) {
                a -= side;
                b += 1;
            }
        }
#pragma unroll
        for (int u = 0; u < PER; u++) {
            const long long k = kk[u] >= 0 ? kk[u] : kt;
            tk[u] = tag[k];
            xv[u] = X1[k];
            yv[u] = Y1[k];
        }
#pragma unroll
        for (int u = 0; u < PER; u++) {
            if (kk[u] < 0 || !tag_valid_before(tk[u], l)) continue;
            count++;
            f.add(aa[u], bb[u], use_n, nxh, nyh, xv[u], yv[u]);
        }
    }
}

// scan window of half-width 2 around target kt = (i, j) read from the maps
// (lane sub of an 8-lane group)
template <typename T, bool N>
__device__ __forceinline__ bool fit2_global(const GridP& g, const Rect& W,
                                            int l, int i, int j, int kt, int sub, bool use_n,
                                            double nxh, double nyh, const int8_t* tag,
                                            const T* X1, const T* Y1, T& xo, T& yo)
{
    using C2 = Win2<T, 1>;
    bool v[C2::NS];
    T xs[C2::NS], ys[C2::NS];
    int tk[C2::NS];
#pragma unroll
    for (int u = 0; u < C2::NS; u++) {
        int ci = i + C2::off_a(sub, u), cj = j + C2::off_b(sub, u);
        v[u] = C2::in(sub, u) && canon(g, ci, cj) && W.has(ci, cj);
        const long long k = v[u] ? pidx(g, ci, cj) : kt;
        tk[u] = tag[k];
        xs[u] = X1[k];
        ys[u] = Y1[k];
    }
#pragma unroll
    for (int u = 0; u < C2::NS; u++) {
        v[u] = v[u] && tag_valid_before(tk[u], l);
        xs[u] = v[u] ? xs[u] : T(0);
        ys[u] = v[u] ? ys[u] : T(0);
    }
    const unsigned mask = C2::mask_of(sub, v);
    if (N && use_n) {
        typename C2::NW w;
        if (!C2::weights_n(sub, __popc(mask), v, nxh, nyh, g.det_rel, w)) return false;
        C2::value_n(sub, w, xs, ys, xo, yo);
    } else {
        const Geo2 G = geo2(mask, g.det_rel);
        if (!G.ok) return false;
        C2::value(sub, G, xs, ys, xo, yo);
    }
    return true;
}

// outward normal of phi^n at target (i, j) for the weights of layers 1 and 2:
// lanes 0..3 of the group load the four neighbours
template <typename T>
__device__ __forceinline__ bool target_normal(const GridP& g, const Rect& D, int l, int i, int j,
                                              int sub, const T* __restrict__ phin, double& nxh,
                                              double& nyh)
{
    nxh = nyh = 0.0;
    if (l > 2) return false;
    double p = INFINITY;
    if (sub < 4) {
        const int di = sub == 0 ? 1 : sub == 1 ? -1 : 0;
        const int dj = sub == 2 ? 1 : sub == 3 ? -1 : 0;
        const long long kq = ref_index(g, D, i + di, j + dj);
        if (kq >= 0) p = (double)phin[kq];
    }
    const double pe = __shfl(p, 0, FIT_LANES), pw = __shfl(p, 1, FIT_LANES);
    const double pn = __shfl(p, 2, FIT_LANES), ps = __shfl(p, 3, FIT_LANES);
    return normal_from(pe, pw, pn, ps, nxh, nyh);
}

// Fit of one target kt = (i, j) of layer l by the FIT_LANES lanes of a group
// (every lane of the group calls it with the same target): the outward normal
// of phi^n for layers 1 and 2, then scan windows of half-width r = 2 .. r_max
// until one holds three valid nodes and a well-posed fit.  N: layers 1 and 2
// (an instance of their own: the other layers' needs fewer registers).
template <typename T, bool N>
__device__ __forceinline__ bool fit_target(const GridP& g, const Rect& W, const Rect& D,
                                           int l, int kt, int i, int j,
                                           int sub, const int8_t* tag,
                                           const T* __restrict__ phin, const T* X1, const T* Y1,
                                           T& xo, T& yo)
{
    double nxh = 0.0, nyh = 0.0;
    const bool use_n = N && target_normal<T>(g, D, l, i, j, sub, phin, nxh, nyh);
    if (fit2_global<T, N>(g, W, l, i, j, kt, sub, use_n, nxh, nyh, tag, X1, Y1, xo, yo))
        return true;
    for (int r = 3; r <= g.r_max; r++) {
        int count = 0;
        Fit<T> f;
        f.zero();
        fit_window<T>(g, W, l, i, j, kt, r, sub, use_n, nxh, nyh, tag, X1, Y1, f, count);
        if (fit_finish<T>(g.det_rel, f, count, xo, yo)) return true;
    }
    return false;
}

// One layer of Sec. 3.2: every target of the layer list is fitted by a group
// of FIT_LANES lanes that share the scan-window nodes; the sums of the normal
// equations are reduced across the group.  Scan windows grow from r = 2 to
// r_max until they hold three valid nodes and a well-posed fit.  Valid nodes
// come only from earlier layers, so targets of one layer never read each
// other.  With displacement storage the fit of d = xi - x gives the fit of xi
// minus x at the target, since the weighted fit reproduces linear fields.
template <typename T, bool N>
__device__ __forceinline__ void layer_fit_body(GridP g, const Win* __restrict__ win,
                                                   int wcur, int wprev, int l, int8_t* tag,
                                                   const int* __restrict__ lists,
                                                   const int* __restrict__ lcount,
                                                   const T* __restrict__ phin, T* X1, T* Y1,
                                                   unsigned* health)
{
    // group g takes sub-list g mod NSUB (the sub-lists come from interleaved
    // distance-transform blocks, so they are of similar length); its first
    // list entry is loaded together with the sub-list's count
    const long long cap = g.lcap;
    const int sub = threadIdx.x % FIT_LANES;
    const int grp = (blockIdx.x * blockDim.x + threadIdx.x) / FIT_LANES;
    const int s = grp % NSUB, a0 = grp / NSUB;
    const int astride = gridDim.x * blockDim.x / FIT_LANES / NSUB;
    const int* list = lists + (l * NSUB + s) * cap;
    const int ns = (int)min((long long)lcount[(l * NSUB + s) * LCOUNT_PAD], cap);
    const int kfirst = a0 < cap ? list[a0] : 0;
    const Rect W = window_of(win, wcur, g);
    const Rect D = window_of(win, wprev, g);
    if (a0 >= ns || !W.ok) return;  // whole groups leave together
    // all lanes of a group run the same trip counts, so shuffles see full groups
    for (int at = a0; at < ns; at += astride) {
        const int kt = at == a0 ? kfirst : list[at];
        const int i = kt % g.pp - PAD, j = kt / g.pp - PAD;
        T xo = T(0), yo = T(0);
        const bool done = fit_target<T, N>(g, W, D, l, kt, i, j, sub, tag, phin, X1, Y1, xo,
                                           yo);
        if (sub == 0) {
            if (done) {
                X1[kt] = xo;
                Y1[kt] = yo;
            } else {
                tag[kt] = (int8_t)(l | TAG_FAIL);
                atomicAdd(&health[1], 1u);
            }
        }
    }
}

template <typename T, bool N>
__global__ __launch_bounds__(256) void k_layer_fit(GridP g, const Win* __restrict__ win,
                                                   int wcur, int wprev, int l, int8_t* tag,
                                                   const int* __restrict__ lists,
                                                   const int* __restrict__ lcount,
                                                   const T* __restrict__ phin, T* X1, T* Y1,
                                                   unsigned* health)
{
    layer_fit_body<T, N>(g, win, wcur, wprev, l, tag, lists, lcount, phin, X1, Y1, health);
}

template <typename T, bool N>
__global__ __launch_bounds__(256) void kb_layer_fit(const FitArgs* __restrict__ args, int l)
{
    const FitArgs& a = args[blockIdx.y];
    if (l > a.g.layers) return;
    layer_fit_body<T, N>(a.g, a.win, a.wcur, a.wprev, l, a.tag, a.lists, a.lcount,
                         (const T*)a.phin, (T*)a.X1, (T*)a.Y1, a.health);
}

// ---- every layer of a region in one block
//
// A region of the window (a tile with its margin, or a whole window) is copied
// into LDS once: tags, and the advected values of the solid nodes.  What the
// fits depend on besides values is then known at once: which nodes are valid
// at layer l is in the tags (solid, or of an earlier layer), so the targets
// of every layer are listed, their validity masks taken and their cofactors
// computed up front, all layers side by side.  A layer is left with the
// dependent part alone: read the window's values, weigh and add them, write
// the result.
//
// A block's time is its instruction count (one VALU instruction of a wave takes
// its SIMD 4 cycles and a layer has 20 to 100 targets), so one lane takes a
// target (a 64-target layer is one wave's work; eight lanes repeated the solve
// eight times and the window's offsets, weights and address arithmetic are
// constants when the slot is a node), and four sets of two waves take the
// layers in turn: one finishes layer l while the others take the coefficients
// and addresses of the next three from their records.  Measured alone, 64^2
// FP64: eight lanes and every sum in double 38.5 us, eight lanes and integer
// normal matrices 27.4, two lanes with records 20.2, this 18.6 (256^2 FP32: 31 to
// 18.5).
//
// A target that the copy cannot serve (its fit needs a scan window wider than
// half-width 2, or fails for good) sets s.cut to its layer: the layers before
// it stand, the caller sees to the others (FIT_TILE).
// A whole window's copy holds every node there is, so it can serve wider scan
// windows too: FIT_WIDE lists such targets (up to FF_WIDE) and searches them in
// the copy as on the maps, eight lanes each, when the others of their layer are
// done; one that fails for good cuts the layers after its own, whose records
// take it for valid.  (60 solids of 44 x 1.8 nodes, us/step FP64 with the layers
// from the first such target on fitted from the maps 207, searched in the copy
// 101; FP32 184, 88.)  The search in its layers costs a solid without such
// targets 2 us a step, so FIT_WHOLE goes first and leaves before its third layer
// with nothing written if there are any.
enum FitMode { FIT_TILE, FIT_WHOLE, FIT_WIDE };
template <typename T>
struct Vec2;
template <>
struct Vec2<double> {
    using V = double2;
};
template <>
struct Vec2<float> {
    using V = float2;
};

// REC uint4: a record of the layers 3 and up holds the mask of valid nodes and
// the normal matrix; unsigned: the mask alone
template <typename T, int NODES, int LN, typename REC = uint4>
struct FitLds {
    typename Vec2<T>::V val[NODES + 1];  // values of node e at e + 1; the first stays zero
    REC rec[(FF_LAYERS - 2) * LN];       // layers >= 3
    unsigned short lst[FF_LAYERS * LN];  // targets of layer l (places in the copy) from (l - 1) LN
    unsigned char st[NODES];             // tags; 255 where there is none
    unsigned short wide[FF_WIDE];        // targets without a fit at half-width 2
    int cnt[FF_LAYERS + 1];
    int nwide, wlayers;                  // their number, and their layers (a bit each)
    int cut;
};

// the region: origin (x0, y0), width rw (rh rows), its own nodes [ox, ox + ow)
// x [oy, oy + oh); targets of layer l are taken within mstep (L - l) of them
struct FitRegion {
    int x0, y0, rw, rh, ox, oy, ow, oh, mstep;
};

template <typename T, int NT, int NODES, int LN, int RWC, FitMode MODE, typename REC>
__device__ __forceinline__ void fit_region(FitLds<T, NODES, LN, REC>& s, const GridP& g,
                                           const Rect& W, const Rect& D, int L,
                                           const FitRegion& R, int8_t* tag,
                                           const T* __restrict__ phin, T* X1, T* Y1,
                                           unsigned* health, int reach)
{
    constexpr bool WIDE = MODE == FIT_WIDE;
    using C2 = Win2<T, 8>;
    constexpr int NS = C2::NS;
    constexpr int NIT = (NODES + NT - 1) / NT;  // staged nodes per thread
    constexpr int NSET = 4, SW = NT / NSET;     // sets of threads, targets per pass
    static_assert(SW % 64 == 0, "whole waves");
    const int rw = RWC > 0 ? RWC : R.rw;
    // (behind an empty asm: what follows from the thread's number is computed
    // here for each region, not ahead of a loop over regions, where it would
    // hold half the registers)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int set = tid / SW, lane = tid % SW;
    // ---- copy: every tag and value of the thread's nodes in flight together;
    // node tid + u NT, stepped along the rows; periodic axes wrap (the region
    // is no wider than a period)
    const int step_y = NT / rw, step_x = NT % rw;
    int tvs[NIT];
    T xs0[NIT], ys0[NIT];
    const int wx = g.px ? g.nx : 0, wy = g.py ? g.ny : 0;
    {
        int x = R.x0 + tid % rw, y = R.y0 + tid / rw;
        const int xe = R.x0 + rw, ye = R.y0 + R.rh;
#pragma unroll
        for (int u = 0; u < NIT; u++) {
            const int xc = x + (x < 0 ? wx : x >= g.nx ? -wx : 0);
            const int yc = y + (y < 0 ? wy : y >= g.ny ? -wy : 0);
            const bool in = y < ye && W.has(xc, yc);
            const int kq = in ? (yc + PAD) * g.pp + xc + PAD : 0;
            const int tv = tag[kq];
            tvs[u] = in ? tv : TAG_NONE;
            xs0[u] = X1[kq];
            ys0[u] = Y1[kq];
            x += step_x;
            y += step_y;
            if (x >= xe) {
                x -= rw;
                y++;
            }
        }
    }
    __syncthreads();  // the previous region's shared state is no longer read
    if (tid <= FF_LAYERS) s.cnt[tid] = 0;
    if (WIDE && tid == FF_LAYERS + 1) s.nwide = s.wlayers = 0;
    if (tid == 0) {
        s.cut = L + 1;
        s.val[0].x = s.val[0].y = T(0);
    }
    __syncthreads();
    // (a layer's targets do not read each other: their order does not matter)
    int pos[NIT];
    {
        int lx = tid % rw, ly = tid / rw;
        const int x0 = R.ox - R.x0, y0 = R.oy - R.y0, x1 = x0 + R.ow - 1, y1 = y0 + R.oh - 1;
#pragma unroll
        for (int u = 0; u < NIT; u++) {
            const int tv = tvs[u];
            pos[u] = LN;
            // distance to the own nodes
            const int d = max(max(x0 - lx, lx - x1), max(y0 - ly, ly - y1));
            if (tv >= 1 && (MODE == FIT_TILE ? d <= R.mstep * (L - tv) : tv <= L && d <= 0)) {
                pos[u] = atomicAdd(&s.cnt[tv], 1);
                // (the check mode: the copy is taken to hold one node less
                // around the targets of each layer)
                if (reach < 2 && tv > 1 && reach + 2 * (L - tv) - d < 2) atomicMin(&s.cut, tv);
            }
            lx += step_x;
            ly += step_y;
            if (lx >= rw) {
                lx -= rw;
                ly++;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < NIT; u++) {
        const int e = tid + u * NT, tv = tvs[u];
        if (u == NIT - 1 && e >= NODES) continue;
        s.st[e] = (unsigned char)tv;
        s.val[e + 1].x = tv == TAG_SOLID ? xs0[u] : T(0);
        s.val[e + 1].y = tv == TAG_SOLID ? ys0[u] : T(0);
        if (pos[u] < LN) s.lst[(tv - 1) * LN + pos[u]] = (unsigned short)e;
    }
    __syncthreads();
    int cn[FF_LAYERS + 1];  // targets of each layer (the same in every thread)
    bool fits = true;
    cn[0] = 0;
#pragma unroll
    for (int l = 1; l <= FF_LAYERS; l++) {
        cn[l] = s.cnt[l];
        fits = fits && cn[l] <= LN;
    }
    if (!fits || (reach < 2 && cn[1] + cn[2] > 64)) {
        if (tid == 0) s.cut = 1;
        __syncthreads();
        return;
    }
    // target q of layer l has no fit at half-width 2
    auto defer = [&](int q, int l) {
        if constexpr (WIDE) {
            const int u = atomicAdd(&s.nwide, 1);
            if (u < FF_WIDE) {
                s.wide[u] = (unsigned short)q;
                atomicOr(&s.wlayers, 1 << l);
                return;
            }
        }
        atomicMin(&s.cut, l);
    };
    // layer l's of them, the rest of the layer being done (as fit_target, the
    // nodes read from the copy); nobody lists meanwhile.  Not those of a layer
    // that is cut (its targets were listed with nodes that have failed since,
    // or not all of them were): the caller's
    auto search = [&](int l) {
        const int nw = s.cut <= l ? 0 : min(s.nwide, FF_WIDE), sub = tid % FIT_LANES;
#pragma unroll 1
        for (int u = tid / FIT_LANES; u < nw; u += NT / FIT_LANES) {
            const int q = s.wide[u];
            if (s.st[q] != l) continue;  // whole groups leave together
            const int i = R.x0 + q % rw, j = R.y0 + q / rw;
            double nxh, nyh;
            const bool use_n = target_normal<T>(g, D, l, i, j, sub, phin, nxh, nyh);
            T xo = T(0), yo = T(0);
            bool ok = false;
#pragma unroll 1
            for (int r = 3; r <= g.r_max && !ok; r++) {
                const int side = 2 * r + 1;
                int count = 0, a = sub % side - r, b = sub / side - r;
                Fit<T> f;
                f.zero();
#pragma unroll 1
                for (int k = sub; k < side * side; k += FIT_LANES) {
                    int x = i + a, y = j + b;
                    if (canon(g, x, y) && W.has(x, y)) {
                        const int e = (y - R.y0) * rw + x - R.x0;
                        if (s.st[e] < l) {
                            count++;
                            f.add(a, b, use_n, nxh, nyh, s.val[e + 1].x, s.val[e + 1].y);
                        }
                    }
                    a += FIT_LANES;
                    while (a > r) {
                        a -= side;
                        b += 1;
                    }
                }
                ok = fit_finish<T>(g.det_rel, f, count, xo, yo);
            }
            if (sub == 0) {
                if (ok) {
                    s.val[q + 1].x = xo;
                    s.val[q + 1].y = yo;
                } else {
                    s.st[q] = (unsigned char)(l | TAG_FAIL);
                    tag[pidx(g, i, j)] = (int8_t)(l | TAG_FAIL);
                    atomicAdd(&health[1], 1u);
                    atomicMin(&s.cut, l + 1);
                }
            }
        }
        __syncthreads();
    };
    // ---- layers 1 and 2 (sets 0 and 1), with the normal of phi^n at the
    // target; the records of the others (sets 2 and 3)
    auto record = [&](int e) {
        // record e of the layers 3 .. L laid end to end
        int l = 3;
#pragma unroll
        for (int k = 3; k < FF_LAYERS; k++)
            if (l == k && e >= cn[k]) {
                e -= cn[k];
                l++;
            }
        const int q = s.lst[(l - 1) * LN + e];
        unsigned m = 0;
#pragma unroll
        for (int k = 0; k < NS; k++)
            if (C2::in(0, k))
                m |= s.st[q + C2::off_b(0, k) * rw + C2::off_a(0, k)] < l ? 1u << k : 0u;
        const Geo2 G = geo2(m, g.det_rel);
        if (!G.ok) defer(q, l);
        // (a record without a fit: no node, or determinant 0)
        if constexpr (sizeof(REC) == 4)
            s.rec[(l - 3) * LN + e] = !WIDE || G.ok ? m : 0u;
        else
            s.rec[(l - 3) * LN + e] =
                make_uint4(m, (unsigned)(G.m00 | G.m11 << 8 | (G.m01 & 0xff) << 16),
                           (unsigned)((G.m02 & 0xff) | (G.m12 & 0xff) << 8),
                           !WIDE || G.ok ? (unsigned)G.det : 0u);
    };
    // layer 1 + set: set 1 takes its weights while set 0 fits layer 1, and
    // weighs the values after the barrier
    {
        typename C2::NW w;
        int q = 0;
        bool have = false, ok = false;
        int nrec = 0, e = tid - 2 * SW;
#pragma unroll
        for (int k = 3; k <= FF_LAYERS; k++) nrec += cn[k];
#pragma unroll 1
        for (int ph = 0; ph < 2; ph++) {
            if (set < 2 && ph <= set) {
                const int l = 1 + set, n = set == 0 ? cn[1] : cn[2];
#pragma unroll 1
                for (int a = lane; a < n; a += SW) {
                    if (!have) {
                        q = s.lst[set * LN + a];
                        const int i = R.x0 + q % rw, j = R.y0 + q / rw;
                        // (D lies in the map's domain: no test of their own)
                        auto at = [&](int x, int y) {
                            x += x < 0 ? wx : x >= g.nx ? -wx : 0;
                            y += y < 0 ? wy : y >= g.ny ? -wy : 0;
                            return D.has(x, y) ? (y + PAD) * g.pp + x + PAD : -1;
                        };
                        const int ke = at(i + 1, j), kw = at(i - 1, j);
                        const int kn = at(i, j + 1), ks = at(i, j - 1);
                        const T pe = phin[ke >= 0 ? ke : 0], pw = phin[kw >= 0 ? kw : 0];
                        const T pn = phin[kn >= 0 ? kn : 0], ps = phin[ks >= 0 ? ks : 0];
                        bool v[NS];
#pragma unroll
                        for (int k = 0; k < NS; k++)
                            v[k] = C2::in(0, k) &&
                                   s.st[q + C2::off_b(0, k) * rw + C2::off_a(0, k)] < l;
                        const unsigned mask = C2::mask_of(0, v);
                        double nxh = 0.0, nyh = 0.0;
                        const bool use_n = normal_from(ke >= 0 ? (double)pe : INFINITY,
                                                       kw >= 0 ? (double)pw : INFINITY,
                                                       kn >= 0 ? (double)pn : INFINITY,
                                                       ks >= 0 ? (double)ps : INFINITY, nxh, nyh);
                        ok = use_n ? C2::weights_n(0, __popc(mask), v, nxh, nyh, g.det_rel, w)
                                   : C2::weights_2(0, mask, g.det_rel, w);
                        have = true;
                    }
                    if (set != ph) break;
                    T xs[NS], ys[NS], xo, yo;
#pragma unroll
                    for (int k = 0; k < NS; k++) {
                        if (!C2::in(0, k)) continue;
                        const int qk = q + C2::off_b(0, k) * rw + C2::off_a(0, k);
                        const auto z = s.val[s.st[qk] < l ? qk + 1 : 0];
                        xs[k] = z.x;
                        ys[k] = z.y;
                    }
                    C2::value_n(0, w, xs, ys, xo, yo);
                    if (ok) {
                        s.val[q + 1].x = xo;
                        s.val[q + 1].y = yo;
                    } else {
                        defer(q, l);
                    }
                    have = false;
                }
            }
            if (set >= 2) {
                const int stop = ph == 0 ? min(nrec, NT) : nrec;
#pragma unroll 1
                for (; e < stop; e += NT - 2 * SW) record(e);
            }
            __syncthreads();
            if (WIDE && (s.wlayers >> (ph + 1) & 1)) search(ph + 1);
        }
    }
    // ---- layers 3 and up
    int pq = -1, adr[NS];
    Geo2 pg{};
    auto prep = [&](int l, int a, int n) {
        pq = -1;
        if (a >= n) return;
        const REC r = s.rec[(l - 3) * LN + a];
        pq = s.lst[(l - 1) * LN + a] + 1;
        unsigned m;
        if constexpr (sizeof(REC) == 4) {
            m = r;
            if (WIDE && m == 0) {
                pq = -1;
                return;
            }
            pg = geo2(m, g.det_rel);
        } else {
            m = r.x;
            if (WIDE && r.w == 0) {
                pq = -1;
                return;
            }
            pg.m00 = (int)(r.y & 0xff);
            pg.m11 = (int)(r.y >> 8 & 0xff);
            pg.m01 = (int)(r.y << 8) >> 24;
            pg.m02 = (int)(r.z << 24) >> 24;
            pg.m12 = (int)(r.z << 16) >> 24;
            pg.det = (int)r.w;
        }
#pragma unroll
        for (int k = 0; k < NS; k++)
            adr[k] = ((int)(m << (31 - k)) >> 31) &
                     (pq + C2::off_b(0, k) * rw + C2::off_a(0, k));
    };
    auto finish = [&]() {
        if (pq < 0) return;
        T xs[NS], ys[NS], xo, yo;
#pragma unroll
        for (int k = 0; k < NS; k++) {
            if (!C2::in(0, k)) continue;
            const auto z = s.val[adr[k]];
            xs[k] = z.x;
            ys[k] = z.y;
        }
        C2::value(0, pg, xs, ys, xo, yo);
        s.val[pq].x = xo;
        s.val[pq].y = yo;
    };
    const int wl = WIDE ? __builtin_amdgcn_readfirstlane(s.wlayers) : 0;
    int last = min(L, s.cut - 1);  // (the same in every thread)
    if (MODE == FIT_WHOLE && last < L) return;
    int lm = 3 + set, n = s.cnt[min(lm, FF_LAYERS)];  // the set's next layer
    if (lm <= last) prep(lm, lane, n);
#pragma unroll 1
    for (int l = 3; l <= last; l++) {
        const bool mine = l == lm;
        if (mine) {
            int a = lane;
#pragma unroll 1
            while (true) {
                finish();
                a += SW;
                if (a >= n) break;
                prep(l, a, n);
            }
        }
        __syncthreads();
        if (WIDE && (wl >> l & 1)) {
            search(l);
            last = min(last, s.cut - 1);
        }
        if (mine) {
            lm += NSET;
            n = s.cnt[min(lm, FF_LAYERS)];
            if (lm <= last) prep(lm, lane, n);
        }
    }
    // ---- the region's own nodes of the layers that stand (the layers touch
    // LDS only, so none of their barriers waits for HBM)
    for (int e = tid; e < R.ow * R.oh; e += NT) {
        const int x = R.ox + e % R.ow, y = R.oy + e / R.ow;
        const int q = (y - R.y0) * rw + x - R.x0, l = s.st[q];
        if (l >= 1 && l <= last && W.has(x, y)) {
            const long long kt = pidx(g, x, y);
            through(&X1[kt], T(s.val[q + 1].x));  // (read by fit_rest, if it runs)
            through(&Y1[kt], T(s.val[q + 1].y));
        }
    }
}

// Can a block's copy hold a whole window (dilated by 2; no two of its nodes
// images of one node)?
__device__ __forceinline__ bool fits_whole(const GridP& g, const Rect& W, int nodes)
{
    const int w = W.i1 - W.i0 + 1, h = W.j1 - W.j0 + 1;
    return (long long)(w + 4) * (h + 4) <= nodes && !(g.px && w + 4 > g.nx) &&
           !(g.py && h + 4 > g.ny);
}

// The layers of one solid, FF_LAYERS at most, in one block on such a copy, laid
// out in unwrapped coordinates, each node holding what its periodic image
// holds.  Returns the first layer that the copy did not serve (the block sees
// what it wrote of the others).  wide: there are targets without a fit at
// half-width 2.
template <typename T, int NT, int NODES, int LN, typename REC>
__device__ __forceinline__ int fit_whole(FitLds<T, NODES, LN, REC>& s, const GridP& g,
                                         const Rect& W, const Rect& D, int8_t* tag,
                                         const T* __restrict__ phin, T* X1, T* Y1,
                                         unsigned* health, bool wide)
{
    const int w = W.i1 - W.i0 + 1, h = W.j1 - W.j0 + 1;
    const FitRegion R{W.i0 - 2, W.j0 - 2, w + 4, h + 4, W.i0, W.j0, w, h, 0};
    const int L = min(g.layers, FF_LAYERS);
    if (!wide)
        fit_region<T, NT, NODES, LN, 0, FIT_WHOLE>(s, g, W, D, L, R, tag, phin, X1, Y1, health, 2);
    if (wide || s.cut <= L)
        fit_region<T, NT, NODES, LN, 0, FIT_WIDE>(s, g, W, D, L, R, tag, phin, X1, Y1, health, 2);
    const int l0 = s.cut;
    if (l0 <= g.layers) {
        // (the copy's results went through the caches)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        __threadfence();
    }
    return l0;
}

// Several solids without the one-launch extrapolation: one block per solid
// (its layers are short), on a copy where that can be.  The layers that the
// copy does not serve are fitted on the maps (layer_fit_body: the same bits).
// (Thirteen layers, 30 solids, us/step FP64 with all of them on the maps 290,
// with the first eleven on the copy 136; FP32 236, 115.)
// Block row y takes table row ord[y] (row y when ord is null).
template <typename T, int NT>
__global__ __launch_bounds__(NT) void kb_fit_lds(const FitArgs* __restrict__ args, int layers,
                                                  const int* __restrict__ ord)
{
    __shared__ FitLds<T, MB_FIT_LDS_NODES, FF_LAYER_MB> s;
    const FitArgs& a = args[ord ? ord[blockIdx.y] : blockIdx.y];
    const GridP& g = a.g;
    const Rect W = window_of(a.win, a.wcur, g);
    const Rect D = window_of(a.win, a.wprev, g);
    if (!W.ok) return;
    int l0 = 1;
    if (fits_whole(g, W, MB_FIT_LDS_NODES))
        l0 = fit_whole<T, NT>(s, g, W, D, a.tag, (const T*)a.phin, (T*)a.X1, (T*)a.Y1, a.health,
                              false);
    for (int l = l0; l <= layers; l++) {
        layer_fit_body<T, true>(g, a.win, a.wcur, a.wprev, l, a.tag, a.lists, a.lcount,
                                (const T*)a.phin, (T*)a.X1, (T*)a.Y1, a.health);
        __syncthreads();
    }
}

// The stopped tiles of a fused extrapolation (one block, the last to end):
// fits, layer by layer from the first to the last, every target that lies in
// a stopped tile at or after the layer where that tile stopped (found by the
// tile's tags; full scan windows up to r_max, the per-layer path's fit).
// cut_tiles null: every tile of the window (nc of them), from layer cut_all.
// The tiles' tags are read twice, to count each layer's targets and to list
// them, for as many layers at a time as the list has room for (lst, room: LDS;
// a layer of its own larger than that goes by shares of the tiles).  (Two solids
// of 200 x 2.4 nodes, us/step FP64 with each tile's tags read in each layer 378,
// so 223; FP32 347, 202.)
template <typename T, int NT>
__device__ void fit_rest(const GridP& g, const Rect& W, const Rect& D, int8_t* tag,
                         const T* __restrict__ phin, T* X1, T* Y1, unsigned* health,
                         const int* cut_tiles, int nc, int cut_all, int* lst, int room)
{
    constexpr int NG = NT / FIT_LANES, TN = FF_TILE * FF_TILE, U = 4;
    __shared__ int cnt[FF_LAYERS + 1], at[FF_LAYERS + 1];
    const int sub = threadIdx.x % FIT_LANES, grp = threadIdx.x / FIT_LANES;
    const int ntx = (W.i1 - W.i0 + FF_TILE) / FF_TILE;
    // f(layer, node) of the targets of layers la .. lb in tiles c0 .. c1 - 1
    auto targets = [&](int c0, int c1, int la, int lb, auto f) {
        for (int e0 = c0 * TN + threadIdx.x; e0 < c1 * TN; e0 += NT * U) {
            int kt[U], tv[U], ct[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int e = min(e0 + u * NT, c1 * TN - 1), c = e / TN, o = e % TN;
                ct[u] = cut_tiles ? cut_tiles[c] : c | cut_all << FF_CUT_SHIFT;
                const int t = ct[u] & FF_CUT_TILE;
                const int x = W.i0 + (t % ntx) * FF_TILE + o % FF_TILE;
                const int y = W.j0 + (t / ntx) * FF_TILE + o / FF_TILE;
                kt[u] = (int)pidx(g, min(x, W.i1), min(y, W.j1));
                tv[u] = tag[kt[u]];
                if (e0 + u * NT >= c1 * TN || !W.has(x, y)) tv[u] = TAG_NONE;
            }
#pragma unroll
            for (int u = 0; u < U; u++)
                if (tv[u] >= la && tv[u] <= lb && tv[u] >= ct[u] >> FF_CUT_SHIFT) f(tv[u], kt[u]);
        }
    };
    for (int la = 1; la <= g.layers;) {
        __syncthreads();
        if (threadIdx.x <= FF_LAYERS) cnt[threadIdx.x] = 0;
        __syncthreads();
        targets(0, nc, la, g.layers, [&](int l, int) { atomicAdd(&cnt[l], 1); });
        __syncthreads();
        int lb = la, n = cnt[la];  // (the same in every thread)
        while (lb < g.layers && n + cnt[lb + 1] <= room) n += cnt[++lb];
        // tiles at a time: all, or (one layer, beyond the room) what surely fits
        const int step = n <= room ? nc : room / TN;
        for (int c0 = 0; c0 < nc; c0 += step) {
            const int c1 = min(nc, c0 + step);
            __syncthreads();
            if (threadIdx.x == 0) {
                int o = 0;
                for (int l = la; l <= lb; l++) {
                    at[l] = o;
                    o += cnt[l];
                }
            }
            __syncthreads();
            // (at[l] runs to the end of layer l's entries)
            targets(c0, c1, la, lb, [&](int l, int kt) { lst[atomicAdd(&at[l], 1)] = kt; });
            __syncthreads();
            int from = 0;
            for (int l = la; l <= lb; l++) {
                const int end = at[l];
                for (int a = from + grp; a < end; a += NG) {
                    const int kt = lst[a];
                    const int i = kt % g.pp - PAD, j = kt / g.pp - PAD;
                    T xo = T(0), yo = T(0);
                    const bool done =
                        fit_target<T, true>(g, W, D, l, kt, i, j, sub, tag, phin, X1, Y1, xo, yo);
                    if (sub == 0) {
                        if (done) {
                            X1[kt] = xo;
                            Y1[kt] = yo;
                        } else {
                            tag[kt] = (int8_t)(l | TAG_FAIL);
                            atomicAdd(&health[1], 1u);
                        }
                    }
                }
                from = end;
                __syncthreads();
            }
        }
        la = lb + 1;
    }
}

// All layers of one solid in one launch.  Block b takes FF_TILE x FF_TILE
// tiles of the window from the list the distance transform made of the tiles
// the zone reaches; for layer l it fits every layer-l target within
// M_l = 2 (L - l) nodes of its tile, its own and those of the tiles around
// (recomputed, with the same arithmetic, so the same bits as their own
// blocks find), on a copy of the tile and a margin of M_1 + 2 nodes: a scan
// window of half-width 2 around a target within M_l of the tile stays within
// M_l + 2 = M_{l-1}, where the copy holds every earlier layer, and layer-1
// windows read solid nodes only, which the copy holds across the margin.  Only
// the tile's own targets are written back.  A tile that the copy cannot serve
// from some layer on (a fit that needs a wider scan window, or fails for good;
// more than FF_LAYER targets in a layer) is listed, with the layer; the block
// that ends last finishes the listed tiles layer by layer (fit_rest) and
// empties both lists.  (A launch of its own for that took 4 us a step, with
// nothing to do but at rare steps; the ticket of the blocks takes ~1 us.)
// reach = 2; reach = 1 stops every tile with a target on the rim of its
// margin, and every tile with more than 64 targets in layers 1 and 2 before
// its first layer (fit_rest then fits most of the zone: a check of it).
// Block b of nb.  Returns the number of listed tiles in the last block, -1 in
// the others.
template <typename T, int NT, int LC, int NODES, int LN, typename REC>
__device__ __forceinline__ int fit_tiles(FitLds<T, NODES, LN, REC>& s, const GridP& g, const Rect& W,
                                         const Rect& D, int8_t* tag, const T* __restrict__ phin,
                                         T* X1, T* Y1, unsigned* health, int* cut_tiles,
                                         int* ncut, const int* __restrict__ ff_list, int ntile,
                                         int t0, unsigned* ticket, int reach, int b, int nb)
{
    constexpr int RW = FF_REGION;
    static_assert(RW * RW <= NODES, "a tile with its margin");
    const int L = LC > 0 ? LC : g.layers;
    const int S = 2 * (L - 1) + 2, rw = FF_TILE + 2 * S;  // margin of the copy, its width
    const int ntx = (W.i1 - W.i0 + FF_TILE) / FF_TILE;
    for (int k = b; k < ntile; k += nb) {
        const int t = k == b ? t0 : ff_list[k];
        const int x0 = W.i0 + (t % ntx) * FF_TILE, y0 = W.j0 + (t / ntx) * FF_TILE;
        const FitRegion R{x0 - S, y0 - S, rw, rw, x0, y0, FF_TILE, FF_TILE, 2};
        fit_region<T, NT, NODES, LN, LC == FF_LAYERS ? RW : 0, FIT_TILE>(
            s, g, W, D, L, R, tag, phin, X1, Y1, health, reach);
        if (threadIdx.x == 0 && s.cut <= L)
            through(&cut_tiles[atomicAdd(ncut, 1)], t | s.cut << FF_CUT_SHIFT);
    }
    static_assert(sizeof(s.val) >= sizeof(int) * FF_TILE * FF_TILE, "fit_rest's list");
    if (!last_arrival(ticket, min(ntile, nb))) return -1;
    const int nc = seen(ncut);
    if (nc > 0) __threadfence();
    return nc;
}

// The tiles left to the maps when fit_whole has returned l0: none, every tile of
// the window from that layer on, or, where it served no layer, the listed ones.
__device__ __forceinline__ int left_tiles(const GridP& g, const Rect& W, int l0, int nc,
                                          const int*& cut_tiles)
{
    if (l0 > g.layers) return 0;
    if (l0 == 1 && cut_tiles) return nc;
    cut_tiles = nullptr;
    return ((W.i1 - W.i0 + FF_TILE) / FF_TILE) * ((W.j1 - W.j0 + FF_TILE) / FF_TILE);
}

// WHOLE: of the tiles that their copies cannot serve, the last block finishes
// the whole solid where its copy holds the window, which takes less than the
// layers on the maps (8 members of 64^2, thin, us/step FP64 113 -> 77, FP32 135 ->
// 91; 32 of 128^2 190 -> 161, 215 -> 171).
template <typename T, int NT, int LC, bool WHOLE, typename REC = uint4>
__device__ __forceinline__ void fit_fused_body(const GridP& g, const Win* __restrict__ win,
                                               int wcur, int wprev, int8_t* tag,
                                               const T* __restrict__ phin, T* X1, T* Y1,
                                               unsigned* health, int* cut_tiles, int* ncut,
                                               const int* __restrict__ ff_list, int* ff_n,
                                               unsigned* ticket, int* wide, int reach)
{
    __shared__ FitLds<T, FF_REGION * FF_REGION, WHOLE ? FF_LAYER_BATCH : FF_LAYER, REC> s;
    // (the first tile is read together with the count; a block beyond the
    // list's room reads its last entry, and leaves)
    const int ntile = *ff_n, t0 = ff_list[ff_first(blockIdx.x, g.nx, g.ny)];
    const Rect W = window_of(win, wcur, g);
    const Rect D = window_of(win, wprev, g);
    if ((int)blockIdx.x >= ntile || !W.ok) return;
    int nc = fit_tiles<T, NT, LC>(s, g, W, D, tag, phin, X1, Y1, health, cut_tiles, ncut, ff_list,
                                  ntile, t0, ticket, reach, blockIdx.x, gridDim.x);
    if (nc < 0) return;
    const int cut = nc;
    const int* left = cut_tiles;
    int l0 = 0;
    if (WHOLE && __builtin_expect(nc > 0 && fits_whole(g, W, FF_REGION * FF_REGION), 0)) {
        l0 = fit_whole<T, NT>(s, g, W, D, tag, phin, X1, Y1, health, true);
        nc = left_tiles(g, W, l0, nc, left);
    }
    // (told unlikely, it costs a launch without such tiles nothing; else 0.3 us at
    // 256^2 FP32)
    if (__builtin_expect(nc > 0, 0))
        fit_rest<T, NT>(g, W, D, tag, phin, X1, Y1, health, left, nc, l0, (int*)s.val,
                        (int)(sizeof(s.val) / (sizeof(int))));
    if (threadIdx.x == 0) {
        *ncut = 0;
        *ff_n = 0;
        *wide = cut;
    }
}

// Several solids: solid row y (ord[y], the largest first).  A solid whose
// window fits one block's copy is one block's, unless tiles is set (few
// solids: whole-solid blocks would leave most of the chip idle); any other's
// listed tiles are shared by the row's blocks.  Of the tiles that their copies
// cannot serve, the last block finishes the whole solid where it can, which
// the layers on the maps take longer than.
template <typename T, int LC>
__global__ __launch_bounds__(FF_THREADS) void kb_fit_mb(const FitArgs* __restrict__ args,
                                                        const int* __restrict__ ord, MbFit f)
{
    constexpr int NT = FF_THREADS;
    __shared__ FitLds<T, MB_FIT_LDS_NODES, FF_LAYER_MB> s;
    // row and block of it
    const int many = f.rows * f.blocks, id = blockIdx.x;
    const int nb = id < many ? f.blocks : f.few, at = id < many ? id : id - many;
    const int row = at / nb + (id < many ? 0 : f.rows), b = at % nb;
    const FitArgs& a = args[ord[row]];
    const GridP& g = a.g;
    const Rect W = window_of(a.win, a.wcur, g);
    const Rect D = window_of(a.win, a.wprev, g);
    if (!W.ok) return;
    const int ntile = *a.ff_n;
    const bool whole = fits_whole(g, W, MB_FIT_LDS_NODES);
    const int* cut_tiles = nullptr;  // the tiles left to the maps, and from which layer
    int nc = 0, l0 = 0;
    if (whole && !f.tiles) {
        if (b != 0) return;
        nc = 1;
    } else {
        if (b >= ntile) return;
        nc = fit_tiles<T, NT, LC>(s, g, W, D, a.tag, (const T*)a.phin, (T*)a.X1, (T*)a.Y1,
                                  a.health, a.cut_tiles, a.ncut, a.ff_list, ntile,
                                  a.ff_list[b], a.ticket, 2, b, nb);
        if (nc < 0) return;
        cut_tiles = a.cut_tiles;
    }
    if (__builtin_expect(nc > 0 && whole, 0)) {
        l0 = fit_whole<T, NT>(s, g, W, D, a.tag, (const T*)a.phin, (T*)a.X1, (T*)a.Y1, a.health,
                              f.tiles != 0);
        nc = left_tiles(g, W, l0, nc, cut_tiles);
    }
    if (__builtin_expect(nc > 0, 0))
        fit_rest<T, NT>(g, W, D, a.tag, (const T*)a.phin, (T*)a.X1, (T*)a.Y1, a.health, cut_tiles,
                        nc, l0, (int*)s.val, (int)(sizeof(s.val) / (sizeof(int))));
    if (threadIdx.x == 0) {
        *a.ncut = 0;
        *a.ff_n = 0;
    }
}

template <typename T, int NT, int LC>
__global__ __launch_bounds__(NT) void k_fit_fused(GridP g, const Win* __restrict__ win, int wcur,
                                                  int wprev, int8_t* tag,
                                                  const T* __restrict__ phin, T* X1, T* Y1,
                                                  unsigned* health, int* cut_tiles, int* ncut,
                                                  const int* __restrict__ ff_list, int* ff_n,
                                                  unsigned* ticket, int* wide, int reach)
{
    __builtin_amdgcn_s_setprio(3);
    fit_fused_body<T, NT, LC, false>(g, win, wcur, wprev, tag, phin, X1, Y1, health, cut_tiles, ncut,
                              ff_list, ff_n, ticket, wide, reach);
}

// A batch: member blockIdx.y.  Where its tiles are many rounds of blocks, and a
// block is bound by its chain of layers, two blocks of 256 threads share a
// compute unit in FP32 (PAIRS), their records short enough (masks alone, the
// matrices counted again) for both copies to fit (96 cavities of 96^2 .. 768^2,
// 2900 tiles: 234 -> 168 us; one block a solid of a suspension, 400 of them, is
// little more than a round, and slower two to a unit: 47 -> 56 us; the line lies
// at BATCH_FIT_TILES).  FP64 copies do not fit twice.
template <bool PAIRS>
struct BatchFit {
    static constexpr int NT = PAIRS ? 256 : FF_THREADS;
    using Rec = typename std::conditional<PAIRS, unsigned, uint4>::type;
};
template <typename T, int LC, bool PAIRS>
__global__ __launch_bounds__(BatchFit<PAIRS>::NT) void kb_fit_fused(const FitArgs* __restrict__ args)
{
    const FitArgs& a = args[blockIdx.y];
    fit_fused_body<T, BatchFit<PAIRS>::NT, LC, true, typename BatchFit<PAIRS>::Rec>(
        a.g, a.win, a.wcur, a.wprev, a.tag, (const T*)a.phin, (T*)a.X1, (T*)a.Y1, a.health,
        a.cut_tiles, a.ncut, a.ff_list, a.ff_n, a.ticket, a.ff_wide, 2);
}

hipError_t launch_extrapolate(const GridP& g, const BandBufs& bb, const StepSlots& s,
                              hipStream_t st, int fused_threads)
{
    if (fused_threads > 0 && fused_fit_ok(g)) {
#define FUSED_L(T, NT, LC)                                                                        \
    k_fit_fused<T, NT, LC><<<FF_BLOCKS, NT, 0, st>>>(                                             \
        g, bb.win, s.wcur, s.wprev, bb.tag, (const T*)bb.phi[s.cur], (T*)bb.X[s.nxt],             \
        (T*)bb.Y[s.nxt], bb.health, bb.cut_tiles, bb.ncut, bb.ff_list, bb.ff_n, bb.ticket,       \
        bb.ff_wide, fused_threads == 1 ? 1 : 2)
#define FUSED(T, NT)                                                                              \
    do {                                                                                          \
        if (g.layers == FF_LAYERS) FUSED_L(T, NT, FF_LAYERS);                                     \
        else FUSED_L(T, NT, 0);                                                                   \
    } while (0)
#define FUSED_T(T)                                                                                \
    do {                                                                                          \
        if (fused_threads == 256) FUSED(T, 256);                                                  \
        else FUSED(T, FF_THREADS);                                                                \
    } while (0)
        if (g.rm32) FUSED_T(float);
        else FUSED_T(double);
#undef FUSED_T
#undef FUSED
#undef FUSED_L
        return hipGetLastError();
    }
#define LAYER(T, N)                                                                            \
    k_layer_fit<T, N><<<FIT_BLOCKS, 256, 0, st>>>(g, bb.win, s.wcur, s.wprev, l, bb.tag,       \
                                                  bb.lists, bb.lcount, (const T*)bb.phi[s.cur], \
                                                  (T*)bb.X[s.nxt], (T*)bb.Y[s.nxt], bb.health)
    for (int l = 1; l <= g.layers; l++)
        if (g.rm32) {
            if (l <= 2) LAYER(float, true);
            else LAYER(float, false);
        } else {
            if (l <= 2) LAYER(double, true);
            else LAYER(double, false);
        }
#undef LAYER
    return hipGetLastError();
}

// ---------------------------------------------------------------- stress and force

constexpr int FTX = 32, FTY = 8;
constexpr int SX = FTX + 2, SY = FTY + 2;

// F = J^{-1} (Eq. (3_3_refmap_deformation)) and the plane-strain
// neo-Hookean deviatoric stress (Eq. (3_3_solid_stress)) scaled by lam
template <typename C>
__device__ __forceinline__ void tau_of(C J0, C J1, C J2, C J3, C det, C G, C lam, C out[3])
{
    const C F00 = J3 / det, F01 = -J1 / det;
    const C F10 = -J2 / det, F11 = J0 / det;
    const C Bxx = F00 * F00 + F01 * F01;
    const C Bxy = F00 * F10 + F01 * F11;
    const C Byy = F10 * F10 + F11 * F11;
    const C tr = Bxx + Byy;
    out[0] = lam * (G * (Bxx - (tr + C(1)) / C(3)));
    out[1] = lam * (G * Bxy);
    out[2] = lam * (G * (Byy - (tr + C(1)) / C(3)));
}

// Blended stress (1 - H(phi_e)) tau_s of one half-edge from the LDS tile.
// a, bb: the two nodes of the edge (a before bb along the normal direction);
// s1..s4: the side nodes of the tangential difference (s1 + s2 - s3 - s4)/4
// (Eq. (3_3_refmap_jacobian), six-node stencil); dir 0: x-edge, 1: y-edge.
// With displacement storage grad xi = I + grad d; where its determinant is
// below kappa_J the inversion is redone in double.
template <typename C>
__device__ void edge_tau(const GridP& g, const BodyP& b, const C* sX, const C* sY, const C* sP,
                         int a, int bb, int s1, int s2, int s3, int s4, int dir, bool count,
                         unsigned* health, C out[3])
{
    constexpr bool DISP = sizeof(C) == 4;
    out[0] = out[1] = out[2] = C(0);
    const C pa = sP[a], pb = sP[bb];
    if (!(pa < C(INFINITY)) || !(pb < C(INFINITY))) return;
    const C phie = C(0.5) * (pa + pb);
    const C lam = C(1) - heaviside<C>(phie, C(g.eps));
    if (!(lam > C(0))) return;
    if (!(sP[s1] < C(INFINITY)) || !(sP[s2] < C(INFINITY)) || !(sP[s3] < C(INFINITY)) ||
        !(sP[s4] < C(INFINITY))) {
        if (count) atomicAdd(&health[2], 1u);
        return;
    }
    const C nX = sX[bb] - sX[a], nY = sY[bb] - sY[a];
    const C tX = (sX[s1] + sX[s2] - sX[s3] - sX[s4]) / C(4);
    const C tY = (sY[s1] + sY[s2] - sY[s3] - sY[s4]) / C(4);
    C J0, J1, J2, J3;  // [dX/dx, dX/dy; dY/dx, dY/dy]
    if (dir == 0) {
        J0 = nX; J1 = tX; J2 = nY; J3 = tY;
    } else {
        J0 = tX; J1 = nX; J2 = tY; J3 = nY;
    }
    if (DISP) {
        J0 += C(1);
        J3 += C(1);
    }
    const C det = J0 * J3 - J1 * J2;
    if (DISP && !(det >= C(g.kappa_J))) {
        // near-singular (or inverted) grad xi: decide and invert in double
        const double dnX = (double)sX[bb] - (double)sX[a], dnY = (double)sY[bb] - (double)sY[a];
        const double dtX =
            ((double)sX[s1] + (double)sX[s2] - (double)sX[s3] - (double)sX[s4]) / 4.0;
        const double dtY =
            ((double)sY[s1] + (double)sY[s2] - (double)sY[s3] - (double)sY[s4]) / 4.0;
        double K0, K1, K2, K3;
        if (dir == 0) {
            K0 = 1.0 + dnX; K1 = dtX; K2 = dnY; K3 = 1.0 + dtY;
        } else {
            K0 = 1.0 + dtX; K1 = dnX; K2 = dtY; K3 = 1.0 + dnY;
        }
        const double dd = K0 * K3 - K1 * K2;
        if (!(dd > g.detJ_min)) {
            if (count) {
                atomicAdd(&health[3], 1u);
                if (lam > C(0.5)) atomicAdd(&health[4], 1u);
            }
            return;
        }
        double o[3];
        tau_of<double>(K0, K1, K2, K3, dd, b.G, (double)lam, o);
        out[0] = C(o[0]);
        out[1] = C(o[1]);
        out[2] = C(o[2]);
        return;
    }
    if (!(det > C(g.detJ_min))) {
        if (count) {
            atomicAdd(&health[3], 1u);
            if (lam > C(0.5)) atomicAdd(&health[4], 1u);
        }
        return;
    }
    tau_of<C>(J0, J1, J2, J3, det, C(b.G), lam, out);
}

// reference-map node k at (i, j) after the extrapolation of a step: its level
// set phi0(xi) in double (it decides the solid set), or +inf if it holds no map
template <typename C>
__device__ __forceinline__ double relabel_phi(const GridP& g, const BodyP& b, int8_t tv, C xv,
                                              C yv, int i, int j)
{
    if (!tag_set(tv)) return INFINITY;
    double X = (double)xv, Y = (double)yv;
    if (sizeof(C) == 4) {  // displacement storage
        X += pos_x(g, b, i);
        Y += pos_y(g, b, j);
    }
    return shape_phi(b, X, Y);
}

// Shared body of the force kernel (MODE 0) and the stress read (MODE 1) over
// interior tiles of region Rg: stage xi, phi of the tile plus a one-node halo
// in LDS (all loads issued first), compute each half-edge once, then combine
// per node.  MODE 0 also relabels (Alg. 1): phi^{n+1} = phi0(xi^{n+1}) is
// evaluated for every staged node from its tag and map, written for the
// tile's own nodes (with the map cleared where none is held), and for the
// window's nodes outside the interior by a strided pass; each block writes the
// partial box of the new interior solid set it saw, which the next lattice
// update (MODE 3: the last block) reduces into the next ring slot.  MODE 2 is
// the relabel alone, node by node (one solid of several: the forces are
// combined over all solids afterwards).  MODE 3 is MODE 0 followed, for each of the tile's own
// nodes, by its lattice Boltzmann update with the force just computed (the
// window's nodes; the lattice update of every other node does not depend on
// the solid's force of this step).
template <int MODE, typename C>
__device__ __forceinline__ void edges_body(GridP g, BodyP b, Win* win, int wvalid,
                                           int* boxpart, int whole_grid, C* X, C* Y,
                                           const C* __restrict__ phi, const int8_t* __restrict__ tag,
                                           C* phi1, double* o0, double* o1, double* o2,
                                           int* lcount, unsigned* health, const LbFuse& lf)
{
    // the force pass ends the reference-map chain of a step: clear the layer
    // counters of the next step's distance transform
    constexpr bool RELABEL = MODE != 1;
    if (RELABEL) clear_lcount(lcount);
    const Rect V = window_of(win, wvalid, g);
    const Rect WP = MODE == 3 ? window_of(win, lf.wprev, g) : Rect{0, -1, 0, -1, false};
    int bi0 = 0x3fffffff, bi1 = -0x3fffffff, bj0 = 0x3fffffff, bj1 = -0x3fffffff;
    // MODE 2: also the box of the nodes with phi < eps (where the solid
    // fraction is positive), partials after the solid box's
    int ei0 = 0x3fffffff, ei1 = -0x3fffffff, ej0 = 0x3fffffff, ej1 = -0x3fffffff;
    if (MODE == 2) {
        // no stencil: every node of the window by itself (400 solids in 4096^2
        // FP32 43 -> 28 us, 25 in 1024^2 FP64 14.3 -> 12.7, against tiles with
        // halos of maps in LDS as the other modes stage them)
        if (V.ok && b.present) {
            const int w = V.i1 - V.i0 + 1, n = w * (V.j1 - V.j0 + 1);
            for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n;
                 e += gridDim.x * blockDim.x) {
                const int i = V.i0 + e % w, j = V.j0 + e / w;
                const int k = (int)pidx(g, i, j);
                const int8_t tv = tag[k];
                const C xv = X[k], yv = Y[k];
                const C p = store_phi<C>(relabel_phi<C>(g, b, tv, xv, yv, i, j));
                if (p < C(INFINITY)) {
                    phi1[k] = p;
                    if (p < C(0) && i >= 0 && i < g.nx && j >= 0 && j < g.ny) {
                        bi0 = min(bi0, i);
                        bi1 = max(bi1, i);
                        bj0 = min(bj0, j);
                        bj1 = max(bj1, j);
                    }
                    if (p < C(g.eps)) {
                        ei0 = min(ei0, i);
                        ei1 = max(ei1, i);
                        ej0 = min(ej0, j);
                        ej1 = max(ej1, j);
                    }
                } else {
                    phi1[k] = C(INFINITY);
                    X[k] = C(NAN);
                    Y[k] = C(NAN);
                }
            }
        }
        block_box(bi0, bi1, bj0, bj1, boxpart + 4 * blockIdx.x);
        block_box(ei0, ei1, ej0, ej1, boxpart + 4 * (gridDim.x + blockIdx.x));
        return;
    }
    __shared__ C sX[SY * SX], sY[SY * SX], sP[SY * SX];
    __shared__ C ex[FTY][FTX + 1][3];
    __shared__ C ey[FTY + 1][FTX][3];
    Rect Rg;
    if (whole_grid) {
        Rg.i0 = 0; Rg.i1 = g.nx - 1; Rg.j0 = 0; Rg.j1 = g.ny - 1;
        Rg.ok = true;
    } else {
        Rg = V;
        Rg.i0 = max(Rg.i0, 0);
        Rg.j0 = max(Rg.j0, 0);
        Rg.i1 = min(Rg.i1, g.nx - 1);
        Rg.j1 = min(Rg.j1, g.ny - 1);
        Rg.ok = V.ok && Rg.i0 <= Rg.i1 && Rg.j0 <= Rg.j1;
    }
    const int ntx = Rg.ok ? (Rg.i1 - Rg.i0) / FTX + 1 : 0;
    const int nty = Rg.ok ? (Rg.j1 - Rg.j0) / FTY + 1 : 0;
    const int tx = threadIdx.x % FTX, ty = threadIdx.x / FTX;
    // MODE 3: blocks beyond lf.nown update the lattice tiles taken along
    const int nown = MODE == 3 ? lf.nown : (int)gridDim.x;
    for (int t = blockIdx.x; t < ntx * nty; t += nown) {
        const int i0 = Rg.i0 + (t % ntx) * FTX, j0 = Rg.j0 + (t / ntx) * FTY;
        for (int e = threadIdx.x; e < SX * SY; e += blockDim.x) {
            int ci = i0 - 1 + e % SX, cj = j0 - 1 + e / SX;
            const bool in = b.present && canon(g, ci, cj) && V.has(ci, cj);
            const long long k = in ? pidx(g, ci, cj) : 0;
            const C xv = X[k], yv = Y[k];
            C p;
            if (RELABEL) p = store_phi<C>(relabel_phi<C>(g, b, tag[k], xv, yv, ci, cj));
            else p = phi[k];
            const bool set = in && p < C(INFINITY);
            sX[e] = set ? xv : C(NAN);
            sY[e] = set ? yv : C(NAN);
            sP[e] = set ? p : C(INFINITY);
        }
        __syncthreads();
        const int i = i0 + tx, j = j0 + ty;
        const bool mine = i <= Rg.i1 && j <= Rg.j1;
        if (RELABEL && mine) {
            // relabel output of the tile's own node
            const long long k = pidx(g, i, j);
            const C p = sP[(ty + 1) * SX + tx + 1];
            if (p < C(INFINITY)) {
                phi1[k] = p;
                if (p < C(0)) {
                    bi0 = min(bi0, i);
                    bi1 = max(bi1, i);
                    bj0 = min(bj0, j);
                    bj1 = max(bj1, j);
                }
            } else if (V.has(i, j)) {
                phi1[k] = C(INFINITY);
                X[k] = C(NAN);
                Y[k] = C(NAN);
            }
        }
        // health counting: an edge is counted once, by the node on its far
        // side, or by its near node when the far node lies outside the region
        const bool rowin = j <= Rg.j1, colin = i <= Rg.i1;
        constexpr bool FORCE = MODE == 0 || MODE == 3;
        const bool cnt_l = FORCE && (mine || (rowin && i == Rg.i1 + 1));
        const bool cnt_b = FORCE && (mine || (colin && j == Rg.j1 + 1));
        // local index of node (i + di, j + dj)
#define LI(di, dj) ((ty + 1 + (dj)) * SX + (tx + 1 + (di)))
        // x-edge (i - 1/2, j): a = (i-1, j), b = (i, j); side (i, j+1), (i-1, j+1), (i, j-1), (i-1, j-1)
        edge_tau<C>(g, b, sX, sY, sP, LI(-1, 0), LI(0, 0), LI(0, 1), LI(-1, 1), LI(0, -1),
                    LI(-1, -1), 0, cnt_l, health, ex[ty][tx]);
        // y-edge (i, j - 1/2): a = (i, j-1), b = (i, j); side (i+1, j), (i+1, j-1), (i-1, j), (i-1, j-1)
        edge_tau<C>(g, b, sX, sY, sP, LI(0, -1), LI(0, 0), LI(1, 0), LI(1, -1), LI(-1, 0),
                    LI(-1, -1), 1, cnt_b, health, ey[ty][tx]);
        if (tx == FTX - 1) {
            // right x-edge (i + 1/2, j) of the last tile column
            edge_tau<C>(g, b, sX, sY, sP, LI(0, 0), LI(1, 0), LI(1, 1), LI(0, 1), LI(1, -1),
                        LI(0, -1), 0, FORCE && mine && i == Rg.i1, health, ex[ty][tx + 1]);
        }
        if (ty == FTY - 1) {
            // top y-edge (i, j + 1/2) of the last tile row
            edge_tau<C>(g, b, sX, sY, sP, LI(0, 0), LI(0, 1), LI(1, 1), LI(1, 0), LI(-1, 1),
                        LI(-1, 0), 1, FORCE && mine && j == Rg.j1, health, ey[ty + 1][tx]);
        }
#undef LI
        __syncthreads();
        if (mine) {
            const C* L = ex[ty][tx];
            const C* Rr = ex[ty][tx + 1];
            const C* B = ey[ty][tx];
            const C* T = ey[ty + 1][tx];
            const long long n = (long long)j * g.pitch + i;
            if (MODE == 0 || MODE == 3) {
                // Eq. (3_3_div_solid_stress) in Eq. (2_4_F_divs)
                C fx = (Rr[0] - L[0]) + (T[1] - B[1]);
                C fy = (Rr[1] - L[1]) + (T[2] - B[2]);
                const C p = sP[(ty + 1) * SX + tx + 1];
                C H = C(1), dr = C(0);
                if (b.present && p < C(INFINITY)) {
                    H = heaviside<C>(p, C(g.eps));
                    const C drs = C(b.rho_s - g.rho_f);
                    fx += (C(1) - H) * drs * C(g.gx);
                    fy += (C(1) - H) * drs * C(g.gy);
                    dr = (C(1) - H) * drs;  // Eq. (2_3_drho)
                }
                fx += H * C(g.fext_x);
                fy += H * C(g.fext_y);
                o0[n] = (double)fx;
                o1[n] = (double)fy;
                o2[n] = (double)dr;
                if (MODE == 3) {
                    // the node's lattice update (Sec. 3.4, 3.5): F^n as just
                    // stored (in double, read back in C as the lattice
                    // kernels do), F^{n-1} inside the previous window
                    const Neigh q = neigh(g, i, j);
                    C fl[NQ];
                    gather<C>(g, q, (const C*)lf.A, fl);
                    C Fpx = C(lf.fpo_x), Fpy = C(lf.fpo_y);
                    if (WP.has(i, j)) {
                        Fpx = C(lf.fpx[n]);
                        Fpy = C(lf.fpy[n]);
                    }
                    lb_finish_node<C, true>(g, (C*)lf.B, q, fl, Fpx, Fpy, C((double)fx),
                                            C((double)fy), C((double)dr), health);
                }
            } else {
                const long long e = (long long)j * g.nx + i;
                o0[e] = (double)((L[0] + Rr[0] + B[0] + T[0]) / C(4));
                o1[e] = (double)((L[1] + Rr[1] + B[1] + T[1]) / C(4));
                o2[e] = (double)((L[2] + Rr[2] + B[2] + T[2]) / C(4));
            }
        }
        __syncthreads();
    }
    if (RELABEL) {
        // relabel of the window's nodes outside the interior (buffer nodes)
        if (V.ok && b.present) {
            const int w = V.i1 - V.i0 + 1, h = V.j1 - V.j0 + 1;
            for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x;
                 e < (long long)w * h; e += (long long)nown * blockDim.x) {
                const int i = V.i0 + (int)(e % w), j = V.j0 + (int)(e / w);
                if (i >= 0 && i < g.nx && j >= 0 && j < g.ny) continue;
                const long long k = pidx(g, i, j);
                const double p = relabel_phi<C>(g, b, tag[k], X[k], Y[k], i, j);
                if (p < INFINITY) {
                    phi1[k] = store_phi<C>(p);
                } else {
                    phi1[k] = C(INFINITY);
                    X[k] = C(NAN);
                    Y[k] = C(NAN);
                }
            }
        }
        if (MODE == 3) {
            // the last of the blocks that took a tile (block 0 if none did)
            // reduces the boxes into ring slot wnext, checks the new window's
            // zone, and counts a box whose lower edge moved down by more than
            // BULK_EARLY_GAP rows from the current one (the early part of the
            // next step's bulk update assumes it does not).  (A launch of its
            // own for that took 4 to 7 us a step.)
            const int nb = max(1, min(ntx * nty, nown));
            if ((int)blockIdx.x >= nb) return;
            block_box(bi0, bi1, bj0, bj1, boxpart + 4 * blockIdx.x);
            if (!last_arrival(lf.ticket, nb)) return;
            const Win r = reduce_boxes<true>(boxpart, nb, &win[lf.wnext], nullptr);
            if (threadIdx.x == 0) {
                const Win cur = win[wvalid];
                check_zone(g, r, health);
                if (r.i0 <= r.i1 && cur.i0 <= cur.i1 && r.j0 < cur.j0 - BULK_EARLY_GAP)
                    atomicAdd(&health[6], 1u);
            }
            return;
        }
        block_box(bi0, bi1, bj0, bj1, boxpart + 4 * blockIdx.x);
    }
}

template <int MODE, typename C>
__global__ __launch_bounds__(256) void k_edges(GridP g, BodyP b, Win* win, int wvalid,
                                               int* boxpart, int whole_grid, C* X, C* Y,
                                               const C* __restrict__ phi,
                                               const int8_t* __restrict__ tag, C* phi1,
                                               double* o0, double* o1, double* o2, int* lcount,
                                               unsigned* health, LbFuse lf)
{
    // beside the bulk lattice update (MODE 3) the force pass is on the
    // critical path: its waves take the issue slots of a SIMD first
    if (MODE == 3) {
        if ((int)blockIdx.x >= lf.nown) {
            lb_along<C>(g, lf, win, wvalid, blockIdx.x - lf.nown, gridDim.x - lf.nown, health);
            return;
        }
        __builtin_amdgcn_s_setprio(3);
    }
    edges_body<MODE, C>(g, b, win, wvalid, boxpart, whole_grid, X, Y, phi, tag, phi1, o0, o1,
                        o2, lcount, health, lf);
}

// window index of lattice column c (row r) in solid grid g; along a
// sub-window axis the offset from the window origin, in [-PAD, lnx - PAD)
__device__ __forceinline__ int win_col(const GridP& g, int c)
{
    if (!g.wx) return c;
    const int d = wrap_axis(c - g.ox, g.lnx);
    return d >= g.lnx - PAD ? d - g.lnx : d;
}
__device__ __forceinline__ int win_row(const GridP& g, int r)
{
    if (!g.wy) return r;
    const int d = wrap_axis(r - g.oy, g.lny);
    return d >= g.lny - PAD ? d - g.lny : d;
}

// rectangle V of a solid's window as lattice nodes {x, dx, y, dy}: columns
// x .. x + dx (x wrapped, the range may run over a periodic seam), rows
// likewise; dx < 0 or dy < 0: empty
__device__ int4 mb_region(const GridP& g, const Rect& V)
{
    int4 r = make_int4(0, -1, 0, -1);
    if (!V.ok) return r;
    if (g.wx) {
        r.x = wrap_axis(V.i0 + g.ox, g.lnx);
        r.y = V.i1 - V.i0;
    } else {
        r.x = max(V.i0, 0);
        r.y = min(V.i1, g.nx - 1) - r.x;
    }
    if (g.wy) {
        r.z = wrap_axis(V.j0 + g.oy, g.lny);
        r.w = V.j1 - V.j0;
    } else {
        r.z = max(V.j0, 0);
        r.w = min(V.j1, g.ny - 1) - r.z;
    }
    return r;
}

// do [a, a + la] and [b, b + lb] meet (on a circle of n nodes if periodic)?
__device__ __forceinline__ bool ranges_meet(int a, int la, int b, int lb, int n, int periodic)
{
    if (!periodic) return a <= b + lb && b <= a + la;
    return wrap_axis(b - a, n) <= la || wrap_axis(a - b, n) <= lb;
}

// One block, solid k: the relabel's partial boxes (SAME: of this launch, by
// the solid's last block) into ring slot wnext, the solid's force region, and
// the force blocks it meets stamped and listed.
template <bool SAME>
__device__ __forceinline__ void mb_mark(const MbMark& m, int k, int nbox, unsigned* health)
{
    MbBody& B = m.bodies[k];
    const int sval = m.dcur ? (int)(*m.dcur + 1) : m.sval;
    __shared__ Win feps, fbox;
    if (nbox > 0) {
        const Win r = reduce_boxes<SAME>(B.boxpart, nbox, &B.win[m.wnext], nullptr);
        if (threadIdx.x == 0) fbox = r;
        reduce_boxes<SAME>(B.boxpart + 4 * nbox, nbox, &feps, nullptr);
    }
    __shared__ int4 reg;
    if (threadIdx.x == 0) {
        const GridP& g = B.g;
        Rect R;
        if (nbox > 0) {
            check_zone(g, fbox, health);
            // the force region of this step: the nodes with phi < eps and
            // their neighbours (elsewhere every solid fraction is zero on the
            // node and its edges, and the force is the uniform one), inside
            // the working window
            const Win e = feps;
            const Rect V = window_of(B.win, m.wcur, g);
            R.i0 = max(e.i0 - 1, V.i0);
            R.i1 = min(e.i1 + 1, V.i1);
            R.j0 = max(e.j0 - 1, V.j0);
            R.j1 = min(e.j1 + 1, V.j1);
            R.ok = V.ok && e.i0 <= e.i1 && R.i0 <= R.i1 && R.j0 <= R.j1;
        } else {
            R = window_of(B.win, m.wcur, g);
        }
        reg = mb_region(g, R);
        B.reg = reg;
    }
    __syncthreads();
    if (reg.y < 0 || reg.w < 0) return;
    // sample columns x, x + FB, ..., x + dx (and rows alike): every block met
    const int nsx = reg.y / FB + 2, nsy = reg.w / FB + 2;
    for (int e = threadIdx.x; e < nsx * nsy; e += blockDim.x) {
        int gx = reg.x + min((e % nsx) * FB, reg.y), gy = reg.z + min((e / nsx) * FB, reg.w);
        if (m.lg.px) gx = wrap_axis(gx, m.lg.nx);
        if (m.lg.py) gy = wrap_axis(gy, m.lg.ny);
        const int blk = (gy >> FB_LOG) * m.nbx + (gx >> FB_LOG);
        if (atomicExch(&m.stamp[blk], sval) != sval) m.list[atomicAdd(m.count, 1)] = blk;
    }
}

// the initial regions (one block per solid)
__global__ __launch_bounds__(256) void k_mb_mark(MbMark m)
{
    mb_mark<false>(m, blockIdx.x, 0, nullptr);
}

template <int MODE, typename C>
__global__ __launch_bounds__(256) void kb_force(const EdgesArgs* __restrict__ args,
                                                const int* __restrict__ ord, MbMark mk)
{
    const int row = ord ? ord[blockIdx.y] : blockIdx.y;
    const EdgesArgs& a = args[row];
    edges_body<MODE, C>(a.g, a.b, a.win, a.wvalid, a.boxpart, 0, (C*)a.X, (C*)a.Y, nullptr,
                        a.tag, (C*)a.phi, a.o0, a.o1, a.o2, a.lcount, a.health, LbFuse{});
    // several solids: the solid's last block marks its region (a launch of
    // its own, one block per solid, took 6 to 12 us)
    if (MODE == 2 && last_arrival(a.ticket, gridDim.x)) mb_mark<true>(mk, row, gridDim.x, a.health);
}

int lb_along_tiles(const GridP& g, int precision)
{
    const int tx = precision == 0 ? LbTile<double>::TX : LbTile<float>::TX, ty = 256 / tx;
    return ((g.nx + tx - 1) / tx) * ((g.ny + ty - 1) / ty);
}

hipError_t launch_force(const GridP& g, const BodyP& b, const BandBufs& bb, const StepSlots& s,
                        double* fx, double* fy, double* drho, hipStream_t st, const LbFuse* lf)
{
    // (MODE 3: no more own blocks than the largest window has tiles, rounded up
    // to the XCDs for the lattice tiles taken along)
    LbFuse f = lf ? *lf : LbFuse{};
    const int tiles = ((g.nx + FTX - 1) / FTX) * ((g.ny + FTY - 1) / FTY);
    f.nown = tiles < RELABEL_BLOCKS ? (tiles + 7) / 8 * 8 : RELABEL_BLOCKS;
    const int blocks = lf ? f.nown + f.along : RELABEL_BLOCKS;
#define KE(MODE, C, LF)                                                                       \
    k_edges<MODE, C><<<blocks, 256, 0, st>>>(                                                 \
        g, b, bb.win, s.wcur, bb.boxpart, 0, (C*)bb.X[s.nxt], (C*)bb.Y[s.nxt], nullptr, bb.tag, \
        (C*)bb.phi[s.nxt], fx, fy, drho, bb.lcount, bb.health, LF)
    if (lf) {
        if (g.rm32) KE(3, float, f);
        else KE(3, double, f);
    } else {
        if (g.rm32) KE(0, float, LbFuse{});
        else KE(0, double, LbFuse{});
    }
#undef KE
    return hipGetLastError();
}

hipError_t launch_read_stress(const GridP& g, const BodyP& b, const BandBufs& bb, int buf,
                              int wvalid, double* sxx, double* sxy, double* syy, hipStream_t st)
{
    if (g.rm32)
        k_edges<1, float><<<2048, 256, 0, st>>>(g, b, bb.win, wvalid, nullptr, 1,
                                                (float*)bb.X[buf], (float*)bb.Y[buf],
                                                (const float*)bb.phi[buf], nullptr, nullptr, sxx,
                                                sxy, syy, nullptr, bb.health, LbFuse{});
    else
        k_edges<1, double><<<2048, 256, 0, st>>>(g, b, bb.win, wvalid, nullptr, 1,
                                                 (double*)bb.X[buf], (double*)bb.Y[buf],
                                                 (const double*)bb.phi[buf], nullptr, nullptr,
                                                 sxx, sxy, syy, nullptr, bb.health, LbFuse{});
    return hipGetLastError();
}

// ---------------------------------------------------------------- reads

template <typename T>
__global__ void k_read_refmap(GridP g, BodyP b, const Win* __restrict__ win, int wvalid,
                              const T* __restrict__ X, const T* __restrict__ Y,
                              const T* __restrict__ phi, double* Xo, double* Yo, double* Po)
{
    constexpr bool DISP = sizeof(T) == 4;
    const Rect V = window_of(win, wvalid, g);
    const long long N = (long long)g.nx * g.ny;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < N;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(e % g.nx), j = (int)(e / g.nx);
        double xv = NAN, yv = NAN, pv = NAN;
        if (V.has(i, j)) {
            const long long k = pidx(g, i, j);
            if (phi[k] < T(INFINITY)) {
                xv = (double)X[k];
                yv = (double)Y[k];
                pv = (double)phi[k];
                if (DISP) {
                    xv += pos_x(g, b, i);
                    yv += pos_y(g, b, j);
                }
            }
        }
        if (Xo) Xo[e] = xv;
        if (Yo) Yo[e] = yv;
        if (Po) Po[e] = pv;
    }
}

hipError_t launch_read_refmap(const GridP& g, const BodyP& b, const BandBufs& bb, int buf,
                              int wvalid, double* X, double* Y, double* phi, hipStream_t st)
{
    if (g.rm32)
        k_read_refmap<float><<<2048, 256, 0, st>>>(g, b, bb.win, wvalid, (const float*)bb.X[buf],
                                                   (const float*)bb.Y[buf],
                                                   (const float*)bb.phi[buf], X, Y, phi);
    else
        k_read_refmap<double><<<2048, 256, 0, st>>>(g, b, bb.win, wvalid, (const double*)bb.X[buf],
                                                    (const double*)bb.Y[buf],
                                                    (const double*)bb.phi[buf], X, Y, phi);
    return hipGetLastError();
}

// ---------------------------------------------------------------- batched launches

// ---------------------------------------------------------------- several solids
//
// Every solid keeps its reference map on a window of its own (the chain
// kernels above run per solid, blockIdx.y = solid, relabelling only).  The
// lattice is cut into FB x FB force blocks; each step every solid stamps the
// blocks of its working window and lists the newly stamped ones, and one
// kernel over the listed blocks combines all solids into the force planes
// (Sec. 3.6): the global half-edge stress is the solids' blend normalised by
// their summed fraction where it exceeds one, plus the contact stress of
// every pair, Eqs. (3_6_global_stress) to (3_6_normal).

hipError_t launch_mb_mark(const MbMark& m, int nb, hipStream_t st)
{
    if (nb > 0) k_mb_mark<<<nb, 256, 0, st>>>(m);
    return hipGetLastError();
}

// (with solids the combine moves the counter on)
__global__ void k_mb_tick(long long* dstep)
{
    if (threadIdx.x == 0) *dstep += 1;
}

hipError_t launch_mb_tick(long long* dstep, hipStream_t st)
{
    k_mb_tick<<<1, 64, 0, st>>>(dstep);
    return hipGetLastError();
}

// xi, phi of solid B on the 3 x 3 nodes around window node (wi, wj), index
// (dj + 1) * 3 + (di + 1); a node without a map holds (NaN, NaN, +inf)
template <typename C>
__device__ __forceinline__ void mb_load3(const MbBody& B, const Rect& V, int buf, int wi, int wj,
                                         C* sX, C* sY, C* sP)
{
    // (pointers read from memory: to device memory, not to any)
    using G = const __attribute__((address_space(1))) C*;
    G X = (G)B.X[buf], Y = (G)B.Y[buf], P = (G)B.phi[buf];
#pragma unroll
    for (int e = 0; e < 9; e++) {
        int ci = wi + e % 3 - 1, cj = wj + e / 3 - 1;
        const bool in = canon(B.g, ci, cj) && V.has(ci, cj);
        const int k = in ? (int)pidx(B.g, ci, cj) : 0;
        const C xv = X[k], yv = Y[k], p = P[k];
        const bool set = in && p < C(INFINITY);
        sX[e] = set ? xv : C(NAN);
        sY[e] = set ? yv : C(NAN);
        sP[e] = set ? p : C(INFINITY);
    }
}

// the half-edges of a node in the 3 x 3 stencil: L, R, B, T as (a, b, s1..s4,
// dir) with a before b along the normal and s1 + s2 - s3 - s4 the tangential
// difference (the stencil of the single-solid force kernel)
constexpr int MB_EDGE[4][7] = {{3, 4, 7, 6, 1, 0, 0},
                                  {4, 5, 8, 7, 2, 1, 0},
                                  {1, 4, 5, 2, 3, 0, 1},
                                  {4, 7, 8, 5, 6, 3, 1}};

// Eq. (3_6_collision_force)
template <typename C>
__device__ __forceinline__ C contact_f(C x, C eps)
{
    return x < eps ? C(0.5) * (C(1) - x / eps) : C(0);
}

// force density and density excess of lattice node (gi, gj) from the solids
// sl[0 .. ns) (index order) of its block.  mode 0: force and density excess
// (fxo, fyo, drho: lattice planes); 1: density excess only; 2: the node
// average of the four global half-edge solid stresses (blend and contact)
// into fxo, fyo, drho as the xx, xy, yy planes of a read ([ny][nx]), with no
// health counts.
template <typename C>
__device__ void mb_node(const GridP& lg, const MbBody* __restrict__ bodies, const int* sl,
                        int ns, int buf, int wcur, int gi, int gj, double* fxo, double* fyo,
                        double* drho, int mode, unsigned* health)
{
    const bool drho_only = mode == 1;
    C acc[4][3], lse[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        lse[e] = C(0);
        acc[e][0] = acc[e][1] = acc[e][2] = C(0);
    }
    C lsum = C(0), dacc = C(0);
    int nset = 0;
    for (int q = 0; q < ns; q++) {
        const MbBody& B = bodies[sl[q]];
        const GridP& g = B.g;
        const int wi = win_col(g, gi), wj = win_row(g, gj);
        const Rect V = window_of(B.win, wcur, g);
        if (!V.has(wi, wj)) continue;
        C sX[9], sY[9], sP[9];
        mb_load3<C>(B, V, buf, wi, wj, sX, sY, sP);
        if (!(sP[4] < C(INFINITY))) continue;
        nset++;
        const C lam = C(1) - heaviside<C>(sP[4], C(g.eps));
        lsum += lam;
        dacc += lam * C(B.b.rho_s - lg.rho_f);
        if (drho_only) continue;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int a = MB_EDGE[e][0], b = MB_EDGE[e][1];
            if (!(sP[a] < C(INFINITY)) || !(sP[b] < C(INFINITY))) continue;
            const C le = C(1) - heaviside<C>(C(0.5) * (sP[a] + sP[b]), C(g.eps));
            if (!(le > C(0))) continue;
            lse[e] += le;
            C t[3];
            // each edge is counted once: by its far node (the L and B edges)
            edge_tau<C>(g, B.b, sX, sY, sP, a, b, MB_EDGE[e][2], MB_EDGE[e][3], MB_EDGE[e][4],
                        MB_EDGE[e][5], MB_EDGE[e][6], mode == 0 && (e == 0 || e == 2), health,
                        t);
            acc[e][0] += t[0];
            acc[e][1] += t[1];
            acc[e][2] += t[2];
        }
    }
    const long long n = (long long)gj * lg.pitch + gi;
    const C dr = lsum > C(1) ? dacc / lsum : dacc;
    if (mode != 2) drho[n] = (double)dr;
    if (drho_only) return;
#pragma unroll
    for (int e = 0; e < 4; e++)
        if (lse[e] > C(1)) {
            acc[e][0] /= lse[e];
            acc[e][1] /= lse[e];
            acc[e][2] /= lse[e];
        }
    if (nset >= 2 && lg.eta != 0.0) {
        // contact stress of every pair (p, q), p < q, on the node's edges
        for (int p = 0; p < ns; p++) {
            const MbBody& Bp = bodies[sl[p]];
            const int pi = win_col(Bp.g, gi), pj = win_row(Bp.g, gj);
            const Rect Vp = window_of(Bp.win, wcur, Bp.g);
            if (!Vp.has(pi, pj)) continue;
            C pX[9], pY[9], pP[9];
            mb_load3<C>(Bp, Vp, buf, pi, pj, pX, pY, pP);
            if (!(pP[4] < C(INFINITY))) continue;
            for (int q = p + 1; q < ns; q++) {
                const MbBody& Bq = bodies[sl[q]];
                const int qi = win_col(Bq.g, gi), qj = win_row(Bq.g, gj);
                const Rect Vq = window_of(Bq.win, wcur, Bq.g);
                if (!Vq.has(qi, qj)) continue;
                C qX[9], qY[9], qP[9];
                mb_load3<C>(Bq, Vq, buf, qi, qj, qX, qY, qP);
                if (!(qP[4] < C(INFINITY))) continue;
                const C cg = C(-lg.eta);
                const C gsum = C(Bp.b.G + Bq.b.G);
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    bool all = true;
#pragma unroll
                    for (int t = 0; t < 6; t++) {
                        const int v = MB_EDGE[e][t];
                        all = all && pP[v] < C(INFINITY) && qP[v] < C(INFINITY);
                    }
                    if (!all) continue;
                    const int a = MB_EDGE[e][0], b = MB_EDGE[e][1];
                    const C fp = contact_f<C>(C(0.5) * (pP[a] + pP[b]), C(lg.eps));
                    const C fq = contact_f<C>(C(0.5) * (qP[a] + qP[b]), C(lg.eps));
                    const C fmin = fp < fq ? fp : fq;
                    if (!(fmin > C(0))) continue;
                    C d[6];
#pragma unroll
                    for (int t = 0; t < 6; t++) {
                        const int v = MB_EDGE[e][t];
                        d[t] = pP[v] - qP[v];
                    }
                    // Eq. (3_6_normal) on the edge stencil
                    const C gn = d[1] - d[0];
                    const C gt = (d[2] + d[3] - d[4] - d[5]) / C(4);
                    const C gx = MB_EDGE[e][6] == 0 ? gn : gt;
                    const C gy = MB_EDGE[e][6] == 0 ? gt : gn;
                    const C gl = sqrt(gx * gx + gy * gy);
                    if (!(gl > C(0))) continue;
                    const C nx = gx / gl, ny = gy / gl;
                    const C c = cg * fmin * gsum;
                    acc[e][0] += c * (nx * nx - C(0.5));
                    acc[e][1] += c * (nx * ny);
                    acc[e][2] += c * (ny * ny - C(0.5));
                }
            }
        }
    }
    if (mode == 2) {
        const long long r = (long long)gj * lg.nx + gi;
        fxo[r] = (double)((acc[0][0] + acc[1][0] + acc[2][0] + acc[3][0]) / C(4));
        fyo[r] = (double)((acc[0][1] + acc[1][1] + acc[2][1] + acc[3][1]) / C(4));
        drho[r] = (double)((acc[0][2] + acc[1][2] + acc[2][2] + acc[3][2]) / C(4));
        return;
    }
    // Eq. (3_3_div_solid_stress) on the node's four edges, buoyancy of the
    // mixture and the fluid's share of the external force
    C fx = (acc[1][0] - acc[0][0]) + (acc[3][1] - acc[2][1]);
    C fy = (acc[1][1] - acc[0][1]) + (acc[3][2] - acc[2][2]);
    fx += dr * C(lg.gx);
    fy += dr * C(lg.gy);
    const C hf = lsum < C(1) ? C(1) - lsum : C(0);
    fx += hf * C(lg.fext_x);
    fy += hf * C(lg.fext_y);
    fxo[n] = (double)fx;
    fyo[n] = (double)fy;
}

// mode as mb_node; list null: every force block (nblk_all of them)
template <typename C>
__global__ __launch_bounds__(256) void k_mb_combine(GridP lg, const MbBody* __restrict__ bodies,
                                                    int nb, int buf, int wcur,
                                                    const int* __restrict__ list,
                                                    const int* __restrict__ count,
                                                    int* count_clear, int nbx, double* fx,
                                                    double* fy, double* drho, int mode,
                                                    unsigned* health, int nblk_all,
                                                    const long long* dcur, long long* dstep)
{
    static_assert(FB * FB == 256, "one thread per node of a force block");
    if (blockIdx.x == 0 && threadIdx.x == 0 && count_clear) *count_clear = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0 && dstep) *dstep = *dcur + 1;
    __shared__ int sl[MB_MAX_PER_BLOCK], hit[MB_HITS], nh;
    const int nblk = list ? *count : nblk_all;
    for (int t = blockIdx.x; t < nblk; t += gridDim.x) {
        const int blk = list ? list[t] : t;
        const int bx0 = (blk % nbx) * FB, by0 = (blk / nbx) * FB;
        if (threadIdx.x == 0) nh = 0;
        __syncthreads();
        // the solids whose region meets this block, as they are found among
        // MB_CHUNK solids at a time: a list that ends holds the first in index
        // order that the block takes
        for (int k0 = 0; k0 < nb; k0 += MB_CHUNK) {
            const int k = k0 + threadIdx.x;
            if (k < nb && (int)threadIdx.x < MB_CHUNK) {
                const int4 r = bodies[k].reg;
                if (r.y >= 0 && r.w >= 0 && ranges_meet(r.x, r.y, bx0, FB - 1, lg.nx, lg.px) &&
                    ranges_meet(r.z, r.w, by0, FB - 1, lg.ny, lg.py)) {
                    const int u = atomicAdd(&nh, 1);
                    if (u < MB_HITS) hit[u] = k;
                }
            }
            __syncthreads();
        }
        // in index order: a solid's place is the number of those before it
        const int all = min(nh, MB_HITS), ns = min(all, MB_MAX_PER_BLOCK);
        if ((int)threadIdx.x < all) {
            const int k = hit[threadIdx.x];
            int place = 0;
            for (int u = 0; u < all; u++) place += hit[u] < k ? 1 : 0;
            if (place < MB_MAX_PER_BLOCK) sl[place] = k;
        }
        if (threadIdx.x == 0 && nh > MB_MAX_PER_BLOCK && mode != 2)
            atomicAdd(&health[7], (unsigned)(nh - MB_MAX_PER_BLOCK));
        __syncthreads();
        const int gi = bx0 + threadIdx.x % FB, gj = by0 + threadIdx.x / FB;
        if (gi < lg.nx && gj < lg.ny)
            mb_node<C>(lg, bodies, sl, ns, buf, wcur, gi, gj, fx, fy, drho, mode, health);
        __syncthreads();
    }
}

hipError_t launch_mb_combine(const GridP& lg, int precision, const MbBody* bodies, int nb,
                             int buf, int wcur, const int* list, const int* count,
                             int* count_clear, int nbx, double* fx, double* fy, double* drho,
                             bool drho_only, unsigned* health, hipStream_t st,
                             const long long* dcur, long long* dstep)
{
    if (precision == 0)
        k_mb_combine<double><<<MB_COMBINE_BLOCKS, 256, 0, st>>>(
            lg, bodies, nb, buf, wcur, list, count, count_clear, nbx, fx, fy, drho,
            drho_only ? 1 : 0, health, 0, dcur, dstep);
    else
        k_mb_combine<float><<<MB_COMBINE_BLOCKS, 256, 0, st>>>(
            lg, bodies, nb, buf, wcur, list, count, count_clear, nbx, fx, fy, drho,
            drho_only ? 1 : 0, health, 0, dcur, dstep);
    return hipGetLastError();
}

hipError_t launch_mb_read_stress(const GridP& lg, int precision, const MbBody* bodies, int nb,
                                 int buf, int wslot, int nbx, int nby, double* sxx, double* sxy,
                                 double* syy, unsigned* health, hipStream_t st)
{
    if (precision == 0)
        k_mb_combine<double><<<MB_COMBINE_BLOCKS, 256, 0, st>>>(
            lg, bodies, nb, buf, wslot, nullptr, nullptr, nullptr, nbx, sxx, sxy, syy, 2, health,
            nbx * nby, nullptr, nullptr);
    else
        k_mb_combine<float><<<MB_COMBINE_BLOCKS, 256, 0, st>>>(
            lg, bodies, nb, buf, wslot, nullptr, nullptr, nullptr, nbx, sxx, sxy, syy, 2, health,
            nbx * nby, nullptr, nullptr);
    return hipGetLastError();
}

// the region boxes and window origins of the solids from a saved copy of the
// solid table (every other field of a table entry is fixed by the context)
__global__ void k_mb_copy_reg(const MbBody* __restrict__ src, MbBody* dst, int nb, MbTabs tabs)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < nb) {
        dst[k].reg = src[k].reg;
        mb_set_origin(dst[k], tabs, k, src[k].g.ox, src[k].g.oy);
    }
}

hipError_t launch_mb_copy_reg(const MbBody* src, MbBody* dst, int nb, const MbTabs& tabs,
                              hipStream_t st)
{
    k_mb_copy_reg<<<(nb + 255) / 256, 256, 0, st>>>(src, dst, nb, tabs);
    return hipGetLastError();
}

// xi and phi of solid k on the lattice nodes (NaN where it holds no map)
template <typename C>
__global__ void k_mb_read_refmap(GridP lg, const MbBody* __restrict__ bodies, int k, int buf,
                                 int wvalid, double* X, double* Y, double* phi)
{
    const MbBody& B = bodies[k];
    const GridP& g = B.g;
    const Rect V = window_of(B.win, wvalid, g);
    const C* Xs = (const C*)B.X[buf];
    const C* Ys = (const C*)B.Y[buf];
    const C* Ps = (const C*)B.phi[buf];
    const long long N = (long long)lg.nx * lg.ny;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < N;
         e += (long long)gridDim.x * blockDim.x) {
        const int gi = (int)(e % lg.nx), gj = (int)(e / lg.nx);
        const int i = win_col(g, gi), j = win_row(g, gj);
        double xv = NAN, yv = NAN, pv = NAN;
        if (V.has(i, j) && i >= 0 && i < g.nx && j >= 0 && j < g.ny) {
            const long long kk = pidx(g, i, j);
            const C p = Ps[kk];
            if (p < C(INFINITY)) {
                xv = (double)Xs[kk];
                yv = (double)Ys[kk];
                if (sizeof(C) == 4) {
                    xv += pos_x(g, B.b, i);
                    yv += pos_y(g, B.b, j);
                }
                pv = (double)p;
            }
        }
        if (X) X[e] = xv;
        if (Y) Y[e] = yv;
        if (phi) phi[e] = pv;
    }
}

hipError_t launch_mb_read_refmap(const GridP& lg, int precision, const MbBody* bodies, int k,
                                 int buf, int wvalid, double* X, double* Y, double* phi,
                                 hipStream_t st)
{
    const long long N = (long long)lg.nx * lg.ny;
    const int blocks = (int)((N + 255) / 256 < 4096 ? (N + 255) / 256 : 4096);
    if (precision == 0)
        k_mb_read_refmap<double><<<blocks, 256, 0, st>>>(lg, bodies, k, buf, wvalid, X, Y, phi);
    else
        k_mb_read_refmap<float><<<blocks, 256, 0, st>>>(lg, bodies, k, buf, wvalid, X, Y, phi);
    return hipGetLastError();
}

// one block per solid: its fraction moments over the interior nodes of its
// window, reduced in a fixed order
template <typename C>
__global__ __launch_bounds__(256) void k_mb_diag(const MbBody* __restrict__ bodies, int buf,
                                                 int wvalid, double* out)
{
    const MbBody& B = bodies[blockIdx.x];
    const GridP& g = B.g;
    const Rect V = window_of(B.win, wvalid, g);
    const C* Xs = (const C*)B.X[buf];
    const C* Ys = (const C*)B.Y[buf];
    const C* Ps = (const C*)B.phi[buf];
    double a[7] = {0, 0, 0, 0, 0, 0, 0};
    if (V.ok) {
        const int i0 = max(V.i0, 0), i1 = min(V.i1, g.nx - 1);
        const int j0 = max(V.j0, 0), j1 = min(V.j1, g.ny - 1);
        const int w = i1 - i0 + 1, h = j1 - j0 + 1;
        if (w > 0 && h > 0)
            for (int e = threadIdx.x; e < w * h; e += blockDim.x) {
                const int i = i0 + e % w, j = j0 + e / w;
                const long long k = pidx(g, i, j);
                const double p = (double)Ps[k];
                if (!(p < INFINITY)) continue;
                a[6] += 1.0;
                if (p < 0.0) a[5] += 1.0;
                const double lam = 1.0 - heaviside<double>(p, g.eps);
                const double x = pos_x(g, B.b, i), y = pos_y(g, B.b, j);
                double dx, dy;
                if (sizeof(C) == 4) {  // displacement storage: x - xi = -d
                    dx = -(double)Xs[k];
                    dy = -(double)Ys[k];
                } else {
                    dx = x - (double)Xs[k];
                    dy = y - (double)Ys[k];
                }
                a[0] += lam;
                a[1] += lam * x;
                a[2] += lam * y;
                a[3] += lam * dx;
                a[4] += lam * dy;
            }
    }
    __shared__ double red[7][256];
    for (int t = 0; t < 7; t++) red[t][threadIdx.x] = a[t];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o)
            for (int t = 0; t < 7; t++) red[t][threadIdx.x] += red[t][threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x < 7) out[7 * blockIdx.x + threadIdx.x] = red[threadIdx.x][0];
}

hipError_t launch_mb_diag(int precision, const MbBody* bodies, int nb, int buf, int wvalid,
                          double* out, hipStream_t st)
{
    if (nb <= 0) return hipSuccess;
    if (precision == 0) k_mb_diag<double><<<nb, 256, 0, st>>>(bodies, buf, wvalid, out);
    else k_mb_diag<float><<<nb, 256, 0, st>>>(bodies, buf, wvalid, out);
    return hipGetLastError();
}

hipError_t launch_batch_band(int precision, const BatchTables& t, int nsim, int layers,
                             hipStream_t st, int dt_blocks, int fit_blocks, int band_blocks,
                             bool fused, bool pairs, const MbStep* mb)
{
    // the reference-map chain of every member of a batch, or (mb) of every
    // solid of a context, which relabels and marks only
    const dim3 gb(band_blocks, nsim), gd(dt_blocks, nsim), gf(fit_blocks, nsim);
    const MbFit mf = mb ? mb->fit : MbFit{};
    const int gm = mf.rows * mf.blocks + (nsim - mf.rows) * mf.few;  // blocks of kb_fit_mb
    const long long* dstep = mb ? mb->dstep : nullptr;
    long long* dcur = mb ? mb->dcur : nullptr;
#define ADB(T, LC, TH) kb_advect_dt<LC, TH, T><<<gd, 256, 0, st>>>(t.adv, t.ord, dstep, dcur)
#define ADB_D(LC, TH) ADB(double, LC, TH)
#define ADB_F(LC, TH) ADB(float, LC, TH)
    // fused: every layer of a member in one launch over its zone tiles (the
    // advection pass lists those tiles); several solids: by solid or by tile
#define CHAIN(T, MB_NT)                                                                        \
    do {                                                                                       \
        if (fused && mb) {                                                                     \
            if (layers == FF_LAYERS)                                                           \
                kb_fit_mb<T, FF_LAYERS><<<gm, FF_THREADS, 0, st>>>(t.fit, t.ord, mf);          \
            else kb_fit_mb<T, 0><<<gm, FF_THREADS, 0, st>>>(t.fit, t.ord, mf);                 \
        } else if (fused) {                                                                    \
            constexpr bool P = sizeof(T) == 4;                                                 \
            if (P && pairs) {                                                                  \
                if (layers == FF_LAYERS) kb_fit_fused<T, FF_LAYERS, P><<<gf, 256, 0, st>>>(t.fit); \
                else kb_fit_fused<T, 0, P><<<gf, 256, 0, st>>>(t.fit);                         \
            } else if (layers == FF_LAYERS) {                                                  \
                kb_fit_fused<T, FF_LAYERS, false><<<gf, FF_THREADS, 0, st>>>(t.fit);           \
            } else {                                                                           \
                kb_fit_fused<T, 0, false><<<gf, FF_THREADS, 0, st>>>(t.fit);                   \
            }                                                                                  \
        } else if (mb) {                                                                       \
            kb_fit_lds<T, MB_NT><<<dim3(1, nsim), MB_NT, 0, st>>>(t.fit, layers, t.ord);       \
        } else {                                                                               \
            for (int l = 1; l <= layers; l++)                                                  \
                if (l <= 2) kb_layer_fit<T, true><<<gf, 256, 0, st>>>(t.fit, l);               \
                else kb_layer_fit<T, false><<<gf, 256, 0, st>>>(t.fit, l);                     \
        }                                                                                      \
        if (mb) kb_force<2, T><<<gb, 256, 0, st>>>(t.edg, t.ord, mb->mark);                    \
        else kb_force<0, T><<<gb, 256, 0, st>>>(t.edg, t.ord, MbMark{});                       \
    } while (0)
    if (precision == 0) {
        DT_DISPATCH(layers, fused, ADB_D);
        CHAIN(double, MB_FIT_THREADS_F64);
    } else {
        DT_DISPATCH(layers, fused, ADB_F);
        CHAIN(float, MB_FIT_THREADS_F32);
    }
#undef CHAIN
#undef ADB_F
#undef ADB_D
#undef ADB
    return hipGetLastError();
}

}  // namespace lbrmt
