// adjoint.hip -- reverse mode of the MPDATA step on the GPU (an extension of
// the method, not in the paper).
//
// Sweep: a forward pass keeps psi at the start of every segment of
// ckpt_every steps; segments are then reversed last to first, recomputing
// their states, and every step is reversed stage by stage.  The forward
// recompute of a step runs the staged kernels and keeps each pass's input
// field, raw and limited pseudo-velocities and limiter coefficients; the
// reverse kernels are the transposes of those stages.  Every transpose
// gathers: each adjoint entry is summed by one thread over the forward
// outputs that read it (through the boundary map), in a fixed order -- the
// pseudo-velocity transpose in 2-D without third-order terms from
// coefficients its workgroup keeps in LDS, otherwise from per-position slots
// each wall writes to workspace -- so the gradients are the same bits on
// every run; no kernel uses atomics.
//
// Conventions at non-differentiable points: d[u]+/du = [u > 0],
// d[u]-/du = [u < 0], d|u|/du = [u > 0] - [u < 0]; max/min pass the
// derivative to the operand they returned, ties to the earliest operand in
// the forward's scan order; zero-denominator fractions and the "no flux"
// limiter branch have zero derivative.  G is a constant.
#include "adjoint.hpp"
#include "common.hpp"
#include "kernels.hpp"

#include <rocprofiler-sdk-roctx/roctx.h>

#include <type_traits>

namespace mp {
namespace {

constexpr int B = 256;

// Named range in rocprofv3's marker trace (--marker-trace), scoped.
struct TraceRange {
    explicit TraceRange(const char *name) { roctxRangePushA(name); }
    ~TraceRange() { roctxRangePop(); }
    TraceRange(const TraceRange &) = delete;
    TraceRange &operator=(const TraceRange &) = delete;
};

struct I3 {
    int v[3];
};

__device__ inline I3 unflat_i3(int64_t t, const int64_t e[3])
{
    I3 p;
    unflat3(t, e, p.v);
    return p;
}

__device__ inline I3 sh1(I3 p, int d, int s)
{
    p.v[d] += s;
    return p;
}

__device__ inline I3 sh2(I3 p, int d, int s, int e, int t)
{
    p.v[d] += s;
    p.v[e] += t;
    return p;
}

__device__ inline int64_t ci(const Geom &g, const I3 &p)
{
    int i = wrap_cell(p.v[0], (int)g.n[0], g.bc[0]);
    int j = wrap_cell(p.v[1], (int)g.n[1], g.bc[1]);
    int k = wrap_cell(p.v[2], (int)g.n[2], g.bc[2]);
    return ((int64_t)i * g.n[1] + j) * g.n[2] + k;
}

__device__ inline int64_t wi(const Geom &g, int d, const I3 &p)
{
    int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
    e[d] += 1;
    int q[3];
    for (int t = 0; t < 3; t++)
        q[t] = (t == d) ? wrap_wall(p.v[t], (int)g.n[t], g.bc[t])
                        : wrap_cell(p.v[t], (int)g.n[t], g.bc[t]);
    return ((int64_t)q[0] * e[1] + q[1]) * e[2] + q[2];
}

template <typename T> __device__ inline T sgnv(T u) { return T((u > T(0)) - (u < T(0))); }

// psi-fraction num / den (num / m under iga; 0 for a zero den) and its
// derivatives d/d num and d/d den, from one reciprocal of den
template <typename T>
__device__ inline void frac_vd(bool iga, T num, T den, T m, T &v, T &dn, T &dd)
{
    if (iga) {
        v = num / m;
        dn = T(1) / m;
        dd = T(0);
    } else if (den == T(0)) {
        v = dn = dd = T(0);
    } else {
        const T r = T(1) / den;
        v = num * r;
        dn = r;
        dd = -v * r;
    }
}

template <typename T> __global__ void k_fill(T *a, int64_t n, T v)
{
    int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t < n) a[t] = v;
}

template <typename T> __global__ void k_add(T *a, const T *b, int64_t n)
{
    int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t < n) a[t] += b[t];
}

// several buffers per launch: clear a[i] (b == nullptr) or add b[i] into
// a[i] and clear b[i]
template <typename T> struct Bufs {
    T *a[8];
    T *b[8];
    int64_t n[8];
    int k = 0;
    int64_t nmax = 0;
    void push(T *x, int64_t m, T *y = nullptr)
    {
        a[k] = x;
        b[k] = y;
        n[k] = m;
        k++;
        if (m > nmax) nmax = m;
    }
};

template <typename T> __global__ void k_clear_n(Bufs<T> f)
{
    int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    for (int i = 0; i < f.k; i++)
        if (t < f.n[i]) f.a[i][t] = T(0);
}

template <typename T> __global__ void k_add_clear_n(Bufs<T> f)
{
    int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    for (int i = 0; i < f.k; i++)
        if (t < f.n[i]) {
            f.a[i][t] += f.b[i][t];
            f.b[i][t] = T(0);
        }
}

template <typename T> __global__ void k_copy(T *a, const T *b, int64_t n)
{
    int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t < n) a[t] = b[t];
}

// Gather form of the donor-cell transpose (no atomics).  Cell i's adjoint
// collects, from every cell q in {i - e_d, i, i + e_d} and each of q's two
// dimension-d walls, the derivative of q's update with respect to x_i
// through that wall's flux (whose left / right cells are read through the
// boundary map, exactly as the forward pass reads them); the advector
// adjoint of a wall collects the same from the cells that read the wall.
template <typename T, int ND>
__global__ void k_donor_adj_cells(Geom g, const T *c0, const T *c1, const T *c2, const T *G,
                                  int flux_is_vel, const T *__restrict__ yb, T *xb)
{
    int64_t N = g.n[0] * g.n[1] * g.n[2];
    int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t >= N) return;
    T acc = yb[t];
    if (!flux_is_vel) {
        const T *c[3] = {c0, c1, c2};
        I3 p = unflat_i3(t, g.n);
#pragma unroll
        for (int d = 0; d < ND; d++) {
            const int n = (int)g.n[d], bc = g.bc[d], pd = p.v[d];
#pragma unroll
            for (int off = -1; off <= 1; off++) {
                int qd = pd + off;
                if (bc == BC_OPEN && (qd < 0 || qd >= n)) continue;
                I3 q = p;
                q.v[d] = qd;
                int64_t kq = ci(g, q);
                T ybg = G ? yb[kq] / G[kq] : yb[kq];
#pragma unroll
                for (int sd = 0; sd < 2; sd++) {
                    int wd = qd + sd;                  // wall of q (before the map)
                    int Ld = wrap_cell(wd - 1, n, bc), Rd = wrap_cell(wd, n, bc);
                    if (Ld != pd && Rd != pd) continue;
                    I3 w = q;
                    w.v[d] = wd;
                    T u = c[d][wi(g, d, w)];
                    T fb = sd ? -ybg : ybg;            // d y_q / d F (times yb_q)
                    if (Ld == pd) acc += pos(u) * fb;
                    if (Rd == pd) acc += neg(u) * fb;
                }
            }
        }
    }
    xb[t] += acc;
}

template <typename T, int ND, int WD>
__global__ void k_donor_adj_walls(Geom g, const T *__restrict__ x, const T *cd, const T *G,
                                  int flux_is_vel, const T *__restrict__ yb, T *cbd)
{
    constexpr int d = WD;
    int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
    e[d] += 1;
    int64_t M = e[0] * e[1] * e[2];
    int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t >= M) return;
    I3 w = unflat_i3(t, e);
    const int n = (int)g.n[d], bc = g.bc[d], wdv = w.v[d];
    T acc = T(0);
#pragma unroll
    for (int sd = 0; sd < 2; sd++) {
        int qd = wdv - sd;                         // cell whose side sd is this wall
        if (bc == BC_OPEN && (qd < 0 || qd >= n)) continue;
        if (wrap_wall(qd + sd, n, bc) != wdv) continue;   // periodic wall n is never read
        I3 q = w;
        q.v[d] = qd;
        int64_t kq = ci(g, q);
        T ybg = G ? yb[kq] / G[kq] : yb[kq];
        T fb = sd ? -ybg : ybg;
        if (flux_is_vel) {
            acc += fb;
        } else {
            T u = cd[wi(g, d, w)];
            I3 L = q, R = q;
            L.v[d] = qd + sd - 1;
            R.v[d] = qd + sd;
            T du = (u > T(0) ? x[ci(g, L)] : T(0)) + (u < T(0) ? x[ci(g, R)] : T(0));
            acc += du * fb;
        }
    }
    if (acc != T(0)) cbd[t] += acc;
}

// Both transposes of a 2-D donor-cell pass (G = 1) in one gather: the
// thread of cell (i, j) owns xb(i, j) and the adjoints of the cell's low
// walls, plus the far edge wall of an open dimension.  The flux adjoint of
// a wall is yb of the cell above it minus yb of the cell below (cells
// outside an open domain read no wall); a cell is the left cell of its high
// wall and the right cell of its low wall, and at an open edge also the
// mapped outside neighbour of the edge wall.  The row is wave-uniform (one
// block per row segment), so no index division per thread.
// It writes xb, plus xadd with XADD, and writes (AC) or adds to the wall
// adjoints (the periodic wall n of a dimension is never written).  z0..z2 (cell fields, NULL when unused, never read here)
// are set to zero at the thread's cell, for the scatter-add kernels that
// follow (in place of separate clearing launches).
// A thread makes DR rows of its column: the rows share their reads of yb, c0
// and x, and all reads of the DR cells are in flight together.  Bound by
// memory (64 to 72 bytes a cell in FP64), but with one cell per thread the
// latency of its reads was two thirds of a wave's time.
constexpr int DR = 4;

template <typename T, bool XADD, bool AC>
__global__ void __launch_bounds__(B)
    k_donor_adj2d(int n0, int n1, int bc0, int bc1, int bpr, int flux_is_vel,
                  const T *__restrict__ x, const T *__restrict__ c0, const T *__restrict__ c1,
                  const T *__restrict__ yb, const T *__restrict__ xadd, T *__restrict__ xb,
                  T *__restrict__ cb0, T *__restrict__ cb1, T *__restrict__ z0,
                  T *__restrict__ z1, T *__restrict__ z2)
{
    // block b runs on XCD b % 8: each XCD takes a contiguous range of row
    // segments, so the rows above and below a segment are read by blocks on
    // the same XCD, through its L2
    int b;
    {
        const int nblk = (int)gridDim.x;
        const int x8 = blockIdx.x & 7, per = nblk >> 3, rem = nblk & 7;
        b = x8 * per + (x8 < rem ? x8 : rem) + (blockIdx.x >> 3);
    }
    const int i0 = b / bpr * DR;
    const int j = (b % bpr) * B + threadIdx.x;
    if (j >= n1) return;
    const bool o0 = bc0 == BC_OPEN, o1 = bc1 == BC_OPEN;
    const bool lft = o1 && j == 0, rgt = o1 && j == n1 - 1;
    const int jm = wrap_cell(j - 1, n1, bc1), jp = wrap_cell(j + 1, n1, bc1);
    const int jw = wrap_wall(j + 1, n1, bc1);
    // rows i0-1 .. i0+DR (through the boundary map; a row past the last one
    // of the grid is read in the place of the last and not used)
    T y[DR + 2], yl[DR], yr[DR], u0[DR + 1], ul[DR], uh[DR], xc[DR + 1], xl[DR];
    T add[DR], old0[DR], old1[DR];
#pragma unroll
    for (int r = 0; r < DR + 2; r++)
        y[r] = yb[(int64_t)wrap_cell(min(i0 + r - 1, n0), n0, bc0) * n1 + j];
#pragma unroll
    for (int r = 0; r < DR; r++) {
        const int64_t k = (int64_t)min(i0 + r, n0 - 1) * n1;
        yl[r] = yb[k + jm];
        yr[r] = yb[k + jp];
        if (XADD) add[r] = xadd[k + j];
        if (!AC) {
            old0[r] = cb0[k + j];
            old1[r] = cb1[k + min(i0 + r, n0 - 1) + j];
        }
    }
    if (!flux_is_vel) {
#pragma unroll
        for (int r = 0; r < DR + 1; r++) {
            u0[r] = c0[(int64_t)wrap_wall(min(i0 + r, n0), n0, bc0) * n1 + j];
            xc[r] = x[(int64_t)wrap_cell(min(i0 + r - 1, n0 - 1), n0, bc0) * n1 + j];
        }
#pragma unroll
        for (int r = 0; r < DR; r++) {
            const int i = min(i0 + r, n0 - 1);
            ul[r] = c1[(int64_t)i * (n1 + 1) + j];
            uh[r] = c1[(int64_t)i * (n1 + 1) + jw];
            xl[r] = x[(int64_t)i * n1 + jm];
        }
    }
#pragma unroll
    for (int r = 0; r < DR; r++) {
        const int i = i0 + r;
        if (i >= n0) return;
        const bool top = o0 && i == 0, bot = o0 && i == n0 - 1;
        const int64_t k = (int64_t)i * n1 + j, k1 = k + i;
        const int64_t w0hi = (int64_t)n0 * n1 + j, w1hi = k1 - j + n1;   // edge walls n0, n1
        if (z0) z0[k] = T(0);
        if (z1) z1[k] = T(0);
        if (z2) z2[k] = T(0);
        const T yc = y[r + 1];
        const T yim = top ? T(0) : y[r], yip = bot ? T(0) : y[r + 2];
        const T yjm = lft ? T(0) : yl[r], yjp = rgt ? T(0) : yr[r];
        const T F0lo = yc - yim, F0hi = yip - yc, F1lo = yc - yjm, F1hi = yjp - yc;
        T acc = yc, f0 = F0lo, f1 = F1lo, f0h = F0hi, f1h = F1hi;
        if (!flux_is_vel) {
            const T u0lo = u0[r], u0hi = u0[r + 1], u1lo = ul[r], u1hi = uh[r];
            acc = yc + (pos(u0hi) * F0hi + neg(u0lo) * F0lo) + (pos(u1hi) * F1hi + neg(u1lo) * F1lo);
            if (top) acc += pos(u0lo) * F0lo;
            if (bot) acc += neg(u0hi) * F0hi;
            if (lft) acc += pos(u1lo) * F1lo;
            if (rgt) acc += neg(u1hi) * F1hi;
            const T xi = xc[r], xo = xc[r + 1], xj = xl[r];
            f0 = ((u0lo > T(0) ? xi : T(0)) + (u0lo < T(0) ? xo : T(0))) * F0lo;
            f1 = ((u1lo > T(0) ? xj : T(0)) + (u1lo < T(0) ? xo : T(0))) * F1lo;
            f0h = ((u0hi > T(0) ? xo : T(0)) + (u0hi < T(0) ? xo : T(0))) * F0hi;
            f1h = ((u1hi > T(0) ? xo : T(0)) + (u1hi < T(0) ? xo : T(0))) * F1hi;
        }
        if (XADD) acc += add[r];
        xb[k] = acc;
        cb0[k] = AC ? f0 : old0[r] + f0;
        cb1[k1] = AC ? f1 : old1[r] + f1;
        if (bot) cb0[w0hi] = AC ? f0h : cb0[w0hi] + f0h;
        if (rgt) cb1[w1hi] = AC ? f1h : cb1[w1hi] + f1h;
    }
}

// Deterministic transpose of the pseudo-velocity (1-D, 3-D, and 2-D with
// the third-order terms), phase 1: every wall of dimension WD sums what it
// sends to each stencil position -- its right cell R = p, left cell
// L = p - e_d, R + e_d, L - e_d, R and L shifted by +-e_o along each other
// dimension o, and (3-D third-order term) R and L shifted by +-e_o1 +-e_o2
// -- into that position's slot, in the order of the terms; its own advector
// adjoint into U and a quarter of each cross-mean adjoint into Q.  Every
// slot entry has one writer.  Phase 2 (k_pseudo_gather_cells / _walls) has
// every cell and wall sum the slots that land on it in a fixed order, so the
// sums are the same bits on every run.  Slots of a wall: 0 R, 1 L, 2 R+e_d,
// 3 L-e_d, then per other dimension (ascending) R+e_o, L+e_o, R-e_o, L-e_o,
// then (3-D) for L and then R: (+o1,+o2), (-o1,+o2), (+o1,-o2), (-o1,-o2).
template <int ND> constexpr int pseudo_slots() { return 4 + 4 * (ND - 1) + (ND == 3 ? 8 : 0); }

// offset from the wall's right cell of slot k (wall dimension d)
template <int ND>
__device__ __forceinline__ void slot_offset(int d, int k, int off[3])
{
    off[0] = off[1] = off[2] = 0;
    if (k < 4) {
        off[d] = k == 0 ? 0 : (k == 1 ? -1 : (k == 2 ? 1 : -2));
        return;
    }
    int o[2] = {0, 0}, n = 0;
    for (int t = 0; t < ND; t++)
        if (t != d) o[n++] = t;
    if (k < 4 + 4 * (ND - 1)) {
        const int oi = (k - 4) >> 2, r = (k - 4) & 3;
        off[d] = (r & 1) ? -1 : 0;               // R, L, R, L
        off[o[oi]] = (r < 2) ? 1 : -1;           // +e_o twice, then -e_o twice
        return;
    }
    const int q = k - 4 - 4 * (ND - 1);           // (3-D) the eight corners
    off[d] = (q < 4) ? -1 : 0;                    // L first, then R
    off[o[0]] = (q & 1) ? -1 : 1;
    off[o[1]] = (q & 2) ? -1 : 1;
}

template <typename T, int ND, int WD>
__global__ void __launch_bounds__(B)
k_pseudo_adj_slots(Geom g, unsigned opts, const T *__restrict__ x, const T *c0, const T *c1,
                   const T *c2, const T *G, const T *__restrict__ Vb, T *__restrict__ S,
                   T *__restrict__ U, T *__restrict__ Q)
{
    constexpr int d = WD;
    constexpr int NS = pseudo_slots<ND>();
    int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
    e[d] += 1;
    const int64_t M = e[0] * e[1] * e[2];
    const int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t >= M) return;
    T acc[NS];
#pragma unroll
    for (int k = 0; k < NS; k++) acc[k] = T(0);
    T ub = T(0);
    T cbar_b[3] = {T(0), T(0), T(0)};
    const T vb = Vb[t];
    if (vb != T(0)) {
        const bool iga = opts & OPT_IGA, tot = opts & OPT_TOT;
        const T *c[3] = {c0, c1, c2};
        const I3 p = unflat_i3(t, e);
        const I3 L = sh1(p, d, -1), R = p;
        const T u = c[d][wi(g, d, p)];
        const T GL = G ? G[ci(g, L)] : T(1), GR = G ? G[ci(g, R)] : T(1);
        const T Gb = T(0.5) * (GL + GR);
        const T iGb = T(1) / Gb, iGb2 = iGb * iGb;
        const T xL = x[ci(g, L)], xR = x[ci(g, R)];
        T fn, fd;
        T A;
        frac_vd(iga, xR - xL, xR + xL, T(2), A, fn, fd);
        ub += (sgnv(u) - T(2) * u * iGb) * A * vb;
        const T Ab = (fabs(u) - u * u * iGb) * vb;
        acc[0] += (fn + fd) * Ab;
        acc[1] += (-fn + fd) * Ab;
        T cbar[3] = {T(0), T(0), T(0)};
        {
            int oi = 0;
#pragma unroll
            for (int o = 0; o < ND; o++) {
                if (o == d) continue;
                cbar[o] = T(0.25) * (c[o][wi(g, o, L)] + c[o][wi(g, o, sh1(L, o, 1))] +
                                     c[o][wi(g, o, R)] + c[o][wi(g, o, sh1(R, o, 1))]);
                const T a = x[ci(g, sh1(R, o, 1))], b = x[ci(g, sh1(L, o, 1))];
                const T ee = x[ci(g, sh1(R, o, -1))], f = x[ci(g, sh1(L, o, -1))];
                T Bv;
                frac_vd(iga, a + b - ee - f, a + b + ee + f, T(4), Bv, fn, fd);
                ub += T(-0.5) * cbar[o] * iGb * Bv * vb;
                cbar_b[o] += T(-0.5) * u * iGb * Bv * vb;
                const T Bb = T(-0.5) * u * cbar[o] * iGb * vb;
                acc[4 + 4 * oi + 0] += (fn + fd) * Bb;
                acc[4 + 4 * oi + 1] += (fn + fd) * Bb;
                acc[4 + 4 * oi + 2] += (-fn + fd) * Bb;
                acc[4 + 4 * oi + 3] += (-fn + fd) * Bb;
                oi++;
            }
        }
        if (tot) {
            const T xR2 = x[ci(g, sh1(R, d, 1))], xL2 = x[ci(g, sh1(L, d, -1))];
            T Dv;
            frac_vd(iga, xR2 - xR - xL + xL2, xR2 + xR + xL + xL2, T(4), Dv, fn, fd);
            const T cD = (T(3) * u * fabs(u) * iGb - T(2) * u * u * u * iGb2 - u) / T(3);
            ub += (T(6) * fabs(u) * iGb - T(6) * u * u * iGb2 - T(1)) / T(3) * Dv * vb;
            const T Db = cD * vb;
            acc[2] += (fn + fd) * Db;
            acc[0] += (-fn + fd) * Db;
            acc[1] += (-fn + fd) * Db;
            acc[3] += (fn + fd) * Db;
            int oi = 0;
#pragma unroll
            for (int o = 0; o < ND; o++) {
                if (o == d) continue;
                const T a = x[ci(g, sh1(R, o, 1))], b = x[ci(g, sh1(L, o, 1))];
                const T ee = x[ci(g, sh1(R, o, -1))], f = x[ci(g, sh1(L, o, -1))];
                T Ev;
                frac_vd(iga, a - b - ee + f, a + b + ee + f, T(4), Ev, fn, fd);
                const T cE = fabs(u) * cbar[o] * iGb - T(2) * u * u * cbar[o] * iGb2;
                ub += (sgnv(u) * cbar[o] * iGb - T(4) * u * cbar[o] * iGb2) * Ev * vb;
                cbar_b[o] += (fabs(u) * iGb - T(2) * u * u * iGb2) * Ev * vb;
                const T Eb = cE * vb;
                acc[4 + 4 * oi + 0] += (fn + fd) * Eb;
                acc[4 + 4 * oi + 1] += (-fn + fd) * Eb;
                acc[4 + 4 * oi + 2] += (-fn + fd) * Eb;
                acc[4 + 4 * oi + 3] += (fn + fd) * Eb;
                oi++;
            }
            if constexpr (ND == 3) {
                constexpr int o1 = (d == 0) ? 1 : 0;
                constexpr int o2 = (d == 2) ? 1 : 2;
                T xs[2][4];
                T num = T(0), den = T(0);
#pragma unroll
                for (int sd = 0; sd < 2; sd++) {
                    const I3 SS = sd ? R : L;
                    xs[sd][0] = x[ci(g, sh2(SS, o1, 1, o2, 1))];
                    xs[sd][1] = x[ci(g, sh2(SS, o1, -1, o2, 1))];
                    xs[sd][2] = x[ci(g, sh2(SS, o1, 1, o2, -1))];
                    xs[sd][3] = x[ci(g, sh2(SS, o1, -1, o2, -1))];
                    num += xs[sd][0] - xs[sd][1] - xs[sd][2] + xs[sd][3];
                    den += xs[sd][0] + xs[sd][1] + xs[sd][2] + xs[sd][3];
                }
                T Tv;
                frac_vd(iga, num, den, T(8), Tv, fn, fd);
                const T k = -(T(2) / T(3)) * iGb2;
                ub += k * cbar[o1] * cbar[o2] * Tv * vb;
                cbar_b[o1] += k * u * cbar[o2] * Tv * vb;
                cbar_b[o2] += k * u * cbar[o1] * Tv * vb;
                const T Tb = k * u * cbar[o1] * cbar[o2] * vb;
                const T sg[4] = {T(1), T(-1), T(-1), T(1)};
#pragma unroll
                for (int sd = 0; sd < 2; sd++)
#pragma unroll
                    for (int q = 0; q < 4; q++) acc[12 + 4 * sd + q] += (sg[q] * fn + fd) * Tb;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NS; k++) S[(int64_t)k * M + t] = acc[k];
    U[t] = ub;
    {
        int oi = 0;
#pragma unroll
        for (int o = 0; o < ND; o++) {
            if (o == d) continue;
            Q[(int64_t)oi * M + t] = T(0.25) * cbar_b[o];
            oi++;
        }
    }
}

// the unmapped coordinates in [-2, n+1] that the boundary map sends to
// cell coordinate q (at most five: an open extent of one cell)
__device__ __forceinline__ int cell_preimages(int q, int n, int bc, int u[5])
{
    int m = 0;
    if (bc == BC_PERIODIC) {
        for (int v = q - 2 * n; v <= q + 2 * n; v += n)
            if (v >= -2 && v <= n + 1) u[m++] = v;
    } else {
        u[m++] = q;
        if (q == 0) {
            u[m++] = -1;
            u[m++] = -2;
        }
        if (q == n - 1) {
            u[m++] = n;
            u[m++] = n + 1;
        }
    }
    return m;
}

// phase 2 for the cells: xb[q] += every slot whose position maps onto q
// (wall dimensions ascending, slots in order, preimages in order)
template <typename T, int ND>
__global__ void __launch_bounds__(B)
k_pseudo_gather_cells(Geom g, const T *__restrict__ S0, const T *__restrict__ S1,
                      const T *__restrict__ S2, T *__restrict__ xb)
{
    constexpr int NS = pseudo_slots<ND>();
    const int64_t N = g.n[0] * g.n[1] * g.n[2];
    const int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t >= N) return;
    const I3 q = unflat_i3(t, g.n);
    int uu[3][5], nu[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        if (a < ND) {
            nu[a] = cell_preimages(q.v[a], (int)g.n[a], g.bc[a], uu[a]);
        } else {
            nu[a] = 1;
            uu[a][0] = 0;
        }
    }
    const T *Sd[3] = {S0, S1, S2};
    T acc = T(0);
#pragma unroll
    for (int d = 0; d < ND; d++) {
        int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
        e[d] += 1;
        const int64_t M = e[0] * e[1] * e[2];
        for (int k = 0; k < NS; k++) {
            int off[3];
            slot_offset<ND>(d, k, off);
            for (int a0 = 0; a0 < nu[0]; a0++)
                for (int a1 = 0; a1 < nu[1]; a1++)
                    for (int a2 = 0; a2 < nu[2]; a2++) {
                        const int p0 = uu[0][a0] - off[0], p1 = uu[1][a1] - off[1],
                                  p2 = uu[2][a2] - off[2];
                        const int pv[3] = {p0, p1, p2};
                        bool ok = true;
#pragma unroll
                        for (int b = 0; b < 3; b++)
                            ok = ok && pv[b] >= 0 && pv[b] < (int)e[b];
                        // a periodic dimension's wall n is wall 0, not a wall of its own
                        if (ok && g.bc[d] == BC_PERIODIC && pv[d] == (int)g.n[d]) ok = false;
                        if (ok) acc += Sd[d][(int64_t)k * M + ((int64_t)p0 * e[1] + p1) * e[2] + p2];
                    }
        }
    }
    xb[t] += acc;
}

// phase 2 for the dimension-o walls: cb[w] += the wall's own share, then the
// cross-mean shares of the other dimensions' walls that land on it (their
// left cell's and right cell's o-walls, low then high)
template <typename T, int ND, int WO>
__global__ void __launch_bounds__(B)
k_pseudo_gather_walls(Geom g, const T *__restrict__ U, const T *__restrict__ Q0,
                      const T *__restrict__ Q1, const T *__restrict__ Q2, T *__restrict__ cb)
{
    constexpr int o = WO;
    int64_t eo[3] = {g.n[0], g.n[1], g.n[2]};
    eo[o] += 1;
    const int64_t M = eo[0] * eo[1] * eo[2];
    const int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t >= M) return;
    const I3 w = unflat_i3(t, eo);
    T v = U[t];
    const T *Qd[3] = {Q0, Q1, Q2};
    // preimages of the wall coordinate along o (walls 0..n) and of the cell
    // coordinates along the other dimensions
    int fo[2], nfo = 0;
    if (g.bc[o] == BC_PERIODIC) {
        if (w.v[o] < (int)g.n[o]) fo[nfo++] = w.v[o];
        if (w.v[o] == 0) fo[nfo++] = (int)g.n[o];
    } else {
        fo[nfo++] = w.v[o];
    }
#pragma unroll
    for (int d = 0; d < ND; d++) {
        if (d == o) continue;
        int oi = 0;   // index of o among the dimensions != d
        for (int t2 = 0; t2 < o; t2++)
            if (t2 != d) oi++;
        int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
        e[d] += 1;
        const int64_t Md = e[0] * e[1] * e[2];
        int ud[5];
        const int nud = cell_preimages(w.v[d], (int)g.n[d], g.bc[d], ud);
        // roles: L (low o-wall), L + e_o, R, R + e_o
        for (int r = 0; r < 4; r++) {
            const int dl = (r < 2) ? 1 : 0;      // L = p - e_d: p_d = u_d + 1
            const int dh = (r & 1) ? 1 : 0;      // o-wall p_o + 1
            for (int a = 0; a < nud; a++)
                for (int b = 0; b < nfo; b++) {
                    int pv[3] = {w.v[0], w.v[1], w.v[2]};
                    pv[d] = ud[a] + dl;
                    pv[o] = fo[b] - dh;
                    bool ok = pv[d] >= 0 && pv[d] <= (int)g.n[d] && pv[o] >= 0 &&
                              pv[o] < (int)g.n[o];
                    if (ok && g.bc[d] == BC_PERIODIC && pv[d] == (int)g.n[d]) ok = false;
                    if (ok)
                        v += Qd[d][(int64_t)oi * Md + ((int64_t)pv[0] * e[1] + pv[1]) * e[2] + pv[2]];
                }
        }
    }
    cb[t] += v;
}

// 2-D boundary map with compile-time boundary types and 32-bit flat indices
// (n0 n1 < 2^31).  The tiled kernels read coordinates from -2 to n + 1
// (a tile's ring of one cell and its neighbours), which one period's shift
// brings into range when a periodic extent is at least 3 (as every plan
// requires, and the launchers check).
template <int BC> __device__ __forceinline__ int wc2(int q, int n)
{
    if constexpr (BC == BC_PERIODIC) {
        return q < 0 ? q + n : (q >= n ? q - n : q);
    } else {
        return q < 0 ? 0 : (q >= n ? n - 1 : q);
    }
}
template <int BC> __device__ __forceinline__ int ww2(int f, int n)
{
    if constexpr (BC == BC_PERIODIC) {
        return f < 0 ? f + n : (f >= n ? f - n : f);
    } else {
        return f < 0 ? 0 : (f > n ? n : f);
    }
}
template <int BC0, int BC1> struct Map2 {
    int n0, n1;
    __device__ __forceinline__ int cell(const I3 &q) const
    {
        return wc2<BC0>(q.v[0], n0) * n1 + wc2<BC1>(q.v[1], n1);
    }
    __device__ __forceinline__ int wall(int d, const I3 &q) const
    {
        return d == 0 ? ww2<BC0>(q.v[0], n0) * n1 + wc2<BC1>(q.v[1], n1)
                      : wc2<BC0>(q.v[0], n0) * (n1 + 1) + ww2<BC1>(q.v[1], n1);
    }
};

// Deterministic 2-D transpose of the pseudo-velocity (no third-order
// terms).  A workgroup owns a tile of GR x GC cells, their low walls of both
// dimensions and, along an open dimension, the far edge walls of its last
// tile.  Phase 1 evaluates, for every wall the tile's cells read (the tile's
// walls plus a one-wall halo, in coordinates before the boundary map), the
// adjoint the wall sends to each of its stencil roles, into LDS; phase 2 has
// every cell sum what its roles receive, and every owned wall its own term
// plus the cross terms, in a fixed order.  Each adjoint entry has one writer
// and one summation order: the same bits on every run.
constexpr int GR = 8, GC = 64, GT = GR * GC;
constexpr int Q0R = GR + 1, Q0C = GC + 2;   // dimension-0 walls: rows i0..i0+GR, cols j0-1..j0+GC
constexpr int Q1R = GR + 2, Q1C = GC + 1;   // dimension-1 walls: rows i0-1..i0+GR, cols j0..j0+GC
constexpr int NQ0 = Q0R * Q0C, NQ1 = Q1R * Q1C;
// what a wall sends: to its right / left cell (the A term), to the cells
// beside them on the +o / -o side (the B term), to the dimension-o walls of
// its cross-advector mean (a quarter each), and to its own advector
enum { KR, KL, KP, KM, KQ, KU, NK };
// halo walls of a tile, dimension 0: the row below it, then the columns at
// its sides; dimension 1: the rows above and below, then the column past it
constexpr int H0 = NQ0 - GT, H1 = NQ1 - GT;
constexpr int H1_FROM = (H0 + 63) / 64 * 64;      // the first thread of dimension 1's (a whole wave)
static_assert(H1_FROM + H1 <= GT, "the halo walls of both dimensions take one round");

template <typename T, int WD, int BC0, int BC1>
__device__ __forceinline__ void pseudo_coef2(const Map2<BC0, BC1> &g, unsigned opts,
                                             const T *__restrict__ x, const T *const c[2],
                                             const T *G, T vb, int i, int j, T k[NK])
{
    constexpr int d = WD, o = 1 - WD;
    const bool iga = opts & OPT_IGA;
    const I3 p{{i, j, 0}};
    const I3 L = sh1(p, d, -1), R = p;
    const T u = c[d][g.wall(d, p)];
    T iGb = T(1);
    if (G) iGb = T(1) / (T(0.5) * (G[g.cell(L)] + G[g.cell(R)]));
    const T xL = x[g.cell(L)], xR = x[g.cell(R)];
    T fn, fd, A;
    frac_vd(iga, xR - xL, xR + xL, T(2), A, fn, fd);
    T ub = (sgnv(u) - T(2) * u * iGb) * A * vb;
    const T Ab = (fabs(u) - u * u * iGb) * vb;
    k[KR] = (fn + fd) * Ab;
    k[KL] = (-fn + fd) * Ab;
    const I3 Lo = sh1(L, o, 1), Ro = sh1(R, o, 1);
    const T cbar = T(0.25) * (c[o][g.wall(o, L)] + c[o][g.wall(o, Lo)] + c[o][g.wall(o, R)] +
                              c[o][g.wall(o, Ro)]);
    const T a = x[g.cell(sh1(R, o, 1))], b = x[g.cell(sh1(L, o, 1))];
    const T e = x[g.cell(sh1(R, o, -1))], f = x[g.cell(sh1(L, o, -1))];
    T Bv;
    frac_vd(iga, a + b - e - f, a + b + e + f, T(4), Bv, fn, fd);
    ub += T(-0.5) * cbar * iGb * Bv * vb;
    const T Bb = T(-0.5) * u * cbar * iGb * vb;
    k[KP] = (fn + fd) * Bb;
    k[KM] = (-fn + fd) * Bb;
    k[KQ] = T(0.25) * (T(-0.5) * u * iGb * Bv * vb);
    k[KU] = ub;
}

template <typename T, int BC0, int BC1>
__global__ void __launch_bounds__(GT)
k_pseudo_adj2g(Geom gg, unsigned opts, const T *__restrict__ x, const T *c0, const T *c1,
               const T *G, const T *__restrict__ Vb0, const T *__restrict__ Vb1, T *xb, T *cb0,
               T *cb1)
{
    const Map2<BC0, BC1> g{(int)gg.n[0], (int)gg.n[1]};
    // (a wall's own adjoint is read by another thread only where a far edge
    // wall is owned by the cell below it)
    constexpr int NK0 = BC0 == BC_OPEN ? NK : KU, NK1 = BC1 == BC_OPEN ? NK : KU;
    __shared__ T K0[NK0][NQ0];
    __shared__ T K1[NK1][NQ1];
    const int n0 = g.n0, n1 = g.n1;
    const int tiles_c = (n1 + GC - 1) / GC;
    const int i0 = (int)(blockIdx.x / tiles_c) * GR, j0 = (int)(blockIdx.x % tiles_c) * GC;
    // the last wall row / column a cell of the tile reads; entries beyond
    // them, and walls an open dimension does not have, hold zeros
    const int ilim = min(i0 + GR, n0), jlim = min(j0 + GC, n1);
    const T *c[2] = {c0, c1};
    // the stencil loads do not wait for the test of vb (a zero vb zeroes
    // the coefficients afterwards)
    auto wall0 = [&](int i, int j) -> T {
        T k[NK] = {T(0), T(0), T(0), T(0), T(0), T(0)};
        bool ok = i <= ilim && j <= jlim;
        if (BC1 == BC_OPEN) ok = ok && j >= 0 && j < n1;
        if (ok) {
            const T vb = Vb0[g.wall(0, I3{{i, j, 0}})];
            pseudo_coef2<T, 0>(g, opts, x, c, G, vb, i, j, k);
            if (vb == T(0))
#pragma unroll
                for (int r = 0; r < NK; r++) k[r] = T(0);
        }
        const int e = (i - i0) * Q0C + (j - (j0 - 1));
#pragma unroll
        for (int r = 0; r < NK0; r++) K0[r][e] = k[r];
        return k[KU];
    };
    auto wall1 = [&](int i, int j) -> T {
        T k[NK] = {T(0), T(0), T(0), T(0), T(0), T(0)};
        bool ok = i <= ilim && j <= jlim;
        if (BC0 == BC_OPEN) ok = ok && i >= 0 && i < n0;
        if (ok) {
            const T vb = Vb1[g.wall(1, I3{{i, j, 0}})];
            pseudo_coef2<T, 1>(g, opts, x, c, G, vb, i, j, k);
            if (vb == T(0))
#pragma unroll
                for (int r = 0; r < NK; r++) k[r] = T(0);
        }
        const int f = (i - (i0 - 1)) * Q1C + (j - j0);
#pragma unroll
        for (int r = 0; r < NK1; r++) K1[r][f] = k[r];
        return k[KU];
    };
    const int tid = (int)threadIdx.x;
    const int qi = i0 + tid / GC, qj = j0 + tid % GC;
    const T own0 = wall0(qi, qj), own1 = wall1(qi, qj);
    if (tid < H0) {
        if (tid < Q0C) (void)wall0(i0 + GR, j0 - 1 + tid);
        else (void)wall0(i0 + (tid - Q0C) / 2, (tid - Q0C) % 2 ? j0 + GC : j0 - 1);
    } else if (tid >= H1_FROM && tid < H1_FROM + H1) {
        const int f = tid - H1_FROM;
        if (f < 2 * Q1C) (void)wall1(f < Q1C ? i0 - 1 : i0 + GR, j0 + (f < Q1C ? f : f - Q1C));
        else (void)wall1(i0 + f - 2 * Q1C, j0 + GC);
    }
    __syncthreads();
    if (qi >= n0 || qj >= n1) return;
    // coefficient kind r of the wall at unmapped (i, j); zero outside the
    // box.  The cell's own position and its neighbours are always inside
    // (unchecked reads, CK false); only the positions past an open edge can
    // fall outside.
    auto k0 = [&](auto CK, int r, int i, int j) -> T {
        const int a = i - i0, b = j - (j0 - 1);
        if (!decltype(CK)::value) return K0[r][a * Q0C + b];
        return (a >= 0 && a < Q0R && b >= 0 && b < Q0C) ? K0[r][a * Q0C + b] : T(0);
    };
    auto k1 = [&](auto CK, int r, int i, int j) -> T {
        const int a = i - (i0 - 1), b = j - j0;
        if (!decltype(CK)::value) return K1[r][a * Q1C + b];
        return (a >= 0 && a < Q1R && b >= 0 && b < Q1C) ? K1[r][a * Q1C + b] : T(0);
    };
    using Un = std::false_type;
    using Ck = std::true_type;
    // the unmapped positions the boundary map sends to row qi / column qj:
    // the cell itself, and past an open edge the position beyond it
    int pr[3], pc[3], nr = 0, nc = 0;
    pr[nr++] = qi;
    if (BC0 == BC_OPEN && qi == 0) pr[nr++] = -1;
    if (BC0 == BC_OPEN && qi == n0 - 1) pr[nr++] = n0;
    pc[nc++] = qj;
    if (BC1 == BC_OPEN && qj == 0) pc[nc++] = -1;
    if (BC1 == BC_OPEN && qj == n1 - 1) pc[nc++] = n1;
    // the cell: every role of every wall that lands on it
    auto roles = [&](auto CK, int X0, int X1, T &acc) {
        acc += k0(CK, KR, X0, X1) + k0(CK, KL, X0 + 1, X1);              // A term, d = 0
        acc += k0(CK, KP, X0, X1 - 1) + k0(CK, KP, X0 + 1, X1 - 1);      // B term, +o side
        acc += k0(CK, KM, X0, X1 + 1) + k0(CK, KM, X0 + 1, X1 + 1);      // B term, -o side
        acc += k1(CK, KR, X0, X1) + k1(CK, KL, X0, X1 + 1);              // A term, d = 1
        acc += k1(CK, KP, X0 - 1, X1) + k1(CK, KP, X0 - 1, X1 + 1);
        acc += k1(CK, KM, X0 + 1, X1) + k1(CK, KM, X0 + 1, X1 + 1);
    };
    T acc = T(0);
    roles(Un{}, qi, qj, acc);
    for (int s = 0; s < nr; s++)
        for (int t = 0; t < nc; t++)
            if (s > 0 || t > 0) roles(Ck{}, pr[s], pc[t], acc);
    xb[(int64_t)qi * n1 + qj] += acc;
    // owned dimension-0 walls: the cell's low wall, and at an open far edge
    // the edge wall; own term plus the cross terms of the dimension-1 walls
    // whose cross-advector mean reads them
    auto cross0 = [&](auto CK, int Y0, int Z1) {
        return k1(CK, KQ, Y0, Z1 + 1) + k1(CK, KQ, Y0 - 1, Z1 + 1) + k1(CK, KQ, Y0, Z1) +
               k1(CK, KQ, Y0 - 1, Z1);
    };
    {
        T v = own0;
        v += cross0(Un{}, qi, qj);
        for (int t = 1; t < nc; t++) v += cross0(Ck{}, qi, pc[t]);
        cb0[(int64_t)qi * n1 + qj] += v;
    }
    if constexpr (BC0 == BC_OPEN) if (qi == n0 - 1) {
        T v = k0(Ck{}, KU, n0, qj);
        for (int t = 0; t < nc; t++) v += cross0(Ck{}, n0, pc[t]);
        cb0[(int64_t)n0 * n1 + qj] += v;
    }
    auto cross1 = [&](auto CK, int Z0, int Y1) {
        return k0(CK, KQ, Z0 + 1, Y1) + k0(CK, KQ, Z0 + 1, Y1 - 1) + k0(CK, KQ, Z0, Y1) +
               k0(CK, KQ, Z0, Y1 - 1);
    };
    {
        T v = own1;
        v += cross1(Un{}, qi, qj);
        for (int s = 1; s < nr; s++) v += cross1(Ck{}, pr[s], qj);
        cb1[(int64_t)qi * (n1 + 1) + qj] += v;
    }
    if constexpr (BC1 == BC_OPEN) if (qj == n1 - 1) {
        T v = k1(Ck{}, KU, qi, n1);
        for (int s = 0; s < nr; s++) v += cross1(Ck{}, pr[s], n1);
        cb1[(int64_t)qi * (n1 + 1) + n1] += v;
    }
}

// ---- atomic-free limiter transposes -------------------------------------
// The limited velocity W = [V]+ up + [V]- dn of a wall routes its adjoint to
// the limiter coefficient of the cell that attains up / dn; the limiter
// coefficients of a cell route theirs to the cell and face neighbours that
// attain the bounds, to the neighbours' fluxes and to the cell's walls.  As
// scatters these need atomics, whose order -- and so the rounding of the
// sums -- changes from run to run.  Here every adjoint entry is written by
// one thread that sums its contributions in a fixed order, so the gradient
// is the same bits on every run.

// the decision of one wall (mapped coordinates w, wall dimension d): its
// cells L, R, which of them attains up and dn (0: the constant 1, 1: L,
// 2: R), the adjoints sent (upb, dnb) and the velocity adjoint
template <typename T> struct LimWall {
    int64_t kL, kR;
    int wu, wd;
    T upb, dnb, vb;
};

template <typename T>
__device__ __forceinline__ LimWall<T> lim_wall(const Geom &g, int d, const I3 &w, const T *V,
                                               const T *bup, const T *bdn, const T *Wb)
{
    LimWall<T> r;
    const int64_t kw = wi(g, d, w);
    r.kL = ci(g, sh1(w, d, -1));
    r.kR = ci(g, w);
    const T wb = Wb[kw];
    const T v = V[kw];
    T up = T(1), dn = T(1);
    r.wu = r.wd = 0;
    if (bdn[r.kL] < up) { up = bdn[r.kL]; r.wu = 1; }
    if (bup[r.kR] < up) { up = bup[r.kR]; r.wu = 2; }
    if (bup[r.kL] < dn) { dn = bup[r.kL]; r.wd = 1; }
    if (bdn[r.kR] < dn) { dn = bdn[r.kR]; r.wd = 2; }
    r.vb = ((v > T(0) ? up : T(0)) + (v < T(0) ? dn : T(0))) * wb;
    r.upb = pos(v) * wb;
    r.dnb = neg(v) * wb;
    if (wb == T(0)) r.wu = r.wd = 0;
    return r;
}

// transpose of the limited velocities of all wall dimensions, one thread per
// cell: it writes the velocity adjoint of the cell's low walls (and of an
// open dimension's far edge wall), and sums into bub, bdb of the cell what
// each of its 2 ND walls sends it (low then high wall, dimension by
// dimension; the right-cell role before the left-cell role, which at an
// open edge wall are the same cell).  bub and bdb are written, not added to.
template <typename T, int ND>
__global__ void __launch_bounds__(B)
k_limit_adj_gather(Geom g, const T *V0, const T *V1, const T *V2, const T *__restrict__ bup,
                   const T *__restrict__ bdn, const T *Wb0, const T *Wb1, const T *Wb2, T *Vb0,
                   T *Vb1, T *Vb2, T *__restrict__ bub, T *__restrict__ bdb)
{
    const int64_t N = g.n[0] * g.n[1] * g.n[2];
    const int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t >= N) return;
    const T *V[3] = {V0, V1, V2}, *Wb[3] = {Wb0, Wb1, Wb2};
    T *Vb[3] = {Vb0, Vb1, Vb2};
    const I3 p = unflat_i3(t, g.n);
    T su = T(0), sd = T(0);
#pragma unroll
    for (int d = 0; d < ND; d++) {
        const int n = (int)g.n[d];
#pragma unroll
        for (int side = 0; side < 2; side++) {
            // one cell along a periodic dimension: its high wall is its low wall
            if (side == 1 && g.bc[d] == BC_PERIODIC && n == 1) continue;
            I3 w = p;
            w.v[d] = wrap_wall(p.v[d] + side, n, g.bc[d]);
            const LimWall<T> r = lim_wall<T>(g, d, w, V[d], bup, bdn, Wb[d]);
            // the cell owns its low wall, and at an open far edge the edge wall
            if (side == 0 || (g.bc[d] == BC_OPEN && p.v[d] == n - 1)) Vb[d][wi(g, d, w)] = r.vb;
            if (r.kR == t) {
                if (r.wu == 2) su += r.upb;
                if (r.wd == 2) sd += r.dnb;
            }
            if (r.kL == t) {
                if (r.wu == 1) sd += r.upb;
                if (r.wd == 1) su += r.dnb;
            }
        }
    }
    bub[t] = su;
    bdb[t] = sd;
}

// limiter-coefficient transpose, phase 1 (one thread per cell): the adjoints
// of the cell's in- and out-flux, of its bounds and of its own value, and
// which cell attains each bound (slot 0 the cell, 1 + 2d + (s > 0) the face
// neighbour -e_d / +e_d; bit 3 / 7: the bound is psi^n's value, not x's),
// stored for phase 2.  F[0..4] = finb, foutb, mxb, mnb, own-value adjoint.
template <typename T, int ND>
__global__ void __launch_bounds__(B)
k_beta_adj_a(Geom g, unsigned opts, const T *__restrict__ psi_n, const T *__restrict__ x,
             const T *V0, const T *V1, const T *V2, const T *G, const T *__restrict__ bub,
             const T *__restrict__ bdb, T *__restrict__ F0, T *__restrict__ F1,
             T *__restrict__ F2, T *__restrict__ F3, T *__restrict__ F4, int *__restrict__ code)
{
    const int64_t N = g.n[0] * g.n[1] * g.n[2];
    const int64_t t = (int64_t)blockIdx.x * B + threadIdx.x;
    if (t >= N) return;
    const T bu_b = bub[t], bd_b = bdb[t];
    if (bu_b == T(0) && bd_b == T(0)) {
        F0[t] = F1[t] = F2[t] = F3[t] = F4[t] = T(0);
        code[t] = 0;
        return;
    }
    const bool iga = opts & OPT_IGA;
    const T *V[3] = {V0, V1, V2};
    const I3 p = unflat_i3(t, g.n);
    T mx = psi_n[t], mn = mx;
    int amx = 0, amn = 0, smx = 0, smn = 0;
    const T v = x[t];
    if (v > mx) { mx = v; smx = 1; }
    if (v < mn) { mn = v; smn = 1; }
    for (int d = 0; d < ND; d++)
        for (int s = -1; s <= 1; s += 2) {
            const int64_t kq = ci(g, sh1(p, d, s));
            const int slot = 1 + 2 * d + (s > 0);
            const T a = psi_n[kq], b = x[kq];
            if (a > mx) { mx = a; amx = slot; smx = 0; }
            if (a < mn) { mn = a; amn = slot; smn = 0; }
            if (b > mx) { mx = b; amx = slot; smx = 1; }
            if (b < mn) { mn = b; amn = slot; smn = 1; }
        }
    const T xi = v;
    T fin = T(0), fout = T(0);
    for (int d = 0; d < ND; d++) {
        const T vlo = V[d][wi(g, d, p)], vhi = V[d][wi(g, d, sh1(p, d, 1))];
        const T wm = iga ? T(1) : x[ci(g, sh1(p, d, -1))];
        const T wp = iga ? T(1) : x[ci(g, sh1(p, d, 1))];
        const T wc = iga ? T(1) : xi;
        fin += pos(vlo) * wm - neg(vhi) * wp;
        fout += pos(vhi) * wc - neg(vlo) * wc;
    }
    const T Gi = G ? G[t] : T(1);
    T finb = T(0), foutb = T(0), mxb = T(0), mnb = T(0), xib = T(0);
    if (fin > T(0) && bu_b != T(0)) {
        const T r = T(1) / fin, gq = Gi * r * bu_b;
        mxb += gq;
        xib -= gq;
        finb -= (mx - xi) * r * gq;
    }
    if (fout > T(0) && bd_b != T(0)) {
        const T r = T(1) / fout, gq = Gi * r * bd_b;
        xib += gq;
        mnb -= gq;
        foutb -= (xi - mn) * r * gq;
    }
    if (!iga)
        for (int d = 0; d < ND; d++) {
            const T vlo = V[d][wi(g, d, p)], vhi = V[d][wi(g, d, sh1(p, d, 1))];
            xib += (pos(vhi) - neg(vlo)) * foutb;
        }
    F0[t] = finb;
    F1[t] = foutb;
    F2[t] = mxb;
    F3[t] = mnb;
    F4[t] = xib;
    code[t] = amx | (smx << 3) | (amn << 4) | (smn << 7);
}

// the cell a bound slot of cell c points at (mapped)
// (selects: no indexing of c by a run-time dimension)
__device__ __forceinline__ int64_t slot_cell(const Geom &g, const I3 &c, int64_t kc, int slot)
{
    if (slot == 0) return kc;
    I3 t = c;
    t.v[0] += slot == 1 ? -1 : (slot == 2 ? 1 : 0);
    t.v[1] += slot == 3 ? -1 : (slot == 4 ? 1 : 0);
    t.v[2] += slot == 5 ? -1 : (slot == 6 ? 1 : 0);
    return ci(g, t);
}

// limiter-coefficient transpose, phase 2 (one thread per cell q): adds to
// xb(q) and pnb(q) what the cells whose bounds or fluxes read q send it, and
// to the velocity adjoint of q's low walls (and an open far edge wall) what
// the wall's two cells send it, in a fixed order.
template <typename T, int ND>
__global__ void __launch_bounds__(B)
k_beta_adj_b(Geom g, unsigned opts, const T *__restrict__ x, const T *V0, const T *V1,
             const T *V2, const T *__restrict__ F0, const T *__restrict__ F1,
             const T *__restrict__ F2, const T *__restrict__ F3, const T *__restrict__ F4,
             const int *__restrict__ code, T *__restrict__ xb, T *__restrict__ pnb, T *Vb0,
             T *Vb1, T *Vb2)
{
    const int64_t N = g.n[0] * g.n[1] * g.n[2];
    const int64_t q = (int64_t)blockIdx.x * B + threadIdx.x;
    if (q >= N) return;
    const bool iga = opts & OPT_IGA;
    const T *V[3] = {V0, V1, V2};
    T *Vb[3] = {Vb0, Vb1, Vb2};
    const I3 pq = unflat_i3(q, g.n);
    T ax = F4[q], ap = T(0);
    // candidates: q itself, then its face neighbours (-e0, +e0, -e1, ...),
    // each cell once; a neighbour that maps onto q is q itself, already
    // counted (the checks below test every role of a candidate)
#pragma unroll
    for (int k = 0; k < 1 + 2 * ND; k++) {
        I3 c = pq;
        int64_t kc = q;
        if (k > 0) {
            const int d = (k - 1) >> 1, s = ((k - 1) & 1) ? 1 : -1;
            // two cells along a periodic dimension: both neighbours are one cell
            if (s > 0 && g.bc[d] == BC_PERIODIC && g.n[d] == 2) continue;
            c = sh1(pq, d, s);
            if (g.bc[d] == BC_OPEN && (c.v[d] < 0 || c.v[d] >= (int)g.n[d])) continue;
            c.v[d] = wrap_cell(c.v[d], (int)g.n[d], g.bc[d]);
            kc = ci(g, c);
            if (kc == q) continue;
        }
        const int cd = code[kc];
        if (slot_cell(g, c, kc, cd & 7) == q) {
            if (cd & 8) ax += F2[kc];
            else ap += F2[kc];
        }
        if (slot_cell(g, c, kc, (cd >> 4) & 7) == q) {
            if (cd & 128) ax += F3[kc];
            else ap += F3[kc];
        }
        if (!iga) {
            const T finb = F0[kc];
#pragma unroll
            for (int d = 0; d < ND; d++) {
                // q is c's -e_d neighbour: c's in-flux through its low wall
                if (ci(g, sh1(c, d, -1)) == q) ax += pos(V[d][wi(g, d, c)]) * finb;
                // q is c's +e_d neighbour: through its high wall
                if (ci(g, sh1(c, d, 1)) == q) ax += -neg(V[d][wi(g, d, sh1(c, d, 1))]) * finb;
            }
        }
    }
    xb[q] += ax;
    pnb[q] += ap;
    // velocity adjoint of q's low walls (and an open far edge wall): from the
    // wall's right cell (whose low wall it is) and its left cell (high wall)
#pragma unroll
    for (int d = 0; d < ND; d++) {
        const int n = (int)g.n[d];
#pragma unroll
        for (int side = 0; side < 2; side++) {
            if (side == 1 && !(g.bc[d] == BC_OPEN && pq.v[d] == n - 1)) continue;
            I3 w = pq;
            w.v[d] = pq.v[d] + side;                  // the wall, unmapped
            const int64_t kw = wi(g, d, w);
            const T vw = V[d][kw];
            T acc = T(0);
            // right cell: the wall is its low wall
            if (w.v[d] < n || g.bc[d] == BC_PERIODIC) {
                I3 R = w;
                R.v[d] = wrap_cell(w.v[d], n, g.bc[d]);
                const int64_t kR = ci(g, R);
                if (wi(g, d, R) == kw) {
                    const T wm = iga ? T(1) : x[ci(g, sh1(R, d, -1))];
                    const T wc = iga ? T(1) : x[kR];
                    acc += (vw > T(0) ? wm : T(0)) * F0[kR] - (vw < T(0) ? wc : T(0)) * F1[kR];
                }
            }
            // left cell: the wall is its high wall
            if (w.v[d] > 0 || g.bc[d] == BC_PERIODIC) {
                I3 L = w;
                L.v[d] = wrap_cell(w.v[d] - 1, n, g.bc[d]);
                const int64_t kL = ci(g, L);
                if (wi(g, d, sh1(L, d, 1)) == kw) {
                    const T wc = iga ? T(1) : x[kL];
                    const T wp = iga ? T(1) : x[ci(g, sh1(L, d, 1))];
                    acc += (vw > T(0) ? wc : T(0)) * F1[kL] - (vw < T(0) ? wp : T(0)) * F0[kL];
                }
            }
            Vb[d][kw] += acc;
        }
    }
}

// 2-D: the limiter transposes (limited velocities, then coefficients) in
// one launch.  A workgroup owns a tile of LR x LC cells (a thread per cell),
// their low walls and, along an open dimension, the far edge walls of its
// last tile.  Phase 1, for the tile and a ring of one cell: what the cell's
// four walls send its limiter coefficients (the limited-velocity transpose),
// then what those coefficients send on -- to the cells attaining the
// bounds, through the in-flux to the face neighbours, and to the cell's
// walls -- into LDS (the cell's own shares stay in registers).  Phase 2, per
// tile cell: the cell and wall adjoints gathered in a fixed order, written
// once.  Periodic extents are at least 3 (as every plan requires), so the
// face neighbours of a cell are four distinct cells.
constexpr int LR = 8, LC = 64, LT = LR * LC;
constexpr int ER = LR + 2, EC = LC + 2, NE = ER * EC;   // tile + ring of one cell
static_assert(NE - LT <= LT, "the ring takes one more entry per thread at most");

template <typename T, int BC0, int BC1>
__global__ void __launch_bounds__(LT)
k_limiter_adj2g(Geom gg, unsigned opts, const T *__restrict__ psi_n, const T *__restrict__ x,
                const T *__restrict__ V0, const T *__restrict__ V1, const T *__restrict__ bup,
                const T *__restrict__ bdn, const T *__restrict__ Wb0, const T *__restrict__ Wb1,
                const T *__restrict__ G, T *__restrict__ Vb0, T *__restrict__ Vb1,
                T *__restrict__ xb, T *__restrict__ pnb)
{
    const Map2<BC0, BC1> g{(int)gg.n[0], (int)gg.n[1]};
    __shared__ int Ecd[NE];                 // bound codes (as k_beta_adj_a)
    __shared__ T Emx[NE], Emn[NE];          // bound adjoints
    __shared__ T Elo[2][NE], Ehi[2][NE];    // in-flux shares to the -e_d / +e_d neighbour
    __shared__ T Eqh[2][NE];                // share to the high wall of dimension d
    const int n0 = g.n0, n1 = g.n1;
    const int tiles_c = (n1 + LC - 1) / LC;
    const int i0 = (int)(blockIdx.x / tiles_c) * LR, j0 = (int)(blockIdx.x % tiles_c) * LC;
    const int ilim = min(i0 + LR, n0), jlim = min(j0 + LC, n1);
    const bool iga = opts & OPT_IGA;
    const T *V[2] = {V0, V1}, *Wb[2] = {Wb0, Wb1};
    const int tid = threadIdx.x;
    // the own cell's shares: its own-value adjoint, to its low walls, and the
    // limited-velocity adjoint of its low walls and (open) far edge walls
    T own_x = T(0), own_ql[2] = {T(0), T(0)}, own_qh[2] = {T(0), T(0)};
    T own_vb[2][2] = {{T(0), T(0)}, {T(0), T(0)}};
#pragma unroll
    for (int it = 0; it < 2; it++) {
        const int e = tid + it * LT;
        if (e >= NE) break;
        int a, b;   // box position: cell (i0 - 1 + a, j0 - 1 + b)
        if (e < LT) {
            a = 1 + e / LC;
            b = 1 + e % LC;
        } else {
            const int k = e - LT;
            if (k < EC) { a = 0; b = k; }
            else if (k < 2 * EC) { a = ER - 1; b = k - EC; }
            else { a = 1 + (k - 2 * EC) / 2; b = ((k - 2 * EC) & 1) ? EC - 1 : 0; }
        }
        const int idx = a * EC + b;
        const I3 c{{i0 - 1 + a, j0 - 1 + b, 0}};
        bool ok = c.v[0] <= ilim && c.v[1] <= jlim;
        if (BC0 == BC_OPEN) ok = ok && c.v[0] >= 0 && c.v[0] < n0;
        if (BC1 == BC_OPEN) ok = ok && c.v[1] >= 0 && c.v[1] < n1;
        int cd = 0;
        T fmx = T(0), fmn = T(0), plo[2] = {T(0), T(0)}, phi[2] = {T(0), T(0)};
        T ql[2] = {T(0), T(0)}, qh[2] = {T(0), T(0)}, xo = T(0);
        if (ok) {
            const int kc = g.cell(c);
            // limited-velocity transpose: what the cell's walls send bub, bdb
            T su = T(0), sd = T(0), vl[2], vh[2];
#pragma unroll
            for (int d = 0; d < 2; d++)
#pragma unroll
                for (int side = 0; side < 2; side++) {
                    const I3 w = sh1(c, d, side);
                    const int kw = g.wall(d, w), kL = g.cell(sh1(w, d, -1)), kR = g.cell(w);
                    const T wb = Wb[d][kw], v = V[d][kw];
                    const T dL = bdn[kL], uR = bup[kR], uL = bup[kL], dR = bdn[kR];
                    T up = T(1), dn = T(1);
                    int wu = 0, wd = 0;
                    if (dL < up) { up = dL; wu = 1; }
                    if (uR < up) { up = uR; wu = 2; }
                    if (uL < dn) { dn = uL; wd = 1; }
                    if (dR < dn) { dn = dR; wd = 2; }
                    const T vb = ((v > T(0) ? up : T(0)) + (v < T(0) ? dn : T(0))) * wb;
                    const T upb = pos(v) * wb, dnb = neg(v) * wb;
                    if (wb == T(0)) wu = wd = 0;
                    if (kR == kc) {
                        if (wu == 2) su += upb;
                        if (wd == 2) sd += dnb;
                    }
                    if (kL == kc) {
                        if (wu == 1) sd += upb;
                        if (wd == 1) su += dnb;
                    }
                    if (side == 0) {
                        vl[d] = v;
                        if (e < LT) own_vb[d][0] = vb;
                    } else {
                        vh[d] = v;
                        if (e < LT) own_vb[d][1] = vb;
                    }
                }
            // coefficient transpose (as k_beta_adj_a)
            if (su != T(0) || sd != T(0)) {
                T mx = psi_n[kc], mn = mx;
                int amx = 0, amn = 0, smx = 0, smn = 0;
                const T xi = x[kc];
                if (xi > mx) { mx = xi; smx = 1; }
                if (xi < mn) { mn = xi; smn = 1; }
                T xm[2], xp[2];
#pragma unroll
                for (int d = 0; d < 2; d++)
#pragma unroll
                    for (int sg = 0; sg < 2; sg++) {
                        const int kq = g.cell(sh1(c, d, sg ? 1 : -1));
                        const int slot = 1 + 2 * d + sg;
                        const T pa = psi_n[kq], pb = x[kq];
                        if (sg) xp[d] = pb; else xm[d] = pb;
                        if (pa > mx) { mx = pa; amx = slot; smx = 0; }
                        if (pa < mn) { mn = pa; amn = slot; smn = 0; }
                        if (pb > mx) { mx = pb; amx = slot; smx = 1; }
                        if (pb < mn) { mn = pb; amn = slot; smn = 1; }
                    }
                T fin = T(0), fout = T(0);
#pragma unroll
                for (int d = 0; d < 2; d++) {
                    const T wm = iga ? T(1) : xm[d], wp = iga ? T(1) : xp[d];
                    const T wc = iga ? T(1) : xi;
                    fin += pos(vl[d]) * wm - neg(vh[d]) * wp;
                    fout += pos(vh[d]) * wc - neg(vl[d]) * wc;
                }
                const T Gi = G ? G[kc] : T(1);
                T finb = T(0), foutb = T(0);
                if (fin > T(0) && su != T(0)) {
                    const T r = T(1) / fin, gq = Gi * r * su;
                    fmx += gq;
                    xo -= gq;
                    finb -= (mx - xi) * r * gq;
                }
                if (fout > T(0) && sd != T(0)) {
                    const T r = T(1) / fout, gq = Gi * r * sd;
                    xo += gq;
                    fmn -= gq;
                    foutb -= (xi - mn) * r * gq;
                }
#pragma unroll
                for (int d = 0; d < 2; d++) {
                    const T wm = iga ? T(1) : xm[d], wp = iga ? T(1) : xp[d];
                    const T wc = iga ? T(1) : xi;
                    ql[d] = (vl[d] > T(0) ? wm : T(0)) * finb - (vl[d] < T(0) ? wc : T(0)) * foutb;
                    qh[d] = (vh[d] > T(0) ? wc : T(0)) * foutb - (vh[d] < T(0) ? wp : T(0)) * finb;
                    if (!iga) {
                        plo[d] = pos(vl[d]) * finb;
                        phi[d] = -neg(vh[d]) * finb;
                        xo += (pos(vh[d]) - neg(vl[d])) * foutb;
                    }
                }
                cd = amx | (smx << 3) | (amn << 4) | (smn << 7);
            }
        }
        Ecd[idx] = cd;
        Emx[idx] = fmx;
        Emn[idx] = fmn;
#pragma unroll
        for (int d = 0; d < 2; d++) {
            Elo[d][idx] = plo[d];
            Ehi[d][idx] = phi[d];
            Eqh[d][idx] = qh[d];
        }
        if (e < LT) {
            own_x = xo;
#pragma unroll
            for (int d = 0; d < 2; d++) {
                own_ql[d] = ql[d];
                own_qh[d] = qh[d];
            }
        }
    }
    __syncthreads();
    const int a = 1 + tid / LC, b = 1 + tid % LC;
    const I3 q{{i0 - 1 + a, j0 - 1 + b, 0}};
    if (q.v[0] >= n0 || q.v[1] >= n1) return;
    const int kq = g.cell(q);
    const int iq = a * EC + b;
    const int nn[2] = {n0, n1};
    const bool op[2] = {BC0 == BC_OPEN, BC1 == BC_OPEN};
    T ax = own_x, ap = T(0);
    // Away from an open edge the boundary map sends no neighbour of a
    // neighbour onto the cell (periodic extents are at least 3), so a bound
    // slot of neighbour k points at the cell exactly when it is the slot
    // back along k's offset; at an open edge the clamped positions are
    // compared.
    const bool edge = (op[0] && (q.v[0] == 0 || q.v[0] == n0 - 1)) ||
                      (op[1] && (q.v[1] == 0 || q.v[1] == n1 - 1));
    // bounds: the cell itself, then its face neighbours (-e0, +e0, -e1, +e1)
#pragma unroll
    for (int k = 0; k < 5; k++) {
        I3 c = q;
        int ic = iq;
        if (k > 0) {
            const int d = (k - 1) >> 1, sg = ((k - 1) & 1) ? 1 : -1;
            c = sh1(q, d, sg);
            if (op[d] && (c.v[d] < 0 || c.v[d] >= nn[d])) continue;
            ic = iq + (d == 0 ? sg * EC : sg);
        }
        const int cd = Ecd[ic];
        const int smx = cd & 7, smn = (cd >> 4) & 7;
        // slot back to the cell from neighbour k: 0, then +e0, -e0, +e1, -e1
        constexpr int back[5] = {0, 2, 1, 4, 3};
        // the cell a bound slot of c points at (selects: no indexing of c by a
        // run-time dimension)
        auto target = [&](int slot) {
            if (!edge) return slot == back[k];
            const int ti = c.v[0] + (slot == 1 ? -1 : (slot == 2 ? 1 : 0));
            const int tj = c.v[1] + (slot == 3 ? -1 : (slot == 4 ? 1 : 0));
            return g.cell(I3{{ti, tj, 0}}) == kq;
        };
        if (target(smx)) {
            if (cd & 8) ax += Emx[ic];
            else ap += Emx[ic];
        }
        if (target(smn)) {
            if (cd & 128) ax += Emn[ic];
            else ap += Emn[ic];
        }
    }
    // in-flux: the +e_d neighbour's share to its -e_d side, the -e_d
    // neighbour's to its +e_d side; at an open edge the cell's own share
    // beyond the edge comes back to it
#pragma unroll
    for (int d = 0; d < 2; d++) {
        const int st = d == 0 ? EC : 1;
        if (!op[d] || q.v[d] < nn[d] - 1) ax += Elo[d][iq + st];
        if (!op[d] || q.v[d] > 0) ax += Ehi[d][iq - st];
        if (op[d] && q.v[d] == 0) ax += Elo[d][iq];
        if (op[d] && q.v[d] == nn[d] - 1) ax += Ehi[d][iq];
    }
    xb[kq] += ax;
    pnb[kq] += ap;
    // velocity adjoints of the owned walls: the limited-velocity share, the
    // cell's share to its low wall and the -e_d neighbour's to its high wall
    T *Vb[2] = {Vb0, Vb1};
#pragma unroll
    for (int d = 0; d < 2; d++) {
        const int st = d == 0 ? EC : 1;
        T v = own_vb[d][0] + own_ql[d];
        if (!op[d] || q.v[d] > 0) v += Eqh[d][iq - st];
        Vb[d][g.wall(d, q)] = v;
        if (op[d] && q.v[d] == nn[d] - 1) Vb[d][g.wall(d, sh1(q, d, 1))] = own_vb[d][1] + own_qh[d];
    }
}

// Run f with the dimension count (and a wall dimension) as compile-time
// constants.
template <typename F> void with_nd(int nd, F f)
{
    if (nd == 1)
        f(std::integral_constant<int, 1>{});
    else if (nd == 2)
        f(std::integral_constant<int, 2>{});
    else
        f(std::integral_constant<int, 3>{});
}

template <typename F> void with_nd_d(int nd, int d, F f)
{
    using N1 = std::integral_constant<int, 1>;
    using N2 = std::integral_constant<int, 2>;
    using N3 = std::integral_constant<int, 3>;
    using D0 = std::integral_constant<int, 0>;
    using D1 = std::integral_constant<int, 1>;
    using D2 = std::integral_constant<int, 2>;
    if (nd == 1)
        f(N1{}, D0{});
    else if (nd == 2) {
        if (d == 0) f(N2{}, D0{}); else f(N2{}, D1{});
    } else {
        if (d == 0) f(N3{}, D0{}); else if (d == 1) f(N3{}, D1{}); else f(N3{}, D2{});
    }
}

// true if the 2-D donor transpose (with its write modes) applies
bool fast_donor_adj(const Geom &g, const void *G)
{
    return g.nd == 2 && !G && g.n[0] * g.n[1] < ((int64_t)1 << 31);
}

// transpose of a donor-cell pass: xb += (dy/dx)^T yb, cb_d += (dy/dc_d)^T yb;
// the 2-D kernel (fast_donor_adj) writes xb (= ... + xadd), and with
// write_walls the wall adjoints, instead of adding
// (2-D kernel only: zero[] cell fields are set to zero, see k_donor_adj2d)
template <typename T>
void donor_adj(const Geom &g, const T *x, const T *const c[3], const T *G, int flux_is_vel,
               const T *yb, T *xb, T *const cb[3], hipStream_t s, bool write_walls = false,
               const T *xadd = nullptr, T *const *zero = nullptr)
{
    const int64_t N = g.n[0] * g.n[1] * g.n[2];
    if (fast_donor_adj(g, G)) {
        const int bpr = (int)cdiv(g.n[1], B);
        auto go = [&](auto kern) {
            kern<<<(unsigned)(bpr * cdiv(g.n[0], DR)), B, 0, s>>>(
                (int)g.n[0], (int)g.n[1], g.bc[0], g.bc[1], bpr, flux_is_vel, x, c[0], c[1], yb,
                xadd, xb, cb[0], cb[1], zero ? zero[0] : nullptr, zero ? zero[1] : nullptr,
                zero ? zero[2] : nullptr);
        };
        if (xadd) go(write_walls ? k_donor_adj2d<T, true, true> : k_donor_adj2d<T, true, false>);
        else go(write_walls ? k_donor_adj2d<T, false, true> : k_donor_adj2d<T, false, false>);
        return;
    }
    with_nd(g.nd, [&](auto ND) {
        k_donor_adj_cells<T, decltype(ND)::value><<<(unsigned)cdiv(N, B), B, 0, s>>>(
            g, c[0], c[1], c[2], G, flux_is_vel, yb, xb);
    });
    for (int d = 0; d < g.nd; d++) {
        int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
        e[d] += 1;
        const int64_t M = e[0] * e[1] * e[2];
        with_nd_d(g.nd, d, [&](auto ND, auto WD) {
            k_donor_adj_walls<T, decltype(ND)::value, decltype(WD)::value>
                <<<(unsigned)cdiv(M, B), B, 0, s>>>(g, x, c[d], G, flux_is_vel, yb, cb[d]);
        });
    }
}

int64_t ncells(const Geom &g);
int64_t nwalls(const Geom &g, int d);

// the deterministic transpose of every other case (see k_pseudo_adj_slots):
// slots of every wall dimension, then the gathers; S / U / Q: per wall
// dimension, pseudo_slots<nd>() / 1 / nd - 1 wall fields of workspace
template <typename T>
void pseudo_adj_slots_launch(const Geom &g, hipStream_t s, unsigned opts, const T *x,
                             const T *const c[3], const T *G, T *const Vb[3], T *xb,
                             T *const cb[3], T *const S[3], T *const U[3], T *const Q[3])
{
    with_nd(g.nd, [&](auto ND) {
        constexpr int nd = decltype(ND)::value;
        for (int d = 0; d < nd; d++) {
            const unsigned wb = (unsigned)cdiv(nwalls(g, d), B);
            with_nd_d(nd, d, [&](auto ND2, auto WD) {
                k_pseudo_adj_slots<T, decltype(ND2)::value, decltype(WD)::value>
                    <<<wb, B, 0, s>>>(g, opts, x, c[0], c[1], c[2], G, Vb[d], S[d], U[d], Q[d]);
            });
        }
        const unsigned cbk = (unsigned)cdiv(ncells(g), B);
        k_pseudo_gather_cells<T, nd><<<cbk, B, 0, s>>>(g, S[0], S[1], S[2], xb);
        for (int o = 0; o < nd; o++) {
            const unsigned wb = (unsigned)cdiv(nwalls(g, o), B);
            with_nd_d(nd, o, [&](auto ND2, auto WO) {
                k_pseudo_gather_walls<T, decltype(ND2)::value, decltype(WO)::value>
                    <<<wb, B, 0, s>>>(g, U[o], Q[0], Q[1], Q[2], cb[o]);
            });
        }
    });
}

// 2-D without third-order terms: both wall dimensions in one launch
// (periodic extents of at least 3: the tiled kernels' boundary map wraps
// once)
bool tiled2_extents(const Geom &g)
{
    for (int d = 0; d < 2; d++)
        if (g.bc[d] == BC_PERIODIC && g.n[d] < 3) return false;
    return (g.n[0] + 1) * (g.n[1] + 1) < ((int64_t)1 << 31);
}

bool pseudo_adj_both(const Geom &g, unsigned opts)
{
    return g.nd == 2 && !(opts & OPT_TOT) && tiled2_extents(g);
}

template <typename T>
void pseudo_adj2_launch(const Geom &g, hipStream_t s, unsigned opts, const T *x, const T *c0,
                        const T *c1, const T *G, const T *Vb0, const T *Vb1, T *xb, T *cb0,
                        T *cb1)
{
    const unsigned tb = (unsigned)(cdiv(g.n[0], GR) * cdiv(g.n[1], GC));
#define MP_K(B0, B1) \
    k_pseudo_adj2g<T, B0, B1><<<tb, GT, 0, s>>>(g, opts, x, c0, c1, G, Vb0, Vb1, xb, cb0, cb1)
    const bool p0 = g.bc[0] == BC_PERIODIC, p1 = g.bc[1] == BC_PERIODIC;
    if (p0 && p1) MP_K(BC_PERIODIC, BC_PERIODIC);
    else if (p0) MP_K(BC_PERIODIC, BC_OPEN);
    else if (p1) MP_K(BC_OPEN, BC_PERIODIC);
    else MP_K(BC_OPEN, BC_OPEN);
#undef MP_K
}

// true if the 2-D one-launch limiter transpose applies
bool limiter_adj_tiled(const Geom &g)
{
    return g.nd == 2 && tiled2_extents(g);
}

// transposes of the limiter (limited velocities, then coefficients), each
// entry gathered by one thread in a fixed order (bub, bdb, F, code: the
// three-kernel path's intermediates, unused by the 2-D one-launch kernel)
template <typename T>
void limiter_adj(const Geom &g, unsigned opts, hipStream_t s, const T *psi_n, const T *x,
                 const T *const V[3], const T *bup, const T *bdn, const T *const Wb[3],
                 const T *G, T *bub, T *bdb, T *const F[5], int *code, T *xb, T *pnb,
                 T *const Vb[3])
{
    if (limiter_adj_tiled(g)) {
        const unsigned tb = (unsigned)(cdiv(g.n[0], LR) * cdiv(g.n[1], LC));
#define MP_L(B0, B1)                                                                          \
    k_limiter_adj2g<T, B0, B1><<<tb, LT, 0, s>>>(g, opts, psi_n, x, V[0], V[1], bup, bdn, Wb[0], \
                                                 Wb[1], G, Vb[0], Vb[1], xb, pnb)
        const bool p0 = g.bc[0] == BC_PERIODIC, p1 = g.bc[1] == BC_PERIODIC;
        if (p0 && p1) MP_L(BC_PERIODIC, BC_PERIODIC);
        else if (p0) MP_L(BC_PERIODIC, BC_OPEN);
        else if (p1) MP_L(BC_OPEN, BC_PERIODIC);
        else MP_L(BC_OPEN, BC_OPEN);
#undef MP_L
        return;
    }
    const unsigned cb = (unsigned)cdiv(g.n[0] * g.n[1] * g.n[2], B);
    with_nd(g.nd, [&](auto ND) {
        constexpr int nd = decltype(ND)::value;
        k_limit_adj_gather<T, nd><<<cb, B, 0, s>>>(g, V[0], V[1], V[2], bup, bdn, Wb[0], Wb[1],
                                                   Wb[2], Vb[0], Vb[1], Vb[2], bub, bdb);
        k_beta_adj_a<T, nd><<<cb, B, 0, s>>>(g, opts, psi_n, x, V[0], V[1], V[2], G, bub, bdb,
                                             F[0], F[1], F[2], F[3], F[4], code);
        k_beta_adj_b<T, nd><<<cb, B, 0, s>>>(g, opts, x, V[0], V[1], V[2], F[0], F[1], F[2],
                                             F[3], F[4], code, xb, pnb, Vb[0], Vb[1], Vb[2]);
    });
}

int64_t ncells(const Geom &g) { return g.n[0] * g.n[1] * g.n[2]; }

int64_t nwalls(const Geom &g, int d)
{
    int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
    e[d] += 1;
    return e[0] * e[1] * e[2];
}

size_t up256(size_t v) { return (v + 255) / 256 * 256; }

// workspace carving for the adjoint (shared by sizing and use).  The pass
// records (X, V, W, bu, bd) are kept for every step of a segment: slot k
// holds step s0 + k's, at a fixed stride from slot 0; select(k) points the
// record pointers at slot k.
template <typename T> struct AdjWs {
    T *ck;          // checkpoints
    T *seg;         // states of one segment
    T *X[8];        // pass inputs 1..n_iters-1 (X[0] is the state itself)
    T *V[8][3];     // raw pseudo-velocities of passes 2..n
    T *W[8][3];     // limited pseudo-velocities (== V without the limiter)
    T *bu[8], *bd[8];
    T *yb, *xb, *pnb, *bub, *bdb;
    T *F[5];        // limiter-coefficient transpose, per cell (k_beta_adj_a)
    int *code;      // which cells attain the bounds (k_beta_adj_a)
    T *Ab[3], *Vb[3], *Cb[3];
    T *PS[3], *PU[3], *PQ[3];   // pseudo-velocity transpose slots (not the 2-D tiled path)
    T *tmp;         // output of a recomputed step
    size_t bytes;
    // slot 0 of the records and the distance between slots (elements)
    T *X0[8], *V0[8][3], *W0[8][3], *bu0[8], *bd0[8];
    size_t rec_stride;
    int nslots;

    void select(int k)
    {
        auto at = [&](T *b) -> T * { return b ? b + (size_t)k * rec_stride : nullptr; };
        for (int p = 0; p < 8; p++) {
            X[p] = at(X0[p]);
            bu[p] = at(bu0[p]);
            bd[p] = at(bd0[p]);
            for (int d = 0; d < 3; d++) {
                V[p][d] = at(V0[p][d]);
                W[p][d] = at(W0[p][d]);
            }
        }
    }
};

template <typename T>
AdjWs<T> carve_adj(const Geom &g, int n_iters, bool fct, int n_steps, int ckpt, char *base,
                   bool slots)
{
    AdjWs<T> w;
    size_t off = 0;
    auto take = [&](size_t n) -> T * {
        T *p = base ? (T *)(base + off) : nullptr;
        off += up256(n * sizeof(T));
        return p;
    };
    int64_t N = ncells(g);
    int nck = (n_steps + ckpt - 1) / ckpt;
    w.ck = take((size_t)N * nck);
    w.seg = take((size_t)N * ckpt);
    for (int p = 0; p < 8; p++) {
        w.X0[p] = nullptr;
        w.bu0[p] = w.bd0[p] = nullptr;
        for (int d = 0; d < 3; d++) w.V0[p][d] = w.W0[p][d] = nullptr;
    }
    const size_t rec_begin = off;
    for (int p = 1; p < n_iters; p++) {
        w.X0[p] = take(N);
        for (int d = 0; d < g.nd; d++) {
            w.V0[p][d] = take(nwalls(g, d));
            w.W0[p][d] = fct ? take(nwalls(g, d)) : w.V0[p][d];
        }
        if (fct) {
            w.bu0[p] = take(N);
            w.bd0[p] = take(N);
        }
    }
    // every take is a multiple of 256 bytes, hence of sizeof(T)
    w.rec_stride = (off - rec_begin) / sizeof(T);
    w.nslots = ckpt < n_steps ? ckpt : (n_steps > 0 ? n_steps : 1);
    off += (off - rec_begin) * (size_t)(w.nslots - 1);
    w.select(0);
    w.yb = take(N);
    w.xb = take(N);
    w.pnb = take(N);
    w.bub = take(N);
    w.bdb = take(N);
    const bool staged_lim = fct && !limiter_adj_tiled(g);
    for (int k = 0; k < 5; k++) w.F[k] = staged_lim ? take(N) : nullptr;
    // N ints, in whole T
    w.code = staged_lim ? (int *)take((size_t)(N * sizeof(int) + sizeof(T) - 1) / sizeof(T))
                        : nullptr;
    w.tmp = take(N);
    for (int d = 0; d < 3; d++) w.Ab[d] = w.Vb[d] = w.Cb[d] = nullptr;
    for (int d = 0; d < g.nd; d++) {
        w.Ab[d] = take(nwalls(g, d));
        w.Vb[d] = take(nwalls(g, d));
        w.Cb[d] = take(nwalls(g, d));
    }
    const int ns = g.nd == 1 ? pseudo_slots<1>() : (g.nd == 2 ? pseudo_slots<2>() : pseudo_slots<3>());
    for (int d = 0; d < 3; d++) {
        w.PS[d] = w.PU[d] = w.PQ[d] = nullptr;
        if (slots && d < g.nd) {
            w.PS[d] = take((size_t)ns * nwalls(g, d));
            w.PU[d] = take(nwalls(g, d));
            if (g.nd > 1) w.PQ[d] = take((size_t)(g.nd - 1) * nwalls(g, d));
        }
    }
    w.bytes = off;
    return w;
}

template <typename T> hipError_t fill(T *a, int64_t n, hipStream_t s)
{
    k_fill<T><<<(unsigned)cdiv(n, B), B, 0, s>>>(a, n, T(0));
    return hipGetLastError();
}

template <typename T> void clear_n(const Bufs<T> &f, hipStream_t s)
{
    if (f.k) k_clear_n<T><<<(unsigned)cdiv(f.nmax, B), B, 0, s>>>(f);
}

// forward recompute of one step from psi_n, keeping the pass records;
// writes the step's result to out when out != nullptr
template <typename T>
hipError_t record_step(const AdjArgs<T> &a, AdjWs<T> &w, const T *psi_n, T *out, hipStream_t s)
{
    const Geom &g = a.g;
    const bool fct = a.opts & OPT_FCT, iga = a.opts & OPT_IGA;
    const int n = a.n_iters;
    hipError_t e;
    const int km = (a.opts & OPT_KAHAN) ? 2 : 0;   // Kahan-compensated donor update
    T *first = n > 1 ? w.X[1] : out;
    // (the separate 2-D donor launch of n_iters = 1 takes G = 1 only)
    if (pass2d_supported(g.nd, n > 1 ? n : 2, a.opts, a.G != nullptr, g.n) && (n > 1 || !a.G)) {
        // 2-D: one launch per corrective pass that also writes the records
        // (raw and limited velocities, coefficients); the first folds the
        // donor pass in and keeps its result as the pass input record
        if (n == 1 && first) {
            e = donor2d_launch<T>(g, a.opts, psi_n, a.c[0], a.c[1], first, nullptr, s);
            if (e != hipSuccess) return e;
        }
        for (int it = 2; it <= n; it++) {
            const bool donor = it == 2;
            const T *x = donor ? psi_n : w.X[it - 1];
            const T *c0 = it == 2 ? a.c[0] : w.W[it - 2][0];
            const T *c1 = it == 2 ? a.c[1] : w.W[it - 2][1];
            PassRecord<T> rec;
            if (fct) {
                rec.v0 = w.V[it - 1][0];
                rec.v1 = w.V[it - 1][1];
                rec.bu = w.bu[it - 1];
                rec.bd = w.bd[it - 1];
            }
            if (donor) rec.xd = w.X[1];
            T *y = (it < n) ? w.X[it] : out;
            e = pass2d_launch<T>(g, a.opts, x, c0, c1, donor ? nullptr : psi_n, a.G, y,
                                 w.W[it - 1][0], w.W[it - 1][1], s, rec);
            if (e != hipSuccess) return e;
        }
        return hipGetLastError();
    }
    if (first) {
        e = launch_donor<T>(g, psi_n, a.c, a.G, km, first, s);
        if (e != hipSuccess) return e;
    }
    for (int it = 2; it <= n; it++) {
        const T *x = w.X[it - 1];
        // advector of the previous pass: the input one for pass 2
        const T *cin[3];
        for (int d = 0; d < 3; d++) cin[d] = (it == 2) ? a.c[d] : w.W[it - 2][d];
        T *V[3] = {w.V[it - 1][0], w.V[it - 1][1], w.V[it - 1][2]};
        T *W[3] = {w.W[it - 1][0], w.W[it - 1][1], w.W[it - 1][2]};
        e = launch_pseudo<T>(g, a.opts, x, cin, a.G, V, s);
        if (e != hipSuccess) return e;
        if (fct) {
            e = launch_fct<T>(g, a.opts, psi_n, x, V, a.G, w.bu[it - 1], w.bd[it - 1], W, s);
            if (e != hipSuccess) return e;
        }
        T *y = (it < n) ? w.X[it] : out;
        if (y) {
            e = launch_donor<T>(g, x, W, a.G, (iga ? 1 : 0) | km, y, s);
            if (e != hipSuccess) return e;
        }
    }
    return hipGetLastError();
}

// reverse of one step from its pass records (the selected slot of w, written
// by record_step from the same psi_n): w.yb = dJ/dpsi_{n+1} on entry,
// dJ/dpsi_n on exit; w.Cb accumulates dJ/dc
template <typename T>
hipError_t reverse_step(const AdjArgs<T> &a, AdjWs<T> &w, const T *psi_n, hipStream_t s)
{
    const Geom &g = a.g;
    const bool fct = a.opts & OPT_FCT, iga = a.opts & OPT_IGA;
    const int n = a.n_iters;
    const int64_t N = ncells(g);
    const unsigned cb = (unsigned)cdiv(N, B);
    hipError_t e = hipSuccess;
    // Buffers whose first writer in a pass assigns need no clearing: the
    // 2-D donor transpose writes xb (and, in the last pass, the advector
    // adjoint); the limiter transpose writes Vb.  The entries of a periodic
    // dimension's wall n are never written and stay zero from adjoint_run.
    // With the 2-D donor transpose, the accumulators the later kernels of a
    // pass scatter into (the limiter coefficients' adjoints, and in the
    // first reversed pass the psi^n adjoint) are zeroed by that pass's donor
    // transpose, which runs before them and reads none of them.
    const bool fast = fast_donor_adj(g, a.G);
    if (!fast) {
        Bufs<T> f;
        f.push(w.pnb, N);
        for (int d = 0; d < g.nd; d++) f.push(w.Ab[d], nwalls(g, d));
        clear_n<T>(f, s);
    }
    for (int it = n; it >= 2; it--) {
        const T *x = w.X[it - 1];
        if (!fast) {
            Bufs<T> f;
            f.push(w.xb, N);
            clear_n<T>(f, s);
        }
        // corrective donor-cell pass
        {
            const T *Wc[3] = {w.W[it - 1][0], w.W[it - 1][1], w.W[it - 1][2]};
            T *const zero[3] = {it == n ? w.pnb : nullptr, nullptr, nullptr};
            donor_adj<T>(g, x, Wc, a.G, iga ? 1 : 0, w.yb, w.xb, w.Ab, s, fast && it == n, nullptr,
                         fast ? zero : nullptr);
        }
        // limiter
        if (fct) {
            const T *V[3] = {w.V[it - 1][0], w.V[it - 1][1], w.V[it - 1][2]};
            const T *Wb[3] = {w.Ab[0], w.Ab[1], w.Ab[2]};
            limiter_adj<T>(g, a.opts, s, psi_n, x, V, w.bu[it - 1], w.bd[it - 1], Wb, a.G,
                           w.bub, w.bdb, w.F, w.code, w.xb, w.pnb, w.Vb);
        } else {
            for (int d = 0; d < g.nd; d++)
                k_copy<T><<<(unsigned)cdiv(nwalls(g, d), B), B, 0, s>>>(w.Vb[d], w.Ab[d],
                                                                        nwalls(g, d));
        }
        // pseudo-velocity: to x and to the previous pass's advector (the
        // first corrective pass reads the input advector: straight into
        // its gradient)
        T *const *tgt = (it == 2) ? w.Cb : w.Ab;
        if (it > 2) {
            Bufs<T> f;
            for (int d = 0; d < g.nd; d++) f.push(w.Ab[d], nwalls(g, d));
            clear_n<T>(f, s);
        }
        const T *cin[3];
        for (int d = 0; d < 3; d++) cin[d] = (it == 2) ? a.c[d] : w.W[it - 2][d];
        if (pseudo_adj_both(g, a.opts))
            pseudo_adj2_launch<T>(g, s, a.opts, x, cin[0], cin[1], a.G, w.Vb[0], w.Vb[1], w.xb,
                                  tgt[0], tgt[1]);
        else
            pseudo_adj_slots_launch<T>(g, s, a.opts, x, cin, a.G, w.Vb, w.xb, tgt, w.PS, w.PU,
                                       w.PQ);
        T *t = w.yb;
        w.yb = w.xb;
        w.xb = t;
    }
    // donor-cell pass of the input field with the input advector, plus the
    // limiter's direct dependence on psi^n
    if (fast) {
        // (pnb was zeroed by the first reversed pass; with no corrective
        // pass there is nothing to add)
        donor_adj<T>(g, psi_n, a.c, a.G, 0, w.yb, w.xb, w.Cb, s, false,
                     n >= 2 ? w.pnb : nullptr);
    } else {
        e = fill<T>(w.xb, N, s);
        donor_adj<T>(g, psi_n, a.c, a.G, 0, w.yb, w.xb, w.Cb, s);
        k_add<T><<<cb, B, 0, s>>>(w.xb, w.pnb, N);
    }
    T *t = w.yb;
    w.yb = w.xb;
    w.xb = t;
    (void)e;
    return hipGetLastError();
}

}  // namespace

size_t adj_extra_bytes(const Geom &g, size_t es, int n_iters, unsigned opts, int n_steps,
                       int ckpt_every)
{
    // FCT on/off changes the layout; size for the larger one
    const bool slots = !pseudo_adj_both(g, opts);
    if (es == 8)
        return carve_adj<double>(g, n_iters, true, n_steps, ckpt_every, nullptr, slots).bytes;
    return carve_adj<float>(g, n_iters, true, n_steps, ckpt_every, nullptr, slots).bytes;
}

template <typename T> hipError_t adjoint_run(const AdjArgs<T> &a, hipStream_t s)
{
    const Geom &g = a.g;
    const int64_t N = ncells(g);
    const size_t nb = (size_t)N * sizeof(T);
    AdjWs<T> w = carve_adj<T>(g, a.n_iters, (a.opts & OPT_FCT) != 0, a.n_steps, a.ckpt_every,
                              a.ws, !pseudo_adj_both(g, a.opts));
    hipError_t e;
    // forward sweep: checkpoint at the start of every segment
    const int ck = a.ckpt_every;
    const int nck = (a.n_steps + ck - 1) / ck;
    T *cur = w.seg, *nxt = w.tmp;
    e = hipMemcpyAsync(cur, a.psi0, nb, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
    for (int st = 0; st < a.n_steps; st++) {
        TraceRange tr("adjoint forward step");
        if (st % ck == 0) {
            e = hipMemcpyAsync(w.ck + (size_t)(st / ck) * N, cur, nb, hipMemcpyDeviceToDevice, s);
            if (e != hipSuccess) return e;
        }
        if (st == (nck - 1) * ck) break;   // the last segment's states are recorded below
        e = a.plain_step ? a.plain_step(a.plain_ctx, cur, nxt) : record_step<T>(a, w, cur, nxt, s);
        if (e != hipSuccess) return e;
        T *t = cur;
        cur = nxt;
        nxt = t;
    }
    for (int d = 0; d < g.nd; d++) {
        e = fill<T>(w.Cb[d], nwalls(g, d), s);
        if (e == hipSuccess) e = fill<T>(w.Ab[d], nwalls(g, d), s);
        if (e == hipSuccess) e = fill<T>(w.Vb[d], nwalls(g, d), s);
        if (e != hipSuccess) return e;
    }
    e = hipMemcpyAsync(w.yb, a.lambda_T, nb, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
    // reverse sweep over segments
    for (int sg = nck - 1; sg >= 0; sg--) {
        TraceRange tr("adjoint reverse segment");
        int s0 = sg * ck;
        int s1 = s0 + ck < a.n_steps ? s0 + ck : a.n_steps;
        e = hipMemcpyAsync(w.seg, w.ck + (size_t)sg * N, nb, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
        // recompute the segment, keeping every step's pass records (the
        // recording launches also produce the next state)
        for (int st = s0; st < s1; st++) {
            const T *in = w.seg + (size_t)(st - s0) * N;
            T *out = st < s1 - 1 ? w.seg + (size_t)(st - s0 + 1) * N : nullptr;
            w.select(st - s0);
            e = record_step<T>(a, w, in, out, s);
            if (e != hipSuccess) return e;
        }
        for (int st = s1 - 1; st >= s0; st--) {
            w.select(st - s0);
            e = reverse_step<T>(a, w, w.seg + (size_t)(st - s0) * N, s);
            if (e != hipSuccess) return e;
        }
    }
    e = hipMemcpyAsync(a.grad_psi0, w.yb, nb, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
    for (int d = 0; d < g.nd; d++) {
        e = hipMemcpyAsync(a.grad_c[d], w.Cb[d], nwalls(g, d) * sizeof(T),
                           hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

template hipError_t adjoint_run<float>(const AdjArgs<float> &, hipStream_t);
template hipError_t adjoint_run<double>(const AdjArgs<double> &, hipStream_t);

}  // namespace mp
