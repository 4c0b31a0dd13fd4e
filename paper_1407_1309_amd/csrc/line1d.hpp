// line1d.hpp -- 1-D MPDATA steps, many per launch (kernel template and its
// launchers; resident1d.hip and resident1d_f32.hip instantiate them).
//
// Design (gfx950, wave64).  A 1-D step is far too little work per cell for a
// launch, or a barrier, per stage: what bounds it is the chain of dependent
// operations and the waits between them.
//   * A lane holds K consecutive cells in registers and a wave 64 K of them;
//     every stage of every pass of a step (donor-cell fluxes, pseudo-velocity,
//     limiter, corrective fluxes) runs in registers, neighbours inside the
//     lane by name and across lanes by DPP wave shifts.  The outer hl lanes
//     of a wave on each side are a halo, recomputed, of at least the step's
//     dependency radius.
//   * Between steps each wave writes the cells it owns to LDS and reads its
//     cells and halo back through the boundary map: one barrier per step
//     (two buffers in turn).
//   * A grid that fits one workgroup of up to 16 waves runs all steps of a
//     call in one launch.  A longer grid is cut into tiles, one workgroup
//     each, with a halo of (steps x radius) cells recomputed, so one launch
//     still makes many steps and reads and writes memory once.
// Boundaries: the LDS reads (and the loads of psi, the advector and G) go
// through the boundary map, so halo cells hold mapped values at the start of
// a step; under periodic boundaries recomputing them is exact.  Under open
// ones a cell outside the domain is, at every stage, a copy of the edge
// cell (a wall, of the edge wall): copied across lanes (readlane) in the
// waves that hold the edge.
// Measured, us per call, against the kernel that kept every stage in LDS
// (about eight barriers a step) and, for the long grid, five launches a step:
// 500 cells FP64, 100 steps 151 -> 40; the 1001-cell oscillator pair, iga +
// fct, 100 steps 812 -> 239; 1000003 cells, fct, 20 steps 713 -> 73.  What is
// left is the chain of one step (0.4 us) or, with full SIMDs, the issue of
// its FP64 operations, the divisions above all.
// Multiply-add contraction is off and divisions are IEEE, so every value is
// the rounded result of the same operations in the same order whatever the
// tiling, K, or steps per launch: the bits do not depend on them.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

#include <type_traits>

#pragma clang fp contract(off)

namespace mp {
namespace {

constexpr int WAVE = 64;

__device__ inline int lane_from_left(int v) { return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true); }
__device__ inline int lane_from_right(int v) { return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true); }
__device__ inline float from_left(float v) { return __int_as_float(lane_from_left(__float_as_int(v))); }
__device__ inline float from_right(float v) { return __int_as_float(lane_from_right(__float_as_int(v))); }
__device__ inline double from_left(double v)
{
    return __hiloint2double(lane_from_left(__double2hiint(v)), lane_from_left(__double2loint(v)));
}
__device__ inline double from_right(double v)
{
    return __hiloint2double(lane_from_right(__double2hiint(v)), lane_from_right(__double2loint(v)));
}
__device__ inline float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ inline double lane_value(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// value of the cell k - 1 / k + 1 of a lane's K cells (l, r: the neighbour
// lanes' last and first cell)
template <int K, typename T> __device__ __forceinline__ T lo(const T (&a)[K], int k, T l)
{
    return k > 0 ? a[k > 0 ? k - 1 : 0] : l;
}
template <int K, typename T> __device__ __forceinline__ T hi(const T (&a)[K], int k, T r)
{
    return k < K - 1 ? a[k < K - 1 ? k + 1 : K - 1] : r;
}

// Positions of the cells of a lane relative to the edges of an open domain,
// and the copies of the edge value across a wave.
struct Edges {
    bool lo, hi, whi;        // wave-uniform: the wave holds cell 0 / cell n-1 / wall n
    int l_lo, l_hi, s_hi;    // lane of cell 0; lane and slot of cell n-1
    int l_w, s_w;            // lane and slot of wall n
    int first, last;         // the lane's first cell position; position of cell n-1

    template <int K, typename T> __device__ __forceinline__ void cells(T (&a)[K], int lane) const
    {
        if (lo) {
            const T e = lane_value(a[0], l_lo);
#pragma unroll
            for (int k = 0; k < K; k++) a[k] = lane < l_lo ? e : a[k];
        }
        if (hi) high(a, l_hi, s_hi, last);
    }
    template <int K, typename T> __device__ __forceinline__ void walls(T (&a)[K], int lane) const
    {
        if (lo) {
            const T e = lane_value(a[0], l_lo);
#pragma unroll
            for (int k = 0; k < K; k++) a[k] = lane < l_lo ? e : a[k];
        }
        if (whi) high(a, l_w, s_w, last + 1);
    }
    template <int K, typename T>
    __device__ __forceinline__ void high(T (&a)[K], int l, int s, int pos) const
    {
        T e = lane_value(a[0], l);
#pragma unroll
        for (int k = 1; k < K; k++) {
            const T v = lane_value(a[k], l);
            e = s == k ? v : e;
        }
#pragma unroll
        for (int k = 0; k < K; k++) a[k] = first + k > pos ? e : a[k];
    }
};

// Options of a step: compile-time in the plain instances (limiter and gauge
// only), read from `opts` in the general one.
template <bool GEN, bool FCT, bool IGA> struct LineOpts {
    unsigned o;
    bool g;
    __device__ __forceinline__ bool fct() const { return GEN ? (o & OPT_FCT) != 0 : FCT; }
    __device__ __forceinline__ bool iga() const { return GEN ? (o & OPT_IGA) != 0 : IGA; }
    __device__ __forceinline__ bool tot() const { return GEN && (o & OPT_TOT); }
    __device__ __forceinline__ bool absf() const { return GEN && (o & OPT_ABS); }
    __device__ __forceinline__ bool dfl() const { return GEN && (o & OPT_DFL); }
    __device__ __forceinline__ bool kahan() const { return GEN && (o & OPT_KAHAN); }
    __device__ __forceinline__ bool has_g() const { return GEN && g; }
};

template <typename T> __device__ __forceinline__ T line_frac(bool iga, T num, T den, T m)
{
    if (iga) return num / m;
    return den == T(0) ? T(0) : num / den;
}

template <typename T, typename O> __device__ __forceinline__ T line_update(const O &o, T x, T acc, T g)
{
    if (o.has_g()) acc = acc / g;
    if (o.kahan()) {
        T s = x, c = T(0);
        kahan_add(s, c, -acc);
        return s;
    }
    return x - acc;
}

// One MPDATA step of the NF fields F (on the lanes' cells) into F; C: the
// advector at the cells' low walls, G: the cells' G.
template <int K, int NF, typename T, typename O>
__device__ __forceinline__ void line_advect(T (&F)[NF][K], const T (&C)[K], const T (&G)[K],
                                            const O &o, int n_iters, bool open, const Edges &ed,
                                            int lane)
{
    T x[NF][K], u[NF][K];
    // donor-cell pass
#pragma unroll
    for (int f = 0; f < NF; f++) {
        const T l = from_left(F[f][K - 1]);
        T fl[K];
#pragma unroll
        for (int k = 0; k < K; k++) fl[k] = upwind_fp(C[k], lo(F[f], k, l), F[f][k]);
        const T r = from_right(fl[0]);
#pragma unroll
        for (int k = 0; k < K; k++) x[f][k] = line_update(o, F[f][k], hi(fl, k, r) - fl[k], G[k]);
        if (open) ed.cells(x[f], lane);
#pragma unroll
        for (int k = 0; k < K; k++) u[f][k] = C[k];
    }
    const T gl = o.has_g() ? from_left(G[K - 1]) : T(1);
#pragma unroll 1
    for (int it = 2; it <= n_iters; it++) {
#pragma unroll
        for (int f = 0; f < NF; f++) {
            const T xl = from_left(x[f][K - 1]), xr = from_right(x[f][0]);
            T V[K];
            // pseudo-velocity at the cells' low walls
            {
                T xl2 = T(0), ul = T(0), ur = T(0);
                if (o.tot()) xl2 = K > 1 ? from_left(x[f][K > 1 ? K - 2 : 0]) : from_left(xl);
                if (o.dfl()) {
                    ul = from_left(u[f][K - 1]);
                    ur = from_right(u[f][0]);
                }
#pragma unroll
                for (int k = 0; k < K; k++) {
                    const T uk = u[f][k];
                    T xL = lo(x[f], k, xl), xR = x[f][k];
                    if (o.absf()) {
                        xL = fabs(xL);
                        xR = fabs(xR);
                    }
                    T Gb = T(1);
                    if (o.has_g()) Gb = T(0.5) * (lo(G, k, gl) + G[k]);
                    T v = (fabs(uk) - (o.has_g() ? uk * uk / Gb : uk * uk)) *
                          line_frac(o.iga(), xR - xL, xR + xL, T(2));
                    if (o.tot()) {
                        T xR2 = hi(x[f], k, xr);
                        T xL2 = k > 1 ? x[f][k > 1 ? k - 2 : 0] : (k == 1 ? xl : xl2);
                        if (o.absf()) {
                            xR2 = fabs(xR2);
                            xL2 = fabs(xL2);
                        }
                        const T D = line_frac(o.iga(), xR2 - xR - xL + xL2, xR2 + xR + xL + xL2, T(4));
                        v += (T(3) * uk * fabs(uk) / Gb - T(2) * uk * uk * uk / (Gb * Gb) - uk) /
                             T(3) * D;
                    }
                    if (o.dfl()) {
                        // divergent-flow term: -c / (2 Gb) times the mean
                        // divergence of the two cells, under iga times the
                        // wall mean of psi (unit-field flux)
                        T dv = (hi(u[f], k, ur) - uk) + (uk - lo(u[f], k, ul));
                        if (o.iga()) dv *= T(0.5) * (xL + xR);
                        v -= T(0.25) * uk / Gb * dv;
                    }
                    V[k] = v;
                }
            }
            if (o.fct()) {
                T m[K], w[K], bu[K], bd[K];
#pragma unroll
                for (int k = 0; k < K; k++) {
                    m[k] = fmax(F[f][k], x[f][k]);
                    w[k] = fmin(F[f][k], x[f][k]);
                }
                const T ml = from_left(m[K - 1]), mr = from_right(m[0]);
                const T wl = from_left(w[K - 1]), wr = from_right(w[0]);
                const T vr = from_right(V[0]);
#pragma unroll
                for (int k = 0; k < K; k++) {
                    const T xi = x[f][k];
                    const T mx = fmax(fmax(m[k], lo(m, k, ml)), hi(m, k, mr));
                    const T mn = fmin(fmin(w[k], lo(w, k, wl)), hi(w, k, wr));
                    const T vlo = V[k], vhi = hi(V, k, vr);
                    const T wm = o.iga() ? T(1) : lo(x[f], k, xl);
                    const T wp = o.iga() ? T(1) : hi(x[f], k, xr);
                    const T wc = o.iga() ? T(1) : xi;
                    const T fin = pos(vlo) * wm - neg(vhi) * wp;
                    const T fout = pos(vhi) * wc - neg(vlo) * wc;
                    const T up = o.has_g() ? G[k] * (mx - xi) : mx - xi;
                    const T dn = o.has_g() ? G[k] * (xi - mn) : xi - mn;
                    bu[k] = fin > T(0) ? up / fin : T(1);
                    bd[k] = fout > T(0) ? dn / fout : T(1);
                }
                if (open) {
                    ed.cells(bu, lane);
                    ed.cells(bd, lane);
                }
                const T bul = from_left(bu[K - 1]), bdl = from_left(bd[K - 1]);
#pragma unroll
                for (int k = 0; k < K; k++) {
                    const T up = fmin(fmin(T(1), lo(bd, k, bdl)), bu[k]);
                    const T dn = fmin(fmin(T(1), lo(bu, k, bul)), bd[k]);
                    u[f][k] = pos(V[k]) * up + neg(V[k]) * dn;
                }
            } else {
#pragma unroll
                for (int k = 0; k < K; k++) u[f][k] = V[k];
            }
            // corrective donor-cell pass
            T fl[K], y[K];
#pragma unroll
            for (int k = 0; k < K; k++)
                fl[k] = o.iga() ? u[f][k] : pos(u[f][k]) * lo(x[f], k, xl) + neg(u[f][k]) * x[f][k];
            const T r = from_right(fl[0]);
#pragma unroll
            for (int k = 0; k < K; k++) y[k] = line_update(o, x[f][k], hi(fl, k, r) - fl[k], G[k]);
#pragma unroll
            for (int k = 0; k < K; k++) x[f][k] = y[k];
            if (open && it < n_iters) {
                ed.cells(x[f], lane);
                if (o.dfl()) ed.walls(u[f], lane);
            }
        }
    }
#pragma unroll
    for (int f = 0; f < NF; f++)
#pragma unroll
        for (int k = 0; k < K; k++) F[f][k] = x[f][k];
}

// n_steps steps of the NF fields (the second one, phi, makes the translating
// oscillator pair: explicit half of the coupling of strength osc_a = dt omega
// / 2, one step of each field, implicit half in closed form).  A workgroup
// makes the `tile` cells from blockIdx.x * tile on (tile >= n: the whole
// grid, in place if asked) from a region with `halo` more cells on each
// side; hl: halo lanes per wave; stride: cells of one field in an LDS buffer
// (at least the region's).
template <typename T, int K, int NF, bool GEN, bool FCT, bool IGA>
__global__ void __launch_bounds__(LINE_WAVES *WAVE)
    k_resident1d(int n, int tile, int halo, int hl, int stride, int bc, int n_iters, unsigned opts,
                 int n_steps, const T *psi, const T *phi, T *psi_out, T *phi_out,
                 const T *__restrict__ cin, const T *__restrict__ Gin, T osc_a)
{
    extern __shared__ __align__(16) char lds_raw[];
    T *buf = (T *)lds_raw;
    const LineOpts<GEN, FCT, IGA> o{opts, Gin != nullptr};
    const bool open = bc == BC_OPEN, whole = tile >= n;
    const int t0 = whole ? 0 : (int)blockIdx.x * tile;
    const int t1 = whole ? n : min(t0 + tile, n);
    // the region: `size` cells from cell `base` on (clipped at an open edge)
    int base = 0, size = n;
    if (!whole) {
        base = open ? max(t0 - halo, 0) : t0 - halo;
        size = (open ? min(t1 + halo, n) : t1 + halo) - base;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    const int lane = threadIdx.x & (WAVE - 1);
    const int own_lanes = WAVE - 2 * hl;
    const int first = (wave * own_lanes + lane - hl) * K;     // region position of cell 0
    const bool own = lane >= hl && lane < WAVE - hl;

    Edges ed;
    ed.first = first;
    ed.last = size - 1;
    ed.l_lo = hl - wave * own_lanes;
    ed.l_hi = (size - 1) / K - wave * own_lanes + hl;
    ed.s_hi = (size - 1) % K;
    ed.l_w = size / K - wave * own_lanes + hl;
    ed.s_w = size % K;
    ed.lo = open && base == 0 && ed.l_lo >= 0 && ed.l_lo < WAVE;
    ed.hi = open && base + size == n && ed.l_hi >= 0 && ed.l_hi < WAVE;
    ed.whi = open && base + size == n && ed.l_w >= 0 && ed.l_w < WAVE;

    // region position (and through it the grid cell) each cell of the lane
    // is read from
    T F[NF][K], C[K], G[K];
    int src[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        int p = first + k;
        if (whole && !open) {
            p %= n;
            p = p < 0 ? p + n : p;
        } else {
            p = min(max(p, 0), size - 1);
        }
        src[k] = p;
        int c = base + p;
        if (!open) c = c < 0 ? c + n : (c >= n ? c - n : c);
        F[0][k] = psi[c];
        if (NF > 1) F[NF - 1][k] = phi[c];
        G[k] = o.has_g() ? Gin[c] : T(1);
        int q = base + first + k;                              // low wall
        if (open) {
            q = min(max(q, 0), n);
        } else {
            q %= n;
            q = q < 0 ? q + n : q;
        }
        C[k] = cin[q];
    }

    const T den = T(1) + osc_a * osc_a;
    for (int s = 0; s < n_steps; s++) {
        if (s > 0) {
            T *b = buf + (s & 1) * NF * stride;
#pragma unroll
            for (int f = 0; f < NF; f++)
#pragma unroll
                for (int k = 0; k < K; k++)
                    if (own && first + k < size) b[f * stride + first + k] = F[f][k];
            __syncthreads();
#pragma unroll
            for (int f = 0; f < NF; f++)
#pragma unroll
                for (int k = 0; k < K; k++) F[f][k] = b[f * stride + src[k]];
        }
        if (NF > 1) {
#pragma unroll
            for (int k = 0; k < K; k++) {
                const T a = F[0][k], b = F[NF - 1][k];
                F[0][k] = a + osc_a * b;
                F[NF - 1][k] = b - osc_a * a;
            }
        }
        line_advect<K, NF>(F, C, G, o, n_iters, open, ed, lane);
        if (NF > 1) {
#pragma unroll
            for (int k = 0; k < K; k++) {
                const T a = F[0][k], b = F[NF - 1][k];
                F[0][k] = (a + osc_a * b) / den;
                F[NF - 1][k] = (b - osc_a * a) / den;
            }
        }
    }
    // (in place, no wave stores before every wave has its inputs; with more
    // steps the barrier between them has seen to that)
    if (n_steps == 1) __syncthreads();
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int c = base + first + k;
        if (own && c >= t0 && c < t1 && first + k < size) {
            psi_out[c] = F[0][k];
            if (NF > 1) phi_out[c] = F[NF - 1][k];
        }
    }
}

inline int line_halo_lanes(int radius, int K) { return (radius + K - 1) / K; }

template <typename T, int K>
hipError_t line_launch(const LineShape &sh, const LineArgs<T> &a, int steps, const T *psi,
                       const T *phi, T *psi_out, T *phi_out, hipStream_t s)
{
    const int radius = line_radius(a.n_iters, a.opts), hl = line_halo_lanes(radius, K);
    const int n = (int)a.n;
    const int region = sh.tile >= n ? n : sh.tile + 2 * sh.halo;
    const int nf = phi ? 2 : 1;
    const size_t lds = sizeof(T) * 2 * nf * (size_t)region;
    hipError_t e = hipSuccess;
    auto go = [&](auto NF, auto GE, auto FC, auto IG) {
        auto kern = k_resident1d<T, K, decltype(NF)::value, decltype(GE)::value,
                                 decltype(FC)::value, decltype(IG)::value>;
        if (lds > 64 * 1024) {
            e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds);
            if (e != hipSuccess) return;
        }
        kern<<<(unsigned)cdiv(n, sh.tile), sh.waves * WAVE, lds, s>>>(
            n, sh.tile, sh.halo, hl, region, a.bc, a.n_iters, a.opts, steps, psi, phi, psi_out,
            phi_out, a.c, a.G, (T)a.osc_a);
        e = hipGetLastError();
    };
    using TT = std::true_type;
    using FF = std::false_type;
    auto by_o = [&](auto NF) {
        const bool fct = a.opts & OPT_FCT, iga = a.opts & OPT_IGA;
        if (a.G || (a.opts & ~(unsigned)(OPT_FCT | OPT_IGA))) go(NF, TT{}, FF{}, FF{});
        else if (fct && iga) go(NF, FF{}, TT{}, TT{});
        else if (fct) go(NF, FF{}, TT{}, FF{});
        else if (iga) go(NF, FF{}, FF{}, TT{});
        else go(NF, FF{}, FF{}, FF{});
    };
    if (phi) by_o(std::integral_constant<int, 2>{});
    else by_o(std::integral_constant<int, 1>{});
    return e;
}

}  // namespace

template <typename T>
hipError_t line1d_launch(const LineShape &sh, const LineArgs<T> &a, int steps, const T *psi,
                         const T *phi, T *psi_out, T *phi_out, hipStream_t s)
{
    // a tile's halo must cover the steps of the launch, and a region its waves
    const int radius = line_radius(a.n_iters, a.opts);
    const int64_t region = sh.tile >= a.n ? a.n : (int64_t)sh.tile + 2 * sh.halo;
    if (steps < 1 || sh.waves < 1 || sh.waves > LINE_WAVES || (phi != nullptr) != (phi_out != nullptr) ||
        (int64_t)sh.waves * line_own(radius, sh.K) < region ||
        (sh.tile < a.n && (psi == psi_out || (int64_t)steps * radius > sh.halo || sh.halo >= a.n)))
        return hipErrorInvalidValue;
    switch (sh.K) {
    case 1: return line_launch<T, 1>(sh, a, steps, psi, phi, psi_out, phi_out, s);
    case 2: return line_launch<T, 2>(sh, a, steps, psi, phi, psi_out, phi_out, s);
    case 4: return line_launch<T, 4>(sh, a, steps, psi, phi, psi_out, phi_out, s);
    case 8:
        if constexpr (sizeof(T) == 4)
            return line_launch<T, 8>(sh, a, steps, psi, phi, psi_out, phi_out, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace mp
