// pass2d.hpp -- one corrective MPDATA pass on a 2-D grid in one launch
// (kernel templates; pass2d_f64_donor.hip and its siblings instantiate them,
// pass2d.hip holds the dispatch and the donor-cell pass alone).
//
// For the 2-D configurations the whole-step fused kernel does not take (open
// boundaries, iga, dfl, variable G, third-order terms): the pseudo-velocities
// of both dimensions (eq. adf_vel with its cross terms, the divergent-flow
// term and the third-order terms of Sect. 3.1.2, with the wall means of G),
// the limiter bounds and coefficients, the limited velocities and the
// corrective donor-cell update (divided by G) are computed in one sweep.
//
// Design (gfx950, wave64), the row march of the fused step kernel applied to
// a single pass whose input lives in HBM:
//   * one wavefront owns a strip of 64 columns and marches down a chunk of
//     rows; every stage is kept in per-lane register rings (one row per
//     iteration), column neighbours come from DPP lane shifts;
//   * the halo is 2 lanes on the left and 3 on the right (the divergent-flow
//     term reaches one wall further right), so a strip emits 59 columns
//     (more halo with the donor pass folded in and the third-order terms,
//     see Lanes);
//   * every load goes through the boundary map of its array (cells: wrap or
//     clamp; walls of the dimension's own advector: wrap, or clamp to the
//     edge wall), so the halo lanes and warm-up rows see exactly what the
//     stage-by-stage path reads.  The one quantity a halo cell may not
//     recompute is the limiter coefficient pair: with open boundaries the
//     coefficient of a cell outside the domain is that of the edge cell (the
//     boundary map applied to the coefficient array), so those lanes and rows
//     take it from the edge lane (readlane) or the edge row (ring slot).
#include "common.hpp"
#include "kernels.hpp"

#include <type_traits>

// Multiply-add contraction only within one source expression, decided by the
// front end, as in the fused step kernel (fused2d.hpp): the expressions the
// two kernels share then round alike, so a corrective pass formed here (the
// adjoint's recording launches) gives the bits of the same pass inside the
// fused step.
#pragma clang fp contract(on)

namespace mp {
namespace {

// Quotients of a stage with the fused step kernel's rule: a kept quotient is
// n * r, r the hardware reciprocal refined by one Newton step, where it is in
// range (FP64: r is a normal number; FP32: the divisor is normal or zero),
// else the IEEE quotient -- lane by lane, so its value depends on its
// operands only.  A wave with no kept quotient out of range (one test per
// set) issues no division.  Quotients not kept are discarded by the caller.
template <int K>
__device__ __forceinline__ void lane_quotients(const double (&n)[K], const double (&d)[K],
                                               const bool (&keep)[K], double (&q)[K])
{
    double r[K];
    bool in[K];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < K; k++) {
        r[k] = __builtin_amdgcn_rcp(d[k]);
        in[k] = __builtin_amdgcn_class(r[k], 0x108);   // +-normal
        ok = ok & (in[k] | !keep[k]);
    }
#pragma unroll
    for (int k = 0; k < K; k++) {
        const double rr = fma(fma(-d[k], r[k], 1.0), r[k], r[k]);
        q[k] = n[k] * rr;
    }
    if (__builtin_amdgcn_ballot_w64(!ok) != 0) {
#pragma unroll
        for (int k = 0; k < K; k++) q[k] = in[k] ? q[k] : n[k] / d[k];
    }
}
template <int K>
__device__ __forceinline__ void lane_quotients(const float (&n)[K], const float (&d)[K],
                                               const bool (&keep)[K], float (&q)[K])
{
    bool in[K];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < K; k++) {
        in[k] = __builtin_amdgcn_classf(d[k], 0x168);   // +-normal or +-zero
        ok = ok & (in[k] | !keep[k]);
        const float r = __builtin_amdgcn_rcpf(d[k]);
        const float q0 = n[k] * r;
        q[k] = fmaf(fmaf(-d[k], q0, n[k]), r, q0);
    }
    if (__builtin_amdgcn_ballot_w64(!ok) != 0) {
#pragma unroll
        for (int k = 0; k < K; k++) q[k] = in[k] ? q[k] : n[k] / d[k];
    }
}

constexpr int WAVE = 64;
constexpr int PF = 2;                    // rows in flight ahead of use

// Halo lanes left / right and output columns per strip.  With the donor
// pass computed in the kernel its result is valid one lane less on each
// side, so the strip needs one more halo lane on the left.  The third-order
// term of V1 reads x two columns to the left of its wall and one to the
// right: one more lane on the left, and with the donor pass (whose result
// the last lane cannot form) one more on the right.
template <bool DONOR, bool TOT> struct Lanes {
    static constexpr int HL = (DONOR ? 3 : 2) + (TOT ? 1 : 0);
    static constexpr int HR = 3 + (DONOR && TOT ? 1 : 0);
    static constexpr int OW = WAVE - HL - HR;
};

// ---- wave-wide lane shifts (DPP wave_shr:1 / wave_shl:1) -------------------
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
// value of v in lane l (l wave-uniform)
__device__ inline float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ inline double lane_value(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

template <typename T> __device__ __forceinline__ T donor_update(bool kahan, T x, T d0, T d1)
{
    if (!kahan) return x - (d0 + d1);
    T s = x, c = T(0);
    kahan_add(s, c, -d0);
    kahan_add(s, c, -d1);
    return s;
}

// the same with the flux differences divided by the cell's G (HG), as
// the stage-by-stage path: x - (d0 + d1) / G, or the two terms d_k / G
// compensated
template <bool HG, typename T>
__device__ __forceinline__ T donor_update_g(bool kahan, T x, T d0, T d1, T g)
{
    if constexpr (!HG) {
        return donor_update(kahan, x, d0, d1);
    } else {
        const bool keep[2] = {true, true};
        if (!kahan) {
            T n[1] = {d0 + d1}, d[1] = {g}, q[1];
            const bool k1[1] = {true};
            lane_quotients<1>(n, d, k1, q);
            return x - q[0];
        }
        T n[2] = {d0, d1}, d[2] = {g, g}, q[2];
        lane_quotients<2>(n, d, keep, q);
        return donor_update(true, x, q[0], q[1]);
    }
}

// ---- register rings (slot of the row pushed `age` iterations ago is a
// compile-time index for each unrolled phase P) ------------------------------
template <int D> __host__ __device__ constexpr int slot(int phase, int age)
{
    return ((phase - age) % D + D) % D;
}

template <typename T, int D> struct Ring {
    T v[D];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int k = 0; k < D; k++) v[k] = T(0);
    }
};
#define AT(ring, depth, age) (ring).v[slot<depth>(P, (age))]

// Row-loop unroll: every ring depth divides it (8 under the third-order
// terms, whose rings are deeper).
template <bool TOT> constexpr int unroll() { return TOT ? 8 : 4; }

// State of one wavefront.  At iteration a (the newest row) it holds
//   x rows a..a-3 (and their left / right neighbours), psi^n row a,
//   dimension-0 walls a+1..a-1, dimension-1 walls of rows a, a-1,
//   raw V0 at walls a, a-1, bounds rows a..a-2, coefficients rows a-1, a-2,
//   limited V0 at walls a-1, a-2 and limited V1 of rows a-1, a-2;
// it computes V0 at wall a, V1 of row a-1, the coefficients of row a-1, the
// limited velocities at wall a-1 / row a-1 and the corrected row a-2.
// TOT: the third-order term of V0 at wall w reads x rows w-2..w+1, so V0 is
// formed at wall a-1 and every later stage one row later (SH = 1): the
// coefficients and limited velocities of row a-2, the corrected row a-3;
// x is kept back to row a-4, and V1 (still formed at row a-1, its
// third-order term reaching one column further left) for one more row.
//
// DONOR: the pass input x is the donor-cell pass of psi^n, computed here
// (row a from psi^n rows a-1..a+1, which are loaded one row ahead like the
// dimension-0 walls); otherwise x is loaded.  With open boundaries the donor
// result of a cell outside the domain is the edge cell's: edge lanes are
// copied across (readlane), rows past the end repeat the last row, and the
// first chunks start at row 0 with the rows above filled with row 0.
// HG: G is an array (loaded with the cell rows, row a at age CO); otherwise
// G = 1.
// VAR: what a launch is asked for beside y (Variant): the plain and
// divergent-flow ones write y only, the walls one the limited velocities for
// a following pass too, the recording one those and every record there is
// (and y if asked), none with Kahan's summation; the general one decides it
// all at run time.  Every run-time choice is a branch in every row, which splits
// the row for the instruction scheduler and adds scalar work that a wave
// issues in order: with the choices, the 64-bit row offsets formed by
// multiplications and (FP32) a branch per quotient, a row of the FP64 iga +
// limiter instance took 212 scalar beside 326 vector instructions.
enum Variant { V_PLAIN = 0, V_DFL = 1, V_WALLS = 2, V_REC = 3, V_ANY = 4 };

template <typename T, bool FCT, bool IGA, bool ABS, bool DONOR, bool HG, bool TOT, int VAR>
struct March {
    static constexpr bool OUT = VAR >= V_WALLS;    // w0, w1
    static constexpr bool REC = VAR >= V_REC;      // the records
    static constexpr bool ASK = VAR == V_ANY;      // whether each is given is asked for
    // what y held before may be kept (the shallow-water fields' option sets:
    // the previous time level, saved here instead of by a copy of its own)
    static constexpr bool SAVE = DONOR && FCT && !HG && !TOT &&
                                 ((IGA && VAR == V_DFL) || (ABS && VAR == V_PLAIN));
    static constexpr int CO = DONOR ? 1 : 0;   // age of row a in the c1 and G rings
    static constexpr int SH = TOT ? 1 : 0;     // row shift of the stages after V0
    static constexpr int XQ = TOT ? 8 : 4;     // x ring depth (ages 0..3+SH used)
    static constexpr int XR = TOT ? 4 : 2;     // right-neighbour ring (ages 0..1+SH)
    static constexpr int GQ = TOT ? 8 : 4;     // G ring (ages 0..CO+2+SH)
    int n0, n1, i0, i1;
    int rr, rw;                        // next cell row and wall row to load (periodic: wrapped)
    int64_t oc, oc1, ow;               // their offsets in cell, c1 and c0 arrays (uniform)
    int64_t ro, ro1;                   // a n1 and a (n1 + 1) of the current row a (uniform)
    int lane_lo, lane_hi;              // lanes of columns 0 and n1-1 (edge strips; else 0)
    bool fix, below, above;            // an edge strip; the lane lies outside an open domain
    bool open0;                        // open along the rows
    bool dfl, kahan, out_lane, w1_lane, prefill;
    int64_t ocol, ccol, wcol;          // per-lane column offsets
    const T *x, *pn, *c0, *c1, *G;
    T *y, *w0, *w1;
    T *v0r, *v1r, *bur, *bdr;          // records: raw velocities, coefficients
    T *xd;                             // record of the donor pass's result (DONOR)
    T *save;                           // SAVE: receives y's old values, or NULL
    T old;                             // SAVE: y's value of the next row to store
    T fx[PF], fp[PF], f0[PF], f1[PF], fg[PF];
    Ring<T, XQ> xq;
    Ring<T, 4> xl, c0q, c1q, mxq, mnq, pq;
    Ring<T, GQ> gq;
    Ring<T, XR> xr;
    Ring<T, 2> v0q, v1q, buq, bdq, aq0, aq1;

    // x (or psi^n), psi^n, c1 and G of the next cell row and the next
    // dimension-0 wall row; then both one row on (open: the edge row is read
    // again outside the domain; periodic: wrapped at n0)
    __device__ __forceinline__ void fetch(T &vx, T &vp, T &v1, T &v0, T &vg)
    {
        vx = (x + oc)[ccol];
        if (FCT && !DONOR) vp = (pn + oc)[ccol];
        v1 = (c1 + oc1)[wcol];
        v0 = (c0 + ow)[ccol];
        if (HG) vg = (G + oc)[ccol];
        rr++;
        rw++;
        const bool wr = !open0 && rr == n0, ww = !open0 && rw == n0;
        const bool sr = !open0 || (rr >= 1 && rr < n0), sw = !open0 || (rw >= 1 && rw <= n0);
        rr = wr ? 0 : rr;
        rw = ww ? 0 : rw;
        oc = wr ? 0 : oc + (sr ? n1 : 0);
        oc1 = wr ? 0 : oc1 + (sr ? n1 + 1 : 0);
        ow = ww ? 0 : ow + (sw ? n1 : 0);
    }
    // the first row to load: cell row r and wall row w
    __device__ __forceinline__ void seek(int r, int w)
    {
        const int bc = open0 ? BC_OPEN : BC_PERIODIC;
        const int64_t mr = map_cell(r, n0, bc), mw = map_wall(w, n0, bc);
        rr = open0 ? r : (int)mr;
        rw = open0 ? w : (int)mw;
        oc = mr * n1;
        oc1 = mr * (n1 + 1);
        ow = mw * n1;
    }
    __device__ __forceinline__ void load(int k) { fetch(fx[k], fp[k], f1[k], f0[k], fg[k]); }

    __device__ __forceinline__ bool with_dfl() const
    {
        return VAR == V_DFL || (VAR == V_ANY && dfl);
    }
    __device__ __forceinline__ bool with_kahan() const { return VAR == V_ANY && kahan; }

    // G of cell row a - k (1 without HG)
    template <int P> __device__ __forceinline__ T g_row(int k) const
    {
        if constexpr (HG) return gq.v[slot<GQ>(P, CO + k)];
        else return T(1);
    }

    // donor result at a lane outside an open domain: the edge lane's
    __device__ __forceinline__ T edge_cols(T v)
    {
        if (fix) v = edge_value(v);
        return v;
    }
    __device__ __forceinline__ T edge_value(T v)
    {
        // (below / above: no lane where the strip does not have that edge)
        const T lo = lane_value(v, lane_lo), hi = lane_value(v, lane_hi);
        return below ? lo : (above ? hi : v);
    }

    // The rows above an open domain are copies of row 0: before the march of a
    // chunk that starts there, every ring slot takes the donor result of row
    // 0 (psi^n rows -1 and 0 are in the rings at phase 0, row 1 is fetched).
    __device__ __forceinline__ void fill_above()
    {
        constexpr int P = 0;
        const T pc = AT(pq, 4, 1), f0lo = upwind_fp(AT(c0q, 4, 1), AT(pq, 4, 2), pc);
        const T f0hi = upwind_fp(f0[0], pc, fx[0]);
        const T f1lo = upwind_fp(AT(c1q, 4, 1), from_left(pc), pc);
        const T f1hi = from_right(f1lo);
        T g = T(1);
        if constexpr (HG) g = AT(gq, GQ, 1);
        const T x0 = edge_cols(donor_update_g<HG>(with_kahan(), pc, f0hi - f0lo, f1hi - f1lo, g));
        const T l = from_left(x0), r = from_right(x0);
#pragma unroll
        for (int k = 0; k < XQ; k++) xq.v[k] = x0;
#pragma unroll
        for (int k = 0; k < XR; k++) xr.v[k] = r;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            xl.v[k] = l;
            mxq.v[k] = fmax(pc, x0);
            mnq.v[k] = fmin(pc, x0);
        }
    }

    // One row.  STAGE: 2, all of it; on the first rows of a chunk, above
    // what any output row reads, 0: the pass input alone, 1: and the raw
    // velocities.
    template <int P, int STAGE> __device__ __forceinline__ void iter(int a)
    {
        constexpr int S = P % PF;
        T x_a, pn_a;
        if (HG) AT(gq, GQ, 0) = fg[S];   // row a + CO
        if (DONOR) {
            // psi^n, c1 of row a+1 and wall a+1 arrive; donor pass of row a
            AT(pq, 4, 0) = fx[S];
            AT(c1q, 4, 0) = f1[S];
            AT(c0q, 4, 0) = f0[S];
            load(S);
            const T pc = AT(pq, 4, 1), pm = AT(pq, 4, 2), pp = AT(pq, 4, 0);
            const T u0lo = AT(c0q, 4, 1), u0hi = AT(c0q, 4, 0), u1 = AT(c1q, 4, 1);
            const T f0lo = upwind_fp(u0lo, pm, pc);
            const T f0hi = upwind_fp(u0hi, pc, pp);
            const T f1lo = upwind_fp(u1, from_left(pc), pc);
            const T f1hi = from_right(f1lo);
            x_a = edge_cols(donor_update_g<HG>(with_kahan(), pc, f0hi - f0lo, f1hi - f1lo,
                                               g_row<P>(0)));
            x_a = open0 && a >= n0 ? AT(xq, XQ, 1) : x_a;   // rows past the end
            pn_a = pc;
            // the donor result of the chunk's own rows and columns
            if (REC && (!ASK || xd) && a >= i0 && a < i1 && out_lane) (xd + ro)[ocol] = x_a;
        } else {
            x_a = fx[S];
            pn_a = fp[S];
            AT(c1q, 4, 0) = f1[S];   // row a
            AT(c0q, 4, 0) = f0[S];   // wall a+1
            load(S);
        }
        AT(xq, XQ, 0) = x_a;
        AT(xl, 4, 0) = from_left(x_a);
        AT(xr, XR, 0) = from_right(x_a);
        if (FCT) {
            AT(mxq, 4, 0) = fmax(pn_a, x_a);
            AT(mnq, 4, 0) = fmin(pn_a, x_a);
        }
        if constexpr (STAGE == 0) {
            ro += n1;
            ro1 += n1 + 1;
            return;
        }

        // psi-fractions: V0 at wall w = a - SH (rows w-1 | w), V1 of row a-1
        // at wall j (columns j-1 | j): A terms and cross (B) terms, with TOT
        // the third-order D and E terms; with HG the reciprocal wall means
        // of G at both walls (the last two quotients)
        auto fa = [](T v) -> T { return ABS ? fabs(v) : v; };
        constexpr int NF = TOT ? 8 : 4;          // psi-fractions
        constexpr int NQ = NF + (HG ? 2 : 0);
        T num[NQ], den[NQ], fr[NQ];
        {
            const T xL = fa(AT(xq, XQ, SH + 1)), xR = fa(AT(xq, XQ, SH));
            num[0] = xR - xL;
            den[0] = xR + xL;
            const T p = fa(AT(xr, XR, SH)), q = fa(AT(xr, XR, SH + 1));
            const T e = fa(AT(xl, 4, SH)), f = fa(AT(xl, 4, SH + 1));
            num[1] = p + q - e - f;
            den[1] = p + q + e + f;
            if constexpr (TOT) {
                const T xR2 = fa(AT(xq, XQ, 0)), xL2 = fa(AT(xq, XQ, 3));
                num[4] = xR2 - xR - xL + xL2;
                den[4] = xR2 + xR + xL + xL2;
                num[5] = p - q - e + f;
                den[5] = den[1];
            }
        }
        {
            const T xL = fa(AT(xl, 4, 1)), xR = fa(AT(xq, XQ, 1));
            num[2] = xR - xL;
            den[2] = xR + xL;
            const T p = fa(AT(xq, XQ, 0)), q = fa(AT(xl, 4, 0));
            const T e = fa(AT(xq, XQ, 2)), f = fa(AT(xl, 4, 2));
            num[3] = p + q - e - f;
            den[3] = p + q + e + f;
            if constexpr (TOT) {
                const T xR2 = fa(AT(xr, XR, 1)), xL2 = fa(from_left(AT(xl, 4, 1)));
                num[6] = xR2 - xR - xL + xL2;
                den[6] = xR2 + xR + xL + xL2;
                num[7] = p - q - e + f;
                den[7] = den[3];
            }
        }
        T ig0 = T(1), ig1 = T(1);    // 1 / wall mean of G: wall a-SH | row a-1, wall j
        if constexpr (HG) {
            const T gw = g_row<P>(SH), gwm = g_row<P>(SH + 1), gm = g_row<P>(1);
            num[NF] = T(1);
            den[NF] = T(0.5) * (gwm + gw);
            num[NF + 1] = T(1);
            den[NF + 1] = T(0.5) * (from_left(gm) + gm);
        }
        if (IGA) {
            fr[0] = num[0] / T(2);
            fr[1] = num[1] / T(4);
            fr[2] = num[2] / T(2);
            fr[3] = num[3] / T(4);
#pragma unroll
            for (int k = 4; k < NF; k++) fr[k] = num[k] / T(4);
            if constexpr (HG) {
                T n2[2] = {num[NF], num[NF + 1]}, d2[2] = {den[NF], den[NF + 1]}, q2[2];
                const bool k2[2] = {true, true};
                lane_quotients<2>(n2, d2, k2, q2);
                ig0 = q2[0];
                ig1 = q2[1];
            }
        } else {
            bool keep[NQ];
#pragma unroll
            for (int k = 0; k < NQ; k++) keep[k] = k >= NF || den[k] != T(0);
            lane_quotients<NQ>(num, den, keep, fr);
#pragma unroll
            for (int k = 0; k < NF; k++) fr[k] = den[k] == T(0) ? T(0) : fr[k];
            if constexpr (HG) {
                ig0 = fr[NF];
                ig1 = fr[NF + 1];
            }
        }
        T v0, v1;
        {
            const T u = AT(c0q, 4, 1 + SH);                  // wall a-SH
            const T s1 = AT(c1q, 4, CO + SH + 1) + AT(c1q, 4, CO + SH);
            const T cb = T(0.25) * (s1 + from_right(s1));
            if constexpr (HG) {
                v0 = (fabs(u) - u * u * ig0) * fr[0];
                v0 -= T(0.5) * u * cb * ig0 * fr[1];
            } else {
                v0 = (fabs(u) - u * u) * fr[0];
                v0 -= T(0.5) * u * cb * fr[1];
            }
            if (with_dfl()) {
                // mean of the divergences of the wall's two cells
                const T c1a = AT(c1q, 4, CO + SH), c1b = AT(c1q, 4, CO + SH + 1);
                T dv = (AT(c0q, 4, 1 + SH) - AT(c0q, 4, 2 + SH)) +
                       (AT(c0q, 4, SH) - AT(c0q, 4, 1 + SH));
                dv += (from_right(c1b) - c1b) + (from_right(c1a) - c1a);
                if (IGA) dv *= T(0.5) * (AT(xq, XQ, SH + 1) + AT(xq, XQ, SH));
                v0 -= T(0.25) * u * ig0 * dv;
            }
            if constexpr (TOT) {
                v0 += (T(3) * u * fabs(u) * ig0 - T(2) * u * u * u * (ig0 * ig0) - u) *
                      (T(1) / T(3)) * fr[4];
                v0 += (fabs(u) * cb * ig0 - T(2) * u * u * cb * (ig0 * ig0)) * fr[5];
            }
        }
        {
            const T u = AT(c1q, 4, CO + 1);                  // row a-1, wall j
            const T s0 = AT(c0q, 4, 2) + AT(c0q, 4, 1);
            const T cb = T(0.25) * (from_left(s0) + s0);
            if constexpr (HG) {
                v1 = (fabs(u) - u * u * ig1) * fr[2];
                v1 -= T(0.5) * u * cb * ig1 * fr[3];
            } else {
                v1 = (fabs(u) - u * u) * fr[2];
                v1 -= T(0.5) * u * cb * fr[3];
            }
            if (with_dfl()) {
                // mean of the divergences of cells (a-1, j-1) and (a-1, j)
                const T d0 = AT(c0q, 4, 1) - AT(c0q, 4, 2);
                T dv = from_left(d0) + d0;
                const T c = AT(c1q, 4, CO + 1);
                dv += (c - from_left(c)) + (from_right(c) - c);
                if (IGA) dv *= T(0.5) * (AT(xl, 4, 1) + AT(xq, XQ, 1));
                v1 -= T(0.25) * u * ig1 * dv;
            }
            if constexpr (TOT) {
                v1 += (T(3) * u * fabs(u) * ig1 - T(2) * u * u * u * (ig1 * ig1) - u) *
                      (T(1) / T(3)) * fr[6];
                v1 += (fabs(u) * cb * ig1 - T(2) * u * u * cb * (ig1 * ig1)) * fr[7];
            }
        }
        AT(v0q, 2, 0) = v0;
        if constexpr (TOT) AT(v1q, 2, 0) = v1;
        if constexpr (STAGE == 1) {
            ro += n1;
            ro1 += n1 + 1;
            return;
        }
        // V1 of the limiter's row rl = a-1-SH
        const T v1l = TOT ? AT(v1q, 2, 1) : v1;
        const int rl = a - 1 - SH;

        T lim0, lim1;
        if (FCT) {
            // bounds over {psi^n, x} at the cell and its face neighbours
            const T m1 = AT(mxq, 4, SH + 1), n1v = AT(mnq, 4, SH + 1);
            const T mx = fmax(fmax(m1, fmax(AT(mxq, 4, SH + 2), AT(mxq, 4, SH))),
                              fmax(from_left(m1), from_right(m1)));
            const T mn = fmin(fmin(n1v, fmin(AT(mnq, 4, SH + 2), AT(mnq, 4, SH))),
                              fmin(from_left(n1v), from_right(n1v)));
            // in / out fluxes of cell (rl, j); unit field under iga
            const T xc = AT(xq, XQ, SH + 1);
            const T v0lo = AT(v0q, 2, 1), v0hi = v0;
            const T v1lo = v1l, v1hi = from_right(v1l);
            T fin, fout;
            if (IGA) {
                fin = (pos(v0lo) - neg(v0hi)) + (pos(v1lo) - neg(v1hi));
                fout = (pos(v0hi) - neg(v0lo)) + (pos(v1hi) - neg(v1lo));
            } else {
                fin = (pos(v0lo) * AT(xq, XQ, SH + 2) - neg(v0hi) * AT(xq, XQ, SH)) +
                      (pos(v1lo) * AT(xl, 4, SH + 1) - neg(v1hi) * AT(xr, XR, SH + 1));
                fout = (pos(v0hi) * xc - neg(v0lo) * xc) + (pos(v1hi) * xc - neg(v1lo) * xc);
            }
            const T gc = g_row<P>(1 + SH);
            T bn[2] = {HG ? gc * (mx - xc) : mx - xc, HG ? gc * (xc - mn) : xc - mn};
            T bdv[2] = {fin, fout}, bq[2];
            const bool bkeep[2] = {fin > T(0), fout > T(0)};
            lane_quotients<2>(bn, bdv, bkeep, bq);
            T bu = fin > T(0) ? bq[0] : T(1);
            T bd = fout > T(0) ? bq[1] : T(1);
            // open columns: a cell left of column 0 / right of column n1-1
            // has the edge cell's coefficients
            if (fix) {
                bu = edge_value(bu);
                bd = edge_value(bd);
            }
            AT(buq, 2, 0) = bu;
            AT(bdq, 2, 0) = bd;
            // limited V1 of row rl at wall j: L = (rl, j-1), R = (rl, j)
            {
                T up = fmin(fmin(T(1), from_left(bd)), bu);
                T dn = fmin(fmin(T(1), from_left(bu)), bd);
                lim1 = pos(v1l) * up + neg(v1l) * dn;
            }
            // limited V0 at wall rl: L = row rl-1, R = row rl; with open rows
            // the row outside the domain takes the edge row's coefficients
            {
                T bu_l = AT(buq, 2, 1), bd_l = AT(bdq, 2, 1);
                T bu_r = AT(buq, 2, 0), bd_r = AT(bdq, 2, 0);
                if (open0 && (rl == 0 || rl == n0)) {
                    if (rl == 0) {
                        bu_l = bu_r;
                        bd_l = bd_r;
                    } else {
                        bu_r = bu_l;
                        bd_r = bd_l;
                    }
                }
                T v = AT(v0q, 2, 1);
                T up = fmin(fmin(T(1), bd_l), bu_r);
                T dn = fmin(fmin(T(1), bu_l), bd_r);
                lim0 = pos(v) * up + neg(v) * dn;
            }
        } else {
            lim0 = AT(v0q, 2, 1);
            lim1 = v1l;
        }
        AT(aq0, 2, 0) = lim0;
        AT(aq1, 2, 0) = lim1;

        // limited velocities for a following pass (and, when asked, the raw
        // velocities and the coefficients): wall rl and row rl
        if (OUT && (!ASK || w0)) {
            const int w = rl;
            if (w >= i0 && (w < i1 || (w == n0 && i1 == n0 && open0))) {
                const int64_t k0 = ro - (int64_t)(1 + SH) * n1;
                const int64_t k1 = ro1 - (int64_t)(1 + SH) * (n1 + 1);
                if (out_lane) {
                    (w0 + k0)[ocol] = lim0;
                    if (REC && (ASK ? v0r != nullptr : FCT)) (v0r + k0)[ocol] = AT(v0q, 2, 1);
                    if (REC && FCT && (!ASK || bur) && w < i1) {
                        (bur + k0)[ocol] = AT(buq, 2, 0);
                        (bdr + k0)[ocol] = AT(bdq, 2, 0);
                    }
                }
                if (w < i1 && w1_lane) {
                    (w1 + k1)[ocol] = lim1;
                    if (REC && (ASK ? v1r != nullptr : FCT)) (v1r + k1)[ocol] = v1l;
                }
            }
        }

        // corrective donor-cell pass at row rl-1 (flux = limited velocity
        // under iga)
        const T xc = AT(xq, XQ, SH + 2);
        T f0lo, f0hi, f1lo;
        if (IGA) {
            f0lo = AT(aq0, 2, 1);
            f0hi = AT(aq0, 2, 0);
            f1lo = AT(aq1, 2, 1);
        } else {
            f0lo = pos(AT(aq0, 2, 1)) * AT(xq, XQ, SH + 3) + neg(AT(aq0, 2, 1)) * xc;
            f0hi = pos(AT(aq0, 2, 0)) * xc + neg(AT(aq0, 2, 0)) * AT(xq, XQ, SH + 1);
            f1lo = pos(AT(aq1, 2, 1)) * AT(xl, 4, SH + 2) + neg(AT(aq1, 2, 1)) * xc;
        }
        const T f1hi = from_right(f1lo);
        const T res =
            donor_update_g<HG>(with_kahan(), xc, f0hi - f0lo, f1hi - f1lo, g_row<P>(2 + SH));
        const int r = rl - 1;
        if constexpr (SAVE) {
            if (save) {
                // the old value of row r arrived with the previous row
                const T was = old;
                const int next = min(max(r + 1, i0), i1 - 1);
                old = (y + (int64_t)next * n1)[ccol];
                if (r >= i0 && r < i1 && out_lane) (save + ro - (int64_t)(2 + SH) * n1)[ocol] = was;
            }
        }
        if ((!REC || y) && r >= i0 && r < i1 && out_lane) (y + ro - (int64_t)(2 + SH) * n1)[ocol] = res;
        ro += n1;
        ro1 += n1 + 1;
    }
};

// N rows from row a on, with phases P0 ..
template <int N, int P0, typename M, int I = 0>
__device__ __forceinline__ void iter_block(M &m, int a)
{
    if constexpr (I < N) {
        m.template iter<P0 + I, 2>(a + I);
        iter_block<N, P0, M, I + 1>(m, a);
    }
}

// The first LEAD rows of a chunk whose first output row is i0 = a + 3: the
// rows i0-3, i0-2 (TOT: and i0-1) feed the rings only, the next one the raw
// velocities (V0 at wall i0-1, V1 of the limiter's first row), and from
// then on every stage counts.
constexpr int LEAD = 4;
constexpr int LEAD_P = 4;          // their first phase: the row loop follows at phase 0 (of 4 or 8)
template <typename M> __device__ __forceinline__ void lead_in(M &m, int a)
{
    m.template iter<LEAD_P, 0>(a);
    m.template iter<LEAD_P + 1, 0>(a + 1);
    if constexpr (M::SH) {
        m.template iter<LEAD_P + 2, 0>(a + 2);
        m.template iter<LEAD_P + 3, 1>(a + 3);
    } else {
        m.template iter<LEAD_P + 2, 1>(a + 2);
        m.template iter<LEAD_P + 3, 2>(a + 3);
    }
}

// DONOR: x is psi^n (the donor pass is done here); otherwise x is the
// previous pass's result and psi_n is psi^n.
template <typename T, bool FCT, bool IGA, bool ABS, bool DONOR, bool HG, bool TOT, int VAR>
__global__ void __launch_bounds__(WAVE)
    k_pass2d(int n0, int n1, int bc0, int bc1, int th, int strips, int dfl, int kahan,
             PassFields<T> fl, const T *__restrict__ c0, const T *__restrict__ c1,
             const T *__restrict__ psi_n, const T *__restrict__ G, T *__restrict__ w0,
             T *__restrict__ w1, T *__restrict__ v0r, T *__restrict__ v1r,
             T *__restrict__ bur, T *__restrict__ bdr, T *__restrict__ xd)
{
    constexpr int HL = Lanes<DONOR, TOT>::HL, HR = Lanes<DONOR, TOT>::HR;
    constexpr int OW = Lanes<DONOR, TOT>::OW;
    const int strip = blockIdx.x % strips, chunk = blockIdx.x / strips;
    const int i0 = chunk * th;
    const int i1 = i0 + th < n0 ? i0 + th : n0;
    const int jstrip0 = strip * OW;
    // several fields under one advector: one after another along the grid
    const T *x = fl.x[blockIdx.y];
    T *y = fl.y[blockIdx.y];
    if (DONOR) psi_n = x;   // (so that the fields of a launch are alike)
    const int lane = threadIdx.x & (WAVE - 1);
    const int col = jstrip0 - HL + lane;

    using M = March<T, FCT, IGA, ABS, DONOR, HG, TOT, VAR>;
    M m;
    m.n0 = n0;
    m.n1 = n1;
    m.i0 = i0;
    m.i1 = i1;
    m.open0 = bc0 == BC_OPEN;
    m.dfl = dfl != 0;
    m.kahan = kahan != 0;
    m.x = x;
    m.pn = psi_n;
    m.c0 = c0;
    m.c1 = c1;
    m.G = G;
    m.y = y;
    m.w0 = w0;
    m.w1 = w1;
    m.v0r = v0r;
    m.v1r = v1r;
    m.bur = bur;
    m.bdr = bdr;
    m.xd = DONOR ? xd : nullptr;
    if constexpr (M::SAVE) {
        m.save = fl.save[blockIdx.y];
        m.old = T(0);
    }
    m.ccol = map_cell(col, n1, bc1);
    m.wcol = map_wall(col, n1, bc1);
    m.ocol = col;
    m.out_lane = lane >= HL && lane < WAVE - HR && col >= 0 && col < n1;
    // walls of dimension 1 written for a following pass: the strip's output
    // columns, plus the edge wall n1 (open) by the last strip
    m.w1_lane = (lane >= HL && lane < WAVE - HR && col >= 0 && col < n1) ||
                (bc1 == BC_OPEN && col == n1 && strip == strips - 1);
    const bool lo = bc1 == BC_OPEN && jstrip0 - HL < 0;
    const bool hi = bc1 == BC_OPEN && jstrip0 - HL + WAVE > n1;
    m.lane_lo = lo ? HL - jstrip0 : 0;
    m.lane_hi = hi ? n1 - 1 - jstrip0 + HL : 0;
    m.fix = lo || hi;
    m.below = lo && lane < m.lane_lo;
    m.above = hi && lane > m.lane_hi;
    m.xq.zero();
    m.xl.zero();
    m.c0q.zero();
    m.pq.zero();
#pragma unroll
    for (int k = 0; k < M::GQ; k++) m.gq.v[k] = T(1);
    m.mxq.zero();
    m.mnq.zero();
    m.xr.zero();
    m.c1q.zero();
    m.v0q.zero();
    m.v1q.zero();
    m.buq.zero();
    m.bdq.zero();
    m.aq0.zero();
    m.aq1.zero();
#pragma unroll
    for (int k = 0; k < PF; k++) m.fp[k] = T(0);

    // iterations a = i0-3 .. i1+1+SH (whole blocks of the unroll; extra
    // rows are not stored).  The first output row i0 needs the limiter coefficients of
    // row i0-1, hence V0 at wall i0-1, whose divergent-flow term reads wall
    // i0-2: loaded as the newest wall at iteration i0-3.  Without the donor
    // pass, cell rows are loaded from a and dimension-0 walls one row
    // ahead; with it, psi^n, c1 and the walls all one row ahead, and the
    // rings start with rows a-1 and a.  A chunk of an open domain whose first
    // iteration would lie above row 0 starts at row 0 (the rows above are
    // copies of row 0).
    m.prefill = DONOR && bc0 == BC_OPEN && i0 < 3;
    const int a_begin = m.prefill ? 0 : i0 - 3;
    const int a_end = i1 + 1 + M::SH;
    m.ro = (int64_t)a_begin * n1;
    m.ro1 = (int64_t)a_begin * (n1 + 1);
    if (DONOR) {
        // (the ring slots of the first phase: LEAD_P with the lead-in, 0
        // without, which differ in rings of eight only)
        T vp;
        m.seek(a_begin - 1, a_begin - 1);
        auto first = [&](auto PH) {
            constexpr int ph = decltype(PH)::value;
            m.fetch(m.pq.v[slot<4>(ph, 2)], vp, m.c1q.v[slot<4>(ph, 2)], m.c0q.v[slot<4>(ph, 2)],
                    m.gq.v[slot<M::GQ>(ph, 2)]);
            m.fetch(m.pq.v[slot<4>(ph, 1)], vp, m.c1q.v[slot<4>(ph, 1)], m.c0q.v[slot<4>(ph, 1)],
                    m.gq.v[slot<M::GQ>(ph, 1)]);
        };
        if (M::GQ == 4 || m.prefill) first(std::integral_constant<int, 0>{});
        else first(std::integral_constant<int, LEAD_P>{});
    } else {
        m.seek(a_begin, a_begin + 1);
    }
#pragma unroll
    for (int k = 0; k < PF; k++) m.load(k);
    // A chunk without the lead-in runs a row loop of its own: one loop
    // entered from both measured 6 % slower (shallow water 1024^2, 67 -> 70 us
    // a step).  Under TOT, whose rows are three times the code, one loop
    // serves both: a launch from cold caches is bound by fetching it (256^2
    // FP64 with G, five steps after other work, 336 -> 200 us).
    constexpr int U = unroll<TOT>();
    int a = a_begin;
    if (DONOR && m.prefill) {
        m.fill_above();
        if constexpr (!TOT) {
            for (; a <= a_end; a += U) iter_block<U, 0>(m, a);
            return;
        }
    } else {
        lead_in(m, a);
        a += LEAD;
    }
    for (; a <= a_end; a += U) iter_block<U, 0>(m, a);
}

template <typename T, bool FCT, bool IGA, bool ABS, bool DONOR, bool HG, bool TOT, int VAR>
hipError_t launch(const PassArgs<T> &p)
{
    const int64_t n0 = p.g.n[0], n1 = p.g.n[1];
    const int64_t strips = cdiv(n1, Lanes<DONOR, TOT>::OW);
    auto kern = k_pass2d<T, FCT, IGA, ABS, DONOR, HG, TOT, VAR>;
    int64_t th = p.tile_rows;
    if (th <= 0) {
        static_assert(LEAD == 4 && unroll<TOT>() == (TOT ? 8 : 4), "what pass2d_rows prices");
        static const Slots slots = slots_of((const void *)kern, WAVE);
        static thread_local ChunkMemo memo;
        th = memo(n0, strips * p.fields, [&] {
            return pass2d_rows(n0, strips * p.fields, slots, TOT, sizeof(T) == 8);
        });
    }
    if (th > n0) th = n0;
    const dim3 blocks((unsigned)(strips * cdiv(n0, th)), (unsigned)p.fields);
    kern<<<blocks, WAVE, 0, p.s>>>(
        (int)n0, (int)n1, p.g.bc[0], p.g.bc[1], (int)th, (int)strips, (p.opts & OPT_DFL) ? 1 : 0,
        (p.opts & OPT_KAHAN) ? 1 : 0, p.fl, p.c0, p.c1, p.psi_n, p.G, p.w0, p.w1, p.rec.v0,
        p.rec.v1, p.rec.bu, p.rec.bd, p.rec.xd);
    return hipGetLastError();
}

}  // namespace

// The instance of a launch.  The variants without run-time choices exist for
// what steps and recordings ask for: y alone (every option), y with the
// divergent-flow term under iga and the limiter (shallow water), y and the
// walls, or the walls and records, without iga or abs; everything else is
// V_ANY.
template <typename T, bool DONOR> hipError_t pass2d_go(const PassArgs<T> &p)
{
    const bool fct = p.opts & OPT_FCT, iga = p.opts & OPT_IGA, absf = p.opts & OPT_ABS;
    const bool tot = p.opts & OPT_TOT, dfl = p.opts & OPT_DFL, kahan = p.opts & OPT_KAHAN;
    const bool out = p.w0 || p.w1 || p.rec.xd || p.rec.v0 || p.rec.bu || !p.fl.y[0];
    const PassRecord<T> &rec = p.rec;
    const bool recs = rec.xd || rec.v0 || rec.v1 || rec.bu || rec.bd;
    const bool all_recs = (!DONOR || rec.xd) && (fct ? rec.v0 && rec.v1 && rec.bu && rec.bd
                                                     : !rec.v0 && !rec.v1);
    auto by_v = [&](auto F, auto I, auto A, auto H, auto O) {
        constexpr bool f = decltype(F)::value, i = decltype(I)::value, a = decltype(A)::value;
        constexpr bool h = decltype(H)::value, o = decltype(O)::value;
        if (!kahan && !dfl && !out) return launch<T, f, i, a, DONOR, h, o, V_PLAIN>(p);
        if constexpr (f && i && !h && !o)
            if (!kahan && !out) return launch<T, f, i, a, DONOR, h, o, V_DFL>(p);
        if constexpr (!i && !a)
            if (!kahan && !dfl && p.w0 && p.w1) {
                if (!recs && p.fl.y[0]) return launch<T, f, i, a, DONOR, h, o, V_WALLS>(p);
                if (all_recs) return launch<T, f, i, a, DONOR, h, o, V_REC>(p);
            }
        return launch<T, f, i, a, DONOR, h, o, V_ANY>(p);
    };
    using TT = std::true_type;
    using FF = std::false_type;
    auto by_t = [&](auto F, auto I, auto A, auto H) {
        return tot ? by_v(F, I, A, H, TT{}) : by_v(F, I, A, H, FF{});
    };
    auto by_g = [&](auto F, auto I, auto A) {
        return p.G ? by_t(F, I, A, TT{}) : by_t(F, I, A, FF{});
    };
    auto by_f = [&](auto I, auto A) { return fct ? by_g(TT{}, I, A) : by_g(FF{}, I, A); };
    // (the infinite gauge has two passes at most, and the second one always
    // comes with the donor pass)
    if constexpr (DONOR) {
        if (iga) return by_f(TT{}, FF{});
    } else if (iga) {
        return hipErrorInvalidValue;
    }
    if (absf) return by_f(FF{}, TT{});
    return by_f(FF{}, FF{});
}

}  // namespace mp
