// sw.hip -- prognosed velocity (Sect. 5.1-5.2) and the pressure-gradient
// forcing of the shallow-water equations (eqs. shw1d, shw2d).
//
// Both kernels are elementwise with small stencils and bound by HBM
// traffic; each thread handles one wall (advector) or one cell (forcing) in
// a grid-stride loop.  Contraction into FMA is off in this file, so in FP64
// every value is the correctly rounded result of the same operations in the
// same order as a plain evaluation of the formulas.
#include "common.hpp"
#include "kernels.hpp"

#pragma clang fp contract(off)

namespace mp {
namespace {

constexpr int SB = 256;

// cell velocity: num / den, 0 where den <= eps; num itself without den
template <typename T>
__device__ inline T vel(const T *__restrict__ num, const T *__restrict__ den, int64_t i, T eps)
{
    if (!den) return num[i];
    T h = den[i];
    return h > eps ? num[i] / h : T(0);
}

// Advector component WD at every wall: the velocity extrapolated to n+1/2,
// 1.5 u^n - 0.5 u^(n-1), averaged over the wall's two cells (through the
// boundary map), times k = dt / dx_WD.
template <typename T, int WD>
__global__ void k_vip(Geom g, const T *__restrict__ num, const T *__restrict__ den,
                      const T *__restrict__ nump, const T *__restrict__ denp, T eps, T k,
                      T *__restrict__ c)
{
    int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
    e[WD] += 1;
    const int64_t M = e[0] * e[1] * e[2];
    const int64_t stride = WD == 2 ? 1 : (WD == 1 ? g.n[2] : g.n[1] * g.n[2]);
    for (int64_t t = (int64_t)blockIdx.x * SB + threadIdx.x; t < M;
         t += (int64_t)gridDim.x * SB) {
        int v[3];
        unflat3(t, e, v);
        const int64_t f = v[WD];
        v[WD] = 0;
        const int64_t base = ((int64_t)v[0] * g.n[1] + v[1]) * g.n[2] + v[2];
        const int64_t iL = base + map_cell(f - 1, g.n[WD], g.bc[WD]) * stride;
        const int64_t iR = base + map_cell(f, g.n[WD], g.bc[WD]) * stride;
        T uL = T(1.5) * vel(num, den, iL, eps) - T(0.5) * vel(nump, denp, iL, eps);
        T uR = T(1.5) * vel(num, den, iR, eps) - T(0.5) * vel(nump, denp, iR, eps);
        c[t] = k * (T(0.5) * (uL + uR));
    }
}

// Momentum forcing: q_d += (dt/2) (-g h dh/dx_d), the derivative as the
// centred difference through the boundary map.  With save set, the
// previous level is taken first: q_prev_d = q_d, h_prev = h.
template <typename T>
__global__ void k_sw_force(Geom g, const T *__restrict__ h, T *__restrict__ h_prev, T *q0,
                           T *q1, T *q2, T *qp0, T *qp1, T *qp2, T ngrav, T tdx0, T tdx1,
                           T tdx2, T half_dt, int save)
{
    const int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
    const int64_t M = e[0] * e[1] * e[2];
    const int64_t st[3] = {e[1] * e[2], e[2], 1};
    T *q[3] = {q0, q1, q2};
    T *qp[3] = {qp0, qp1, qp2};
    const T tdx[3] = {tdx0, tdx1, tdx2};
    for (int64_t t = (int64_t)blockIdx.x * SB + threadIdx.x; t < M;
         t += (int64_t)gridDim.x * SB) {
        int v[3];
        unflat3(t, e, v);
        const T hc = h[t];
        if (save) h_prev[t] = hc;
#pragma unroll
        for (int d = 0; d < 3; d++) {
            if (d >= g.nd) break;
            const int64_t base = t - (int64_t)v[d] * st[d];
            const T hp = h[base + map_cell(v[d] + 1, e[d], g.bc[d]) * st[d]];
            const T hm = h[base + map_cell(v[d] - 1, e[d], g.bc[d]) * st[d]];
            const T f = ngrav * hc * (hp - hm) / tdx[d];
            const T qc = q[d][t];
            if (save) qp[d][t] = qc;
            q[d][t] = qc + half_dt * f;
        }
    }
}

// The save-phase forcing of one momentum component d written elsewhere: out
// = q + (dt/2)(-g h dh/dx_d) (the same expressions as above), q itself left
// at level n and copied to qp; h_prev, when given, receives h.  The step
// then advects out into q, with no copy of q into the workspace.
template <typename T>
__global__ void k_sw_force1(Geom g, int d, const T *__restrict__ h, T *__restrict__ h_prev,
                            const T *__restrict__ q, T *__restrict__ qp, T *__restrict__ out,
                            T ngrav, T tdx, T half_dt)
{
    const int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
    const int64_t M = e[0] * e[1] * e[2];
    const int64_t st[3] = {e[1] * e[2], e[2], 1};
    for (int64_t t = (int64_t)blockIdx.x * SB + threadIdx.x; t < M;
         t += (int64_t)gridDim.x * SB) {
        int v[3];
        unflat3(t, e, v);
        const T hc = h[t];
        if (h_prev) h_prev[t] = hc;
        const int64_t base = t - (int64_t)v[d] * st[d];
        const T hp = h[base + map_cell(v[d] + 1, e[d], g.bc[d]) * st[d]];
        const T hm = h[base + map_cell(v[d] - 1, e[d], g.bc[d]) * st[d]];
        const T f = ngrav * hc * (hp - hm) / tdx;
        const T qc = q[t];
        qp[t] = qc;
        out[t] = qc + half_dt * f;
    }
}

// 2-D, one thread per cell of a row (blockIdx.y: the row, so no division of
// a flat index): everything that precedes the advection of a shallow-water
// step.  The advector at the cell's low walls (and by the last row and
// column at the far edge walls) with k_vip's expressions, and the fields to
// advect: the depth copied, the momenta with the explicit half of the
// forcing (k_sw_force1's expressions).  Bound by memory: levels n and n-1 of
// three fields in, the advector and three fields out (88 bytes a cell in
// FP64), where k_vip per dimension and k_sw_force1 per component read them
// three times over.  1024^2 FP64: 34 us in four launches before, 19 now; the
// whole step 111 -> 67.
template <typename T>
__global__ void __launch_bounds__(SB)
    k_sw_pre2d(int n0, int n1, int bc0, int bc1, const T *__restrict__ h,
               const T *__restrict__ q0, const T *__restrict__ q1, const T *__restrict__ hp,
               const T *__restrict__ qp0, const T *__restrict__ qp1, T eps, T k0, T k1, T ngrav,
               T tdx0, T tdx1, T half_dt, T *__restrict__ c0, T *__restrict__ c1,
               T *__restrict__ hc, T *__restrict__ qs0, T *__restrict__ qs1)
{
    const int j = blockIdx.x * SB + threadIdx.x;
    if (j >= n1) return;
    for (int i = blockIdx.y; i < n0; i += gridDim.y) {
        const int64_t t = (int64_t)i * n1 + j;
        const int64_t up = (int64_t)wrap_cell(i - 1, n0, bc0) * n1 + j;
        const int64_t dn = (int64_t)wrap_cell(i + 1, n0, bc0) * n1 + j;
        const int64_t lf = (int64_t)i * n1 + wrap_cell(j - 1, n1, bc1);
        const int64_t rt = (int64_t)i * n1 + wrap_cell(j + 1, n1, bc1);
        auto vext = [&](const T *q, const T *qp, int64_t m) {
            return T(1.5) * vel(q, h, m, eps) - T(0.5) * vel(qp, hp, m, eps);
        };
        const T u0 = vext(q0, qp0, t), u1 = vext(q1, qp1, t);
        c0[t] = k0 * (T(0.5) * (vext(q0, qp0, up) + u0));
        c1[t + i] = k1 * (T(0.5) * (vext(q1, qp1, lf) + u1));
        if (i == n0 - 1) c0[t + n1] = k0 * (T(0.5) * (u0 + vext(q0, qp0, dn)));
        if (j == n1 - 1) c1[t + i + 1] = k1 * (T(0.5) * (u1 + vext(q1, qp1, rt)));
        const T hm = h[t];
        hc[t] = hm;
        const T f0 = ngrav * hm * (h[dn] - h[up]) / tdx0;
        const T f1 = ngrav * hm * (h[rt] - h[lf]) / tdx1;
        qs0[t] = q0[t] + half_dt * f0;
        qs1[t] = q1[t] + half_dt * f1;
    }
}

// 2-D, the forcing after the advection (k_sw_force without the save)
template <typename T>
__global__ void __launch_bounds__(SB)
    k_sw_force2d(int n0, int n1, int bc0, int bc1, const T *__restrict__ h, T *__restrict__ q0,
                 T *__restrict__ q1, T ngrav, T tdx0, T tdx1, T half_dt)
{
    const int j = blockIdx.x * SB + threadIdx.x;
    if (j >= n1) return;
    for (int i = blockIdx.y; i < n0; i += gridDim.y) {
        const int64_t t = (int64_t)i * n1 + j;
        const T hm = h[t];
        const T f0 = ngrav * hm * (h[(int64_t)wrap_cell(i + 1, n0, bc0) * n1 + j] -
                                   h[(int64_t)wrap_cell(i - 1, n0, bc0) * n1 + j]) / tdx0;
        const T f1 = ngrav * hm * (h[(int64_t)i * n1 + wrap_cell(j + 1, n1, bc1)] -
                                   h[(int64_t)i * n1 + wrap_cell(j - 1, n1, bc1)]) / tdx1;
        q0[t] = q0[t] + half_dt * f0;
        q1[t] = q1[t] + half_dt * f1;
    }
}

dim3 grid2d(const Geom &g)
{
    return dim3((unsigned)cdiv(g.n[1], SB), (unsigned)(g.n[0] < 65535 ? g.n[0] : 65535));
}

unsigned blocks_for(int64_t n)
{
    int64_t b = cdiv(n, SB);
    return (unsigned)(b < 16384 ? (b > 0 ? b : 1) : 16384);
}

}  // namespace

template <typename T>
hipError_t vip_launch(const Geom &g, const T *const num[3], const T *den, const T *const nump[3],
                      const T *denp, double eps, const double k[3], T *const c[3], hipStream_t s)
{
    for (int d = 0; d < g.nd; d++) {
        int64_t e[3] = {g.n[0], g.n[1], g.n[2]};
        e[d] += 1;
        const unsigned nb = blocks_for(e[0] * e[1] * e[2]);
        if (d == 0)
            k_vip<T, 0><<<nb, SB, 0, s>>>(g, num[0], den, nump[0], denp, (T)eps, (T)k[0], c[0]);
        else if (d == 1)
            k_vip<T, 1><<<nb, SB, 0, s>>>(g, num[1], den, nump[1], denp, (T)eps, (T)k[1], c[1]);
        else
            k_vip<T, 2><<<nb, SB, 0, s>>>(g, num[2], den, nump[2], denp, (T)eps, (T)k[2], c[2]);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

template <typename T>
hipError_t sw_pre2d_launch(const Geom &g, const T *h, const T *const q[3], const T *hp,
                           const T *const qp[3], double eps, const double k[3], double grav,
                           const double dx[3], double dt, T *const c[3], T *hc, T *const qs[2],
                           hipStream_t s)
{
    if (g.nd != 2) return hipErrorInvalidValue;
    k_sw_pre2d<T><<<grid2d(g), SB, 0, s>>>((int)g.n[0], (int)g.n[1], g.bc[0], g.bc[1], h, q[0],
                                           q[1], hp, qp[0], qp[1], (T)eps, (T)k[0], (T)k[1],
                                           (T)(-grav), (T)(2.0 * dx[0]), (T)(2.0 * dx[1]),
                                           (T)(0.5 * dt), c[0], c[1], hc, qs[0], qs[1]);
    return hipGetLastError();
}

template <typename T>
hipError_t sw_force_launch(const Geom &g, const T *h, T *h_prev, T *const q[3],
                           T *const q_prev[3], double grav, const double dx[3], double dt,
                           int save, hipStream_t s)
{
    if (g.nd == 2 && !save) {
        k_sw_force2d<T><<<grid2d(g), SB, 0, s>>>((int)g.n[0], (int)g.n[1], g.bc[0], g.bc[1], h,
                                                 q[0], q[1], (T)(-grav), (T)(2.0 * dx[0]),
                                                 (T)(2.0 * dx[1]), (T)(0.5 * dt));
        return hipGetLastError();
    }
    const int64_t M = g.n[0] * g.n[1] * g.n[2];
    k_sw_force<T><<<blocks_for(M), SB, 0, s>>>(g, h, h_prev, q[0], q[1], q[2], q_prev[0],
                                               q_prev[1], q_prev[2], (T)(-grav),
                                               (T)(2.0 * dx[0]), (T)(2.0 * dx[1]),
                                               (T)(2.0 * dx[2]), (T)(0.5 * dt), save);
    return hipGetLastError();
}

template <typename T>
hipError_t sw_force1_launch(const Geom &g, int d, const T *h, T *h_prev, const T *q, T *q_prev,
                            T *out, double grav, const double dx[3], double dt, hipStream_t s)
{
    if (d < 0 || d >= g.nd || !q || !q_prev || !out) return hipErrorInvalidValue;
    const int64_t M = g.n[0] * g.n[1] * g.n[2];
    k_sw_force1<T><<<blocks_for(M), SB, 0, s>>>(g, d, h, h_prev, q, q_prev, out, (T)(-grav),
                                                (T)(2.0 * dx[d]), (T)(0.5 * dt));
    return hipGetLastError();
}

template hipError_t vip_launch<float>(const Geom &, const float *const[3], const float *,
                                      const float *const[3], const float *, double,
                                      const double[3], float *const[3], hipStream_t);
template hipError_t vip_launch<double>(const Geom &, const double *const[3], const double *,
                                       const double *const[3], const double *, double,
                                       const double[3], double *const[3], hipStream_t);
template hipError_t sw_pre2d_launch<float>(const Geom &, const float *, const float *const[3],
                                         const float *, const float *const[3], double,
                                         const double[3], double, const double[3], double,
                                         float *const[3], float *, float *const[2], hipStream_t);
template hipError_t sw_force_launch<float>(const Geom &, const float *, float *, float *const[3],
                                           float *const[3], double, const double[3], double,
                                           int, hipStream_t);
template hipError_t sw_pre2d_launch<double>(const Geom &, const double *, const double *const[3],
                                         const double *, const double *const[3], double,
                                         const double[3], double, const double[3], double,
                                         double *const[3], double *, double *const[2], hipStream_t);
template hipError_t sw_force_launch<double>(const Geom &, const double *, double *,
                                            double *const[3], double *const[3], double,
                                            const double[3], double, int, hipStream_t);
template hipError_t sw_force1_launch<float>(const Geom &, int, const float *, float *,
                                            const float *, float *, float *, double,
                                            const double[3], double, hipStream_t);
template hipError_t sw_force1_launch<double>(const Geom &, int, const double *, double *,
                                             const double *, double *, double *, double,
                                             const double[3], double, hipStream_t);

}  // namespace mp
