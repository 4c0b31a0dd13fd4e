// pass2d.hip -- the 2-D donor-cell pass, and the dispatch of the single
// corrective passes (pass2d.hpp; one file per element type and per whether
// the donor pass is folded in, so that they compile in parallel).
#include "common.hpp"
#include "kernels.hpp"

#pragma clang fp contract(on)

namespace mp {
namespace {

template <typename T> __device__ __forceinline__ T donor_update(bool kahan, T x, T d0, T d1)
{
    if (!kahan) return x - (d0 + d1);
    T s = x, c = T(0);
    kahan_add(s, c, -d0);
    kahan_add(s, c, -d1);
    return s;
}

// Donor-cell pass of a 2-D grid (eqs. upstream, F; G = 1): one thread per
// cell, a block of 256 threads per row segment (the row is wave-uniform, so
// no division per thread).  With `copy`, psi^n is also written there (for
// an in-place step whose corrective passes still need psi^n).
constexpr int DB = 256;

template <typename T>
__global__ void __launch_bounds__(DB)
    k_donor2d(int n0, int n1, int bc0, int bc1, int bpr, int kahan, const T *__restrict__ x,
              const T *__restrict__ c0, const T *__restrict__ c1, T *__restrict__ out,
              T *__restrict__ copy)
{
    const int row = blockIdx.x / bpr;
    const int j = (blockIdx.x - row * bpr) * DB + threadIdx.x;
    if (j >= n1) return;
    const int64_t r = (int64_t)row * n1;
    const int64_t rm = (int64_t)wrap_cell(row - 1, n0, bc0) * n1;
    const int64_t rp = (int64_t)wrap_cell(row + 1, n0, bc0) * n1;
    const int jm = wrap_cell(j - 1, n1, bc1), jp = wrap_cell(j + 1, n1, bc1);
    const T xc = x[r + j];
    const T u0lo = c0[r + j];
    const T u0hi = c0[(int64_t)wrap_wall(row + 1, n0, bc0) * n1 + j];
    const int64_t r1 = (int64_t)row * (n1 + 1);
    const T u1lo = c1[r1 + j];
    const T u1hi = c1[r1 + wrap_wall(j + 1, n1, bc1)];
    const T f0lo = upwind_fp(u0lo, x[rm + j], xc);
    const T f0hi = upwind_fp(u0hi, xc, x[rp + j]);
    const T f1lo = upwind_fp(u1lo, x[r + jm], xc);
    const T f1hi = upwind_fp(u1hi, xc, x[r + jp]);
    out[r + j] = donor_update(kahan != 0, xc, f0hi - f0lo, f1hi - f1lo);
    if (copy) copy[r + j] = xc;
}
}  // namespace

bool pass2d_supported(int nd, int n_iters, unsigned opts, int has_g, const int64_t n[3])
{
    (void)has_g;   // G = 1 and variable G alike
    if (nd != 2 || n_iters < 2) return false;
    if ((opts & OPT_ABS) && (opts & OPT_IGA)) return false;
    // 32-bit row / column arithmetic
    return n[0] < (1 << 30) && n[1] < (1 << 30) && n[0] * (n[1] + 1) < ((int64_t)1 << 31);
}

template <typename T>
hipError_t pass2d_launch(const Geom &g, unsigned opts, const T *x, const T *c0, const T *c1,
                         const T *psi_n, const T *G, T *y, T *w0, T *w1, hipStream_t s,
                         const PassRecord<T> &rec, int tile_rows)
{
    // psi_n NULL: the first corrective pass with the donor pass folded in
    // (x = psi^n)
    const PassArgs<T> p{g, opts, 1, {{x}, {y}, {}}, c0, c1, psi_n,
                        G, w0, w1, rec, tile_rows, s};
    return psi_n ? pass2d_go<T, false>(p) : pass2d_go<T, true>(p);
}

// the option sets of the shallow-water examples (Sect. 5.4), whose variants
// of the pass carry the saving store; another set's fields are advected by a
// launch each
bool pass2d_saves(unsigned opts)
{
    return opts == (OPT_FCT | OPT_IGA | OPT_DFL) || opts == (OPT_FCT | OPT_ABS);
}

template <typename T>
hipError_t pass2d_fields_launch(const Geom &g, unsigned opts, int nf, const PassFields<T> &fl,
                                const T *c0, const T *c1, int tile_rows, hipStream_t s)
{
    if (nf < 1 || nf > 3 || !pass2d_saves(opts)) return hipErrorInvalidValue;
    for (int f = 0; f < nf; f++)
        if (!fl.x[f] || !fl.y[f] || fl.x[f] == fl.y[f]) return hipErrorInvalidValue;
    return pass2d_go<T, true>(PassArgs<T>{g, opts, nf, fl, c0, c1, nullptr, nullptr, nullptr,
                                          nullptr, PassRecord<T>(), tile_rows, s});
}

template <typename T>
hipError_t donor2d_launch(const Geom &g, unsigned opts, const T *x, const T *c0, const T *c1,
                          T *out, T *copy, hipStream_t s)
{
    const int bpr = (int)cdiv(g.n[1], DB);
    k_donor2d<T><<<(unsigned)(bpr * g.n[0]), DB, 0, s>>>((int)g.n[0], (int)g.n[1], g.bc[0],
                                                         g.bc[1], bpr,
                                                         (opts & OPT_KAHAN) ? 1 : 0, x, c0, c1,
                                                         out, copy);
    return hipGetLastError();
}

template hipError_t donor2d_launch<float>(const Geom &, unsigned, const float *, const float *,
                                          const float *, float *, float *, hipStream_t);
template hipError_t donor2d_launch<double>(const Geom &, unsigned, const double *,
                                           const double *, const double *, double *, double *,
                                           hipStream_t);
template hipError_t pass2d_fields_launch<float>(const Geom &, unsigned, int,
                                                const PassFields<float> &, const float *,
                                                const float *, int, hipStream_t);
template hipError_t pass2d_launch<float>(const Geom &, unsigned, const float *, const float *,
                                         const float *, const float *, const float *, float *,
                                         float *, float *, hipStream_t, const PassRecord<float> &,
                                         int);
template hipError_t pass2d_fields_launch<double>(const Geom &, unsigned, int,
                                                const PassFields<double> &, const double *,
                                                const double *, int, hipStream_t);
template hipError_t pass2d_launch<double>(const Geom &, unsigned, const double *, const double *,
                                          const double *, const double *, const double *,
                                          double *, double *, double *, hipStream_t,
                                          const PassRecord<double> &, int);

}  // namespace mp
