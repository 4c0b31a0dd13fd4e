// resident1d.hip -- FP64 instances of the 1-D steps (line1d.hpp) and the
// rules that choose their launch shapes.
#include "line1d.hpp"

namespace mp {

int line_radius(int n_iters, unsigned opts)
{
    const int per = ((opts & OPT_FCT) ? 2 : 1) + ((opts & OPT_TOT) ? 1 : 0);
    return 1 + (n_iters - 1) * per;
}

int line_own(int radius, int K) { return (WAVE - 2 * line_halo_lanes(radius, K)) * K; }

bool resident1d_supported(int nd, int64_t n, int dtype_is_f64, int has_g, int two_fields)
{
    // The grids that run every step of a call in one launch, in place (what
    // KERNEL_FUSED admits, and where the cancel flag is read once a call).
    // One workgroup's waves hold 3328 FP64 or 7424 FP32 cells at the largest
    // radius; the bound is lower, that of a kernel that kept nine fields in
    // LDS, so that the same grids run this way as did with it.  It is not
    // where the two ways cross: one workgroup is the faster one for a few
    // steps, on either side of it, and tiles are for many.  us per call,
    // limiter, two passes, one workgroup / tiles: 2275 cells FP64 1 step 9.3 /
    // 11.7, 5 steps 15 / 12, 20 steps 50 / 13, 100 steps 237 / 51; 1000 cells
    // 1 step 9.0 / 11.6, 20 steps 28 / 13, 100 steps 131 / 50; 4550 cells
    // FP32 1 step 10.2 / 11.7, 100 steps 352 / 45; 6000 cells FP32 1 step
    // 12.6 / 11.4.
    if (nd != 1 || n < 1 || n > (1 << 20)) return false;
    const size_t fields = 9 + (has_g ? 1 : 0) + (two_fields ? 1 : 0);
    return (dtype_is_f64 ? 8 : 4) * (fields * (size_t)n + 4) <= 160 * 1024;
}

LineShape line1d_whole(int64_t n, int n_iters, unsigned opts)
{
    const int radius = line_radius(n_iters, opts);
    LineShape sh{1, 0, (int)n, 0};
    for (; sh.K < 8; sh.K *= 2)
        if (cdiv(n, line_own(radius, sh.K)) <= LINE_WAVES) break;
    sh.waves = (int)cdiv(n, line_own(radius, sh.K));
    return sh;
}

static LineShape tiled_shape(int64_t n, int f64, int n_iters, unsigned opts, int fields,
                             int n_steps, int *launches)
{
    // cost in microseconds: a launch, a step's chain of dependent operations
    // and its barrier, and the issue of a step's operations for one cell per
    // lane of one wave on a SIMD
    const double LAUNCH = 5.0, COPY = 6.0, CHAIN = 0.4;
    const double issue = (f64 ? 0.2 : 0.12) * fields * (n_iters > 1 ? n_iters - 1 : 1) *
                         ((opts & OPT_FCT) ? 1.0 : 0.6);
    const int radius = line_radius(n_iters, opts);
    static const int64_t cus = slots_of(nullptr, 0).cus;
    LineShape best{0, 0, 0, 0};
    double best_cost = 0.0;
    for (int L = 1; L <= n_steps; L += L == 1 ? 1 : 2) {
        // an even number of launches ends in the caller's buffer
        const int steps = (int)cdiv(n_steps, L);
        const int64_t halo = (int64_t)steps * radius;
        if (halo >= n) continue;
        for (int K = 1; K <= (f64 ? 4 : 8); K *= 2) {
            const int64_t own = line_own(radius, K), room = LINE_WAVES * own - 2 * halo;
            if (room < 1) continue;
            const int64_t r0 = cdiv(n, cus * room);        // rounds that fit
            for (int64_t r = r0; r < r0 + 8; r++) {
                const int64_t tile = cdiv(n, cus * r), waves = cdiv(tile + 2 * halo, own);
                if (waves > LINE_WAVES) continue;
                const double cost = L * LAUNCH + (L == 1 ? COPY : 0.0) +
                                    n_steps * (CHAIN + K * issue * (double)cdiv(r * waves, 4));
                if (best.K == 0 || cost < best_cost) {
                    best_cost = cost;
                    best = LineShape{K, (int)waves, (int)tile, (int)halo};
                    *launches = L;
                }
            }
        }
        if (best.K && L * LAUNCH > best_cost) break;
    }
    return best;
}

LineShape line1d_tiled(int64_t n, int f64, int n_iters, unsigned opts, int fields, int n_steps,
                       int *launches)
{
    // the last choice, kept by each thread (see ChunkMemo)
    struct Memo {
        int64_t n = -1;
        int f64, n_iters, fields, n_steps, launches;
        unsigned opts;
        LineShape sh;
    };
    static thread_local Memo m;
    if (m.n != n || m.f64 != f64 || m.n_iters != n_iters || m.opts != opts ||
        m.fields != fields || m.n_steps != n_steps) {
        m = Memo{n, f64, n_iters, fields, n_steps, 0, opts, LineShape{}};
        m.sh = tiled_shape(n, f64, n_iters, opts, fields, n_steps, &m.launches);
    }
    *launches = m.launches;
    return m.sh;
}

template hipError_t line1d_launch<double>(const LineShape &, const LineArgs<double> &, int,
                                          const double *, const double *, double *, double *,
                                          hipStream_t);

}  // namespace mp
