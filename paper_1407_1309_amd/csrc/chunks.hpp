// chunks.hpp -- how many rows of a 2-D grid one wave marches when the caller
// set none (host code only; results never depend on the choice).
#pragma once

#include <stdint.h>

namespace mp {

// What the chip holds of a kernel at once: compute units and workgroups per
// unit (from the runtime's occupancy query; the figures of a gfx950, 256
// units and one workgroup, if it fails).  For the rules that choose how much
// of a grid one workgroup takes.
struct Slots {
    int cus, per_cu;
};

// A kind of row march, one wave per strip and chunk: a chunk of th rows costs
// its wave th + extra iterations, in whole blocks of `unit`, and `lead` more
// before them.
struct March2D {
    int extra, unit, min_rows;
    double lead;
    double wait;        // time an iteration waits on its own dependencies, in
                        // units of the issue time of a wave's iteration
};

inline int64_t parts_of(int64_t n, int64_t th) { return (n + th - 1) / th; }

// Rows per chunk.  With w waves on each SIMD an iteration takes wait + w
// units of time (the part that waits on its own dependencies, and the issue
// slots the waves share).  Waves beyond what the chip holds wait for others to
// end: not quite in whole rounds, since a slot is refilled at once, so the
// price is three parts whole rounds and one part the mean load.  Priced for
// every number of waves per SIMD up to what fits and for some more rounds; the
// cheapest wins, ties to the longer chunk.  `usual` is the chunk of a fixed
// number of waves, kept unless another is priced 5 % below it, which is what
// the price is good for.
// wait: 0.375 in FP64, whose iterations fill the issue slots, 0.75 in FP32, 1
// with third-order terms; 0, and whole rounds only, for the one-pass step,
// which memory bounds.  Fitted to sweeps of 20 to 25 chunk lengths over 2562
// combinations of size (48 to 3000 a side, most of them ragged), precision,
// passes and options: the choice is 0.6 % slower than the best chunk in the
// geometric mean, takes 0.72 of `usual`'s time, and is more than 1.5 % slower
// than `usual` at 9 of them (6 % at the worst).  One wait of 1.5 for every
// kernel, whole rounds and no look at `usual`: 1.3 %, 0.72, and 157 of them
// (60 % at the worst, the one-pass step).
inline int64_t march_rows(int64_t n0, int64_t strips, const Slots &sl, const March2D &m,
                          int64_t usual)
{
    constexpr int SIMDS = 4, MORE = 8;
    const int64_t per_round = (int64_t)sl.cus * sl.per_cu, simds = (int64_t)sl.cus * SIMDS;
    const int wps = sl.per_cu >= SIMDS ? sl.per_cu / SIMDS : 1;
    if (strips < 1) strips = 1;
    auto price = [&](int64_t th) {
        const int64_t all = strips * parts_of(n0, th), rest = all % per_round;
        const double rounds = (double)(all / per_round) * (m.wait + wps) +
                              (rest ? m.wait + (double)parts_of(rest, simds) : 0.0);
        const double least = m.wait + 1.0, mean = (double)all / per_round * (m.wait + wps);
        const double load = m.wait > 0.0
                                ? 0.75 * rounds + 0.25 * (mean > least ? mean : least)
                                : rounds;
        return ((double)(parts_of(th + m.extra, m.unit) * m.unit) + m.lead) * load;
    };
    int64_t best = n0;
    double best_cost = 0.0;
    for (int k = 1; k <= wps + MORE; k++) {
        const int64_t waves = k <= wps ? k * simds : (int64_t)(k - wps + 1) * per_round;
        int64_t chunks = waves / strips;
        if (chunks < 1) chunks = 1;
        int64_t th = parts_of(n0, chunks);
        if (th < m.min_rows) th = m.min_rows;
        th = parts_of(th + m.extra, m.unit) * m.unit - m.extra;
        const double cost = price(th);
        if (k == 1 || cost < best_cost || (cost == best_cost && th > best)) {
            best_cost = cost;
            best = th;
        }
    }
    if (price(usual < n0 ? usual : n0) <= 1.05 * best_cost) best = usual;
    return best < n0 ? best : n0;
}

// about `waves` waves in all, at least `least` rows
inline int64_t usual_rows(int64_t n0, int64_t strips, int64_t waves, int64_t least)
{
    const int64_t chunks = waves / (strips > 0 ? strips : 1);
    const int64_t th = parts_of(n0, chunks > 0 ? chunks : 1);
    return th < least ? least : th;
}

// shortest chunk of a fused step that also forms the step's diagnostics: their
// partials' buffer is sized by it
constexpr int FUSED2D_DIAG_ROWS = 16;

// The fused step of n_iters passes: a chunk runs th + 2 LAG + 1 iterations,
// of which the warm-up ones (W) do part of the work.
inline int64_t fused2d_rows(int64_t n0, int64_t strips, const Slots &sl, int n_iters, bool f64,
                            bool diag)
{
    const int np = n_iters - 1, lag = 1 + 2 * np, w = np == 0 ? 0 : 4 * np - 1;
    const March2D m{2 * lag + 1 - w, n_iters <= 3 ? 4 : 8, diag ? FUSED2D_DIAG_ROWS : 4, 0.75 * w,
                    np == 0 ? 0.0 : f64 ? 0.375 : 0.75};
    return march_rows(n0, strips, sl, m, usual_rows(n0, strips, 2048, 16));
}

// The single pass: a chunk runs th + 5 iterations (one more with third-order
// terms, in blocks of 8), of which the first four do part of the work.
inline int64_t pass2d_rows(int64_t n0, int64_t strips, const Slots &sl, bool tot, bool f64)
{
    const March2D m{tot ? 2 : 1, tot ? 8 : 4, 1, 2.0, tot ? 1.0 : f64 ? 0.375 : 0.75};
    const int all = m.extra + 4;
    const int64_t usual = usual_rows(n0, strips, 4096, 11);
    return march_rows(n0, strips, sl, m, parts_of(usual + all, m.unit) * m.unit - all);
}

}  // namespace mp
