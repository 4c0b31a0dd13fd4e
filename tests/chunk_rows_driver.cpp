// Reads lines "kind n0 strips cus per_cu passes f64 diag" (kind 0: the fused
// 2-D step, 1: the single pass, with passes = 1 for third-order terms) and
// prints the rows per chunk the library would choose.
#include <cstdio>

#include "chunks.hpp"

int main()
{
    long long kind, n0, strips, cus, per_cu, passes, f64, diag;
    while (std::scanf("%lld %lld %lld %lld %lld %lld %lld %lld", &kind, &n0, &strips, &cus, &per_cu,
                      &passes, &f64, &diag) == 8) {
        const mp::Slots sl{(int)cus, (int)per_cu};
        std::printf("%lld\n", (long long)(kind == 0 ? mp::fused2d_rows(n0, strips, sl, (int)passes,
                                                                      f64 != 0, diag != 0)
                                                    : mp::pass2d_rows(n0, strips, sl, passes != 0,
                                                                      f64 != 0)));
    }
    return 0;
}
