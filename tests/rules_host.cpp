// The kernels' arithmetic rules (eik_rules.hpp), compiled for the host.
#include <stdint.h>

#include "eik_rules.hpp"

using namespace eik;

extern "C" {

#define EIK_SHAPES(X) \
    X(32, 8, 4) X(16, 8, 8) X(8, 8, 8) X(64, 4, 4) X(16, 8, 4) X(8, 8, 4) X(8, 4, 4) \
    X(32, 32, 1) X(64, 16, 1) X(128, 8, 1) X(16, 16, 1) X(16, 8, 1)

int rule_offsets_fit_32(int tx, int ty, int tz, int64_t nx, int64_t plane) {
#define EIK_ONE(a, b, c) \
    if (tx == a && ty == b && tz == c) return offsets_fit_32<a, b, c>(nx, plane);
    EIK_SHAPES(EIK_ONE)
#undef EIK_ONE
    return -1;
}

int rule_few_tiles(int tx, int ty, int tz, int what, int64_t most, int64_t total) {
#define EIK_ONE(a, b, c)                                    \
    if (tx == a && ty == b && tz == c) {                    \
        using F = FewTiles<a, b, c>;                        \
        return what == 0 ? F::solve(most, total) : (what == 1 ? F::rect(total) : F::adjoint(most, total)); \
    }
    EIK_SHAPES(EIK_ONE)
#undef EIK_ONE
    return -1;
}

int rule_claim_window(int lookahead, int strict, int64_t idle) { return claim_window(lookahead, strict != 0, idle); }

int rule_last_not_above(int n, const int* values, int bound, int* rounds) {
    *rounds = 0;
    return last_not_above(n, [&](int first, int step, int m) {
        ++*rounds;
        int k = 0;
        for (long long i = 0; i < 64 && i * step < m; ++i) k += values[first + i * step] <= bound;
        return k;
    });
}

uint64_t rule_stall_ticks() { return kStallTicks; }
StallWatch* stall_new() { return new StallWatch(); }
void stall_delete(StallWatch* w) { delete w; }
int stall_gives_up(StallWatch* w, uint64_t progress, int another, uint64_t now) {
    return w->gives_up(progress, another != 0, now);
}

}  // extern "C"
