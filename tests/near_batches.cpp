// Every regular near-field rule through the batch size of both forms of the kernel
// (built and run by tests/test_near_batches.py): prints one line per rule whose batch
// is empty or runs past the rows of its points or its 1-D basis.
#include <cstdio>
#include <initializer_list>
#include "near_rules.h"
using namespace igb;
int main() {
    for (int mx : {REG_POINTS_SMALL, REG_POINTS_MAX})
        for (int nu = 1; nu <= REG_ORDER_MAX; ++nu)
            for (int nv = 1; nv <= REG_ORDER_MAX; ++nv) {
                // (the form for more points also takes smaller source rules, beside a larger test rule)
                if (nu * nv > mx) continue;
                const int nb = regular_batch(mx, nu, nv);
                if (nb < 1 || nb > REG_BATCH_MAX || nb * regular_padded(nu * nv) > regular_batch_points(mx) ||
                    nb * (nu + nv) > REG_BASIS_ROWS)
                    std::printf("form %d, rule %d x %d: %d sources\n", mx, nu, nv, nb);
            }
    std::puts("walked");
}
