// Assembly on a host-only context while one host allocation after another fails (built
// and run by tests/test_assembly_without_memory.py, linked with the library): this
// program's operator new throws at the chosen allocation, whatever thread makes it, and
// assemble_nearfield must return an error or succeed, then succeed again.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>
#include "igafmm.h"

static std::atomic<long> count{0}, fail_at{-1};
void* operator new(std::size_t n) {
    if (fail_at.load() >= 0 && count.fetch_add(1) == fail_at.load()) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main() {
    // the six bilinear faces of a cube, outward
    const double f[6][3][3] = {{{1, 0, 0}, {0, 1, 0}, {0, 0, 1}},  {{-1, 0, 0}, {0, 0, 1}, {0, 1, 0}},
                               {{0, 1, 0}, {0, 0, 1}, {1, 0, 0}},  {{0, -1, 0}, {1, 0, 0}, {0, 0, 1}},
                               {{0, 0, 1}, {1, 0, 0}, {0, 1, 0}},  {{0, 0, -1}, {0, 1, 0}, {1, 0, 0}}};
    const double knots[4] = {0, 0, 1, 1};
    double net[6][2][2][4];
    igb_patch P[6];
    for (int j = 0; j < 6; ++j) {
        for (int v = 0; v < 2; ++v)
            for (int u = 0; u < 2; ++u) {
                for (int c = 0; c < 3; ++c)
                    net[j][v][u][c] = f[j][0][c] + (2 * u - 1) * f[j][1][c] + (2 * v - 1) * f[j][2][c];
                net[j][v][u][3] = 1;
            }
        P[j] = igb_patch{1, 1, 2, 2, knots, knots, &net[j][0][0][0]};
    }
    igb_ctx ctx;
    igb_geom g;
    if (igb_ctx_create(IGB_HOST_ONLY, 0, &ctx) || build_geometry(ctx, P, 6, 3, 1, &g)) return 1;
    igb_op_params prm{};
    prm.kappa = 2;
    prm.q = 3;
    prm.eta_adm = 1.6;
    int refused = 0;
    for (int separate = 0; separate < 2; ++separate)
        for (int bc = 0; bc < 2; ++bc) {
            prm.bc = bc;
            prm.separate = separate;
            prm.leaf_depth = separate ? 1 : 3;   // (3: all pairs near, enough for the plan's threads)
            igb_op op;
            count = 0;
            fail_at = 1L << 40;
            if (assemble_nearfield(ctx, g, &prm, &op)) return 1;
            fail_at = -1;
            igb_op_destroy(op);
            const long n = count;
            // every early and late allocation, and 150 between them
            for (long k = 0; k < n; k += k < 40 || k > n - 20 ? 1 : 1 + n / 150) {
                count = 0;
                fail_at = k;
                op = nullptr;
                const igb_status st = assemble_nearfield(ctx, g, &prm, &op);
                fail_at = -1;
                if (st == 0) {
                    igb_op_destroy(op);   // (a thread that could not be had is done without)
                } else {
                    if (st != IGB_ERR_ARG || op || !std::strstr(igb_last_error(), "memory")) {
                        std::printf("allocation %ld of %ld: status %d, %s\n", k, n, st, igb_last_error());
                        return 2;
                    }
                    ++refused;
                }
            }
            if (assemble_nearfield(ctx, g, &prm, &op)) return 3;
            igb_op_destroy(op);
        }
    igb_geom_destroy(g);
    igb_ctx_destroy(ctx);
    std::printf("%d refused\n", refused);
    return refused > 100 ? 0 : 4;
}
