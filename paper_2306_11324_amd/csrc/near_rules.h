// Limits of the regular near-field rules: the orders and points that near_classify
// gives a pair, and the batches in which near_regular takes a rule's source elements
// (plain C++, so that the bounds can be walked without a device).
#pragma once

namespace igb {

constexpr int REG_ORDER_MAX = 12;      // Gauss order per direction
constexpr int REG_POINTS_MAX = 100;    // Gauss points per element
constexpr int REG_POINTS_SMALL = 36;   // rules of up to this many points (6 x 6) take the form with less LDS
constexpr int REG_BATCH_MAX = 16;      // source elements per batch
constexpr int REG_BASIS_ROWS = 64;     // 1-D basis rows (u and v nodes of every source) per batch

// points rounded up to the matrix cores' steps of 4
constexpr int regular_padded(int points) { return (points + 3) & ~3; }

// rows of the batch's source points in the form for rules of up to mx points
constexpr int regular_batch_points(int mx) { return mx <= 64 ? 64 : mx; }

// source elements of a rule with nyu x nyv source points per batch: as many as the
// point rows and the 1-D basis rows hold (a rule of 2 x 4 points has 8 points and 6
// basis rows a source: 12 sources fill the larger form's points, but 10 its basis rows)
constexpr int regular_batch(int mx, int nyu, int nyv) {
    int nb = regular_batch_points(mx) / regular_padded(nyu * nyv);
    if (nb > REG_BASIS_ROWS / (nyu + nyv)) nb = REG_BASIS_ROWS / (nyu + nyv);
    return nb < REG_BATCH_MAX ? nb : REG_BATCH_MAX;
}

}  // namespace igb
