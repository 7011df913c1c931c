// Which form of a solve a group of problems takes: the on-chip or the streaming scaled solve, and the workgroup size of
// the FP64 fused solve.  Each form is priced per problem by a line fitted to measurements and the problems are put on
// the workgroups that are resident at once, longest first, as the device's queue does; the shorter schedule wins.
#include <algorithm>
#include <functional>
#include <vector>

#include "ssp_host.h"

namespace ssp {

namespace {

// Jobs of these costs, longest first, each on the machine that is free first: when the last one ends, and bounds of that
// which need no walk over the jobs.
struct Schedule {
    std::vector<double> cost;
    int machines;
    double sum = 0.0;
    explicit Schedule(int m) : machines(std::max(m, 1)) {}
    void add(double c) {
        cost.push_back(c);
        sum += c;
    }
    double least() const { return cost.empty() ? 0.0 : std::max(cost[0], sum / machines); }
    double most() const { return cost.empty() ? 0.0 : cost[0] + sum / machines; }
    double end() const {
        std::vector<double> free(cost.begin(), cost.begin() + std::min<size_t>(cost.size(), machines));
        if (free.empty()) return 0.0;
        std::make_heap(free.begin(), free.end(), std::greater<double>());  // the machine that is free first on top
        for (size_t j = free.size(); j < cost.size(); ++j) {
            std::pop_heap(free.begin(), free.end(), std::greater<double>());
            free.back() += cost[j];
            std::push_heap(free.begin(), free.end(), std::greater<double>());
        }
        return *std::max_element(free.begin(), free.end());
    }
};

// One problem of N knots in microseconds.  On chip, a workgroup per CU: a start, then a solve that grows with the knots,
// faster past the `held` ones in registers.  Streaming, three workgroups per CU: a solve that grows with the steps of
// `step` knots and with the knots.  Short horizons converge in fewer iterations: both solves are scaled by min(N, 5) / 5.
struct ScaledCost {
    int nx, step, held;
    double chip0, chip, chip_knot, chip_more, stream, stream_step, stream_knot;
};
constexpr ScaledCost kScaledCost[] = {{6, 40, 160, 1, 73, 0.67, 1.05, 23, 29, 0.8},
                                      {14, 16, 128, 7, 61, 0.67, 1.5, 24, 54, 2.4},
                                      {26, 8, 32, 17, 51, 3.4, 4.2, 33, 60, 11}};

}  // namespace

// The lines were fitted to 633 measured pairs (symmetric stair, block-Jacobi and degree 3 at nx 6, 14, 26; 1 to 768
// knots, uniform and ragged; 16 to 4096 problems): the form they choose is at most 5% slower than streaming and 14%
// slower than the better one at any of them.  On chip and streaming, us: nx 14, 4096 problems of 16 knots 1166 and 625,
// of 32 1299 and 1239, of 64 1712 and 2275; 256 of 16 104 and 128; nx 26, 4096 of 8 1454 and 872, of 16 1700 and 1730;
// 2048 of 64 2097 and 3200; 512 of 8 225 and 186; nx 6, 256 of 32 113 and 100, of 64 129 and 160; 512 of 128 321 and 286;
// 640 of 32 to 256 428 and 449, 1365 781 and 513.
//
// `too_long` leading problems stream in any case, and the on-chip grid follows them on the group's stream, so a few of
// them would hold up all others: 16 problems of 400 knots before 480 of 300 at nx 26 take 8.2 ms, 256 of 400 before 256 of
// 300 7.7 and 6.2 when all stream, 600 of 400 before 600 of 200 10.2 and 10.4.  (On a stream of its own the on-chip grid
// overlaps them, 5.95 ms for the first, but only where the runtime gives the two streams different hardware queues: in a
// process with many streams it took 8.2 again.)
bool chip_pays(int nx, const int32_t *N, int count, int too_long, int cus) {
    const ScaledCost *c = nullptr;
    for (const auto &q : kScaledCost)
        if (q.nx == nx) c = &q;
    if (!c || too_long >= count) return false;
    Schedule chip(cus), all(3 * cus), longest(3 * cus);
    for (int j = 0; j < count; ++j) {
        const double n = N[j], early = std::min(n, 5.0) / 5.0;
        const double stream =
            early * (c->stream + c->stream_step * ((N[j] + (int64_t)c->step - 1) / c->step) + c->stream_knot * n);
        all.add(stream);
        if (j < too_long)
            longest.add(stream);
        else
            chip.add(c->chip0 + early * (c->chip + c->chip_knot * std::min<double>(n, c->held) +
                                         c->chip_more * std::max<double>(n - c->held, 0)));
    }
    if (longest.most() + chip.most() <= all.least()) return true;
    if (longest.least() + chip.least() > all.most()) return false;
    return longest.end() + chip.end() <= all.end();
}

// A step of the fused pass costs about the same at any state size, 1.07 and 1.6 times as much with 256 and 512 threads
// as with 128, and holds more knots then; a CU holds 3 to 6, 2 to 3 and 1 of these workgroups.  Of 416 measured cases
// (nx 4 to 31, 1 to 128 knots, 16 to 4096 problems) the choice is at most 17% slower than the best one, and 10% at all
// but two of them.  128, 256 and 512 threads in ms: nx 26, 1024 problems of 128 knots and condition 1e6 156, 120 and 53,
// 512 of 4 knots 0.418, 0.267 and 0.376, 4096 of 2 0.584, 0.797 and 1.729; nx 14, 4096 of 4 0.522, 0.907 and 1.964,
// 16 of 128 2.96, 1.59 and 0.81; nx 6, 512 of 32 0.266, 0.172 and 0.312, 16 of 128 0.729, 0.471 and 0.321.
int fused_fp64_threads(int nx, const int32_t *N, int count, int cus, const int32_t *resident) {
    int best = 128;
    double shortest = 0.0;
    for (int t : {128, 256, 512}) {
        const int lds = pcg2_lds(nx, false, t), knots = lds ? pcg2_steps_for(nx, false, t, lds) : 0;
        if (knots < 1) continue;
        Schedule q(cus * std::max(resident[t >> 8], 1));
        for (int j = 0; j < count; ++j)
            q.add((t == 128 ? 1.0 : t == 256 ? 1.07 : 1.6) * ((N[j] + (int64_t)knots - 1) / knots));
        if (shortest > 0.0 && q.least() >= shortest) continue;
        const double end = q.end();
        if (shortest == 0.0 || end < shortest) {
            shortest = end;
            best = t;
        }
    }
    return best;
}

}  // namespace ssp
