// How structured instances are cut into work (host only): strips and segments
// of the marching step, or boxes of the form with several steps per launch, and
// which of the two takes a step sooner.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "device.h"
#include "mesh.h"

namespace sdg {

// Times in us that the choice rests on, measured on this chip (256 CUs of four
// SIMDs) on cavities of 48 to 1024 cells an edge: a launch, what every round of
// boxes adds to it (the load of the state), and a row of the march or a step of
// the boxes with one, two (and, with FP32 arithmetic, three) waves on every
// SIMD, the most that the registers allow.
struct CartTimes {
    double launch, row[2], box_launch, round, step[3];
    int32_t waves;                      // of boxes on a SIMD
};
inline CartTimes cart_times(int precision)
{
    if (precision == SDUGKS_FP32DEV) return {2.5, {1.7, 2.35}, 1.8, 1.4, {1.9, 2.5, 3.3}, 3};
    return {2.5, {1.8, 2.6}, 1.8, 1.6, {2.1, 3.3, 3.3}, 2};
}
constexpr int64_t kSimds = 1024;
constexpr int32_t kWholeSteps = 1000;   // steps per launch of a mesh in one box, at most

// Time of `waves` equal waves, `at_once` of them on the chip, which take one + time[k]
// times `units` with up to k + 1 of them on a SIMD.
inline double cart_rounds(int64_t waves, int64_t at_once, double one, const double *time, double units)
{
    const int64_t most = (at_once + kSimds - 1) / kSimds, full = waves / at_once, rest = (waves % at_once + kSimds - 1) / kSimds;
    return (double)full * (one + units * time[most - 1]) + (rest > 0 ? one + units * time[rest - 1] : 0.0);
}

struct CartPlan {
    int32_t rows = 0;                   // the march: rows of a segment, at most
    int32_t threads = 0, K = 0;         // boxes: threads per box, steps per launch (0: the march)
    double us = 0.0;                    // time per step
};

inline void cart_cut(DevCart &c, int32_t rows)
{
    c.strips = (c.nx + kCartCols - 1) / kCartCols;
    c.strip_w = c.nx / c.strips;
    c.strip_more = c.nx % c.strips;
    // Where rows are whole sectors of 32 bytes (8 floats) the strips begin at sectors too, if that
    // takes at most a tenth more of them: a sector shared by two strips is written twice in part.
    // FP32 deviations: 1024 x 1024 cells 33.6 -> 31.9 us, 2048 x 2048 143 -> 128.
    const int32_t whole = kCartCols / 8 * 8, strips = (c.nx + whole - 1) / whole;
    if (c.nx % 8 == 0 && 10 * strips <= 11 * c.strips) {
        c.strip_w = ((c.nx + strips - 1) / strips + 7) / 8 * 8;
        c.strip_more = 0;
        c.strips = (c.nx + c.strip_w - 1) / c.strip_w;
    }
    c.segs = (c.ny + rows - 1) / rows;
    c.seg_h = c.ny / c.segs;
    c.seg_more = c.ny % c.segs;
    c.inv_segs = (uint32_t)std::min<uint64_t>(((uint64_t)1 << 32) / (uint64_t)c.segs, UINT32_MAX);
}

// The march over all members: segments of nearly `rows` rows each, such that
// the waves fill the SIMDs in whole rounds and are not much longer than their
// start (about three rows' time: the two rows before and after a segment take
// part of a row's work).  Long segments read few rows twice, but at a wall their
// boundary states take LDS: in FP64 eight waves of 23 rows fit a CU and seven of 38
// (2048 x 2048 cells: one round of 38 rows was planned, and took two).  Times are
// those of a state that the memory-side cache holds; a larger one is bound by memory
// whatever the cut, 2048 x 2048 cells by a factor of 2 in FP64 and 1.3 in FP32 deviations.
inline CartPlan plan_march(const std::vector<DevCart> &members, int32_t n_bc, int precision)
{
    const CartTimes t = cart_times(precision);
    CartPlan best;
    for (int32_t rows = 1; rows <= 64; rows++) {
        int64_t waves = 0;
        int32_t longest = 0;
        size_t lds = 0;
        for (const DevCart &m : members) {
            DevCart c = m;
            cart_cut(c, rows);
            waves += (int64_t)c.strips * c.segs;
            longest = std::max(longest, (c.ny + c.segs - 1) / c.segs);
            lds = std::max(lds, march_lds_bytes(c, n_bc, precision));
        }
        const int64_t at_once = (int64_t)march_waves_per_cu(march_ring_bytes(precision) + lds) * (kSimds / 4);
        const double us = t.launch + cart_rounds(waves, at_once, 0.0, t.row, longest + 3.0);
        if (best.rows == 0 || us < best.us) best = {rows, 0, 0, us};
    }
    return best;
}

// Boxes of n cells along an axis, B cells each, after K steps, with `pad` ghost
// cells at a wall (0: boxes too small).
inline int32_t cart_boxes(int32_t n, bool per, int32_t B, int32_t pad, int32_t K)
{
    if (per ? n <= B : n + 2 * pad <= B) return 1;
    const int32_t T = B - 4 * K, first = B - pad - 2 * K;
    if (T < 1) return 0;
    if (per) return (n + T - 1) / T;
    return n <= 2 * first ? 2 : 2 + (n - 2 * first + T - 1) / T;
}

// The box shape with the fewest boxes for an instance (threads 0: none fits).
inline CartBlock cart_block(const DevCart &c, int32_t threads, int32_t K)
{
    CartBlock best{};
    int64_t fewest = 0;
    for (int32_t lb = 2; lb <= 6; lb++) {
        const int32_t by = threads >> lb;
        if (by < 1) break;
        const int64_t x = cart_boxes(c.nx, c.per_x, 1 << lb, 1, K), y = cart_boxes(c.ny, c.per_y, by, 0, K);
        if (x * y == 0 || x * y > (1 << 20)) continue;
        if (best.threads == 0 || x * y < fewest) {
            best = {lb, threads, K, (int32_t)x, (int32_t)y};
            fewest = x * y;
        }
    }
    return best;
}

// Boxes over all members, or the march where that takes less time.
inline CartPlan plan_cart(const std::vector<DevCart> &members, int32_t n_bc, int precision)
{
    const CartTimes t = cart_times(precision);
    CartPlan best = plan_march(members, n_bc, precision);
    for (int32_t threads : {128, 256, 512})
        for (int32_t K : {1, 2, 3, 4, 5, 6, 32}) {      // 32: only where every mesh fits one box
            int64_t boxes = 0;
            bool fits = true;
            for (const DevCart &m : members) {
                const CartBlock b = cart_block(m, threads, K);
                if (b.threads == 0) { fits = false; break; }
                boxes += (int64_t)b.nbx * b.nby;
            }
            if (!fits) continue;
            // a workgroup of eight waves takes two on each of a CU's SIMDs, and a CU holds one,
            // with nothing beside it while it loads
            const double us = (t.box_launch + (threads == 512 ? cart_rounds((boxes + 255) / 256 * 256 * 8, 2 * kSimds, t.round + 0.6, t.step, K)
                                                              : cart_rounds(boxes * (threads / 64), t.waves * kSimds, t.round, t.step, K))) / K;
            if (us < best.us) best = {best.rows, threads, K, us};
        }
    return best;
}

}  // namespace sdg
