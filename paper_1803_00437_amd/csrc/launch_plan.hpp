// Which launches n consecutive steps of a grid are dealt to.  Host arithmetic only, done in full at
// creation (the times of a launch) and in a few operations per call (the deal).  A step can be taken
// by three kinds of launches, all with the same bits:
//   one    the sweep, one step per launch
//   fused  the sweep of several steps per launch (fd_fused.hip, mrt.hip)
//   tiles  tiles held in registers for several steps (fd_tile.hip, mrt.hip)
// and the fastest depends on the grid and on n: tiles and fused sweeps spend their start, their loads
// and their halo once per launch, so they lose to single steps where n leaves them one step each.
// Measured (us per step): 1024^2 FP64 3-point, n = 1 or 2: one 14.1, tiles 20; n = 50: one 14.1, fused
// 12.1, tiles 12.6.  384^2 FP32 MRT: 4.6 and 6.9; n = 50: one 4.6, tiles 1.9.  800^2 FP64 5-point, any
// n: one 10.1, fused 11.1, tiles 13.6.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace fdlbm {

constexpr int MAX_FUSED = 5;

// Time of one launch in us: of one step, and of the fused sweep of k steps (with the rows per wavefront
// that it takes); most: steps that one launch may take.
struct LaunchTimes {
    int most = 1;
    double one = 0.0, fused[MAX_FUSED + 1] = {};
    int rows[MAX_FUSED + 1] = {};
};

// Small and medium grids: a block advances a tile of 64 cols columns by 16 rows rows up to `steps`
// steps in registers (an odd number: see deal_tiles()).  steps = 0: no tiles.
struct TileShape {
    int cols, rows;
};
struct TilePlan {
    int cols = 0, rows = 0, steps = 0;
};

// Time of a launch of tiles.  A block's launch, loads and stores take start_us and 0.85 us (FP64 1.2)
// per row and column of a lane; a step takes 0.3 us and row_us per row and column of a lane.  A compute
// unit gets one block of 256 after the other, two at once where the shape's registers and its LDS
// (lds bytes per column of a lane, of 160 KB) allow: FP64 with 5-point differences or walls takes one.
// reach: rows and columns a step loses on each side.  floor_us: a launch that is bound by memory.
// Measured against the estimate (us per step): 64^2 FP64 2.3 (2.4), 256^2 FP32 2.3 (2.4), 1024^2 6.7
// (7.4), 1001 x 777 5-point 9.0 (9.0), where the sweep takes 4.5, 6.1, 10.2 and 12.
struct TileCost {
    int nx = 0, ny = 0, reach = 1, elem_bytes = 4;
    size_t lds = 0;
    double row_us = 1.0, start_us = 2.5, floor_us = 0.0;
    // of `steps` steps; negative: the halo leaves nothing to store
    double us(TileShape s, int steps) const
    {
        const int cols = 64 * s.cols - 2 * reach * steps, rows = 16 * s.rows - 2 * reach * steps;
        if (cols < 1 || rows < 1) return -1.0;
        const int64_t blocks = (int64_t)((nx + cols - 1) / cols) * ((ny + rows - 1) / rows);
        const int area = s.cols * s.rows;
        const bool two = area * elem_bytes <= 8 && 2 * lds * s.cols <= 160 * 1024;
        const int64_t each = (blocks + 255) / 256, rounds = two ? (each + 1) / 2 : each;
        const double start = start_us + 0.2 * area * (elem_bytes == 8 ? 6 : 4.25) + 0.3 * steps;
        return std::max(floor_us, double(rounds) * start + double(each) * steps * area * row_us);
    }
};

// The fastest shape and number of steps, or none if the sweep's `sweep_us` (per step) is less.
inline TilePlan plan_tiles(const TileCost &c, const TileShape *shapes, int count, int most, double sweep_us)
{
    TilePlan best;
    double best_us = 0.95 * sweep_us;
    for (int i = 0; i < count; ++i)
        for (int steps = 1; steps <= most; steps += 2) {
            const double us = c.us(shapes[i], steps) / steps;
            if (us < 0.0) break;
            if (us < best_us) {
                best_us = us;
                best.cols = shapes[i].cols;
                best.rows = shapes[i].rows;
                best.steps = steps;
            }
        }
    return best;
}

// `n` steps in launches of five, three, two and one steps, the largest first; or, where `tiles` is not
// zero, in so many launches of tiles, the first `high` of `low` + 2 steps and the others of `low`.
struct Deal {
    int64_t fives = 0, threes = 0, twos = 0, ones = 0;
    int64_t tiles = 0, high = 0;
    int low = 0;
    int64_t count() const { return tiles ? tiles : fives + threes + twos + ones; }
    int steps(int64_t i) const
    {
        if (tiles) return i < high ? low + 2 : low;
        return i < fives ? 5 : i < fives + threes ? 3 : i < fives + threes + twos ? 2 : 1;
    }
};

// In launches of up to `most` steps.  A launch reads one state buffer and writes the other whatever its
// steps, and the current state has to lie in state_a after an even number of steps: launches of five,
// three and one steps keep that, those of two come in pairs.  One or two fives give way where that
// leaves no single steps.
inline Deal deal_steps(int64_t n, int most)
{
    Deal l;
    if (most >= 5) {
        l.fives = n / 5;
        for (int64_t back = 0; back <= 2 && back <= n / 5; ++back)
            if ((n % 5 + 5 * back) % 3 == 0) {
                l.fives -= back;
                break;
            }
        n -= 5 * l.fives;
    }
    if (most >= 3) l.threes = n / 3;
    if (most == 2) l.twos = n / 4 * 2;
    l.ones = n - 3 * l.threes - 2 * l.twos;
    return l;
}

// In launches of tiles of up to `most` steps (an odd number): odd numbers of steps, as even as they can
// be, and as many launches as keep the buffer's parity.
inline Deal deal_tiles(int64_t n, int most)
{
    Deal l;
    l.tiles = (n + most - 1) / most;
    l.tiles += (l.tiles ^ n) & 1;
    l.low = int(n / l.tiles);
    l.low -= l.low % 2 == 0;
    l.high = (n - l.tiles * l.low) / 2;
    return l;
}

// The fastest deal of n steps.  The estimates miss by up to 10 %, so where two kinds come close the
// one that is more often the faster counts as it: the fused sweep up to 16 % behind single steps,
// tiles up to 4 % behind either.  Of 1032 grids and schemes timed, 146 were slower than in single steps
// for n = 1 and 2 and 16 for n = 50 (by up to 1.8 and 1.6 times) when the kind was that of the fastest
// long run; by this rule one (6 %) and three (4 %).
inline Deal deal(int64_t n, const LaunchTimes &t, const TilePlan &p, const TileCost &c)
{
    Deal ones;
    ones.ones = n;
    Deal best = deal_steps(n, t.most);
    double best_us = double(best.ones) * t.one + double(best.twos) * t.fused[2] + double(best.threes) * t.fused[3] +
                     double(best.fives) * t.fused[5];
    if (best_us > 1.16 * double(n) * t.one) {
        best = ones;
        best_us = double(n) * t.one;
    }
    if (p.steps > 0) {
        const Deal l = deal_tiles(n, p.steps);
        const TileShape s{p.cols, p.rows};
        const double us = double(l.tiles - l.high) * c.us(s, l.low) + (l.high ? double(l.high) * c.us(s, l.low + 2) : 0.0);
        if (us < 1.04 * std::min(best_us, double(n) * t.one)) best = l;
    }
    return best;
}

// The batch: launches of three, two and one steps of all its instances, the fastest of three deals: threes
// with two or four twos in place of single steps, twos in pairs, or single steps (each has to be 5 %
// faster by the estimates than the one before).  Every launch changes the buffer, and each deal keeps the
// parity of as many single steps.  Measured (us per step, one, two and three at once): FP32 8 x 1024^2 46,
// 37, 40; FP16 of widths that are multiples of four, whose one-step kernel takes four columns per lane
// instead of two, 37, 39, 43, but other FP16 widths 24, 17, 17; FP64 8 x (64 x 4000) 27, 28, 33.
inline Deal deal_batch(int64_t n, const LaunchTimes &t)
{
    Deal a, b, c;
    a.threes = n / 3;
    if (n % 3 == 1 && a.threes >= 1) {
        a.threes -= 1;
        a.twos = 2;
    } else if (n % 3 == 2 && a.threes >= 1) {
        a.twos = a.threes >= 2 ? 4 : 2;
        a.threes -= a.threes >= 2 ? 2 : 1;
    }
    a.ones = n - 3 * a.threes - 2 * a.twos;
    b.twos = n / 4 * 2;
    b.ones = n - 2 * b.twos;
    c.ones = n;
    auto us = [&](const Deal &d) {
        return double(d.threes) * t.fused[3] + double(d.twos) * t.fused[2] + double(d.ones) * t.one;
    };
    const Deal &ab = us(b) < 0.95 * us(a) ? b : a;
    return us(c) < 0.95 * us(ab) ? c : ab;
}

}  // namespace fdlbm
