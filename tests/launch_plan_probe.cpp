// Prints how steps are dealt to launches, for tests/test_launch_plan.py: per line of input
//   stencil (9: MRT) dtype walls force disk nx ny n
//   0 and the times of a batch's launches of one, two and three steps, 0 0 0, n
// one line: tile columns, rows and steps, then the launches of n steps: tiles, fives, threes, twos, ones,
// and the steps and launches they add up to.
#include <cstdio>

#include "../paper_1803_00437_amd/csrc/internal.hpp"

using namespace fdlbm;

int main()
{
    int st, dt, walls, force, disk, nx, ny;
    long long n;
    while (std::scanf("%d %d %d %d %d %d %d %lld", &st, &dt, &walls, &force, &disk, &nx, &ny, &n) == 8) {
        const double f = force ? 1e-5 : 0.0;
        LaunchTimes t;
        TilePlan p;
        TileCost c;
        Deal d;
        if (st == 0) {
            t.one = dt;
            t.fused[2] = walls;
            t.fused[3] = force;
        } else if (st == 9) {
            const MrtArgs a{nx, ny, walls, dt, 1.1, 1.5, 1.2, 1.3, f, 0.0, FDLBM_KERNEL_AUTO, 0, 0.5};
            t = mrt_launch_times(a);
            c = mrt_tile_cost(a);
            p = mrt_tile_plan(a, t);
        } else {
            const FdArgs a{nx, ny, st, walls, dt, 1.5, 1.0, f, 0.0, 0.5};
            t = fd_launch_times(a);
            c = fd_tile_cost(a);
            p = fd_tile_plan(a, t, disk != 0);
        }
        if (disk) t.most = 1;
        d = st == 0 ? deal_batch(n, t) : disk && p.steps > 0 ? deal_tiles(n, 1) : deal(n, t, p, c);
        long long sum = 0;
        for (int64_t i = 0; i < d.count(); ++i) sum += d.steps(i);
        std::printf("%d %d %d %lld %lld %lld %lld %lld %lld %lld\n", p.cols, p.rows, p.steps, (long long)d.tiles,
                    (long long)d.fives, (long long)d.threes, (long long)d.twos, (long long)d.ones, sum,
                    (long long)d.count());
    }
    return 0;
}
