// FD-LBM and LW-ACM steps of one grid, K time steps per launch (the mapping is described in
// fd_fused_body.hpp): dispatch over storage, stencil, walls, force and width, and the rows per
// wavefront.
//
// Measured (us per step, one by one and here): FP32 8192^2 294 and 190, now bound by instruction
// issue (94 % of the rate at 2.4 GHz; 105 instructions per node and step of which the halo lanes, the
// part-filled last strip and the rows formed twice are 10); FP64 4096^2 148 and 98 (80 % busy at a
// clock that falls to 2.1-2.2 GHz); FP16 6002 x 4095 89 and 76; walls and force 16384 x 1024 FP32 82
// and 60; LW-ACM 8192^2 FP32 283 and 123; 5-point 1001 x 777 FP32 22.7 and 12.8.
#include <algorithm>

#include "fd_fused_body.hpp"
#include "internal.hpp"

namespace fdlbm {
namespace {
using namespace sweep;

template <typename T, int CPL, int ST, bool WALLS, bool FORCE, int AM, int K, int KR, int KC>
__global__ void __launch_bounds__(64 * WV, fused_waves<ST>()) fd_fused_kernel(FusedArgs<T, K> a)
{
    using C = typename Storage<T>::C;
    constexpr int H = Stencil<ST>::H;
    using G = FusedStrip<CPL, H, K>;
    constexpr int nslots = fused_lds_slots<H, WALLS, K, KR, KC>();
    __shared__ Group<C, CPL> lds[nslots > 0 ? WV : 1][nslots > 0 ? nslots : 1][64];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.x * WV + wv;
    if (tile >= a.ntiles) return;  // uniform over the wavefront; there is no barrier
    const int band = tile / a.strips_x, sx = tile - band * a.strips_x;
    int x0 = sx * a.stride;
    if ((AM == AM_UNAL || AM == AM_SEAM) && sx == a.strips_x - 1 && a.nx > G::S) x0 = a.nx - G::S;
    const int xl = x0 - G::P * CPL + CPL * lane;
    const LaneCols<CPL, AM> lc = make_lane_cols<T, CPL, AM>(xl, a.nx, lane >= G::P && lane < 64 - G::P);
    const int y0 = band * a.rows, y1 = min(y0 + a.rows, a.ny);
    Group<C, CPL>(*ldsw)[64] = lds[nslots > 0 ? wv : 0];
    if constexpr (WALLS)
        if (band == 0) {
            fused_tile<-1, T, CPL, ST, WALLS, FORCE, AM, K, KR, KC>(a, ldsw, lane, xl, lc, y0, y1);
            return;
        }
    fused_tile<1, T, CPL, ST, WALLS, FORCE, AM, K, KR, KC>(a, ldsw, lane, xl, lc, y0, y1);
}

// Rows per wavefront: as for the fused MRT launch, the time goes as the wavefronts each SIMD gets
// times the rows each of them forms (R + 2 + (K - 1) (H + 1) per stage on average).
// With walls no band may reach both: the first has to be K (H + 1) rows from the top, the others as
// far from the bottom.
int fused_rows(int strips_x, int ny, int K, int H, bool walls, int waves_per_simd)
{
    const int least = walls ? K * (H + 1) : 1, most = walls ? ny - least : ny;
    int best = least;
    long best_cost = -1;
    for (int rows = least; rows <= 256 && rows <= most; ++rows) {
        const long waves = (long)strips_x * ((ny + rows - 1) / rows);
        const long each = (waves + 1023) / 1024;
        // one wavefront alone on its SIMD issues three cycles in four
        const long cost = (each == 1 || waves_per_simd == 1 ? 13 * each : 10 * each) * (rows + 2 + (K - 1) * (H + 1));
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = rows;
        }
    }
    return best;
}

template <typename T, int CPL, int ST, bool WALLS, bool FORCE, int AM, int K, int KR, int KC>
hipError_t run(const FdArgs &fa, int rows, const void *src, void *dst, hipStream_t s)
{
    constexpr int H = Stencil<ST>::H;
    using G = FusedStrip<CPL, H, K>;
    FusedArgs<T, K> a;
    a.in = static_cast<const T *>(src);
    a.out = static_cast<T *>(dst);
    a.nx = fa.nx;
    a.ny = fa.ny;
    a.strips_x = (fa.nx + G::S - 1) / G::S;
    a.stride = G::S;
    if (AM == AM_SEAM) a.stride = seam_stride(fa.nx, G::S, G::P, CPL, sizeof(T));
    // no band may reach both walls: see fused_rows()
    if (rows < 1 || (WALLS && (rows < K * (H + 1) || rows > fa.ny - K * (H + 1)))) return hipErrorInvalidValue;
    a.rows = rows;
    a.ntiles = a.strips_x * ((fa.ny + a.rows - 1) / a.rows);
    a.k = make_coef<typename Storage<T>::C>(ST, fa.s_xx, fa.s_e, fa.fx, fa.fy);
    a.gr = ghost_rules<typename Storage<T>::C>(fa.xi);
    hipLaunchKernelGGL((fd_fused_kernel<T, CPL, ST, WALLS, FORCE, AM, K, KR, KC>), (a.ntiles + WV - 1) / WV, 64 * WV, 0, s,
                       a);
    return hipGetLastError();
}

template <typename T, int CPL, int ST, bool WALLS, bool FORCE, int K, int KR, int KC>
hipError_t dispatch_width(const FdArgs &a, int rows, const void *src, void *dst, hipStream_t s)
{
    if (a.nx % CPL == 0) return run<T, CPL, ST, WALLS, FORCE, AM_VEC, K, KR, KC>(a, rows, src, dst, s);
    using G = FusedStrip<CPL, Stencil<ST>::H, K>;
    if (seam_stride(a.nx, G::S, G::P, CPL, sizeof(T)) > 0)
        return run<T, CPL, ST, WALLS, FORCE, AM_SEAM, K, KR, KC>(a, rows, src, dst, s);
    return run<T, CPL, ST, WALLS, FORCE, sizeof(T) >= 4 ? AM_UNAL : AM_COL, K, KR, KC>(a, rows, src, dst, s);
}

template <typename T, int CPL, int ST, bool WALLS, int K, int KR, int KC>
hipError_t dispatch(const FdArgs &a, int rows, const void *src, void *dst, hipStream_t s)
{
    if constexpr (ST != 1)
        if (a.fx != 0.0 || a.fy != 0.0) return dispatch_width<T, CPL, ST, WALLS, true, K, KR, KC>(a, rows, src, dst, s);
    return dispatch_width<T, CPL, ST, WALLS, false, K, KR, KC>(a, rows, src, dst, s);
}

}  // namespace

// Two steps per launch with differences, three without (LW-ACM): more take two halo lanes a side
// or registers that are not there (FP32 8192^2 188 us per step in threes against 190, but walls,
// body forces and smaller grids lose).  Stochastic rounding is bound by its hashes: 127 us per step
// at 8192 x 4096 one by one, 128 in twos.
int fd_max_fused(const FdArgs &a)
{
    if (a.dtype == FDLBM_F16DEV_SR) return 1;
    if (a.stencil == 1) return 3;
    if (a.walls && (a.xi < 0.5 || a.ny < 16 || a.stencil == 5)) return 1;  // see fused_rows() and ghost_rules()
    return 2;
}

// Times of a launch.  One step: blocks of 4 x R rows (the defaults of fd_sweep.hip), one of 256 after
// the other on a compute unit, R + 4 rows of `one` us each and 3 us; or the state's bytes at 6 TB/s.
// K steps: the wavefronts each SIMD gets times the rows each takes through K stages of `row` us each,
// and 3 us.  By stencil and dtype, fitted to 40 grids of 8 to 2048 nodes a side and narrow ones, which they
// meet within 10 % (the middle half of them), widths that are no multiple of a lane's columns included.
LaunchTimes fd_launch_times(const FdArgs &a)
{
    const bool f64 = a.dtype == FDLBM_F64, force = a.fx != 0.0 || a.fy != 0.0;
    const int st = a.stencil == 1 ? 0 : a.stencil == 3 ? 1 : 2, CPL = f64 ? 2 : 4, eb = int(dtype_bytes(a.dtype));
    // FP64, FP32, FP16, FP16 rounded stochastically
    static const double one_us[3][4] = {{0.33, 0.40, 0.50, 0.66}, {0.52, 0.63, 0.78, 0.76}, {0.57, 0.82, 0.83, 0.90}};
    static const double row_us[3][4] = {{0.31, 0.40, 0.40, 0.0}, {0.49, 0.61, 0.61, 0.0}, {0.56, 0.65, 0.65, 0.0}};
    const double extra = a.walls ? 1.15 : force && !f64 ? 1.05 : 1.0;
    const double bytes_us = 6.0 * eb * a.nx * a.ny / 6e6;
    LaunchTimes t;
    {
        const int rows = f64 ? 6 : is_f16(a.dtype) || a.stencil == 5 ? 16 : a.stencil == 1 ? 4 : 8, S = f64 ? 124 : 248;
        const long blocks = (long)((a.nx + S - 1) / S) * ((a.ny + 4 * rows - 1) / (4 * rows)), each = (blocks + 255) / 256;
        double us = one_us[st][a.dtype] * extra;
        if (a.nx % CPL != 0 && !f64) us *= a.dtype == FDLBM_F32 ? 1.17 : a.nx % 2 ? 1.27 : 0.75;
        t.one = 3.0 + std::max(double((rows + 4) * each) * us, bytes_us);
    }
    t.most = fd_max_fused(a);
    if (t.most > 1) {
        const int K = t.most, H = st, P = (K * (H + 1) + CPL - 1) / CPL, S = (64 - 2 * P) * CPL, strips = (a.nx + S - 1) / S;
        const int rows = fused_rows(strips, a.ny, K, H, a.walls != 0, a.stencil == 5 ? 1 : 2);
        const long each = ((long)strips * ((a.ny + rows - 1) / rows) + 1023) / 1024;
        double us = row_us[st][a.dtype] * extra;
        if (a.nx % CPL != 0 && seam_stride(a.nx, S, P, CPL, eb) == 0) us *= 1.4;
        t.rows[K] = rows;
        t.fused[K] = 3.0 + std::max(double(K * each) * (rows + 2 * K * (H + 1)) * us, bytes_us);
    }
    return t;
}

template <typename T, int CPL> static hipError_t launch(const FdArgs &a, int rows, const void *src, void *dst, hipStream_t s)
{
    if (a.stencil == 1) return dispatch<T, CPL, 1, false, 3, 1, sizeof(T) == 8 ? 2 : 3>(a, rows, src, dst, s);
    if (a.stencil == 5) return dispatch<T, CPL, 5, false, 2, 1, 2>(a, rows, src, dst, s);
    if (a.walls) return dispatch<T, CPL, 3, true, 2, 1, 2>(a, rows, src, dst, s);
    return dispatch<T, CPL, 3, false, 2, 1, 2>(a, rows, src, dst, s);
}

hipError_t launch_fd_fused(const FdArgs &a, int rows, const void *src, void *dst, hipStream_t s)
{
    switch (a.dtype) {
    case FDLBM_F64: return launch<double, 2>(a, rows, src, dst, s);
    case FDLBM_F32: return launch<float, 4>(a, rows, src, dst, s);
    case FDLBM_F16DEV: return launch<__half, 4>(a, rows, src, dst, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fdlbm
