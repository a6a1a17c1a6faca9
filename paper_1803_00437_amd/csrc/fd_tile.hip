// FD-LBM and LW-ACM steps on small and medium grids: a block keeps a tile of the grid in registers
// for several steps.
//
// A grid of a few hundred nodes a side leaves the sweep kernels with few wavefronts, each of which
// takes its rows one after another: a launch lasts as long as one such chain (64^2 FP64 6.6 us per
// step) whatever the grid.  Here a block of 16 wavefronts loads a tile of 64*CPL columns by 16*R
// rows once, R rows per wavefront, advances it K steps and stores its inner part: every step loses
// H + 1 rows and columns on each side of the tile, which the neighbouring blocks also form (the
// same bits: the operations and their order are those of fd_node_fstar, fd_partial, fd_finish).
// Rows exchange with the wavefronts above and below through LDS, twice a step: the stored rows that
// the differences reach, then the sums that cross.  Columns come from the adjacent lanes (DPP).
//
// What bounds it: a step is 4 R CPL rows of vector instructions per SIMD plus two barriers, and a
// launch costs its start, the loads and the stores besides; TileCost weighs the rows and columns
// formed twice against that.
#include <algorithm>

#include "fd_sweep_body.hpp"
#include "internal.hpp"

namespace fdlbm {
namespace {
using sweep::from_left;
using sweep::from_right;

constexpr int TW = 16;  // wavefronts per block

template <typename T> struct TileStepArgs {
    const T *in;
    T *out;
    int nx, ny, steps, tiles_x, halo;  // halo = steps (H + 1)
    uint32_t step0;     // stochastic rounding: the step count before the first step
    TileDisk disk;      // DISK
    FdCoef<typename Storage<T>::C> k;
    GhostRules<typename Storage<T>::C> gr;
};

template <typename T, int CPL, int R, int ST, bool WALLS, bool FORCE, bool DISK>
__global__ void __launch_bounds__(64 * TW) fd_tile_kernel(TileStepArgs<T> a)
{
    using C = typename Storage<T>::C;
    using S = Stencil<ST>;
    constexpr int H = S::H, HH = H > 0 ? H : 1;
    constexpr bool LW = ST == 1;
    constexpr int E = H < R ? H : R;  // rows a wavefront shows its neighbours at each end
    __shared__ C edge[TW][2][HH][3][CPL][64];   // first and last rows of each wavefront
    __shared__ C cross[TW][4][CPL][64];         // sums sent up (s, x) by the last row, down by the first
    __shared__ C wall[WALLS ? 2 : 1][2][3][CPL][64];  // rows 0, 1 and ny - 1, ny - 2

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny;
    const int ty = blockIdx.x / a.tiles_x, tx = blockIdx.x - ty * a.tiles_x;
    const int cols = 64 * CPL - 2 * a.halo, rows = TW * R - 2 * a.halo;  // stored by a tile
    const int x0 = tx * cols - a.halo + CPL * lane, y0 = ty * rows - a.halo + wv * R;

    // columns and rows within the grid (periodic; rows beyond a wall are formed below)
    size_t col[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) col[c] = (size_t)(((x0 + c) % nx + nx) % nx);
    auto grid_row = [&](int y) { return WALLS ? min(max(y, 0), ny - 1) : (y % ny + ny) % ny; };
    C v[R][3][CPL];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int y = grid_row(y0 + i);
        const T *row = a.in + fd_elem(0, y, 0, nx);
        // the curved wall: ghost nodes from the fluid, as disk_fill_kernel sets them, and rest
        // nodes at rest (the fill and the step in one launch)
        const int dr = DISK ? y - a.disk.row0 : 0;
        const bool drow = DISK && dr >= 0 && dr < a.disk.nrows;  // this row has ghosts
        int ga = 0, gb = -1, glo = 0, ghi = -1, g0 = 0;
        if (drow) {
            const int32_t *d = a.disk.rows + DISK_ROW * dr;
            ga = d[0];
            gb = d[1];
            glo = d[2];
            ghi = d[3];
            g0 = d[4];
        }
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            // every lane loads its node while the row's numbers are on their way
#pragma unroll
            for (int f = 0; f < 3; ++f) v[i][f][c] = Storage<T>::load(row[(size_t)f * nx + col[c]]);
            if constexpr (!DISK) continue;
            const int x = (int)col[c];
            if (x < ga || x > gb) {
#pragma unroll
                for (int f = 0; f < 3; ++f) v[i][f][c] = C(0);
            } else if (x < glo || x > ghi) {
                const int g = g0 + (x < glo ? x - ga : (glo - ga) + (x - ghi - 1));
                const unsigned src = (unsigned)a.disk.src[g], sy = src / (unsigned)nx, sx = src - sy * (unsigned)nx;
                const C wx = C(a.disk.w[3 * g]), wy = C(a.disk.w[3 * g + 1]), sj = C(a.disk.w[3 * g + 2]);
                const C ux = C(1) - wx, uy = C(1) - wy;
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    const T *q = a.in + fd_elem(sx, sy, f, nx);  // the cell's corners
                    const C lower = ux * Storage<T>::load(q[0]) + wx * Storage<T>::load(q[1]);
                    const C upper = ux * Storage<T>::load(q[3 * (size_t)nx]) + wx * Storage<T>::load(q[3 * (size_t)nx + 1]);
                    const C m = uy * lower + wy * upper;
                    v[i][f][c] = Storage<T>::load(Storage<T>::store(f == 0 ? m : sj * m));
                }
            }
        }
    }
    // ghost row y beyond a wall, from the rows next to the wall
    auto ghost_row = [&](int y, C(&g)[3][CPL]) __attribute__((always_inline)) {
        const int side = y < 0 ? 0 : 1;
        const GhostRule<C> q = ghost_rule(a.gr, y < 0 ? -y : y - ny + 1);
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                g[f][c] = (f == 0 ? q.car : q.caj) * wall[WALLS ? side : 0][q.sa & 1][f][c][lane];
                if (q.sb >= 0) g[f][c] = g[f][c] + (f == 0 ? q.cbr : q.cbj) * wall[WALLS ? side : 0][1][f][c][lane];
            }
    };

    for (int step = 0; step < a.steps; ++step) {
        if constexpr (H > 0) {
#pragma unroll
            for (int e = 0; e < E; ++e)
#pragma unroll
                for (int f = 0; f < 3; ++f)
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        edge[wv][0][e][f][c][lane] = v[e][f][c];
                        edge[wv][1][e][f][c][lane] = v[R - 1 - e][f][c];
                    }
            if constexpr (WALLS) {
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const int y = y0 + i;
                    const int bottom = y, top = ny - 1 - y;
                    if (bottom == 0 || bottom == 1)
#pragma unroll
                        for (int f = 0; f < 3; ++f)
#pragma unroll
                            for (int c = 0; c < CPL; ++c) wall[0][bottom][f][c][lane] = v[i][f][c];
                    if (top == 0 || top == 1)
#pragma unroll
                        for (int f = 0; f < 3; ++f)
#pragma unroll
                            for (int c = 0; c < CPL; ++c) wall[WALLS ? 1 : 0][top][f][c][lane] = v[i][f][c];
                }
            }
            __syncthreads();
        }
        // rows y0 - H .. y0 + R - 1 + H (a tile's outermost rows see themselves: never stored)
        C w[R + 2 * H > 0 ? R + 2 * H : 1][3][CPL];
#pragma unroll
        for (int i = 0; i < R + 2 * H; ++i) {
            const int j = i - H;  // row y0 + j
            const bool own = j >= 0 && j < R;
            if (WALLS && (y0 + j < 0 || y0 + j >= ny) && y0 + j >= -2 && y0 + j < ny + 2) {
                ghost_row(y0 + j, w[i]);
            } else if (own) {
#pragma unroll
                for (int f = 0; f < 3; ++f)
#pragma unroll
                    for (int c = 0; c < CPL; ++c) w[i][f][c] = v[own ? j : 0][f][c];
            } else {
                // d rows beyond the first or last row: wavefront (d - 1) / R + 1 away
                const int d = j < 0 ? -j : j - R + 1, far = (d - 1) / R + 1, e = (d - 1) % R;
                const int nb = j < 0 ? max(wv - far, 0) : min(wv + far, TW - 1);
#pragma unroll
                for (int f = 0; f < 3; ++f)
#pragma unroll
                    for (int c = 0; c < CPL; ++c) w[i][f][c] = edge[nb][j < 0 ? 1 : 0][e][f][c][lane];
            }
        }
        // f* row by row; row i is complete once f* of row i + 1 is known, the first and last ones
        // once the sums from the wavefronts below and above are
        C pc[R][CPL], pcx[R][CPL], pu[R][CPL], pux[R][CPL], ld[R][CPL], ldx[R][CPL];
        C up[CPL], upx[CPL], lu0[CPL], lux0[CPL], dn[R][CPL], dnx[R][CPL];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const C(&me)[3][CPL] = w[i + H];
            C f[CPL][9];
            if constexpr (LW) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) lw_node_g<C>(me[0][c], me[1][c], me[2][c], a.k.lin, f[c]);
            } else {
                auto yfield = [&](int q, int k, int c) __attribute__((always_inline)) -> C {
                    const C(&u)[3][CPL] = w[i + H + k];
                    const C xa = plus_force<FORCE>(u[1][c], a.k.hfx), ya = plus_force<FORCE>(u[2][c], a.k.hfy);
                    return q == 0 ? u[0][c] : q == 1 ? u[2][c] : q == 2 ? u[1][c] : q == 3 ? xa * ya : ya * ya;
                };
                C xf[5][CPL], jxa[CPL], jya[CPL];
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    jxa[c] = plus_force<FORCE>(me[1][c], a.k.hfx);
                    jya[c] = plus_force<FORCE>(me[2][c], a.k.hfy);
                    xf[0][c] = me[0][c];
                    xf[1][c] = me[1][c];
                    xf[2][c] = me[2][c];
                    xf[3][c] = jxa[c] * jxa[c];
                    xf[4][c] = jxa[c] * jya[c];
                }
                C l1[5], r1[5], l2[5], r2[5];
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    l1[q] = from_left(xf[q][CPL - 1]);
                    r1[q] = from_right(xf[q][0]);
                    // two columns away: the neighbour's other column, or the lane after it
                    l2[q] = H == 2 ? (CPL >= 2 ? from_left(xf[q][CPL >= 2 ? CPL - 2 : 0]) : from_left(l1[q])) : C(0);
                    r2[q] = H == 2 ? (CPL >= 2 ? from_right(xf[q][CPL >= 2 ? 1 : 0]) : from_right(r1[q])) : C(0);
                }
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    C dd[10];
#pragma unroll
                    for (int q = 0; q < 5; ++q) {
                        const C m1 = c > 0 ? xf[q][c > 0 ? c - 1 : 0] : l1[q];
                        const C p1 = c < CPL - 1 ? xf[q][c < CPL - 1 ? c + 1 : 0] : r1[q];
                        C m2 = C(0), p2 = C(0), ym2 = C(0), yp2 = C(0);
                        if constexpr (H == 2) {
                            m2 = c >= 2 ? xf[q][c >= 2 ? c - 2 : 0] : (c == 1 ? l1[q] : l2[q]);
                            p2 = c + 2 < CPL ? xf[q][c + 2 < CPL ? c + 2 : 0] : (c + 2 == CPL ? r1[q] : r2[q]);
                            ym2 = yfield(q, -2, c);
                            yp2 = yfield(q, 2, c);
                        }
                        dd[2 * q] = S::diff(m2, m1, p1, p2);
                        dd[2 * q + 1] = S::diff(ym2, yfield(q, -1, c), yfield(q, 1, c), yp2);
                    }
                    fd_node_fstar<C, FORCE>(me[0][c], jxa[c], jya[c], dd, a.k, f[c]);
                }
            }
            const C f1l = from_left(f[CPL - 1][1]), f5l = from_left(f[CPL - 1][5]), f8l = from_left(f[CPL - 1][8]);
            const C f3r = from_right(f[0][3]), f6r = from_right(f[0][6]), f7r = from_right(f[0][7]);
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int cl = c > 0 ? c - 1 : 0, cn = c < CPL - 1 ? c + 1 : 0;
                const C c1 = c > 0 ? f[cl][1] : f1l, u5 = c > 0 ? f[cl][5] : f5l, d8 = c > 0 ? f[cl][8] : f8l;
                const C c3 = c < CPL - 1 ? f[cn][3] : f3r, u6 = c < CPL - 1 ? f[cn][6] : f6r,
                        d7 = c < CPL - 1 ? f[cn][7] : f7r;
                const C nup = row_sum(f[c][2], u5, u6), nupx = u5 - u6;
                dn[i][c] = row_sum(f[c][4], d8, d7);
                dnx[i][c] = d8 - d7;
                const C lu = row_sum(f[c][2], f[c][5], f[c][6]), lux = f[c][5] - f[c][6];
                ld[i][c] = row_sum(f[c][4], f[c][8], f[c][7]);
                ldx[i][c] = f[c][8] - f[c][7];
                same_row_part<C>(c1 - f[c][1], c3 - f[c][3], pc[i][c], pcx[i][c]);
                if (i == 0) {
                    lu0[c] = lu;
                    lux0[c] = lux;
                } else {
                    pu[i][c] = up[c] - lu;
                    pux[i][c] = upx[c] - lux;
                }
                up[c] = nup;
                upx[c] = nupx;
            }
        }
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            cross[wv][0][c][lane] = up[c];
            cross[wv][1][c][lane] = upx[c];
            cross[wv][2][c][lane] = dn[0][c];
            cross[wv][3][c][lane] = dnx[0][c];
        }
        __syncthreads();
        const int wb = max(wv - 1, 0), wa = min(wv + 1, TW - 1);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            pu[0][c] = cross[wb][0][c][lane] - lu0[c];
            pux[0][c] = cross[wb][1][c][lane] - lux0[c];
        }
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int n = i + 1 < R ? i + 1 : 0;
                const C fd = i + 1 < R ? dn[n][c] : cross[wa][2][c][lane];
                const C fdx = i + 1 < R ? dnx[n][c] : cross[wa][3][c][lane];
                const C(&old)[3][CPL] = w[i + H];
                C r, x, y;
                fd_finish<C, FORCE>(fd_partial<C>(pc[i][c], pcx[i][c], pu[i][c], pux[i][c]), fd - ld[i][c], fdx - ldx[i][c],
                                    old[0][c], old[1][c], old[2][c], a.k.dfx, a.k.dfy, r, x, y);
                // rounded for storage, as a step of its own would (FP16)
                uint32_t rb[3] = {0u, 0u, 0u};
                if constexpr (Storage<T>::STOCHASTIC)
                    sr_draw(uint32_t(grid_row(y0 + i)) * uint32_t(nx) + uint32_t(col[c]), pcg_hash(a.step0 + uint32_t(step)), rb);
                v[i][0][c] = Storage<T>::load(Storage<T>::store_r(r, rb[0]));
                v[i][1][c] = Storage<T>::load(Storage<T>::store_r(x, rb[1]));
                v[i][2][c] = Storage<T>::load(Storage<T>::store_r(y, rb[2]));
            }
        if constexpr (H == 0) __syncthreads();  // the sums are read before the next step's are written
    }

    // the inner part of the tile
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int j = wv * R + i, y = y0 + i;
        if (j < a.halo || j >= TW * R - a.halo || y >= ny) continue;
        T *row = a.out + fd_elem(0, y, 0, nx);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int t = CPL * lane + c;
            if (t >= a.halo && t < 64 * CPL - a.halo && x0 + c < nx)
#pragma unroll
                for (int f = 0; f < 3; ++f) row[(size_t)f * nx + x0 + c] = Storage<T>::store(v[i][f][c]);
        }
    }
}

template <typename T, int CPL, int R, int ST, bool WALLS, bool FORCE, bool DISK>
hipError_t run(const FdArgs &fa, const TilePlan &p, const TileDisk &disk, const void *src, void *dst, hipStream_t s)
{
    constexpr int H = Stencil<ST>::H;
    TileStepArgs<T> a;
    a.in = static_cast<const T *>(src);
    a.out = static_cast<T *>(dst);
    a.nx = fa.nx;
    a.ny = fa.ny;
    a.steps = p.steps;
    a.halo = p.steps * (H + 1);
    a.step0 = fa.step;
    a.disk = disk;
    const int cols = 64 * CPL - 2 * a.halo, rows = TW * R - 2 * a.halo;
    if (cols < 1 || rows < 1 || (DISK && p.steps != 1)) return hipErrorInvalidValue;
    a.tiles_x = (fa.nx + cols - 1) / cols;
    a.k = sweep::make_coef<typename Storage<T>::C>(ST, fa.s_xx, fa.s_e, fa.fx, fa.fy);
    a.gr = ghost_rules<typename Storage<T>::C>(fa.xi);
    const int tiles = a.tiles_x * ((fa.ny + rows - 1) / rows);
    hipLaunchKernelGGL((fd_tile_kernel<T, CPL, R, ST, WALLS, FORCE, DISK>), tiles, 64 * TW, 0, s, a);
    return hipGetLastError();
}

template <typename T, int CPL, int R, int ST, bool WALLS, bool DISK>
hipError_t force(const FdArgs &a, const TilePlan &p, const TileDisk &disk, const void *src, void *dst, hipStream_t s)
{
    if constexpr (ST != 1)
        if (a.fx != 0.0 || a.fy != 0.0) return run<T, CPL, R, ST, WALLS, true, DISK>(a, p, disk, src, dst, s);
    return run<T, CPL, R, ST, WALLS, false, DISK>(a, p, disk, src, dst, s);
}

template <typename T, int CPL, int R>
hipError_t dispatch(const FdArgs &a, const TilePlan &p, const TileDisk &disk, const void *src, void *dst, hipStream_t s)
{
    if constexpr (CPL == 1)
        if (disk.rows) {
            if (a.stencil == 1) return force<T, CPL, R, 1, false, true>(a, p, disk, src, dst, s);
            if (a.stencil == 5) return force<T, CPL, R, 5, false, true>(a, p, disk, src, dst, s);
            return force<T, CPL, R, 3, false, true>(a, p, disk, src, dst, s);
        }
    if (disk.rows) return hipErrorInvalidValue;
    if (a.stencil == 1) return force<T, CPL, R, 1, false, false>(a, p, disk, src, dst, s);
    if (a.stencil == 5) return force<T, CPL, R, 5, false, false>(a, p, disk, src, dst, s);
    if (a.walls) return force<T, CPL, R, 3, true, false>(a, p, disk, src, dst, s);
    return force<T, CPL, R, 3, false, false>(a, p, disk, src, dst, s);
}

template <typename T>
hipError_t shapes(const FdArgs &a, const TilePlan &p, const TileDisk &disk, const void *src, void *dst, hipStream_t s)
{
    if (p.cols == 1 && p.rows == 1) return dispatch<T, 1, 1>(a, p, disk, src, dst, s);
    if (p.cols == 1 && p.rows == 2) return dispatch<T, 1, 2>(a, p, disk, src, dst, s);
    if (p.cols == 1 && p.rows == 4) return dispatch<T, 1, 4>(a, p, disk, src, dst, s);
    if constexpr (sizeof(T) < 8)
        if (p.cols == 2 && p.rows == 4) return dispatch<T, 2, 4>(a, p, disk, src, dst, s);
    return hipErrorInvalidValue;
}

}  // namespace

// In the disk the wall acts between the steps: one step per launch, which spares the launch of the
// fill (72^2 FP64: 7.0 + 2.8 us).
TileCost fd_tile_cost(const FdArgs &a)
{
    const bool f64 = a.dtype == FDLBM_F64, force = a.fx != 0.0 || a.fy != 0.0;
    const int H = a.stencil == 1 ? 0 : a.stencil == 3 ? 1 : 2;
    TileCost c;
    c.nx = a.nx;
    c.ny = a.ny;
    c.reach = H + 1;
    c.elem_bytes = int(compute_bytes(a.dtype));
    c.lds = size_t(6 * TW * std::max(H, 1) + 4 * TW + (a.walls ? 12 : 0)) * 64 * c.elem_bytes;  // edge, cross, wall
    c.row_us = a.stencil == 1 ? (f64 ? 0.55 : 0.45)
                              : (a.stencil == 3 ? (f64 ? 0.9 : 0.65) : (f64 ? 1.3 : 0.85)) + (force ? 0.08 : 0.0);
    if (a.dtype == FDLBM_F16DEV_SR) c.row_us += 0.12;  // two hashes per node
    return c;
}

TilePlan fd_tile_plan(const FdArgs &a, const LaunchTimes &t, bool disk)
{
    // ghost rows come from the two rows next to a wall
    if (a.walls && (a.xi < 0.5 || a.stencil != 3)) return TilePlan();
    const TileShape shapes[] = {{1, 1}, {1, 2}, {1, 4}, {2, 4}};
    // the disk: the sweep in single steps, and the fill's launch less what the gathers take
    const double sweep_us = disk ? t.one + 2.0 : std::min(t.one, t.most > 1 ? t.fused[t.most] / t.most : t.one);
    return plan_tiles(fd_tile_cost(a), shapes, a.dtype == FDLBM_F64 || disk ? 3 : 4, disk ? 1 : 25, sweep_us);
}

hipError_t launch_fd_tile(const FdArgs &a, const TilePlan &p, const TileDisk &disk, const void *src, void *dst,
                          hipStream_t s)
{
    switch (a.dtype) {
    case FDLBM_F64: return shapes<double>(a, p, disk, src, dst, s);
    case FDLBM_F32: return shapes<float>(a, p, disk, src, dst, s);
    case FDLBM_F16DEV_SR: return shapes<HalfSR>(a, p, disk, src, dst, s);
    default: return shapes<__half>(a, p, disk, src, dst, s);
    }
}

}  // namespace fdlbm
