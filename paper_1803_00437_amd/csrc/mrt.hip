// MRT D2Q9 stream-collide step (section 1, eqs. 1-2; equilibria and rates of the table
// in section 1-a), the scheme the FD-LBM is compared against.
//
// Storage: the nine deviations f_k - w_k from the rest populations, row-interleaved (row j
// of population k at element (9 j + k) nx, pop_elem): the nine rows a node row reads are
// adjacent in memory, and so are the rows it writes.  Three kernels: one thread per node
// (mrt_kernel, the reference), and over lane groups of columns the fused sweep
// (mrt_fused_kernel, the default: one, three or five steps per launch) and the sweep for walls
// at a general distance (mrt_xi_kernel).  Each relaxes the non-conserved moments of a node and
// pushes f*_k to x + e_k in the other buffer.  A population whose destination lies beyond
// a wall returns with the opposite velocity: halfway bounce-back (the wall half-way
// between the last fluid row and the next one, section 3-c), or the interpolated
// bounce-back of Bouzidi et al. for a wall at another distance xi (all kernels agree bit for
// bit).  Traffic: 9 values read + 9 written per node and launch.
#include <algorithm>

#include "fd_sweep_body.hpp"
#include "fdlbm_device.hpp"
#include "internal.hpp"

namespace fdlbm {
namespace {

template <typename C> struct MrtCoef {
    C se, sxx, sq, seps;
    C hfx, hfy, fx, fy;
};

// m = M f for the deviations (rows rho, Jx, Jy, E, XX, XY, qx, qy, eps of section 1).
template <typename C> __device__ __forceinline__ void moments(const C (&f)[9], C (&m)[9])
{
    const C ax = (f[1] + f[2]) + (f[3] + f[4]);
    const C dg = (f[5] + f[6]) + (f[7] + f[8]);
    const C x13 = f[1] - f[3], y24 = f[2] - f[4];
    const C dxp = (f[5] - f[6]) - (f[7] - f[8]);  // sum e_x over diagonals
    const C dyp = (f[5] + f[6]) - (f[7] + f[8]);  // sum e_y over diagonals
    m[0] = (f[0] + ax) + dg;
    m[1] = x13 + dxp;
    m[2] = y24 + dyp;
    m[3] = fmac(C(-4), f[0], fmac(C(2), dg, -ax));
    m[4] = (f[1] + f[3]) - (f[2] + f[4]);
    m[5] = (f[5] + f[7]) - (f[6] + f[8]);
    m[6] = fmac(C(-2), x13, dxp);
    m[7] = fmac(C(-2), y24, dyp);
    m[8] = fmac(C(4), f[0], fmac(C(-2), ax, dg));
}

// f = M^{-1} m, M^{-1} = M^T diag(1/9, 1/6, 1/6, 1/36, 1/4, 1/4, 1/12, 1/12, 1/36).
template <typename C> __device__ __forceinline__ void populations(const C (&m)[9], C (&f)[9])
{
    const C r9 = m[0] * C(1.0 / 9.0);
    const C e36 = m[3] * C(1.0 / 36.0), p36 = m[8] * C(1.0 / 36.0);
    f[0] = fmac(C(-4), e36, fmac(C(4), p36, r9));
    const C ax = fmac(C(-2), p36, r9 - e36);            // rho/9 - E/36 - eps/18
    const C dg = fmac(C(2), e36, r9 + p36);             // rho/9 + E/18 + eps/36
    const C xx = m[4] * C(0.25), xy = m[5] * C(0.25);
    const C jx6 = m[1] * C(1.0 / 6.0), jy6 = m[2] * C(1.0 / 6.0);
    const C qx6 = m[6] * C(1.0 / 6.0), qy6 = m[7] * C(1.0 / 6.0);
    const C ux = jx6 - qx6, uy = jy6 - qy6;             // axis: J/6 - q/6 (M_q = -2e on axes)
    const C vx = fmac(qx6, C(0.5), jx6), vy = fmac(qy6, C(0.5), jy6);  // diagonal: J/6 + q/12
    f[1] = (ax + xx) + ux;
    f[3] = (ax + xx) - ux;
    f[2] = (ax - xx) + uy;
    f[4] = (ax - xx) - uy;
    f[5] = (dg + xy) + (vx + vy);
    f[7] = (dg + xy) - (vx + vy);
    f[6] = (dg - xy) + (vy - vx);
    f[8] = (dg - xy) - (vy - vx);
}

// f += M^{-1} d for a moment increment d that leaves the mass unchanged (d[0] is not read).
// Adding the small change to the stored deviations, instead of rebuilding f from the
// relaxed moments, keeps the FP32 rounding relative to the change rather than to f: in a
// slow steady flow the rebuilt form's rounding biases every step the same way.
template <typename C> __device__ __forceinline__ void add_increment(const C (&d)[9], C (&f)[9])
{
    const C e36 = d[3] * C(1.0 / 36.0), p36 = d[8] * C(1.0 / 36.0);
    f[0] = f[0] + C(4) * (p36 - e36);
    const C ax = -fmac(C(2), p36, e36);                 // -E/36 - eps/18
    const C dg = fmac(C(2), e36, p36);                  // E/18 + eps/36
    const C xx = d[4] * C(0.25), xy = d[5] * C(0.25);
    const C jx6 = d[1] * C(1.0 / 6.0), jy6 = d[2] * C(1.0 / 6.0);
    const C qx6 = d[6] * C(1.0 / 6.0), qy6 = d[7] * C(1.0 / 6.0);
    const C ux = jx6 - qx6, uy = jy6 - qy6;
    const C vx = fmac(qx6, C(0.5), jx6), vy = fmac(qy6, C(0.5), jy6);
    f[1] = f[1] + ((ax + xx) + ux);
    f[3] = f[3] + ((ax + xx) - ux);
    f[2] = f[2] + ((ax - xx) + uy);
    f[4] = f[4] + ((ax - xx) - uy);
    f[5] = f[5] + ((dg + xy) + (vx + vy));
    f[7] = f[7] + ((dg + xy) - (vx + vy));
    f[6] = f[6] + ((dg - xy) + (vy - vx));
    f[8] = f[8] + ((dg - xy) - (vy - vx));
}

// Equilibrium moments of section 1-a as deviations from the rest moments.
template <typename C>
__device__ __forceinline__ void equilibrium(C dr, C jx, C jy, C &E, C &XX, C &XY, C &qx, C &qy, C &eps)
{
    const C rinv = recip(C(1) + dr);
    const C p = jx * jx, q = jy * jy;
    const C K3 = C(3) * ((p + q) * rinv);
    E = fmac(C(-2), dr, K3);
    XX = (p - q) * rinv;
    XY = (jx * jy) * rinv;
    qx = -jx;
    qy = -jy;
    eps = dr - K3;
}

// Collision of one node: moments, relaxation of the non-conserved ones toward the
// equilibria (eq. 1) with the force split half before and half after (Strang), and the
// post-collision populations f* = f + M^{-1} (m* - m).  Every MRT kernel calls this, so
// all of them agree bit for bit.
template <typename C> __device__ __forceinline__ void collide(C (&f)[9], const MrtCoef<C> &k)
{
    C m[9];
    moments<C>(f, m);
    // Strang splitting: half the force before the collision ...
    const C jax = m[1] + k.hfx, jay = m[2] + k.hfy;
    C E, XX, XY, qx, qy, eps;
    equilibrium<C>(m[0], jax, jay, E, XX, XY, qx, qy, eps);
    C d[9];
    d[0] = C(0);
    // ... the whole force over the step (the other half after the collision) ...
    d[1] = k.fx;
    d[2] = k.fy;
    // ... and eq. 1 for the non-conserved moments
    d[3] = k.se * (E - m[3]);
    d[4] = k.sxx * (XX - m[4]);
    d[5] = k.sxx * (XY - m[5]);
    d[6] = k.sq * (qx - m[6]);
    d[7] = k.sq * (qy - m[7]);
    d[8] = k.seps * (eps - m[8]);
    add_increment<C>(d, f);
}

// Reference MRT step: one thread per node.  With walls, a population whose destination
// lies beyond a wall returns to its node with the opposite velocity.  The wall cuts that
// link at the fraction xi of its length (walls at y = -xi and ny - 1 + xi), and the
// returning population is the linear interpolation of Bouzidi, Firdaouss and Lallemand:
//   xi <  1/2:  f_kbar(x) = 2 xi f*_k(x) + (1 - 2 xi) f*_k(x - e_k)
//   xi >= 1/2:  f_kbar(x) = f*_k(x) / (2 xi) + (2 xi - 1) / (2 xi) f*_kbar(x)
// which is halfway bounce-back at xi = 1/2.  For xi < 1/2 the thread collides the node
// behind it, x - e_k, once more.
template <typename T, bool WALLS>
__global__ void __launch_bounds__(256) mrt_kernel(const T *__restrict__ in, T *__restrict__ out, int nx, int ny,
                                                  MrtCoef<typename Storage<T>::C> k, typename Storage<T>::C xi)
{
    using C = typename Storage<T>::C;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    if (i >= nx || j >= ny) return;
    C f[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) f[q] = Storage<T>::load(in[pop_elem(i, j, q, nx)]);
    collide<C>(f, k);
    // propagation, eq. 2 (push)
    const int ip = i + 1 == nx ? 0 : i + 1, im = i == 0 ? nx - 1 : i - 1;
    int jp = j + 1, jm = j - 1;
    if (!WALLS) {
        if (jp == ny) jp = 0;
        if (jm < 0) jm = ny - 1;
    }
    // post-collision population q at node (ii, jj), collided again (interpolated bounce-back)
    auto post_at = [&](int ii, int jj, int q) -> C {
        ii = ii < 0 ? ii + nx : (ii >= nx ? ii - nx : ii);
        C g[9];
#pragma unroll
        for (int r = 0; r < 9; ++r) g[r] = Storage<T>::load(in[pop_elem(ii, jj, r, nx)]);
        collide<C>(g, k);
        C v = g[0];
#pragma unroll
        for (int r = 1; r < 9; ++r)
            if (r == q) v = g[r];
        return v;
    };
    // population kq leaving toward the wall along (ex, ey), returning as kb
    auto back = [&](int kq, int kb, int ex, int ey) -> C {
        if (xi == C(0.5)) return f[kq];
        if (xi > C(0.5)) return f[kq] / (C(2) * xi) + (C(2) * xi - C(1)) / (C(2) * xi) * f[kb];
        return C(2) * xi * f[kq] + (C(1) - C(2) * xi) * post_at(i - ex, j - ey, kq);
    };
    out[pop_elem(i, j, 0, nx)] = Storage<T>::store(f[0]);
    out[pop_elem(ip, j, 1, nx)] = Storage<T>::store(f[1]);
    out[pop_elem(im, j, 3, nx)] = Storage<T>::store(f[3]);
    if (!WALLS || jp < ny) {
        out[pop_elem(i, jp, 2, nx)] = Storage<T>::store(f[2]);
        out[pop_elem(ip, jp, 5, nx)] = Storage<T>::store(f[5]);
        out[pop_elem(im, jp, 6, nx)] = Storage<T>::store(f[6]);
    } else {  // bounce-back at the upper wall
        out[pop_elem(i, j, 4, nx)] = Storage<T>::store(back(2, 4, 0, 1));
        out[pop_elem(i, j, 7, nx)] = Storage<T>::store(back(5, 7, 1, 1));
        out[pop_elem(i, j, 8, nx)] = Storage<T>::store(back(6, 8, -1, 1));
    }
    if (!WALLS || jm >= 0) {
        out[pop_elem(i, jm, 4, nx)] = Storage<T>::store(f[4]);
        out[pop_elem(im, jm, 7, nx)] = Storage<T>::store(f[7]);
        out[pop_elem(ip, jm, 8, nx)] = Storage<T>::store(f[8]);
    } else {  // bounce-back at the lower wall
        out[pop_elem(i, j, 2, nx)] = Storage<T>::store(back(4, 2, 0, -1));
        out[pop_elem(i, j, 5, nx)] = Storage<T>::store(back(7, 5, -1, -1));
        out[pop_elem(i, j, 6, nx)] = Storage<T>::store(back(8, 6, 1, -1));
    }
}

// Walls at a distance xi, one step per launch.  A wavefront owns 64*CPL consecutive columns (CPL per lane, one
// aligned vector access per population row) of R rows.  After the collision, the
// populations moving along +x / -x are shifted by one column across lanes with DPP
// whole-wave shifts, so every store is an aligned vector too; the outermost lane on each
// side has no neighbour to take from and only feeds its neighbour, so strips overlap by
// one lane on each side.  Populations moving along y go to the row above or below (or
// bounce back at a wall).  Wavefronts are dealt out row band after row band.
//
// The nine population rows of the next grid row are loaded while the current one is collided (two row
// buffers, the loop unrolled by two so that they alternate without copies).  Loads and
// stores go through range-checked buffer resources: the halo lanes' stores and the
// prefetch past the last row use an offset beyond the row and are dropped, so every row
// issues the same memory operations without branches.
//
// The bounce-back is interpolated with the same expressions as in mrt_kernel; for xi < 1/2
// the row next to the wall row is loaded and collided once more for f*_k(x - e_k), the
// populations at x - e_k coming from the neighbouring lane with the same DPP shifts.
template <typename T, int CPL>
__global__ void __launch_bounds__(256) mrt_xi_kernel(const T *__restrict__ in, T *__restrict__ out, int nx, int ny,
                                                        int rows, int strips_x, int ntiles,
                                                        MrtCoef<typename Storage<T>::C> k, typename Storage<T>::C xi)
{
    using C = typename Storage<T>::C;
    using namespace sweep;
    constexpr int S = 64 * CPL - 2 * CPL;  // stored columns per strip
    const int lane = threadIdx.x & 63;
    const int tile = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tile >= ntiles) return;  // uniform over the wavefront
    const int band = tile / strips_x, sx = tile - band * strips_x;
    const int xl = sx * S - CPL + CPL * lane;  // first column of this lane (unwrapped)
    const unsigned col = ((xl % nx) + nx) % nx;
    const bool store_ok = lane >= 1 && lane <= 62 && xl < nx;
    const unsigned voff = col * (unsigned)sizeof(T);
    const unsigned soff = store_ok ? voff : OFF_NONE;  // halo lanes do not store
    const int y0 = band * rows, y1 = min(y0 + rows, ny);

    auto load_row = [&](int y, bool use, Group<T, CPL>(&g)[9]) {
        const int yy = min(y, ny - 1);
#pragma unroll
        for (int q = 0; q < 9; ++q)
            g[q] = buf_load_group<T, CPL>(row_rsrc(in + pop_elem(0, 0, q, nx), yy, 9 * nx, nx), use ? voff : OFF_NONE);
    };
    auto put = [&](int q, int y, const Group<T, CPL> &g) {
        buf_store_group<T, CPL>(row_rsrc(out + pop_elem(0, 0, q, nx), y, 9 * nx, nx), soff, g);
    };
    // post-collision populations of row yy (the row next to a wall, collided once more)
    auto collide_row = [&](int yy, C(&h)[CPL][9]) {
        Group<T, CPL> g[9];
        load_row(yy, true, g);
#pragma unroll
        for (int q = 0; q < 9; ++q)
#pragma unroll
            for (int c = 0; c < CPL; ++c) h[c][q] = Storage<T>::load(g[q].v[c]);
#pragma unroll
        for (int c = 0; c < CPL; ++c) collide<C>(h[c], k);
    };
    // populations returning from a wall into this row: kq leaves along (ex, ey) (ey = +1 at
    // the top wall, -1 at the bottom one) and returns as kb; ynb is the row behind the node
    auto bounce = [&](const C(&f)[CPL][9], int kq, int kb, int ex, int ynb, Group<T, CPL> &b) {
        if (xi == C(0.5)) {  // a distance that rounds to 1/2 in the arithmetic type
#pragma unroll
            for (int c = 0; c < CPL; ++c) b.v[c] = Storage<T>::store(f[c][kq]);
        } else if (xi > C(0.5)) {
#pragma unroll
            for (int c = 0; c < CPL; ++c)
                b.v[c] = Storage<T>::store(f[c][kq] / (C(2) * xi) + (C(2) * xi - C(1)) / (C(2) * xi) * f[c][kb]);
        } else {
            C h[CPL][9];
            collide_row(ynb, h);
            // f*_kq at x - e_kq: column - ex, i.e. from the left for ex = +1, the right for -1
            const C edge = ex > 0 ? from_left(h[CPL - 1][kq]) : ex < 0 ? from_right(h[0][kq]) : C(0);
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const C behind = ex == 0 ? h[c][kq]
                                 : ex > 0 ? (c > 0 ? h[c > 0 ? c - 1 : 0][kq] : edge)
                                          : (c < CPL - 1 ? h[c < CPL - 1 ? c + 1 : 0][kq] : edge);
                b.v[c] = Storage<T>::store(C(2) * xi * f[c][kq] + (C(1) - C(2) * xi) * behind);
            }
        }
    };
    // collide row y (populations in `cur`) and push its post-collision populations
    auto process = [&](int y, const Group<T, CPL>(&cur)[9]) {
        C f[CPL][9];
#pragma unroll
        for (int q = 0; q < 9; ++q)
#pragma unroll
            for (int c = 0; c < CPL; ++c) f[c][q] = Storage<T>::load(cur[q].v[c]);
#pragma unroll
        for (int c = 0; c < CPL; ++c) collide<C>(f[c], k);
        // destination rows (wave-uniform); a population leaving the channel
        // returns to its own node with the opposite velocity
        const int yp = y + 1, ym = y - 1;
        const bool top_wall = yp == ny, bottom_wall = ym < 0;
        Group<T, CPL> g[9];
        // velocities (0,0), (0,+1), (0,-1) keep their column
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            g[0].v[c] = Storage<T>::store(f[c][0]);
            g[2].v[c] = Storage<T>::store(f[c][2]);
            g[4].v[c] = Storage<T>::store(f[c][4]);
        }
        // +x movers (1, 5, 8) arrive from the column on the left, -x movers (3, 6, 7) from
        // the column on the right
        const int rq[3] = {1, 5, 8}, lq[3] = {3, 6, 7};
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const C fl = from_left(f[CPL - 1][rq[t]]), fr = from_right(f[0][lq[t]]);
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                g[rq[t]].v[c] = Storage<T>::store(c > 0 ? f[c > 0 ? c - 1 : 0][rq[t]] : fl);
                g[lq[t]].v[c] = Storage<T>::store(c < CPL - 1 ? f[c < CPL - 1 ? c + 1 : 0][lq[t]] : fr);
            }
        }
        put(0, y, g[0]);
        put(1, y, g[1]);
        put(3, y, g[3]);
        if (top_wall) {
            // the upward movers return into this row's downward populations, unshifted
            Group<T, CPL> b2, b5, b6;
            bounce(f, 2, 4, 0, y - 1, b2);
            bounce(f, 5, 7, 1, y - 1, b5);
            bounce(f, 6, 8, -1, y - 1, b6);
            put(4, y, b2);
            put(7, y, b5);
            put(8, y, b6);
        } else {
            put(2, yp, g[2]);
            put(5, yp, g[5]);
            put(6, yp, g[6]);
        }
        if (bottom_wall) {
            Group<T, CPL> b4, b7, b8;
            bounce(f, 4, 2, 0, y + 1, b4);
            bounce(f, 7, 5, -1, y + 1, b7);
            bounce(f, 8, 6, 1, y + 1, b8);
            put(2, y, b4);
            put(5, y, b7);
            put(6, y, b8);
        } else {
            put(4, ym, g[4]);
            put(7, ym, g[7]);
            put(8, ym, g[8]);
        }
    };

    Group<T, CPL> A[9], B[9];
    load_row(y0, true, A);
    for (int y = y0; y < y1; y += 2) {
        load_row(y + 1, y + 1 < y1, B);
        process(y, A);
        if (y + 1 >= y1) break;
        load_row(y + 2, y + 2 < y1, A);
        process(y + 1, B);
    }
}

// MRT steps: K time steps in one pass over memory (K = 1, 3 or 5).  One step moves 18 words per node
// and keeps the vector units 24 % busy; here a wavefront reads a row once, takes it through K
// stages it holds on chip and writes the populations of K steps later.
//
// A wavefront owns a strip of 64*CPL columns (CPL per lane) for R output rows and walks up the rows,
// one input row per tick, the next row's nine loads in flight.  At tick t stage s collides row
// ya + t - s.  Streaming between stages needs the rows on both sides: stage s keeps, of the row it
// collided last, the populations that stay in that row (0, 1, 3) and those on their way up (2, 5,
// 6; also the row's before), already shifted along x with DPP whole-wave shifts; the next row it
// collides brings the three that come down, and the row below it enters stage s + 1.  The last
// stage stores each population in the row it moves to.  Every stage widens the input by one row and
// one column on each side: R + 2 (K - 1) rows are read for R written (the rows beyond are collided
// again by the neighbouring wavefronts, from the same values in the same order, so every node keeps
// its bits), and the K columns each side fit in the halo lanes of the strip (K columns rounded up to
// whole lanes).
//
// Walls half-way between rows (xi = 1/2): a bounced population stays in its row, so at the bottom
// row the three "from below" are that row's own downward ones, and at the top row the three on
// their way up wait for the next tick as that row's downward ones.
//
// What bounds it (8192^2 FP32): one step moved 18 words per node and took 866 us; five take 5 x 232 us,
// 109 vector instructions per node and step with the halo (80 % of the issue rate at 2.4 GHz) and 4.2 TB/s.  What a stage keeps is 9 CPL
// registers; with every stage in registers three steps spilled (349 us per step against 340), so
// the first one or two stages stay there and the others in LDS (9 KB per stage and wavefront: two
// blocks of four wavefronts fit a compute unit up to two such stages).
template <int K> constexpr int mrt_reg_stages() { return K > 4 ? 2 : 1; }
template <typename T, int CPL, int K> struct MrtStrip {
    static constexpr int P = (K + CPL - 1) / CPL;  // halo lanes on each side
    static constexpr int S = (64 - 2 * P) * CPL;   // stored columns
};

template <typename T, int CPL, int AM, int K, bool WALLS>
__global__ void __launch_bounds__(256, K > 1 ? 2 : 1) mrt_fused_kernel(const T *__restrict__ in, T *__restrict__ out, int nx, int ny,
                                                        int rows, int strips_x, int stride, int ntiles,
                                                        MrtCoef<typename Storage<T>::C> k)
{
    using C = typename Storage<T>::C;
    using namespace sweep;
    using G = MrtStrip<T, CPL, K>;
    const int lane = threadIdx.x & 63;
    const int tile = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tile >= ntiles) return;  // uniform over the wavefront
    const int band = tile / strips_x, sx = tile - band * strips_x;
    // element-aligned accesses: the last strip ends at column nx - 1 (see sweep_tile)
    const bool shift_last = (AM == AM_UNAL || AM == AM_SEAM) && sx == strips_x - 1 && nx > G::S;
    const int xl = (shift_last ? nx - G::S : sx * stride) - G::P * CPL + CPL * lane;
    const LaneCols<CPL, AM> lc = make_lane_cols<T, CPL, AM>(xl, nx, lane >= G::P && lane < 64 - G::P);
    const int y0 = band * rows, y1 = min(y0 + rows, ny);
    // stage s collides rows max(y0 - (K-1-s), 0 with walls) .. min(y1-1 + (K-1-s), ny-1 with walls)
    const int ya = WALLS ? max(y0 - (K - 1), 0) : y0 - (K - 1);
    const int yb = WALLS ? min(y1 - 1 + (K - 1), ny - 1) : y1 - 1 + (K - 1);
    const int nticks = y1 - 1 - ya + K;  // the last stage reaches row y1 - 1 at the last one

    auto load_row = [&](int y, Group<T, CPL>(&g)[9]) {
        const bool use = y <= yb;
        int yy = y < 0 ? y + ny : (y >= ny ? y - ny : y);
        yy = min(max(yy, 0), ny - 1);
#pragma unroll
        for (int q = 0; q < 9; ++q) g[q] = row_load<T, CPL, AM>(row_rsrc(in + pop_elem(0, 0, q, nx), yy, 9 * nx, nx), lc, use);
    };
    auto put = [&](int q, int y, const C(&v)[CPL]) {
        Group<T, CPL> g;
#pragma unroll
        for (int c = 0; c < CPL; ++c) g.v[c] = Storage<T>::store(v[c]);
        row_store<T, CPL, AM>(row_rsrc(out + pop_elem(0, 0, q, nx), y, 9 * nx, nx), lc, true, g);
    };

    // Kept between rows, per stage but the last: slots 0..2 the populations 0, 1, 3 of the row
    // collided last, 3..5 and 6..8 the 2, 5, 6 of the last two rows (by the row's parity, which is
    // static in the loop below).  The first KR stages keep them in registers, the others in LDS.
    constexpr int KR = K - 1 < mrt_reg_stages<K>() ? K - 1 : mrt_reg_stages<K>(), KL = K - 1 - KR;
    using V = Group<C, CPL>;
    V reg[KR > 0 ? KR : 1][9];
    __shared__ V lds[KL > 0 ? 4 : 1][KL > 0 ? KL : 1][9][KL > 0 ? 64 : 1];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto keep = [&](int s, int slot, const C(&v)[CPL]) {
        V g;
#pragma unroll
        for (int c = 0; c < CPL; ++c) g.v[c] = v[c];
        if (s < KR)
            reg[s < KR ? s : 0][slot] = g;
        else
            lds[wv][s < KR ? 0 : s - KR][slot][lane] = g;
    };
    auto kept = [&](int s, int slot, C(&v)[CPL]) {
        const V g = s < KR ? reg[s < KR ? s : 0][slot] : lds[wv][s < KR ? 0 : s - KR][slot][lane];
#pragma unroll
        for (int c = 0; c < CPL; ++c) v[c] = g.v[c];
    };
#pragma unroll
    for (int s = 0; s < KR; ++s)
#pragma unroll
        for (int q = 0; q < 9; ++q)
#pragma unroll
            for (int c = 0; c < CPL; ++c) reg[s][q].v[c] = C(0);

    auto tick = [&](int t, int ph, const Group<T, CPL>(&cur)[9]) {  // ph = t & 1
        C f[9][CPL];  // the row entering the stage, then its shifted post-collision populations
#pragma unroll
        for (int q = 0; q < 9; ++q)
#pragma unroll
            for (int c = 0; c < CPL; ++c) f[q][c] = Storage<T>::load(cur[q].v[c]);
#pragma unroll
        for (int s = 0; s < K; ++s) {
            const int y = ya + t - s;  // row of this stage
            // a stage starts with the first row it needs: the rows before it are not complete
            if (s > 0 && y < (WALLS ? max(y0 - (K - 1 - s), 0) : y0 - (K - 1 - s))) return;
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                C p[9];
#pragma unroll
                for (int q = 0; q < 9; ++q) p[q] = f[q][c];
                collide<C>(p, k);
#pragma unroll
                for (int q = 0; q < 9; ++q) f[q][c] = p[q];
            }
            // populations returning from a wall, unshifted: stored at once by the last stage
            C b[3][CPL];
            const bool bottom = WALLS && y == 0, top = WALLS && y == ny - 1;
            if (s == K - 1) {
                if (top) {
                    put(4, y, f[2]);
                    put(7, y, f[5]);
                    put(8, y, f[6]);
                }
                if (bottom) {
                    put(2, y, f[4]);
                    put(5, y, f[7]);
                    put(6, y, f[8]);
                }
            } else if (bottom || top)
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    b[0][c] = bottom ? f[4][c] : f[2][c];
                    b[1][c] = bottom ? f[7][c] : f[5][c];
                    b[2][c] = bottom ? f[8][c] : f[6][c];
                }
            // +x movers (1, 5, 8) arrive from the column on the left, -x movers (3, 6, 7) from
            // the column on the right
            const int rq[3] = {1, 5, 8}, lq[3] = {3, 6, 7};
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const C fl = from_left(f[rq[i]][CPL - 1]), fr = from_right(f[lq[i]][0]);
#pragma unroll
                for (int c = CPL - 1; c > 0; --c) f[rq[i]][c] = f[rq[i]][c - 1];
                f[rq[i]][0] = fl;
#pragma unroll
                for (int c = 0; c < CPL - 1; ++c) f[lq[i]][c] = f[lq[i]][c + 1];
                f[lq[i]][CPL - 1] = fr;
            }
            if (s < K - 1) {
                const int u = 3 + 3 * ((ph + s) & 1), v = 9 - u;  // slots of rows y and y - 2; of row y - 1
                const int stay[3] = {0, 1, 3}, rising[3] = {2, 5, 6}, falling[3] = {4, 7, 8};
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    C own[CPL], below[CPL];
                    kept(s, i, own);
                    kept(s, u + i, below);
                    keep(s, i, f[stay[i]]);
                    if (top)
                        keep(s, u + i, b[i]);
                    else
                        keep(s, u + i, f[rising[i]]);
                    if (bottom) keep(s, v + i, b[i]);
                    if (WALLS && y == ny) kept(s, v + i, f[falling[i]]);  // the top row has its own
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        f[stay[i]][c] = own[c];
                        f[rising[i]][c] = below[c];
                    }
                }
            } else {
                // the last stage: push (rows y0 .. y1 - 1; the guard above starts it at y0)
                put(0, y, f[0]);
                put(1, y, f[1]);
                put(3, y, f[3]);
                if (!top) {
                    const int yp = !WALLS && y + 1 == ny ? 0 : y + 1;
                    put(2, yp, f[2]);
                    put(5, yp, f[5]);
                    put(6, yp, f[6]);
                }
                if (!bottom) {
                    const int ym = !WALLS && y == 0 ? ny - 1 : y - 1;
                    put(4, ym, f[4]);
                    put(7, ym, f[7]);
                    put(8, ym, f[8]);
                }
            }
        }
    };

    Group<T, CPL> A[9], B[9];
    load_row(ya, A);
    for (int t = 0; t < nticks; t += 2) {
        load_row(ya + t + 1, B);
        tick(t, 0, A);
        if (t + 1 >= nticks) break;
        load_row(ya + t + 2, A);
        tick(t + 1, 1, B);
    }
}

// Small and medium grids: a block of 16 wavefronts keeps a tile of 64 columns by 16 R rows in
// registers (R rows per wavefront) for K steps, as fd_tile_kernel does for FD-LBM.  Every step
// loses one row and one column on each side of the tile.  Columns come from the adjacent lanes;
// the populations that cross to the wavefronts above and below go through LDS, in two buffers used
// in turn, so one barrier a step is enough.
constexpr int MRT_TW = 16;  // wavefronts per block

template <typename T, int R, bool WALLS>
__global__ void __launch_bounds__(64 * MRT_TW) mrt_tile_kernel(const T *__restrict__ in, T *__restrict__ out, int nx,
                                                               int ny, int steps, int tiles_x,
                                                               MrtCoef<typename Storage<T>::C> k)
{
    using C = typename Storage<T>::C;
    using sweep::from_left;
    using sweep::from_right;
    __shared__ C cross[2][MRT_TW][6][64];  // 2, 5, 6 of the last row, 4, 7, 8 of the first
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ty = blockIdx.x / tiles_x, tx = blockIdx.x - ty * tiles_x;
    const int cols = 64 - 2 * steps, rows = MRT_TW * R - 2 * steps;  // stored by a tile
    const int x = tx * cols - steps + lane, y0 = ty * rows - steps + wv * R;
    const size_t col = (size_t)((x % nx + nx) % nx);
    C f[R][9];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int y = y0 + i, yy = WALLS ? min(max(y, 0), ny - 1) : (y % ny + ny) % ny;
#pragma unroll
        for (int q = 0; q < 9; ++q) f[i][q] = Storage<T>::load(in[pop_elem(col, yy, q, nx)]);
    }
    const int rising[3] = {2, 5, 6}, falling[3] = {4, 7, 8};
    for (int step = 0; step < steps; ++step) {
        C b[R][3];  // with walls: the populations that return into their row
#pragma unroll
        for (int i = 0; i < R; ++i) {
            collide<C>(f[i], k);
            if (WALLS) {
                const bool bottom = y0 + i == 0;
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const C lo = f[i][falling[t]], hi = f[i][rising[t]];
                    b[i][t] = bottom ? lo : hi;
                }
            }
            f[i][1] = from_left(f[i][1]);
            f[i][5] = from_left(f[i][5]);
            f[i][8] = from_left(f[i][8]);
            f[i][3] = from_right(f[i][3]);
            f[i][6] = from_right(f[i][6]);
            f[i][7] = from_right(f[i][7]);
        }
        C(&lds)[MRT_TW][6][64] = cross[step & 1];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            lds[wv][t][lane] = f[R - 1][rising[t]];
            lds[wv][3 + t][lane] = f[0][falling[t]];
        }
        __syncthreads();
        const int wb = max(wv - 1, 0), wa = min(wv + 1, MRT_TW - 1);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
#pragma unroll
            for (int i = R - 1; i > 0; --i) f[i][rising[t]] = f[i - 1][rising[t]];
            f[0][rising[t]] = lds[wb][t][lane];
#pragma unroll
            for (int i = 0; i < R - 1; ++i) f[i][falling[t]] = f[i + 1][falling[t]];
            f[R - 1][falling[t]] = lds[wa][3 + t][lane];
        }
        if (WALLS)
#pragma unroll
            for (int i = 0; i < R; ++i) {
                if (y0 + i == 0)
#pragma unroll
                    for (int t = 0; t < 3; ++t) f[i][rising[t]] = b[i][t];
                if (y0 + i == ny - 1)
#pragma unroll
                    for (int t = 0; t < 3; ++t) f[i][falling[t]] = b[i][t];
            }
    }
    if (lane < steps || lane >= 64 - steps || x >= nx) return;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int j = wv * R + i, y = y0 + i;
        if (j < steps || j >= MRT_TW * R - steps || y >= ny) continue;
#pragma unroll
        for (int q = 0; q < 9; ++q) out[pop_elem(x, y, q, nx)] = Storage<T>::store(f[i][q]);
    }
}

// Equilibrium populations of host-order FP64 planes (drho, Jx, Jy; node (i, j) at j nx + i),
// stored row-interleaved; one block row of columns per grid row.
template <typename T>
__global__ void __launch_bounds__(256) mrt_init_kernel(const double *__restrict__ dr, const double *__restrict__ jx,
                                                       const double *__restrict__ jy, T *__restrict__ pop, int nx, int ny)
{
    using C = typename Storage<T>::C;
    for (int j = blockIdx.x; j < ny; j += gridDim.x)
        for (int i = threadIdx.x; i < nx; i += blockDim.x) {
            const size_t p = (size_t)j * (size_t)nx + (size_t)i;
            C m[9], f[9];
            m[0] = C(dr[p]);
            m[1] = C(jx[p]);
            m[2] = C(jy[p]);
            equilibrium<C>(m[0], m[1], m[2], m[3], m[4], m[5], m[6], m[7], m[8]);
            populations<C>(m, f);
#pragma unroll
            for (int q = 0; q < 9; ++q) pop[pop_elem(i, j, q, nx)] = Storage<T>::store(f[q]);
        }
}

// Conserved moments of the stored populations, summed in FP64 whatever the storage dtype,
// into host-order planes.
template <typename T>
__global__ void __launch_bounds__(256) mrt_moments_kernel(const T *__restrict__ pop, double *__restrict__ dr,
                                                          double *__restrict__ jx, double *__restrict__ jy, int nx,
                                                          int ny)
{
    for (int j = blockIdx.x; j < ny; j += gridDim.x)
        for (int i = threadIdx.x; i < nx; i += blockDim.x) {
            const size_t p = (size_t)j * (size_t)nx + (size_t)i;
            double f[9], m[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) f[q] = double(Storage<T>::load(pop[pop_elem(i, j, q, nx)]));
            moments<double>(f, m);
            dr[p] = m[0];
            jx[p] = m[1];
            jy[p] = m[2];
        }
}

// Rows per wavefront of a fused launch.  A wavefront of R rows collides R + K - 1 rows per stage on
// average, and the work is dealt to 1024 SIMDs: the time goes as ceil(wavefronts / 1024) (R + K - 1),
// whose minimum balances the rows collided twice against a last wave that is nearly empty.
int fused_rows(int strips_x, int ny, int K)
{
    int best = 1;
    long best_cost = -1;
    for (int rows = 1; rows <= 128 && rows <= ny; ++rows) {
        const long waves = (long)strips_x * ((ny + rows - 1) / rows);
        const long cost = (waves + 1023) / 1024 * (rows + K - 1);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = rows;
        }
    }
    return best;
}

template <typename T, int CPL, int AM, int K, bool WALLS>
hipError_t run_fused(const MrtArgs &a, MrtCoef<typename Storage<T>::C> k, int fused_rows, const void *src, void *dst, hipStream_t s)
{
    constexpr int S = MrtStrip<T, CPL, K>::S;
    const int strips_x = (a.nx + S - 1) / S;
    // one step: 1 row per wavefront measured best at 8192^2 (1 % over 2)
    const int rows = K == 1 ? (a.tile_rows > 0 ? a.tile_rows : 1) : fused_rows;
    if (rows < 1) return hipErrorInvalidValue;
    const int ntiles = strips_x * ((a.ny + rows - 1) / rows);
    const int stride = AM == sweep::AM_SEAM ? sweep::seam_stride(a.nx, S, MrtStrip<T, CPL, K>::P, CPL, sizeof(T)) : S;
    hipLaunchKernelGGL((mrt_fused_kernel<T, CPL, AM, K, WALLS>), (ntiles + 3) / 4, 256, 0, s, static_cast<const T *>(src),
                       static_cast<T *>(dst), a.nx, a.ny, rows, strips_x, stride, ntiles, k);
    return hipGetLastError();
}

template <typename T, int CPL, int K>
hipError_t run_width(const MrtArgs &a, MrtCoef<typename Storage<T>::C> k, int rows, const void *src, void *dst, hipStream_t s)
{
    using namespace sweep;
    using G = MrtStrip<T, CPL, K>;
    if (a.nx % CPL == 0)
        return a.walls ? run_fused<T, CPL, AM_VEC, K, true>(a, k, rows, src, dst, s)
                       : run_fused<T, CPL, AM_VEC, K, false>(a, k, rows, src, dst, s);
    // other widths: element-aligned accesses (through AM_UNAL's edge branches 6001 x 4097 FP32 takes 247 us
    // per step, 3001^2 FP64 83, here 103 and 74; 1021 x 770 the same), but single steps of a state that the
    // last-level cache holds take aligned accesses of fewer columns (FP32 1021 x 770 14.2 us and 12.7,
    // 191^2 6.3 and 3.6; 6001 x 4097 356 and 371)
    const bool seam = seam_stride(a.nx, G::S, G::P, CPL, sizeof(T)) > 0;
    if constexpr (K == 1) {
        if (!seam || 9 * sizeof(T) * (size_t)a.nx * (size_t)a.ny < (size_t(256) << 20)) {
            if constexpr (CPL > 2)
                if (a.nx % 2 == 0)
                    return a.walls ? run_fused<T, 2, AM_VEC, 1, true>(a, k, rows, src, dst, s)
                                   : run_fused<T, 2, AM_VEC, 1, false>(a, k, rows, src, dst, s);
            return a.walls ? run_fused<T, 1, AM_VEC, 1, true>(a, k, rows, src, dst, s)
                           : run_fused<T, 1, AM_VEC, 1, false>(a, k, rows, src, dst, s);
        }
    }
    if (seam)
        return a.walls ? run_fused<T, CPL, AM_SEAM, K, true>(a, k, rows, src, dst, s)
                       : run_fused<T, CPL, AM_SEAM, K, false>(a, k, rows, src, dst, s);
    if constexpr (K > 1)
        return a.walls ? run_fused<T, CPL, AM_UNAL, K, true>(a, k, rows, src, dst, s)
                       : run_fused<T, CPL, AM_UNAL, K, false>(a, k, rows, src, dst, s);
    return hipErrorInvalidValue;
}

template <typename T, int CPL>
hipError_t run_steps(const MrtArgs &a, MrtCoef<typename Storage<T>::C> k, int steps, int rows, const void *src, void *dst, hipStream_t s)
{
    switch (steps) {
    case 1: return run_width<T, CPL, 1>(a, k, rows, src, dst, s);
    case 3: return run_width<T, CPL, 3>(a, k, rows, src, dst, s);
    case 5: return run_width<T, CPL, 5>(a, k, rows, src, dst, s);
    default: return hipErrorInvalidValue;
    }
}

// Walls at a general distance: one step per launch, aligned accesses only.
template <typename T, int CPL>
hipError_t run_xi(const MrtArgs &a, MrtCoef<typename Storage<T>::C> k, const void *src, void *dst, hipStream_t s)
{
    constexpr int S = 64 * CPL - 2 * CPL;
    const int rows = a.tile_rows > 0 ? a.tile_rows : 1;
    const int strips_x = (a.nx + S - 1) / S;
    const int ntiles = strips_x * ((a.ny + rows - 1) / rows);
    using C = typename Storage<T>::C;
    hipLaunchKernelGGL((mrt_xi_kernel<T, CPL>), (ntiles + 3) / 4, 256, 0, s, static_cast<const T *>(src),
                       static_cast<T *>(dst), a.nx, a.ny, rows, strips_x, ntiles, k, C(a.xi));
    return hipGetLastError();
}

template <typename T, int R>
hipError_t run_tile(const MrtArgs &a, MrtCoef<typename Storage<T>::C> k, int steps, const void *src, void *dst, hipStream_t s)
{
    const int cols = 64 - 2 * steps, rows = MRT_TW * R - 2 * steps;
    if (steps < 1 || cols < 1 || rows < 1) return hipErrorInvalidValue;
    const int tiles_x = (a.nx + cols - 1) / cols, tiles = tiles_x * ((a.ny + rows - 1) / rows);
    if (a.walls)
        hipLaunchKernelGGL((mrt_tile_kernel<T, R, true>), tiles, 64 * MRT_TW, 0, s, static_cast<const T *>(src),
                           static_cast<T *>(dst), a.nx, a.ny, steps, tiles_x, k);
    else
        hipLaunchKernelGGL((mrt_tile_kernel<T, R, false>), tiles, 64 * MRT_TW, 0, s, static_cast<const T *>(src),
                           static_cast<T *>(dst), a.nx, a.ny, steps, tiles_x, k);
    return hipGetLastError();
}

template <typename T> hipError_t run_tile(const MrtArgs &a, const TilePlan &p, const void *src, void *dst, hipStream_t s)
{
    using C = typename Storage<T>::C;
    const MrtCoef<C> k{C(a.s_e), C(a.s_xx), C(a.s_q), C(a.s_eps), C(0.5 * a.fx), C(0.5 * a.fy), C(a.fx), C(a.fy)};
    if (p.rows == 1) return run_tile<T, 1>(a, k, p.steps, src, dst, s);
    if (p.rows == 2) return run_tile<T, 2>(a, k, p.steps, src, dst, s);
    if constexpr (sizeof(T) < 8)
        if (p.rows == 4) return run_tile<T, 4>(a, k, p.steps, src, dst, s);
    return hipErrorInvalidValue;
}

template <typename T> hipError_t run(const MrtArgs &a, int steps, int rows, const void *src, void *dst, hipStream_t s)
{
    using C = typename Storage<T>::C;
    MrtCoef<C> k{C(a.s_e), C(a.s_xx), C(a.s_q), C(a.s_eps), C(0.5 * a.fx), C(0.5 * a.fy), C(a.fx), C(a.fy)};
    if (a.kernel != FDLBM_KERNEL_REFERENCE) {
        constexpr int CPL = sizeof(T) == 8 ? 2 : 4;
        if (a.walls && a.xi != 0.5) {
            if (a.nx % CPL == 0) return run_xi<T, CPL>(a, k, src, dst, s);
            if (a.nx % 2 == 0) return run_xi<T, 2>(a, k, src, dst, s);
            return run_xi<T, 1>(a, k, src, dst, s);
        }
        return run_steps<T, CPL>(a, k, steps, rows, src, dst, s);
    }
    dim3 blk(64, 4), grd((a.nx + 63) / 64, (a.ny + 3) / 4);
    if (a.walls)
        hipLaunchKernelGGL((mrt_kernel<T, true>), grd, blk, 0, s, static_cast<const T *>(src), static_cast<T *>(dst),
                           a.nx, a.ny, k, C(a.xi));
    else
        hipLaunchKernelGGL((mrt_kernel<T, false>), grd, blk, 0, s, static_cast<const T *>(src), static_cast<T *>(dst),
                           a.nx, a.ny, k, C(0.5));
    return hipGetLastError();
}

inline unsigned rows_grid(int ny) { return (unsigned)(ny < 65536 ? ny : 65536); }

}  // namespace

// Steps per launch.  Five where the state streams from HBM: 8192^2 FP32 866 us per step one by one,
// 340 in threes, 234 in fives; 2500^2 82, 39, 31.  A smaller state stays in the caches, a launch
// lasts R + 2 (K - 1) ticks of one wavefront per SIMD, and three are as fast or faster: 1200^2 FP32
// 21, 9.3, 10.7 us; 1021 x 770 FP64 22.9, 9.1, 9.7.  The two meet between 60 and 90 MB in both types.
int mrt_max_fused(const MrtArgs &a)
{
    if (a.kernel == FDLBM_KERNEL_REFERENCE || (a.walls && a.xi != 0.5)) return 1;
    return 9 * (size_t)a.nx * (size_t)a.ny * dtype_bytes(a.dtype) >= (size_t(80) << 20) ? 5 : 3;
}

// Times of a launch (as in fd_launch_times()).  One step is bound by the state's bytes at 6 TB/s, on narrow
// grids by the wavefronts, one per row and strip.  K steps: one stage of one row of 64 CPL columns takes
// 0.9 us in FP32, 0.74 in FP64 (512^2, 1024^2, 2048^2); through AM_UNAL's edge branches twice as much.
LaunchTimes mrt_launch_times(const MrtArgs &a)
{
    const bool f64 = a.dtype == FDLBM_F64;
    const int CPL = f64 ? 2 : 4, eb = int(dtype_bytes(a.dtype));
    const double bytes_us = 18.0 * eb * a.nx * a.ny / 6e6;
    LaunchTimes t;
    t.most = mrt_max_fused(a);
    t.one = 3.0 + std::max(bytes_us, 0.9 / 1024.0 * a.ny * ((a.nx + 62 * CPL - 1) / (62 * CPL)));
    for (int K = 3; K <= t.most; K += 2) {
        const int P = (K + CPL - 1) / CPL, S = (64 - 2 * P) * CPL, strips = (a.nx + S - 1) / S;
        const int rows = fused_rows(strips, a.ny, K);
        const long each = ((long)strips * ((a.ny + rows - 1) / rows) + 1023) / 1024;
        double us = (f64 ? 0.74 : 0.9) * (a.walls ? 1.15 : 1.0);
        if (a.nx % CPL != 0 && sweep::seam_stride(a.nx, S, P, CPL, eb) == 0) us *= 2.0;
        t.rows[K] = rows;
        t.fused[K] = 3.0 + std::max(double(K * each) * (rows + K - 1) * us, bytes_us);
    }
    return t;
}

TileCost mrt_tile_cost(const MrtArgs &a)
{
    TileCost c;
    c.nx = a.nx;
    c.ny = a.ny;
    c.elem_bytes = int(dtype_bytes(a.dtype));
    c.lds = size_t(2 * MRT_TW * 6) * 64 * c.elem_bytes;
    c.row_us = a.dtype == FDLBM_F64 ? 0.9 : 0.7;
    c.start_us = 2.8;
    c.floor_us = 3.0 + 1.1 * 18.0 * c.elem_bytes * a.nx * a.ny / 6e6;
    return c;
}

TilePlan mrt_tile_plan(const MrtArgs &a, const LaunchTimes &t)
{
    if (a.kernel != FDLBM_KERNEL_AUTO || (a.walls && a.xi != 0.5)) return TilePlan();
    const TileShape shapes[] = {{1, 1}, {1, 2}, {1, 4}};
    const double sweep_us = std::min(t.one, t.most > 1 ? t.fused[t.most] / t.most : t.one);
    return plan_tiles(mrt_tile_cost(a), shapes, a.dtype == FDLBM_F64 ? 2 : 3, 25, sweep_us);
}

hipError_t launch_mrt_tile(const MrtArgs &a, const TilePlan &p, const void *src, void *dst, hipStream_t s)
{
    return a.dtype == FDLBM_F64 ? run_tile<double>(a, p, src, dst, s) : run_tile<float>(a, p, src, dst, s);
}

hipError_t launch_mrt(const MrtArgs &a, int steps, int rows, const void *src, void *dst, hipStream_t s)
{
    return a.dtype == FDLBM_F64 ? run<double>(a, steps, rows, src, dst, s) : run<float>(a, steps, rows, src, dst, s);
}

hipError_t launch_mrt_init(int dtype, const double *dr, const double *jx, const double *jy, void *pop, int nx, int ny,
                           hipStream_t s)
{
    if (dtype == FDLBM_F64)
        hipLaunchKernelGGL(mrt_init_kernel<double>, rows_grid(ny), 256, 0, s, dr, jx, jy, static_cast<double *>(pop), nx,
                           ny);
    else
        hipLaunchKernelGGL(mrt_init_kernel<float>, rows_grid(ny), 256, 0, s, dr, jx, jy, static_cast<float *>(pop), nx,
                           ny);
    return hipGetLastError();
}

hipError_t launch_mrt_moments(int dtype, const void *pop, double *dr, double *jx, double *jy, int nx, int ny,
                              hipStream_t s)
{
    if (dtype == FDLBM_F64)
        hipLaunchKernelGGL(mrt_moments_kernel<double>, rows_grid(ny), 256, 0, s, static_cast<const double *>(pop), dr,
                           jx, jy, nx, ny);
    else
        hipLaunchKernelGGL(mrt_moments_kernel<float>, rows_grid(ny), 256, 0, s, static_cast<const float *>(pop), dr,
                           jx, jy, nx, ny);
    return hipGetLastError();
}

}  // namespace fdlbm
