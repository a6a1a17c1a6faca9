// FD-LBM and LW-ACM steps, K time steps in one pass over memory: the part of one wavefront, shared
// by the single-grid kernel (fd_fused.hip) and the batch (fd_batch.hip).
//
// One step moves 6 words per node; in FP32 that and the vector work take about the same time, in
// FP64 the memory takes twice as long.  Here a wavefront reads a row once, takes it through K
// stages it holds on chip and stores the row of K steps later.
//
// Mapping: a wavefront owns a strip of 64*CPL columns (CPL per lane, lane shifts with DPP as in
// fd_sweep_body.hpp) for R output rows and walks up the rows, one input row per tick, the next
// row's loads in flight.  Stage s holds the newest row n_s it was given and the 2H rows below it,
// forms f* of row n_s - H - D, completes the output row below that one and hands it to stage
// s + 1 as its newest row (the last stage stores it).  Between rows a stage carries, per column,
// the sums going up, its own downward sums and the partial update of the row below.
//
// Every stage widens the input by H + 1 rows and columns on each side: R + 2 K (H + 1) rows are
// read for R stored, and the neighbouring wavefronts form the rows in between again, from the
// same values with the same operations in the same order (fd_node_fstar, row_sum, same_row_part,
// fd_partial, fd_finish), so every node keeps the bits of single steps.
//
// Walls: a band that reaches a wall sweeps towards it (the bottom one downwards, the others
// upwards), so that the rows a ghost row is formed from have come in before it.  The first stage
// reads its ghost rows by the rule of ghost_rules(), as the one-step kernel does; a later stage
// forms both of its when the first is due and sets the second aside for the next tick.  That
// covers the rules that reach the two rows next to the wall only (H = 1, xi >= 1/2); nearer walls
// take single steps.
#pragma once

#include "fd_sweep_body.hpp"

namespace fdlbm {
namespace sweep {

template <int CPL, int H, int K> struct FusedStrip {
    static constexpr int P = (K * (H + 1) + CPL - 1) / CPL;  // halo lanes on each side
    static constexpr int S = (64 - 2 * P) * CPL;             // stored columns
};

template <typename T, int K> struct FusedArgs {
    const T *in;
    T *out;
    int nx, ny, rows, strips_x, ntiles;
    int stride;  // columns from one strip to the next (AM_SEAM: the last one ends at column nx - 1)
    FdCoef<typename Storage<T>::C> k;
    GhostRules<typename Storage<T>::C> gr;
};

// Rows of a window that lives in LDS: those before the newest one, which comes in registers.
template <int H> constexpr int fused_ring() { return H > 0 ? 2 * H : 1; }
// Unrolling of the row loop, a multiple of the ring, so that every slot is static; a window in
// registers needs no more than its live rows.
template <int H, int K, int KR> constexpr int fused_unroll() { return H == 2 ? (KR < K ? 8 : 6) : 4; }

// Input rows in flight ahead of the one being worked on.  Two measured 1-2 % faster in FP32 (8192^2:
// 189.5 us per step against 192.7) and FP16, and no faster in FP64 or without differences.
template <typename T, int ST> constexpr int fused_ahead() { return sizeof(T) < 8 && ST == 3 ? 2 : 1; }
// Wavefronts per SIMD.  Two stages of 5-point windows do not fit 256 registers (1001 x 777 FP32: 13.9
// us per step with spills, 12.8 with one wavefront and 512 registers; 4096^2 FP64 221 and 132).
template <int ST> constexpr int fused_waves() { return ST == 5 ? 1 : 2; }
// Whether the compiler schedules one stage at a time: across stages it overlaps more (FP32 2-3 %),
// but where registers are short it spills.
template <typename C, int ST, bool FORCE, int AM> constexpr bool fused_fence()
{
    return sizeof(C) == 8 || ST == 5 || FORCE || AM == AM_UNAL || AM == AM_COL;
}

// What one stage carries from row to row, per column: the sums the last row sends on (fw, fwx), its
// own sums in the other direction (lb, lbx), and of its update what is known: sweeping up, the
// partial update (a: q, b: qx, c: pu); sweeping down, the same-row part (a, b) and the part from the
// row above (c, d).
enum { C_FW, C_FWX, C_LB, C_LBX, C_A, C_B, C_C, C_D, NCARRY };

// LDS of one wavefront, in groups of CPL values per lane: the windows of the stages from KR on,
// with walls the ghost rows they set aside, and the carries of the stages from KC on.
template <int H, bool WALLS, int K, int KR, int KC> constexpr int fused_lds_slots()
{
    return (K - KR) * 3 * (fused_ring<H>() + (WALLS ? 1 : 0)) + (K - KC) * NCARRY;
}

template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

template <int DIR, typename T, int CPL, int ST, bool WALLS, bool FORCE, int AM, int K, int KR, int KC>
__device__ __forceinline__ void fused_tile(const FusedArgs<T, K> &a, Group<typename Storage<T>::C, CPL> (*ldsw)[64],
                                           int lane, int xl, const LaneCols<CPL, AM> &lc, int y0, int y1)
{
    using C = typename Storage<T>::C;
    using S = Stencil<ST>;
    constexpr int H = S::H;
    constexpr bool LW = ST == 1;
    constexpr int U = fused_unroll<H, K, KR>();
    constexpr int RING = fused_ring<H>();
    static_assert(U % RING == 0 && U > 2 * H + 1, "window");
    static_assert(!WALLS || (H == 1 && KR == 1), "later stages set ghost rows aside in LDS");
    using V = Group<C, CPL>;
    const int nx = a.nx, ny = a.ny;

    // the first stage completes the rows ext beyond the band: first and last row of input, ticks
    constexpr int ext = (K - 1) * (H + 1);
    const int i0 = DIR > 0 ? y0 - ext - 1 - H : y1 + ext + H;
    const int ilast = DIR > 0 ? y1 + ext + H : y0 - ext - 1 - H;
    const int nticks = y1 - y0 + 2 * K * (H + 1);

    // windows and carries
    C w[KR][U][3][CPL], cr[KC > 0 ? KC : 1][NCARRY][CPL];
#pragma unroll
    for (int s = 0; s < KC; ++s)
#pragma unroll
        for (int q = 0; q < NCARRY; ++q)
#pragma unroll
            for (int c = 0; c < CPL; ++c) cr[s][q][c] = C(0);
#pragma unroll
    for (int s = 0; s < KR; ++s)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int c = 0; c < CPL; ++c) w[s][u][f][c] = C(0);
    // LDS: the windows (and ghost rows set aside, row RING), then the carries
    constexpr int WSLOTS = 3 * (RING + (WALLS ? 1 : 0)), CBASE = (K - KR) * WSLOTS;
    auto lds_put = [&](int slot, const C(&v)[CPL]) __attribute__((always_inline)) {
        V g;
#pragma unroll
        for (int c = 0; c < CPL; ++c) g.v[c] = v[c];
        ldsw[slot][lane] = g;
    };
    auto lds_get = [&](int slot, C(&v)[CPL]) __attribute__((always_inline)) {
        const V g = ldsw[slot][lane];
#pragma unroll
        for (int c = 0; c < CPL; ++c) v[c] = g.v[c];
    };
    auto put_row = [&](int s, int slot, const C(&v)[3][CPL]) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < 3; ++f)
            if (s < KR) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) w[s < KR ? s : 0][slot][f][c] = v[f][c];
            } else {
                lds_put((s < KR ? 0 : s - KR) * WSLOTS + 3 * (slot % RING) + f, v[f]);
            }
    };
    auto get_row = [&](int s, int slot, C(&v)[3][CPL]) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < 3; ++f)
            if (s < KR) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) v[f][c] = w[s < KR ? s : 0][slot][f][c];
            } else {
                lds_get((s < KR ? 0 : s - KR) * WSLOTS + 3 * (slot % RING) + f, v[f]);
            }
    };

    // loads of one input row; with walls, its factors and second row (as in sweep_wave)
    constexpr int PD = fused_ahead<T, ST>();
    static_assert(U % PD == 0, "a load's group must not depend on the loop iteration");
    Group<T, CPL> raw[PD][3];
    C rca[PD], rcj[PD], rbr[PD], rbj[PD];
    int rsb[PD];
    auto fetch = [&](int j, int u) __attribute__((always_inline)) {
        const bool use = DIR > 0 ? j <= ilast : j >= ilast;
        int src = j;
        rsb[u] = -1;
        rca[u] = rcj[u] = C(1);
        rbr[u] = rbj[u] = C(0);
        if (WALLS) {
            if (j < 0 || j >= ny) {  // ghost row beyond a wall
                const GhostRule<C> q = ghost_rule(a.gr, j < 0 ? -j : j - ny + 1);
                src = j < 0 ? q.sa : ny - 1 - q.sa;
                if (q.sb >= 0) rsb[u] = min(max(j < 0 ? q.sb : ny - 1 - q.sb, 0), ny - 1);
                rca[u] = q.car;
                rcj[u] = q.caj;
                rbr[u] = q.cbr;
                rbj[u] = q.cbj;
            }
        } else {
            src = j < 0 ? j + ny : (j >= ny ? j - ny : j);
        }
        src = min(max(src, 0), ny - 1);
#pragma unroll
        for (int f = 0; f < 3; ++f)
            raw[u][f] = row_load<T, CPL, AM>(row_rsrc(a.in + fd_elem(0, 0, f, nx), src, 3 * nx, nx), lc, use);
    };
    auto arrive = [&](int u, C(&v)[3][CPL]) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int c = 0; c < CPL; ++c)
                v[f][c] = WALLS ? (f == 0 ? rca[u] : rcj[u]) * Storage<T>::load(raw[u][f].v[c])
                                : Storage<T>::load(raw[u][f].v[c]);
        if (WALLS && rsb[u] >= 0) {
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                const Group<T, CPL> g =
                    row_load<T, CPL, AM>(row_rsrc(a.in + fd_elem(0, 0, f, nx), rsb[u], 3 * nx, nx), lc, true);
#pragma unroll
                for (int c = 0; c < CPL; ++c) v[f][c] = v[f][c] + (f == 0 ? rbr[u] : rbj[u]) * Storage<T>::load(g.v[c]);
            }
        }
    };
    // ghost row at distance g beyond a wall of a later stage, from its rows 0 and 1 off the wall
    auto ghost = [&](int g, const C(&w0)[3][CPL], const C(&w1)[3][CPL], C(&v)[3][CPL]) __attribute__((always_inline)) {
        const GhostRule<C> q = ghost_rule(a.gr, g);
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                v[f][c] = (f == 0 ? q.car : q.caj) * (q.sa == 0 ? w0[f][c] : w1[f][c]);
                if (q.sb >= 0) v[f][c] = v[f][c] + (f == 0 ? q.cbr : q.cbj) * w1[f][c];
            }
    };

    // One stage: f* of the row r that lies H rows before the newest one (nrow, whose slot is ph), and
    // the completed row before r, returned in nrow.
    auto stage = [&](int s, int ph, C(&nrow)[3][CPL]) __attribute__((always_inline)) {
        // rows r - H .. r + H in sweep order (LW-ACM: the row before r, and r)
        constexpr int LO = H > 0 ? H : 1;
        C wr[LO + H + 1][3][CPL];
#pragma unroll
        for (int k = -LO; k < H; ++k) get_row(s, (ph - H + k + 2 * U) % U, wr[k + LO]);
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int c = 0; c < CPL; ++c) wr[LO + H][f][c] = nrow[f][c];
        put_row(s, ph, nrow);
        const C(&me)[3][CPL] = wr[LO];
        C f[CPL][9];
        if constexpr (LW) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) lw_node_g<C>(me[0][c], me[1][c], me[2][c], a.k.lin, f[c]);
        } else {
            auto yfield = [&](int q, int k, int c) -> C {
                const C(&v)[3][CPL] = wr[DIR * k + LO];  // k rows up the grid
                const C xa = plus_force<FORCE>(v[1][c], a.k.hfx), ya = plus_force<FORCE>(v[2][c], a.k.hfy);
                return q == 0 ? v[0][c] : q == 1 ? v[2][c] : q == 2 ? v[1][c] : q == 3 ? xa * ya : ya * ya;
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
            C xl1[5], xr1[5], xl2[5], xr2[5];
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                xl1[q] = from_left(xf[q][CPL - 1]);
                xr1[q] = from_right(xf[q][0]);
                xl2[q] = H == 2 ? from_left(xf[q][CPL >= 2 ? CPL - 2 : 0]) : C(0);
                xr2[q] = H == 2 ? from_right(xf[q][CPL > 1 ? 1 : 0]) : C(0);
            }
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                C dd[10];
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    const C m1 = c > 0 ? xf[q][c > 0 ? c - 1 : 0] : xl1[q];
                    const C p1 = c < CPL - 1 ? xf[q][c < CPL - 1 ? c + 1 : 0] : xr1[q];
                    C m2 = C(0), p2 = C(0), ym2 = C(0), yp2 = C(0);
                    if constexpr (H == 2) {
                        m2 = c >= 2 ? xf[q][c >= 2 ? c - 2 : 0] : (c == 1 ? xl1[q] : xl2[q]);
                        p2 = c + 2 < CPL ? xf[q][c + 2 < CPL ? c + 2 : 0] : (c + 2 == CPL ? xr1[q] : xr2[q]);
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
        constexpr int NC = DIR > 0 ? C_D : NCARRY;  // carried values in use
        C cin[NCARRY][CPL], co[NCARRY][CPL];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            if (s < KC) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) cin[q][c] = cr[s < KC ? s : 0][q][c];
            } else {
                lds_get(CBASE + (s < KC ? 0 : s - KC) * NCARRY + q, cin[q]);
            }
        }
        const C(&old)[3][CPL] = wr[LO - 1];  // the stored row that is completed
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int cl = c > 0 ? c - 1 : 0, cn = c < CPL - 1 ? c + 1 : 0;
            const C c1 = c > 0 ? f[cl][1] : f1l;
            const C u5 = c > 0 ? f[cl][5] : f5l;
            const C d8 = c > 0 ? f[cl][8] : f8l;
            const C c3 = c < CPL - 1 ? f[cn][3] : f3r;
            const C u6 = c < CPL - 1 ? f[cn][6] : f6r;
            const C d7 = c < CPL - 1 ? f[cn][7] : f7r;
            // sums leaving row r up and down, and the same groups of the node's own populations
            const C up = row_sum(f[c][2], u5, u6), upx = u5 - u6;
            const C dn = row_sum(f[c][4], d8, d7), dnx = d8 - d7;
            const C lu = row_sum(f[c][2], f[c][5], f[c][6]), lux = f[c][5] - f[c][6];
            const C ld = row_sum(f[c][4], f[c][8], f[c][7]), ldx = f[c][8] - f[c][7];
            C pc, pcx;
            same_row_part<C>(c1 - f[c][1], c3 - f[c][3], pc, pcx);
            if constexpr (DIR > 0) {
                const FdPartial<C> qp{cin[C_A][c], cin[C_B][c], cin[C_C][c]};
                fd_finish<C, FORCE>(qp, dn - cin[C_LB][c], dnx - cin[C_LBX][c], old[0][c], old[1][c], old[2][c], a.k.dfx,
                                    a.k.dfy, nrow[0][c], nrow[1][c], nrow[2][c]);
                const FdPartial<C> np = fd_partial<C>(pc, pcx, cin[C_FW][c] - lu, cin[C_FWX][c] - lux);
                co[C_A][c] = np.q;
                co[C_B][c] = np.qx;
                co[C_C][c] = np.pu;
                co[C_FW][c] = up;
                co[C_FWX][c] = upx;
                co[C_LB][c] = ld;
                co[C_LBX][c] = ldx;
            } else {
                const FdPartial<C> qp =
                    fd_partial<C>(cin[C_A][c], cin[C_B][c], up - cin[C_LB][c], upx - cin[C_LBX][c]);
                fd_finish<C, FORCE>(qp, cin[C_C][c], cin[C_D][c], old[0][c], old[1][c], old[2][c], a.k.dfx, a.k.dfy,
                                    nrow[0][c], nrow[1][c], nrow[2][c]);
                co[C_A][c] = pc;
                co[C_B][c] = pcx;
                co[C_C][c] = cin[C_FW][c] - ld;
                co[C_D][c] = cin[C_FWX][c] - ldx;
                co[C_FW][c] = dn;
                co[C_FWX][c] = dnx;
                co[C_LB][c] = lu;
                co[C_LBX][c] = lux;
            }
        }
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            if (s < KC) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) cr[s < KC ? s : 0][q][c] = co[q][c];
            } else {
                lds_put(CBASE + (s < KC ? 0 : s - KC) * NCARRY + q, co[q]);
            }
        }
    };

    // one row in, through the first NS stages (the last stage stores)
    auto tick = [&](int t, int ph, auto stages) __attribute__((always_inline)) {
        constexpr int NS = decltype(stages)::value;
        C row[3][CPL];
        arrive(ph % PD, row);
        fetch(i0 + DIR * (t + PD), ph % PD);
        int n = i0 + DIR * t;  // newest row of the stage
#pragma unroll
        for (int s = 0; s < (NS < K ? NS + 1 : K); ++s) {
            if (WALLS && s > 0) {
                const int beyond = DIR > 0 ? n - ny : -1 - n;  // rows past the first ghost row
                const int aside = (s < KR ? 0 : s - KR) * WSLOTS + 3 * RING;
                if (beyond == 0) {
                    C w0[3][CPL], w1[3][CPL], g2[3][CPL];
                    get_row(s, (ph + U - 1) % U, w0);
                    get_row(s, (ph + U - 2) % U, w1);
                    ghost(1, w0, w1, row);
                    ghost(2, w0, w1, g2);
#pragma unroll
                    for (int f = 0; f < 3; ++f) lds_put(aside + f, g2[f]);
                } else if (beyond > 0) {
#pragma unroll
                    for (int f = 0; f < 3; ++f) lds_get(aside + f, row[f]);
                }
            }
            if (s >= NS) {
                put_row(s, ph, row);
                break;
            }
            stage(s, ph, row);
            if (fused_fence<C, ST, FORCE, AM>()) __builtin_amdgcn_sched_barrier(0);
            n -= DIR * (H + 1);  // the completed row
            // rounded for storage, as a step of its own would (FP16)
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
#pragma unroll
                for (int f = 0; f < 3; ++f)
                    if constexpr (!std::is_same_v<T, C>)
                        row[f][c] = Storage<T>::load(Storage<T>::store(row[f][c]));
            }
        }
        if (NS < K) return;
        const bool use = n >= y0 && n < y1;
        const int orow = min(max(n, 0), ny - 1);
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            Group<T, CPL> g;
#pragma unroll
            for (int c = 0; c < CPL; ++c) g.v[c] = Storage<T>::store(row[f][c]);
            row_store<T, CPL, AM>(row_rsrc(a.out + fd_elem(0, 0, f, nx), orow, 3 * nx, nx), lc, use, g);
        }
    };

    // Stage s has a full window from tick first(s) on.  Whole rounds of the window before the last
    // stage's run the stages that have one; the few ticks left over form values nobody uses.
    // (Skipping them by a branch in the loop would keep every slot of every window live.)
    constexpr int step = 2 * (H + 1), T0 = (2 * H + (K - 1) * step) / U * U;
#pragma unroll
    for (int u = 0; u < PD; ++u) fetch(i0 + DIR * u, u);
    static_for<T0>([&](auto t) __attribute__((always_inline)) {
        constexpr int ns = t.value < 2 * H ? 0 : (t.value - 2 * H) / step + 1;
        tick(t.value, t.value % U, std::integral_constant<int, ns>{});
    });
    for (int t0 = T0; t0 < nticks; t0 += U) {
#pragma unroll
        for (int ph = 0; ph < U; ++ph) {
            if (t0 + ph >= nticks) break;
            tick(t0 + ph, ph, std::integral_constant<int, K>{});
        }
    }
}

}  // namespace sweep
}  // namespace fdlbm
