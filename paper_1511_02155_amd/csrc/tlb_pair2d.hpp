// S D2Q9 steps (two, or four in FP64) in one launch: u_t -> u_{t+S} with the states between kept on the compute
// unit.
//
// What bounds the one-step kernel is the traffic of the state: it reads and writes every population
// once per step, and at 1024^2 it moves these bytes as fast as their access pattern allows.  Here a
// workgroup of S wavefronts owns a strip of columns and sweeps a chunk of rows.  The first wavefront
// advances the rows by a step, the second advances them by another, a few rows behind it, and so on; a row
// goes from each wavefront to the next through LDS, where it is read with the column shifts of the pull.  S
// steps then read the state once and write it once.
//
// Columns.  A wavefront's 64 lanes are neighbouring columns (periodic in x); the concentrations of the
// columns beside a lane come from the wavefront's own LDS rows.  The first step is right in lanes 1 .. 62
// (its stencils need both neighbours), each later one in two lanes less at either end (pull and stencil), so
// a strip has up to 58 columns for two steps and 50 for four.
//
// Rows.  Virtual row v of an item is lattice row yfirst + v*DIR; rows 0 .. L-1 are its output.  In
// iteration k the first wavefront takes the pulled row v = k - (2S-1), forms its concentrations and collides
// row v-1; wavefront r > 0 takes row w = k - (2S+1) - 3(r-1) from the link before it, which completes the
// pull of row w-1, forms the concentrations of that row, and collides and passes on row w-2 (the last one
// stores it).  An item so takes L + 5S - 3 iterations, one barrier each (a link holds two rows in turn: one
// is written while the other is read).  The pulled row v+1 is in flight during iteration k.  Neighbouring
// chunks sweep in opposite directions, so that they reach the rows they both read at the same time, and
// every other launch reverses all of them, as in the one-step sweep.
//
// Measured on MI355X, per step, against the one-step kernel: two steps at 1024^2 FP32 30.5 us (42.4), 512^2
// FP64 15.4 (23.1), 1024^2 of five components FP64 98.5 (168); four steps at 1024^2 FP64 45.8 (89.7; 57 with
// two), 2048^2 157 (353; 244), 700 x 900 of four components with several relaxation times 41.3 (76.9; 43).
// Two FP64 steps at 1024^2 move their bytes at 5.0 TB/s; four steps need a third fewer bytes per step and are
// bound by the 1.7 us an iteration takes at one wavefront per SIMD (registers and links leave room for one
// item per compute unit).  FP32 holds two wavefronts per SIMD and is bound by their instructions (2.2 us per
// iteration), so that the columns four steps would give up cost more than their bytes save.  The
// iterations have no branches but those at walls (rows that do not exist are computed and never used),
// which took the two-step FP64 kernel from 780 to 560 instructions per iteration and wavefront.
//
// Every value is formed by the operations of the one-step kernel in the same order, so the results are
// bitwise those of single steps.
#pragma once

#include "tlb_sweep2d.hpp"

namespace tlb {

// Orders a wavefront's own LDS accesses across its lanes.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

__device__ __forceinline__ void link_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <typename T, int NC, int S>
struct PairLds {
    T link[S - 1][2][9 * NC][64];  // rows on their way from each wavefront to the next
    double row[S][3][NC][64];      // per wavefront: the concentration deviations of its last three rows
};

// Directions by their y component relative to the sweep: lead come from the row after (e_y = -DIR), level
// from the same row, trail from the row before.
template <int DIR>
struct Classes {
    static constexpr int lead[3] = {DIR > 0 ? 4 : 3, DIR > 0 ? 6 : 5, DIR > 0 ? 8 : 7};
    static constexpr int level[3] = {0, 1, 2};
    static constexpr int trail[3] = {DIR > 0 ? 3 : 4, DIR > 0 ? 5 : 6, DIR > 0 ? 7 : 8};
};

// Columns of a strip and iterations of an item beyond its rows, for S steps.
constexpr int pair_cols(int S) { return 64 - 2 * (2 * S - 1); }
constexpr int pair_fill(int S) { return 5 * S - 3; }

template <typename T, int DIR, bool MRT, int NC, int S>
__device__ __forceinline__ void pair_sweep(const StepArgs<T>& A, int x0, int ncols, int y0, int L, PairLds<T, NC, S>& M)
{
    using C = double;
    constexpr int J = 9 * NC, H = 2 * S - 1;
    const int lane = threadIdx.x & 63;
    const int nx = A.nx, ny = A.ny;
    const bool walls = A.walls != 0;
    const int yfirst = DIR > 0 ? y0 : y0 + L - 1;
    // virtual rows that exist (all of them without walls)
    const int vlo = walls ? (DIR > 0 ? -y0 : yfirst - (ny - 1)) : -(1 << 29);
    const int vhi = walls ? (DIR > 0 ? ny - 1 - y0 : yfirst) : (1 << 29);
    const int K = L + pair_fill(S);
    const uint32_t rowb = (uint32_t)nx * (uint32_t)sizeof(T);           // bytes of a row
    const uint32_t arrb = (uint32_t)A.N * (uint32_t)sizeof(T);          // bytes of a population array
    const uint32_t state = arrb * (uint32_t)J;
    // lattice row of virtual row v, and the step to the next one
    auto row_of = [&](int v) {
        const int y = (yfirst + v * DIR) % ny;
        return y < 0 ? y + ny : y;
    };
    auto next_row = [&](int y) { return DIR > 0 ? (y == ny - 1 ? 0 : y + 1) : (y == 0 ? ny - 1 : y - 1); };
    // columns of the lane and of its neighbours, periodic
    int x = (x0 - H + lane) % nx;
    x = x < 0 ? x + nx : x;
    // wetting offsets beyond the wall that the sweep enters at and the one it ends at
    const T* wet_in = A.wet + (size_t)(DIR > 0 ? 0 : 1) * NC * nx + x;
    const T* wet_out = A.wet + (size_t)(DIR > 0 ? 1 : 0) * NC * nx + x;
    // rows of concentrations: the wavefront's own, in turn (the previous, this and the next one)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double(*const rows)[NC][64] = M.row[wave];
    const int lf = lane == 0 ? 0 : lane - 1, rt = lane == 63 ? 63 : lane + 1;
    auto ghost = [&](int of, const T* wt, int to) {
#pragma unroll
        for (int m = 0; m < NC; ++m) rows[to][m][lane] = rows[of][m][lane] + C(wt[(size_t)m * nx]);
    };
    auto stencils = [&](int a, int b, int c, C (&dc)[NC], C (&g)[NC][3], C (&lap)[NC]) {
        wave_fence();
#pragma unroll
        for (int m = 0; m < NC; ++m) {
            const C al = rows[a][m][lf], ar = rows[a][m][rt], bl = rows[b][m][lf], br = rows[b][m][rt],
                    cl = rows[c][m][lf], cr = rows[c][m][rt];
            dc[m] = rows[b][m][lane];
            stencil9<C>(rows[a][m][lane], al + ar, ar - al, dc[m], bl + br, br - bl, rows[c][m][lane], cl + cr, cr - cl,
                        DIR, g[m], lap[m]);
        }
        wave_fence();
    };
    auto concentrations = [&](const T* p, Moments<C, NC>& mo, int to) {
        mo = moments<L9, NC>(p, p + 9, p + 18);
        C c[NC];
        conc_dev<C, NC>(mo, c);
#pragma unroll
        for (int m = 0; m < NC; ++m) rows[to][m][lane] = c[m];
    };

    // the deviations of psi_l are those of C_l, which come back from LDS: they need not be held as moments
    auto psi_of = [&](Moments<C, NC>& mo, const C (&dc)[NC]) {
        mo.dpsi = dc[2];
#pragma unroll
        for (int l = 0; l < NC - 3; ++l) mo.dpsx[l] = dc[3 + l];
    };

    if (wave == 0) {
        // ---- first step ----
        const uint32_t vo[3] = {(uint32_t)x * (uint32_t)sizeof(T),
                                (uint32_t)(x == 0 ? nx - 1 : x - 1) * (uint32_t)sizeof(T),
                                (uint32_t)(x == nx - 1 ? 0 : x + 1) * (uint32_t)sizeof(T)};
        const Rsrc src = make_rsrc(A.src, state);
        // the pull of row y: per-lane offsets of the three rows and columns it comes from, uniform ones of the
        // population arrays; at a wall the populations that would come from beyond it are loaded once more
        auto pull = [&](int y, T* p) {
            const uint32_t at[3] = {(uint32_t)y * rowb, (uint32_t)(y == 0 ? ny - 1 : y - 1) * rowb,
                                    (uint32_t)(y == ny - 1 ? 0 : y + 1) * rowb};
            uint32_t off[3][3];
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int q = 0; q < 3; ++q) off[r][q] = vo[q] + at[r];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int r = L9::ey[i] == 0 ? 0 : (L9::ey[i] == 1 ? 1 : 2), q = L9::ex[i] == 0 ? 0 : (L9::ex[i] == 1 ? 1 : 2);
#pragma unroll
                for (int s = 0; s < NC; ++s) p[9 * s + i] = bload<T>(src, off[r][q], (uint32_t)(9 * s + i) * arrb);
            }
            if (walls && (y == 0 || y == ny - 1)) {
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    if (L9::ey[i] != 0 && (L9::ey[i] == 1 ? y == 0 : y == ny - 1))
#pragma unroll
                        for (int s = 0; s < NC; ++s)
                            p[9 * s + i] = bload<T>(src, off[0][0], (uint32_t)(9 * s + L9::opp[i]) * arrb);
            }
        };
        T P0[J], P1[J], P2[J];
#pragma unroll
        for (int i = 0; i < J; ++i) P0[i] = P1[i] = P2[i] = T(0);
        Moments<C, NC> m0 = {}, m1 = {}, m2 = {};
        auto exists = [&](int v) { return v >= vlo && v <= vhi; };
        int yn = row_of(-H);  // the row to load next
        if (exists(-H)) pull(yn, P0);
        // rows v, v-1 and v+1 of the populations; a, b, c: LDS rows of v-2, v-1 and v
        auto step = [&](int k, int a, int b, int c, T* Pc, T* Pb, T* Pn, Moments<C, NC>& Mc, Moments<C, NC>& Mb) {
            const int v = k - H;
            yn = next_row(yn);
            if (v + 1 < L + H && exists(v + 1)) pull(yn, Pn);
            concentrations(Pc, Mc, c);
            if (walls) {
                if (v == vlo) ghost(c, wet_in, b);
                if (v == vhi + 1) ghost(b, wet_out, c);
            }
            C dc[NC], gC[NC][3], lC[NC];
            stencils(a, b, c, dc, gC, lC);
            psi_of(Mb, dc);
            collide<L9, MRT, NC>(A.P, Mb, dc, gC, lC, Pb, Pb + 9, Pb + 18);
            T(*out)[64] = M.link[0][k & 1];
#pragma unroll
            for (int j = 0; j < J; ++j) out[j][lane] = Pb[j];
            link_barrier();
        };
        for (int k = 0; k < K; k += 3) {
            step(k, 1, 2, 0, P0, P2, P1, m0, m2);
            if (k + 1 < K) step(k + 1, 2, 0, 1, P1, P0, P2, m1, m0);
            if (k + 2 < K) step(k + 2, 0, 1, 2, P2, P1, P0, m2, m1);
        }
    } else {
        // ---- the later steps ----
        const bool last = S == 2 || wave == S - 1;
        using CL = Classes<DIR>;
        const Rsrc dst = make_rsrc(A.dst, state);
        const bool active = lane >= H && lane < H + ncols;
        const uint32_t vo = (uint32_t)x * (uint32_t)sizeof(T);
        // lanes that hold the columns x, x-1 and x+1 (the wavefront's end lanes are never used)
        const int from[3] = {lane, lane == 0 ? 0 : lane - 1, lane == 63 ? 63 : lane + 1};
        T Q0[J], Q1[J], Q2[J];
#pragma unroll
        for (int i = 0; i < J; ++i) Q0[i] = Q1[i] = Q2[i] = T(0);
        Moments<C, NC> m0 = {}, m1 = {}, m2 = {};
        int ye = yfirst;  // the row to store next
        // rows w-1 (completed now), w-2 (collided) and w of the populations; ra, rb, rc: LDS rows of w-3, w-2, w-1
        auto step = [&](int k, int ra, int rb, int rc, T* Qc, T* Qb, T* Qn, Moments<C, NC>& Mc, Moments<C, NC>& Mb) {
            const int w = k - (2 * S + 1) - 3 * (wave - 1);
            T(*in)[64] = M.link[wave - 1][(k - 1) & 1];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int s = 0; s < NC; ++s) {
                    // pull: x - e_x; q = 0, 1, 2 are e_x = 0, +1, -1 in each class
                    if (!(walls && w == vhi + 1)) Qc[9 * s + CL::lead[q]] = in[9 * s + CL::lead[q]][from[q]];
                }
            const int c = w - 1;
            concentrations(Qc, Mc, rc);
            if (walls) {
                if (c == vlo) ghost(rc, wet_in, rb);
                if (c == vhi + 1) ghost(rb, wet_out, rc);
            }
            const int e = w - 2;
            if (e >= -2 * (S - 1 - wave)) {
                C dc[NC], gC[NC][3], lC[NC];
                stencils(ra, rb, rc, dc, gC, lC);
                psi_of(Mb, dc);
                collide<L9, MRT, NC>(A.P, Mb, dc, gC, lC, Qb, Qb + 9, Qb + 18);
                if (!last) {
                    T(*out)[64] = M.link[S == 2 ? 0 : wave][k & 1];
#pragma unroll
                    for (int j = 0; j < J; ++j) out[j][lane] = Qb[j];
                }
                const uint32_t off = vo + (uint32_t)ye * rowb;
                if (last) ye = next_row(ye);
                if (last && active) {
#pragma unroll
                    for (int i = 0; i < 9; ++i)
#pragma unroll
                        for (int s = 0; s < NC; ++s) bstore<T>(Qb[9 * s + i], dst, off, (uint32_t)(9 * s + i) * arrb);
                }
            }
            // row w takes the populations of its own level, and the row after it its trailing ones (into the
            // registers just stored).  At the first row there is, and at the last one, the wall row's own
            // populations, turned back, complete it.
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int s = 0; s < NC; ++s) {
                    Qn[9 * s + CL::level[q]] = in[9 * s + CL::level[q]][from[q]];
                    Qb[9 * s + CL::trail[q]] = in[9 * s + CL::trail[q]][from[q]];
                }
            if (walls && w == vlo) {
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int s = 0; s < NC; ++s) Qn[9 * s + CL::trail[q]] = in[9 * s + L9::opp[CL::trail[q]]][lane];
            }
            if (walls && w == vhi) {
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int s = 0; s < NC; ++s) Qn[9 * s + CL::lead[q]] = in[9 * s + L9::opp[CL::lead[q]]][lane];
            }
            link_barrier();
        };
        // nothing of use has come through the link before this iteration
        const int k0 = 5 * wave - 2;
        for (int k = 0; k < k0; ++k) link_barrier();
        for (int k = k0; k < K; k += 3) {
            step(k, 1, 2, 0, Q0, Q2, Q1, m0, m2);
            if (k + 1 < K) step(k + 1, 2, 0, 1, Q1, Q0, Q2, m1, m0);
            if (k + 2 < K) step(k + 2, 0, 1, 2, Q2, Q1, Q0, m2, m1);
        }
    }
}

}  // namespace tlb
