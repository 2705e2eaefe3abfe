// Two D2Q9 steps in one launch: u_t -> u_{t+2} with u_{t+1} kept on the compute unit.
//
// What bounds the one-step kernel is the traffic of the state: it reads and writes every population
// once per step, and at 1024^2 it moves these bytes as fast as their access pattern allows.  Here a
// workgroup of two wavefronts owns a strip of columns and sweeps a chunk of rows.  The first wavefront
// advances the rows from u_t to u_{t+1}, the second from u_{t+1} to u_{t+2}, a few rows behind it; a row
// of u_{t+1} goes from the one to the other through LDS, where the second wavefront reads it with the
// column shifts of the pull.  Two steps then read the state once and write it once.
//
// Columns.  A wavefront's 64 lanes are neighbouring columns (periodic in x), and the values of the
// columns beside a lane come from its neighbours (cross-lane moves, no LDS).  The first step is right in
// lanes 1 .. 62 (its stencils need both neighbours), the second in lanes 3 .. 60 (pull and stencil), so a
// strip has up to 58 columns.
//
// Rows.  Virtual row v of an item is lattice row yfirst + v*DIR; rows 0 .. L-1 are its output.  In
// iteration k the first wavefront takes the pulled row v = k-3, forms its concentrations and collides row
// v-1; the second takes row w = k-5 of u_{t+1}, which completes the pull of row w-1, forms the
// concentrations of that row, and collides and stores row w-2.  An item so takes L + 7 iterations, one
// barrier each (the link holds two rows in turn: one is written while the other is read).  The pulled row
// v+1 is in flight during iteration k.  Neighbouring chunks sweep in opposite directions, so that they
// reach the rows they both read at the same time, and every other launch reverses all of them, as in the
// one-step sweep.
//
// Measured on MI355X, per step, against the one-step kernel: 1024^2 FP64 60.4 us (89.7), FP32 33.9 (42.4),
// 700 x 900 of four components with several relaxation times FP64 55.0 (76.9), 512^2 FP64 18.9 (23.1),
// 64^2 FP64 6.5 (6.7).  In FP64 an iteration of the 1024 items in flight moves 110 KB per compute unit
// through the L2 in 4.6 us, which bounds it; in FP32 (2.6 us) the instructions of two wavefronts per SIMD do.
// Columns and rows that are computed twice (7 of 64 lanes, 7 of 26 iterations) take the rest.
//
// Every value is formed by the operations of the one-step kernel in the same order, so the results are
// bitwise those of two single steps.
#include <algorithm>

#include "tlb_sweep2d.hpp"

namespace tlb {

namespace {

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

template <typename T, int NC>
struct PairLds {
    T link[2][9 * NC][64];       // rows of u_{t+1} on their way from the first wavefront to the second
    double row[2][3][NC][64];    // per wavefront: the concentration deviations of its last three rows
};

// Directions by their y component relative to the sweep: lead come from the row after (e_y = -DIR), level
// from the same row, trail from the row before.
template <int DIR>
struct Classes {
    static constexpr int lead[3] = {DIR > 0 ? 4 : 3, DIR > 0 ? 6 : 5, DIR > 0 ? 8 : 7};
    static constexpr int level[3] = {0, 1, 2};
    static constexpr int trail[3] = {DIR > 0 ? 3 : 4, DIR > 0 ? 5 : 6, DIR > 0 ? 7 : 8};
};

template <typename T, int DIR, bool MRT, int NC>
__device__ __forceinline__ void pair_sweep(const StepArgs<T>& A, int x0, int ncols, int y0, int L, PairLds<T, NC>& S)
{
    using C = double;
    constexpr int J = 9 * NC;
    const int lane = threadIdx.x & 63;
    const int nx = A.nx, ny = A.ny;
    const bool walls = A.walls != 0;
    const int yfirst = DIR > 0 ? y0 : y0 + L - 1;
    // virtual rows that exist (all of them without walls)
    const int vlo = walls ? (DIR > 0 ? -y0 : yfirst - (ny - 1)) : -(1 << 29);
    const int vhi = walls ? (DIR > 0 ? ny - 1 - y0 : yfirst) : (1 << 29);
    const int K = L + 7;
    auto row_of = [&](int v) {
        int y = (yfirst + v * DIR) % ny;
        return y < 0 ? y + ny : y;
    };
    // columns of the lane and of its neighbours, periodic
    int x = (x0 - 3 + lane) % nx;
    x = x < 0 ? x + nx : x;
    // wetting offsets beyond the wall that the sweep enters at and the one it ends at
    const T* wet_in = A.wet + (size_t)(DIR > 0 ? 0 : 1) * NC * nx + x;
    const T* wet_out = A.wet + (size_t)(DIR > 0 ? 1 : 0) * NC * nx + x;
    // rows of concentrations: the wavefront's own, in turn (the previous, this and the next one)
    double(*const rows)[NC][64] = S.row[threadIdx.x >> 6];
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

    if (threadIdx.x < 64) {
        // ---- first step ----
        const uint32_t vo[3] = {(uint32_t)x * (uint32_t)sizeof(T),
                                (uint32_t)(x == 0 ? nx - 1 : x - 1) * (uint32_t)sizeof(T),
                                (uint32_t)(x == nx - 1 ? 0 : x + 1) * (uint32_t)sizeof(T)};
        const StateAddr<T, false> src(A.src, A.N, NC);
        T P0[J], P1[J], P2[J];
#pragma unroll
        for (int i = 0; i < J; ++i) P0[i] = P1[i] = P2[i] = T(0);
        Moments<C, NC> Mb = {};
        auto exists = [&](int v) { return v >= vlo && v <= vhi; };
        if (exists(-3)) pull2d<T, NC, false>(A, src, vo, row_of(-3), P0);
        auto step = [&](int k, int a, int b, int c, T* Pc, T* Pb, T* Pn) {  // rows v, v-1 and v+1
            const int v = k - 3;
            if (v + 1 <= L + 2 && exists(v + 1)) pull2d<T, NC, false>(A, src, vo, row_of(v + 1), Pn);
            Moments<C, NC> Mc = {};
            if (v <= L + 2 && exists(v)) {
                concentrations(Pc, Mc, c);
                if (walls && v == vlo) ghost(c, wet_in, b);
            } else if (walls && v == vhi + 1) {
                ghost(b, wet_out, c);
            }
            const int e = v - 1;
            if (e >= -2 && e <= L + 1 && exists(e)) {
                C dc[NC], gC[NC][3], lC[NC];
                stencils(a, b, c, dc, gC, lC);
                collide<L9, MRT, NC>(A.P, Mb, dc, gC, lC, Pb, Pb + 9, Pb + 18);
                T(*out)[64] = S.link[k & 1];
#pragma unroll
                for (int j = 0; j < J; ++j) out[j][lane] = Pb[j];
            }
            Mb = Mc;
            link_barrier();
        };
        for (int k = 0; k < K; k += 3) {
            step(k, 1, 2, 0, P0, P2, P1);
            if (k + 1 < K) step(k + 1, 2, 0, 1, P1, P0, P2);
            if (k + 2 < K) step(k + 2, 0, 1, 2, P2, P1, P0);
        }
    } else {
        // ---- second step ----
        using CL = Classes<DIR>;
        const StateAddr<T, false> dst(A.dst, A.N, NC);
        const bool active = lane >= 3 && lane < 3 + ncols;
        const uint32_t vo = (uint32_t)x * (uint32_t)sizeof(T);
        // lanes that hold the columns x, x-1 and x+1 (the wavefront's end lanes are never used)
        const int from[3] = {lane, lane == 0 ? 0 : lane - 1, lane == 63 ? 63 : lane + 1};
        T Q0[J], Q1[J], Q2[J];
#pragma unroll
        for (int i = 0; i < J; ++i) Q0[i] = Q1[i] = Q2[i] = T(0);
        Moments<C, NC> Mb = {};
        auto step = [&](int k, int ra, int rb, int rc, T* Qc, T* Qb, T* Qn) {  // rows w-1 (completed now), w-2 (collided) and w
            const int w = k - 5;
            T(*in)[64] = S.link[(k - 1) & 1];
            const bool got = w >= -2 && w <= L + 1 && w >= vlo && w <= vhi;
            if (got) {
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int s = 0; s < NC; ++s) {
                        // pull: x - e_x; q = 0, 1, 2 are e_x = 0, +1, -1 in each class
                        Qc[9 * s + CL::lead[q]] = in[9 * s + CL::lead[q]][from[q]];
                        Qn[9 * s + CL::level[q]] = in[9 * s + CL::level[q]][from[q]];
                    }
                if (walls && w == vlo) {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int s = 0; s < NC; ++s)
                            Qn[9 * s + CL::trail[q]] = in[9 * s + L9::opp[CL::trail[q]]][lane];
                }
            } else if (walls && w == vhi + 1) {
                // the wall row's own values, turned back, were put into the row after it
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int s = 0; s < NC; ++s) Qc[9 * s + CL::lead[q]] = Qn[9 * s + CL::lead[q]];
            }
            const int c = w - 1;
            Moments<C, NC> Mc = {};
            if (c >= -1 && c <= L && c >= vlo && c <= vhi) {
                concentrations(Qc, Mc, rc);
                if (walls && c == vlo) ghost(rc, wet_in, rb);
            } else if (walls && c == vhi + 1) {
                ghost(rb, wet_out, rc);
            }
            const int e = w - 2;
            if (e >= 0 && e < L) {
                C dc[NC], gC[NC][3], lC[NC];
                stencils(ra, rb, rc, dc, gC, lC);
                collide<L9, MRT, NC>(A.P, Mb, dc, gC, lC, Qb, Qb + 9, Qb + 18);
                if (active) {
                    const uint32_t row = (uint32_t)row_of(e) * (uint32_t)nx;
#pragma unroll
                    for (int i = 0; i < 9; ++i)
#pragma unroll
                        for (int s = 0; s < NC; ++s) bstore<T>(Qb[9 * s + i], dst.rsrc(9 * s + i), vo, dst.soff(9 * s + i, row));
                }
            }
            if (got) {
                // the row after w takes its trailing populations now (into the registers just stored); beyond
                // the last row, w's own ones turned back, for the row itself
                const bool end = walls && w == vhi;
                if (!end) {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int s = 0; s < NC; ++s) Qb[9 * s + CL::trail[q]] = in[9 * s + CL::trail[q]][from[q]];
                } else {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int s = 0; s < NC; ++s) Qb[9 * s + CL::lead[q]] = in[9 * s + L9::opp[CL::lead[q]]][lane];
                }
            }
            Mb = Mc;
            link_barrier();
        };
        for (int k = 0; k < K; k += 3) {
            step(k, 1, 2, 0, Q0, Q2, Q1);
            if (k + 1 < K) step(k + 1, 2, 0, 1, Q1, Q0, Q2);
            if (k + 2 < K) step(k + 2, 0, 1, 2, Q2, Q1, Q0);
        }
    }
}

template <typename T, bool MRT, int NC>
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(NC > 3 ? 1 : 2))) void k_pair2d(StepArgs<T> A)
{
    __shared__ PairLds<T, NC> S;
    const int item = xcd_item(blockIdx.x, A.nitems);
    const int chunk = item / A.ntx;
    const int strip = item - chunk * A.ntx;
    const int x0 = strip * A.cols;
    const int ncols = min(A.cols, A.nx - x0);
    const int y0 = chunk * A.chunk;
    const int L = min(A.chunk, A.ny - y0);
    if (((chunk ^ A.flip) & 1) == 0)
        pair_sweep<T, 1, MRT, NC>(A, x0, ncols, y0, L, S);
    else
        pair_sweep<T, -1, MRT, NC>(A, x0, ncols, y0, L, S);
}

}  // namespace

// Strips and chunks.  An item takes chunk + 7 iterations of about the same length whatever its size, and
// the chip holds `slots` items at once (two wavefronts per SIMD, one in FP64 with four components), so the
// chunk is the one with the fewest iterations in all: rounds of items times iterations of an item.
// Measured at 1024^2 FP64: 19 rows (972 items in one round) 60.4 us per step, 20 rows 63.1, 26 rows 64.0;
// FP32 33.4, 34.5, 37.0; 700 x 900 of four components FP64: 24 rows 55.0, 26 rows 57.1, 12 rows 62.5.
template <typename T>
void pair2d_shape(StepArgs<T>& a, int nc, int cus)
{
    constexpr int kCols = 58, kFill = 7;
    a.ntx = (a.nx + kCols - 1) / kCols;
    a.cols = (a.nx + a.ntx - 1) / a.ntx;
    a.nty = 1;
    const int64_t slots = (int64_t)(cus > 0 ? cus : 256) * (sizeof(T) == 8 && nc > 3 ? 2 : 4);
    // with n rounds at most n * slots items: the longest round count worth a look halves the chunk each time
    int64_t best = INT64_MAX;
    for (int64_t rounds = 1; rounds <= 64; ++rounds) {
        const int64_t nch = std::min<int64_t>(a.ny, std::max<int64_t>(1, rounds * slots / a.ntx));
        const int chunk = (int)((a.ny + nch - 1) / nch);
        const int nchunks = (a.ny + chunk - 1) / chunk;
        const int64_t cost = (((int64_t)a.ntx * nchunks + slots - 1) / slots) * (chunk + kFill);
        if (cost < best) {
            best = cost;
            a.chunk = chunk;
            a.nchunks = nchunks;
        }
    }
    a.nitems = a.ntx * a.nchunks;
}

template <typename T>
hipError_t launch_pair2d(const StepArgs<T>& a, bool mrt, int nc, hipStream_t s)
{
    const dim3 grid(a.nitems), block(128);
#define TLB_P2(M, NC)                                                            \
    if (mrt == M && nc == NC) {                                                  \
        hipLaunchKernelGGL((k_pair2d<T, M, NC>), grid, block, 0, s, a);          \
        return hipGetLastError();                                                \
    }
    TLB_P2(false, 3)
    TLB_P2(true, 3)
    TLB_P2(false, 4)
    TLB_P2(true, 4)
#undef TLB_P2
    return hipErrorInvalidValue;
}

template void pair2d_shape<float>(StepArgs<float>&, int, int);
template void pair2d_shape<double>(StepArgs<double>&, int, int);
template hipError_t launch_pair2d<float>(const StepArgs<float>&, bool, int, hipStream_t);
template hipError_t launch_pair2d<double>(const StepArgs<double>&, bool, int, hipStream_t);

}  // namespace tlb
