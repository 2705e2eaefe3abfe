// Several D2Q9 steps in one launch for small lattices: a workgroup owns a TX x TY tile and advances it
// STEPS steps in LDS.
//
// A step of a lattice that does not fill the chip is bound by the latency of its stages and of its launch,
// not by bytes: 64^2 takes 7 us per one-step launch and 12 us per two-step launch of the sweep
// (tlb_pair2d.hip), whose rows pass through eight iterations.  Here every lane has one node, the stages
// follow one another once per step, and the launch is shared by STEPS steps (64^2 FP64: 2.8 us per step).
// The price is the nodes around the tile that are computed again, a ring of two nodes per step: with three
// steps an 8 x 4 tile pulls 18 x 14 nodes from memory and collides 16 x 12, 12 x 8 and 8 x 4 of them.
//
// Per step: pull (the first from memory, the others from the tile's populations in LDS), moments and
// concentrations to LDS, barrier, stencils and collision, populations to LDS (the last to memory), barrier.
// The populations are stored in LDS in the storage type, so that each step rounds as if it went through
// memory, and every value is formed by the operations of the one-step kernel: results are bitwise those of
// single steps.
#include <math.h>

#include "tlb_sweep2d.hpp"

namespace tlb {

namespace {

template <typename T, int TX, int TY, int STEPS, int NC>
struct TileLds {
    static constexpr int H = 2 * STEPS - 1;             // ring of nodes around the tile
    static constexpr int W = TX + 2 * H, R = TY + 2 * H;  // nodes whose concentrations the first step needs
    double conc[NC][R][W];
    T pop[9 * NC][R - 2][W - 2];
};

template <typename T, int TX, int TY, int STEPS, int NC>
constexpr int tile_threads()
{
    using S = TileLds<T, TX, TY, STEPS, NC>;
    return (S::W * S::R + 63) / 64 * 64;
}

template <typename T, int TX, int TY, int STEPS, bool MRT, int NC>
__global__ __launch_bounds__((tile_threads<T, TX, TY, STEPS, NC>())) void k_tile2d(StepArgs<T> A)
{
    using C = double;
    using Lds = TileLds<T, TX, TY, STEPS, NC>;
    constexpr int J = 9 * NC, H = Lds::H;
    __shared__ Lds S;
    const int item = xcd_item(blockIdx.x, A.nitems);
    const int tyi = item / A.ntx, txi = item - tyi * A.ntx;
    const int x0 = txi * TX - H, y0 = tyi * TY - H;  // lattice node of the region's corner
    const int nx = A.nx, ny = A.ny;
    const bool walls = A.walls != 0;
    const bool wall_tile = walls && (y0 <= 0 || y0 + Lds::R >= ny);
    const int t = threadIdx.x;
    const uint32_t rowb = (uint32_t)nx * (uint32_t)sizeof(T), arrb = (uint32_t)A.N * (uint32_t)sizeof(T);
    const Rsrc src = make_rsrc(A.src, arrb * (uint32_t)J), dst = make_rsrc(A.dst, arrb * (uint32_t)J);
    auto wrap = [](int a, int n) {
        a %= n;
        return a < 0 ? a + n : a;
    };

    T p[J];
    Moments<C, NC> mo;
    int lx = 0, ly = 0, gx = 0, gy = 0;
    bool in = false;
    // the lane's node among those that step s pulls
    auto place = [&](int s) {
        const int w = Lds::W - 4 * s, h = Lds::R - 4 * s;
        in = t < w * h;
        const int k = in ? t : w * h - 1;
        ly = k / w;
        lx = k - ly * w + 2 * s;
        ly += 2 * s;
        gx = wrap(x0 + lx, nx);
        gy = y0 + ly;
        if (!walls) gy = wrap(gy, ny);  // with walls, rows beyond them are computed and never used
    };
    auto concentrations = [&]() {
        mo = moments<L9, NC>(p, p + 9, p + 18);
        C c[NC];
        conc_dev<C, NC>(mo, c);
        if (in) {
#pragma unroll
            for (int m = 0; m < NC; ++m) S.conc[m][ly][lx] = c[m];
        }
    };
    auto collision = [&]() {
        C dc[NC], gC[NC][3], lC[NC];
#pragma unroll
        for (int m = 0; m < NC; ++m) {
            C al = S.conc[m][ly - 1][lx - 1], ac = S.conc[m][ly - 1][lx], ar = S.conc[m][ly - 1][lx + 1];
            const C bl = S.conc[m][ly][lx - 1], bc = S.conc[m][ly][lx], br = S.conc[m][ly][lx + 1];
            C cl = S.conc[m][ly + 1][lx - 1], cc = S.conc[m][ly + 1][lx], cr = S.conc[m][ly + 1][lx + 1];
            if (wall_tile) {  // rows beyond a wall: the wall row's values and the wetting offsets
                const int xl = gx == 0 ? nx - 1 : gx - 1, xr = gx == nx - 1 ? 0 : gx + 1;
                if (gy == 0) {
                    const T* __restrict__ wt = A.wet + (size_t)m * nx;
                    al = bl + C(wt[xl]);
                    ac = bc + C(wt[gx]);
                    ar = br + C(wt[xr]);
                }
                if (gy == ny - 1) {
                    const T* __restrict__ wt = A.wet + (size_t)(NC + m) * nx;
                    cl = bl + C(wt[xl]);
                    cc = bc + C(wt[gx]);
                    cr = br + C(wt[xr]);
                }
            }
            dc[m] = bc;
            stencil9<C>(ac, al + ar, ar - al, bc, bl + br, br - bl, cc, cl + cr, cr - cl, 1, gC[m], lC[m]);
        }
        collide<L9, MRT, NC>(A.P, mo, dc, gC, lC, p, p + 9, p + 18);
    };

    // first step: pull from memory
    place(0);
    {
        const int y = walls ? min(max(gy, 0), ny - 1) : gy;
        const uint32_t row[3] = {(uint32_t)y * rowb, (uint32_t)(y == 0 ? ny - 1 : y - 1) * rowb,
                                 (uint32_t)(y == ny - 1 ? 0 : y + 1) * rowb};
        const uint32_t col[3] = {(uint32_t)gx * (uint32_t)sizeof(T), (uint32_t)(gx == 0 ? nx - 1 : gx - 1) * (uint32_t)sizeof(T),
                                 (uint32_t)(gx == nx - 1 ? 0 : gx + 1) * (uint32_t)sizeof(T)};
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int r = L9::ey[i] == 0 ? 0 : (L9::ey[i] == 1 ? 1 : 2), q = L9::ex[i] == 0 ? 0 : (L9::ex[i] == 1 ? 1 : 2);
#pragma unroll
            for (int s = 0; s < NC; ++s) p[9 * s + i] = bload<T>(src, row[r] + col[q], (uint32_t)(9 * s + i) * arrb);
        }
        if (wall_tile) {
#pragma unroll
            for (int i = 0; i < 9; ++i)
                if (L9::ey[i] != 0 && (L9::ey[i] == 1 ? y == 0 : y == ny - 1))
#pragma unroll
                    for (int s = 0; s < NC; ++s)
                        p[9 * s + i] = bload<T>(src, row[0] + col[0], (uint32_t)(9 * s + L9::opp[i]) * arrb);
        }
    }
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        if (s > 0) {
            place(s);
#pragma unroll
            for (int i = 0; i < 9; ++i)
#pragma unroll
                for (int q = 0; q < NC; ++q) p[9 * q + i] = S.pop[9 * q + i][ly - L9::ey[i] - 1][lx - L9::ex[i] - 1];
            if (wall_tile) {
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    if (L9::ey[i] != 0 && (L9::ey[i] == 1 ? gy == 0 : gy == ny - 1))
#pragma unroll
                        for (int q = 0; q < NC; ++q) p[9 * q + i] = S.pop[9 * q + L9::opp[i]][ly - 1][lx - 1];
            }
        }
        concentrations();
        __syncthreads();
        // the nodes one further in are collided
        const int e = 2 * s + 1;
        if (in && lx >= e && lx < Lds::W - e && ly >= e && ly < Lds::R - e) {
            collision();
            if (s < STEPS - 1) {
#pragma unroll
                for (int j = 0; j < J; ++j) S.pop[j][ly - 1][lx - 1] = p[j];
            } else if (x0 + lx < nx && y0 + ly < ny) {
                const uint32_t off = (uint32_t)gy * rowb + (uint32_t)gx * (uint32_t)sizeof(T);
#pragma unroll
                for (int j = 0; j < J; ++j) bstore<T>(p[j], dst, off, (uint32_t)j * arrb);
            }
        }
        if (s < STEPS - 1) __syncthreads();
    }
}

// The tiles and their times, in us per launch: with up to one tile per compute unit, and for each further
// tile a compute unit works through.  FP32 and FP64 of three components, measured on lattices of 32^2 to
// 512^2 (64^2 FP64: 2.82 us per step in 8 x 4 tiles of three steps, 3.1 in 8 x 8 of four, 3.9 in 16 x 8 of
// two; 160^2: 4.0 in 16 x 8 of three, 4.8 in 12 x 8 of two; 240^2: 5.4 in 32 x 8, 5.7 in 12 x 8; 333 x 217
// FP32: 6.3 in 12 x 8, 8.0 in 32 x 8, 9.2 in sweeps).  Four and five components take 1.2 and 1.4 times the
// first figure and, with fewer tiles on a compute unit at once, 1.7 and 3.2 times the second.
struct TileShape {
    int tx, ty, steps, most_nc;
    double first[2], more[2];
};
constexpr TileShape kTiles[] = {
    {8, 4, 3, 5, {8.0, 8.6}, {3.5, 4.0}},
    {16, 8, 3, 3, {10.4, 12.1}, {7.7, 8.0}},
    {12, 8, 2, 5, {6.45, 7.15}, {2.05, 2.35}},
    {32, 8, 2, 3, {9.25, 10.75}, {6.75, 9.5}},
};
constexpr int kTileShapes = sizeof(kTiles) / sizeof(kTiles[0]);

}  // namespace

int tile2d_steps(int shape) { return kTiles[shape].steps; }

// The fastest tiles for the lattice (of `steps` steps where steps != 0) and their time per step.
int tile2d_best(int nx, int ny, int nc, bool f64, int cus, int steps, double* us)
{
    int found = -1;
    if (cus < 1) cus = 256;
    for (int k = 0; k < kTileShapes; ++k) {
        const TileShape& q = kTiles[k];
        if (nc > q.most_nc || (steps != 0 && q.steps != steps)) continue;
        const double items = (double)((nx + q.tx - 1) / q.tx) * ((ny + q.ty - 1) / q.ty);
        const double share = ceil(items / cus);
        const double f = nc == 3 ? 1.0 : nc == 4 ? 1.2 : 1.4, m = nc == 3 ? 1.0 : nc == 4 ? 1.7 : 3.2;
        const double t = (q.first[f64] * f + q.more[f64] * m * (share - 1.0)) / q.steps;
        if (found < 0 || t < *us) {
            found = k;
            *us = t;
        }
    }
    return found;
}

template <typename T>
hipError_t launch_tile2d(const StepArgs<T>& a, int shape, bool mrt, int nc, hipStream_t s)
{
    StepArgs<T> b = a;
    b.ntx = (a.nx + kTiles[shape].tx - 1) / kTiles[shape].tx;
    b.nty = (a.ny + kTiles[shape].ty - 1) / kTiles[shape].ty;
    b.nitems = b.ntx * b.nty;
#define TLB_T2(K, M, NC)                                                                                       \
    if (shape == K && mrt == M && nc == NC) {                                                                  \
        constexpr TileShape Q = kTiles[K];                                                                     \
        hipLaunchKernelGGL((k_tile2d<T, Q.tx, Q.ty, Q.steps, M, NC>), dim3(b.nitems),                          \
                           dim3(tile_threads<T, Q.tx, Q.ty, Q.steps, NC>()), 0, s, b);                         \
        return hipGetLastError();                                                                              \
    }
#define TLB_T2N(K, NC) TLB_T2(K, false, NC) TLB_T2(K, true, NC)
    TLB_T2N(0, 3) TLB_T2N(0, 4) TLB_T2N(0, 5)
    TLB_T2N(1, 3)
    TLB_T2N(2, 3) TLB_T2N(2, 4) TLB_T2N(2, 5)
    TLB_T2N(3, 3)
#undef TLB_T2N
#undef TLB_T2
    return hipErrorInvalidValue;
}

template hipError_t launch_tile2d<float>(const StepArgs<float>&, int, bool, int, hipStream_t);
template hipError_t launch_tile2d<double>(const StepArgs<double>&, int, bool, int, hipStream_t);

}  // namespace tlb
