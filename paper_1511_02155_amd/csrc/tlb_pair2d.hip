// Launches of two or four steps of one D2Q9 lattice: the kernel around the sweep of tlb_pair2d.hpp (which the
// batch shares), and its strips and chunks.
#include <algorithm>

#include "tlb_pair2d.hpp"

namespace tlb {

namespace {

// Two steps of three components are held to two wavefronts per SIMD (256 registers), which leaves values in scratch
// memory: FP64 16 (52 bytes per lane), with several relaxation times 65 (108), and FP32 with several 27 (56).
template <typename T, bool MRT, int NC, int S>
__global__ __launch_bounds__(64 * S) __attribute__((amdgpu_waves_per_eu(NC > 3 || S > 2 ? 1 : 2))) void k_pair2d(StepArgs<T> A)
{
    __shared__ PairLds<T, NC, S> M;
    const int item = xcd_item(blockIdx.x, A.nitems);
    const int chunk = item / A.ntx;
    const int strip = item - chunk * A.ntx;
    const int x0 = strip * A.cols;
    const int ncols = min(A.cols, A.nx - x0);
    const int y0 = chunk * A.chunk;
    const int L = min(A.chunk, A.ny - y0);
    if (((chunk ^ A.flip) & 1) == 0)
        pair_sweep<T, 1, MRT, NC, S>(A, x0, ncols, y0, L, M);
    else
        pair_sweep<T, -1, MRT, NC, S>(A, x0, ncols, y0, L, M);
}

}  // namespace

// Strips and chunks.  An item takes chunk + 5 S - 3 iterations for S steps, and an iteration takes the longer
// the more items share a compute unit; of two-step items it holds four (two wavefronts per SIMD), of those
// with four or five components two (one), of four-step items one.  Measured, in us per iteration with 1, 2, 3
// and 4 two-step items on a compute unit (lattices of 58 to 1024 columns, 45 to 512 rows, chunks of 1 to 24
// rows): FP32 1.55, 1.9, 2.1, 2.2; FP64 1.6, 1.9, 2.35, 2.6; four components 2.1, 2.4; five 2.7, 3.2; a
// four-step item 1.7, with four components 2.35.  Where that is longer, the time is that of the bytes: the
// state written once and read with the rows and columns around the items, at 6.5 TB/s where both buffers fit
// the Infinity Cache and 5.0 TB/s beyond.  The chunk is the one with the least time by these figures: 512^2
// FP64 5 rows (927 items) 15.4 us per step against 15.8 at 8 rows and 20.1 at 4 (1152 items, a second
// round); 333 x 217 FP32 2 rows 9.0 against 14.7 at one.
// Returns the time per step in us.
template <typename T>
double pair2d_shape(StepArgs<T>& a, int nc, int cus, int steps)
{
    const int most_cols = pair_cols(steps), fill = pair_fill(steps);
    const double f32[4] = {1.55, 1.9, 2.1, 2.2}, f64[4] = {1.6, 1.9, 2.35, 2.6}, four[2] = {2.1, 2.4}, five[2] = {2.7, 3.2};
    const double f64_4[1] = {1.7}, four_4[1] = {2.35};
    const double* per = steps == 4 ? (nc > 3 ? four_4 : f64_4) : nc > 4 ? five : nc > 3 ? four : (sizeof(T) == 4 ? f32 : f64);
    const int most = steps == 4 ? 1 : nc > 3 ? 2 : 4;
    if (cus < 1) cus = 256;
    a.ntx = (a.nx + most_cols - 1) / most_cols;
    a.cols = (a.nx + a.ntx - 1) / a.ntx;
    a.nty = 1;
    const double state = 9.0 * nc * (double)a.N * sizeof(T);
    const double per_us = 2.0 * state <= (double)kStreamStoreBytes ? 6.5e6 : 5.0e6;  // bytes
    double best = 1e300;
    for (int q = 1; q <= 64; ++q) {  // about q items per compute unit in all
        const int64_t want = std::min<int64_t>(a.ny, std::max<int64_t>(1, (int64_t)q * cus / a.ntx));
        const int chunk = (int)((a.ny + want - 1) / want);
        const int nchunks = (a.ny + chunk - 1) / chunk;
        const int64_t share = ((int64_t)a.ntx * nchunks + cus - 1) / cus;
        const int rest = (int)(share % most);
        const double iterations = ((double)(share / most) * per[most - 1] + (rest ? per[rest - 1] : 0.0)) * (chunk + fill);
        const double bytes = state * (1.0 + 64.0 * a.ntx / a.nx * (chunk + 2.0 * steps + 2.0) / chunk) / per_us;
        const double cost = std::max(iterations, bytes);
        if (cost < best) {
            best = cost;
            a.chunk = chunk;
            a.nchunks = nchunks;
        }
    }
    a.nitems = a.ntx * a.nchunks;
    return (best + 0.8) / steps;
}

template <typename T>
hipError_t launch_pair2d(const StepArgs<T>& a, int steps, bool mrt, int nc, hipStream_t s)
{
    const dim3 grid(a.nitems), block(64 * steps);
#define TLB_P2(M, NC)                                                            \
    if (mrt == M && nc == NC && steps == 2) {                                    \
        hipLaunchKernelGGL((k_pair2d<T, M, NC, 2>), grid, block, 0, s, a);       \
        return hipGetLastError();                                                \
    }
    TLB_P2(false, 3)
    TLB_P2(true, 3)
    TLB_P2(false, 4)
    TLB_P2(true, 4)
    TLB_P2(false, 5)
    TLB_P2(true, 5)
#undef TLB_P2
    if constexpr (sizeof(T) == 8) {
#define TLB_P4(M, NC)                                                            \
    if (mrt == M && nc == NC && steps == 4) {                                    \
        hipLaunchKernelGGL((k_pair2d<T, M, NC, 4>), grid, block, 0, s, a);       \
        return hipGetLastError();                                                \
    }
        TLB_P4(false, 3)
        TLB_P4(true, 3)
        TLB_P4(false, 4)
        TLB_P4(true, 4)
#undef TLB_P4
    }
    return hipErrorInvalidValue;
}

template double pair2d_shape<float>(StepArgs<float>&, int, int, int);
template double pair2d_shape<double>(StepArgs<double>&, int, int, int);
template hipError_t launch_pair2d<float>(const StepArgs<float>&, int, bool, int, hipStream_t);
template hipError_t launch_pair2d<double>(const StepArgs<double>&, int, bool, int, hipStream_t);

}  // namespace tlb
