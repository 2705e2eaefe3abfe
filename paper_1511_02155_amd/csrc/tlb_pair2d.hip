// Two-step launches of one D2Q9 lattice: the kernel around the sweep of tlb_pair2d.hpp (which the batch shares),
// and its strips and chunks.
#include <algorithm>

#include "tlb_pair2d.hpp"

namespace tlb {

namespace {

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

// Strips and chunks.  An item takes chunk + 7 iterations, and an iteration takes the longer the more items
// share a compute unit; the chip holds four per compute unit (two wavefronts per SIMD), two of four or
// five components (one).  Measured, in us per iteration with 1, 2, 3 and 4 items on a compute unit (lattices of
// 58 to 1024 columns, 45 to 512 rows, chunks of 1 to 24 rows): FP32 1.55, 1.9, 2.1, 2.2; FP64 1.6, 1.9,
// 2.35, 2.6; four components 2.1, 2.4; five 2.7, 3.2.  The chunk is the one with the least time by these figures: 512^2
// FP64 5 rows (927 items) 15.4 us per step against 15.8 at 8 rows and 20.1 at 4 (1152 items, a second
// round); 333 x 217 FP32 2 rows 9.0 against 14.7 at one.
template <typename T>
double pair2d_shape(StepArgs<T>& a, int nc, int cus)
{
    constexpr int kCols = 58, kFill = 7;
    const double f32[4] = {1.55, 1.9, 2.1, 2.2}, f64[4] = {1.6, 1.9, 2.35, 2.6}, four[2] = {2.1, 2.4}, five[2] = {2.7, 3.2};
    const double* per = nc > 4 ? five : nc > 3 ? four : (sizeof(T) == 4 ? f32 : f64);
    const int most = nc > 3 ? 2 : 4;
    if (cus < 1) cus = 256;
    a.ntx = (a.nx + kCols - 1) / kCols;
    a.cols = (a.nx + a.ntx - 1) / a.ntx;
    a.nty = 1;
    double best = 1e300;
    for (int q = 1; q <= 64; ++q) {  // about q items per compute unit in all
        const int64_t want = std::min<int64_t>(a.ny, std::max<int64_t>(1, (int64_t)q * cus / a.ntx));
        const int chunk = (int)((a.ny + want - 1) / want);
        const int nchunks = (a.ny + chunk - 1) / chunk;
        const int64_t share = ((int64_t)a.ntx * nchunks + cus - 1) / cus;
        const int rest = (int)(share % most);
        const double cost = ((double)(share / most) * per[most - 1] + (rest ? per[rest - 1] : 0.0)) * (chunk + kFill);
        if (cost < best) {
            best = cost;
            a.chunk = chunk;
            a.nchunks = nchunks;
        }
    }
    a.nitems = a.ntx * a.nchunks;
    return 0.5 * best + 0.4;
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
    TLB_P2(false, 5)
    TLB_P2(true, 5)
#undef TLB_P2
    return hipErrorInvalidValue;
}

template double pair2d_shape<float>(StepArgs<float>&, int, int);
template double pair2d_shape<double>(StepArgs<double>&, int, int);
template hipError_t launch_pair2d<float>(const StepArgs<float>&, bool, int, hipStream_t);
template hipError_t launch_pair2d<double>(const StepArgs<double>&, bool, int, hipStream_t);

}  // namespace tlb
