// warm.hip -- the stored column state of a warm start.
//
// Algorithm 1 starts each regression from beta = 0, sigma = 1; a caller may
// instead start it from earlier coefficients and noise levels (a previous
// solve at another penalty, or one stopped by an iteration cap).  The
// minimiser of Eq. (eq:spmesl) is unique, so the start changes the work,
// not the result.  This kernel turns a dense B0 (p x p, row-major, column k
// the coefficients of response k) into the per-column working sets the
// column solves resume from.
//
// A block owns 16 consecutive columns, whose rows are split over 64 segments:
// 16 waves of four, a lane per column and segment, so a load takes 128
// consecutive bytes of four rows.  Two passes over the block's column strip:
// the first counts each segment's nonzeros per column, the second (out of the
// caches) writes them at the offsets of a scan over the segments, so each
// column's list is in ascending row order (the order the solver keeps its
// working sets in).  What bounds it is the latency of B0's reads: with 64
// columns per block, p = 2000 had 32 blocks and one load per wave in flight
// (155 us); with 125 blocks and 16 rows of a lane in flight 18 us.
#include "common.hpp"

namespace spmesl {

constexpr int kWarmWaves = 16;
constexpr int kWarmCols = 16;                                   // columns per block
constexpr int kWarmSegs = kWarmWaves * (kWave / kWarmCols);     // row segments of a column
constexpr int kWarmRows = 16;                                   // rows of a lane in flight

template <typename T>
__global__ __launch_bounds__(kWave *kWarmWaves) void k_warm_start(
    const double *__restrict__ B0, const double *__restrict__ sigma0, int64_t p,
    const double *__restrict__ scale, int original, double lambda0, int *__restrict__ w_cnt,
    int *__restrict__ w_idx, T *__restrict__ w_beta, double *__restrict__ sigma,
    double *__restrict__ lam_used, int *__restrict__ col_status)
{
    __shared__ int cnt[kWarmSegs][kWarmCols];
    const int c = threadIdx.x & (kWarmCols - 1), seg = threadIdx.x / kWarmCols;
    const int64_t k = (int64_t)blockIdx.x * kWarmCols + c;
    const bool col = k < p;
    const int64_t kc = col ? k : p - 1;
    const int64_t rows = (p + kWarmSegs - 1) / kWarmSegs;
    const int64_t j0 = (int64_t)seg * rows;
    const int64_t j1 = j0 + rows < p ? j0 + rows : p;
    const double ck = scale[kc];
    // the value stored for (j, k), or 0 when (j, k) is not kept
    auto value = [&](int64_t j, double b) -> T {
        if (j == k || b == 0.0) return T(0);
        const double v = original ? b * ck / scale[j] : b;
        return (T)v;
    };
    // f(j, value) for the kept entries of the segment, in order
    auto each = [&](auto f) {
        for (int64_t j = j0; j < j1; j += kWarmRows) {
            double b[kWarmRows];
#pragma unroll
            for (int u = 0; u < kWarmRows; ++u) b[u] = B0[(j + u < p ? j + u : p - 1) * p + kc];
            unsigned nz = 0u;
#pragma unroll
            for (int u = 0; u < kWarmRows; ++u) nz |= b[u] != 0.0 && j + u < j1 ? 1u << u : 0u;
            for (; nz; nz &= nz - 1) {  // (few: read again rather than indexed)
                const int64_t ju = j + __builtin_ctz(nz);
                const T v = value(ju, B0[ju * p + kc]);
                if (v != T(0)) f(ju, v);
            }
        }
    };
    int own = 0;
    if (B0) each([&](int64_t, T) { ++own; });
    cnt[seg][c] = own;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll 8
    for (int g = 0; g < kWarmSegs; ++g) {
        const int x = cnt[g][c];
        off += g < seg ? x : 0;
        tot += x;
    }
    if (col && own > 0 && off < kWMax)
        each([&](int64_t j, T v) {
            if (off < kWMax) {
                w_idx[k * kWMax + off] = (int)j;
                w_beta[k * kWMax + off] = v;
            }
            ++off;
        });
    if (seg == 0 && col) {
        double sg = 1.0;
        if (sigma0) {
            const double v = original ? sigma0[k] * ck : sigma0[k];
            if (v > 0.0 && v < 1e300) sg = v;
        }
        w_cnt[k] = tot < kWMax ? tot : kWMax;
        sigma[k] = sg;
        lam_used[k] = sg * lambda0;
        col_status[k] = kColWarm;
    }
}

template <typename T>
void launch_warm_start(const double *B0, const double *sigma0, int64_t p, const double *scale, int original,
                       double lambda0, int *w_cnt, int *w_idx, T *w_beta, double *sigma, double *lam_used,
                       int *col_status, hipStream_t s)
{
    const unsigned blocks = (unsigned)((p + kWarmCols - 1) / kWarmCols);
    hipLaunchKernelGGL(k_warm_start<T>, dim3(blocks), dim3(kWave * kWarmWaves), 0, s, B0, sigma0, p, scale,
                       original, lambda0, w_cnt, w_idx, w_beta, sigma, lam_used, col_status);
}

template void launch_warm_start<double>(const double *, const double *, int64_t, const double *, int, double,
                                        int *, int *, double *, double *, double *, int *, hipStream_t);
template void launch_warm_start<float>(const double *, const double *, int64_t, const double *, int, double,
                                       int *, int *, float *, double *, double *, int *, hipStream_t);

} // namespace spmesl
