// dense.hip -- the regressions whose working sets outgrow the LDS tiers.
//
// A column whose working set would exceed the 128 coordinates an LDS tier
// holds is finished here.  Algorithm 1 puts no bound on the support, so
// neither does this tier: it runs the paper's row-wise PCD (Proposition 2,
// Algorithm 3) in covariance form on a group of up to 16 such columns at
// once, restricted to the union V of their working sets:
//
//   R = S[V, K] - S[V, V] B[V, K]          (gradients of the group's columns K)
//   for each block J of b consecutive rows of V (ascending):
//       every column sweeps J in order on its own: a = R_j + B_j,
//       B_j <- Soft_lambda(a), R_J -= S[J, j] delta_j  (in-wave, S[J, J] in LDS)
//       R -= S[V, J] dB[J, K]                 (the delayed rank-b update,
//                                              on the matrix cores)
//
// Within a column this is the cyclic order of Algorithm 1 exactly (the rows
// of V are visited in ascending order and every coordinate sees every
// earlier change), so the iterates are the same as coordinate descent on V;
// only the gradients of rows outside the current block are brought up to
// date once per block.  Each column keeps its own inner stop (largest
// change of a sweep < tol), noise update sigma^2 = 1 - B'(s + R) (Eq.
// (eq:sigma) from S) and outer stop; columns that are done stay in the group
// with zero changes.  When every column is done, one pass over all p rows
// computes the full gradient g = s_k - S[:, V] B[V, k] (again on the matrix
// cores) and every j outside V with |g_j| > lambda + tol joins V; the group
// repeats until no column has a violator.
//
// Two sources of S:
//   * the covariance S itself (double or float forms, and the float stage of
//     the mixed form): entries are gathered from S;
//   * the standardised data Xt (p x n, double) for the double polish of the
//     mixed form: S[V, V] and s are formed once per V on the matrix cores, and
//     the full gradient is taken in the data form of Algorithm 3,
//     E = x_K - X_V B[V, K] and g = X^T E / n (so no double S is needed).
//
// A workgroup of 16 waves (one column of the group each) takes one group at a
// time.  What bounds it is latency: the chain of dependent
// coordinate updates of a column, and the memory round trips between them.
// So the gradients and coefficients of V live in LDS while the columns iterate
// (up to kVLds rows), the operands of the delayed update and the next block's
// S[J, J] are loaded before the sweep they follow, every product has 8 or more
// loads in flight per wave with no branch between them, and a V of one block
// (up to 64 rows) is solved column by column with no barrier at all.
// One column per wave and 16 waves rather than two and 8: a barrier waits for
// the slowest wave, and the sweeps of a wave's columns follow one another.
// Measured, against 8 waves with gradients and coefficients in global memory
// and each operand waited for:
//   n = 1500, p = 300, double (19 groups, V about 300): a group's sweeps and
//     updates 10.9 -> 6.1 ms, the solve 15.9 -> 11.6 ms, 8.5 with the LDS
//     tiers' shorter steps, and 6.5 with blocks of 64 rows (of 32: 7.3, of 16:
//     10.2; half the barriers, each waiting for its slowest column);
//   n = 400, p = 2500, data form (157 groups, V about 40): 6.0 -> 1.1 to 1.3 ms
//     a solve, by the box: a group's iterations 450 -> 40 us, a full gradient
//     870 -> 290 us (its 2 GB of Xt reads a pass come from the caches at 4.4
//     TB/s).
#include <type_traits>

#include "colsolve_dev.hpp"

namespace spmesl {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
template <typename T> struct DAcc;
template <> struct DAcc<double> { typedef d4 type; };
template <> struct DAcc<float> { typedef f4 type; };

__device__ __forceinline__ d4 dmfma(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 dmfma(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Row of accumulator element r of `lane` in a 16 x 16 block: D[4r + l/16]
// for the double MFMA, D[4(l/16) + r] for the float one (lane l holds
// column l % 16; it supplies row l % 16 of A and column l % 16 of B at
// k-block l / 16).
template <typename T> __device__ __forceinline__ int drow(int lane, int r);
template <> __device__ __forceinline__ int drow<double>(int lane, int r) { return 4 * r + (lane >> 4); }
template <> __device__ __forceinline__ int drow<float>(int lane, int r) { return 4 * (lane >> 4) + r; }

// acc[t] += A_t (16 x K) B (K x 16) for NA row tiles that share B: fa(t, k)
// gives A_t at this lane's row (l % 16), fb(k) B at its column (l % 16), for
// 0 <= k < K.  U steps of 4 k per round, every load of a round in flight
// before its products.
template <typename T, int NA, int U, typename FA, typename FB>
__device__ __forceinline__ void tiles_mma(typename DAcc<T>::type (&acc)[NA], int64_t K, FA fa, FB fb)
{
    const int kq = lane_id() >> 4;
    int64_t k0 = 0;
    for (; k0 + 4 * U <= K; k0 += 4 * U) {
        T a[U][NA], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = k0 + 4 * u + kq;
#pragma unroll
            for (int t = 0; t < NA; ++t) a[u][t] = fa(t, k);
            b[u] = fb(k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < NA; ++t) acc[t] = dmfma(a[u][t], b[u], acc[t]);
    }
    if (k0 < K) {
        // past K the last k again, against a zero of B (loads without
        // branches between them stay in flight together)
        T a[U][NA], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = k0 + 4 * u + kq, kc = k < K ? k : K - 1;
#pragma unroll
            for (int t = 0; t < NA; ++t) a[u][t] = fa(t, kc);
            b[u] = fb(kc);
            b[u] = k < K ? b[u] : T(0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + 4 * u < K) {
#pragma unroll
                for (int t = 0; t < NA; ++t) acc[t] = dmfma(a[u][t], b[u], acc[t]);
            }
    }
}

// Two consecutive values of a row of the data, loaded together: 4 lanes then
// take 64 consecutive bytes of a row (rows are only 8-byte aligned when n is
// odd).  A lane at k-block q holds samples 8 u + 2 q and 8 u + 2 q + 1, so one
// product takes the even and one the odd samples of every 8.
typedef double dpair __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ dpair load_pair(const double *row, int64_t k)
{
    return *reinterpret_cast<const dpair *>(row + k);
}
// ... near the end of the row: the last value in the place of those past it
// (the caller zeroes the other operand there)
__device__ __forceinline__ dpair load_pair_end(const double *row, int64_t k, int64_t n)
{
    const double x = row[k < n ? k : n - 1], y = row[k + 1 < n ? k + 1 : n - 1];
    return dpair{x, y};
}
__device__ __forceinline__ dpair zero_past(dpair v, int64_t k, int64_t n)
{
    return dpair{k < n ? v.x : 0.0, k + 1 < n ? v.y : 0.0};
}

// acc[h][g] += sum over the n samples of rows a[h] times rows b[g] of the data
// (lane l: rows l % 16), 16 samples per round.
template <int NA, int NB>
__device__ __forceinline__ void rows_mma(d4 (&acc)[NA][NB], const double *const (&ra)[NA],
                                         const double *const (&rb)[NB], int64_t n)
{
    const int kq = lane_id() >> 4;
    for (int64_t k0 = 0; k0 < n; k0 += 16) {
        dpair a[2][NA], b[2][NB];
        if (k0 + 16 <= n) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int64_t k = k0 + 8 * u + 2 * kq;
#pragma unroll
                for (int h = 0; h < NA; ++h) a[u][h] = load_pair(ra[h], k);
#pragma unroll
                for (int g = 0; g < NB; ++g) b[u][g] = load_pair(rb[g], k);
            }
        } else {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int64_t k = k0 + 8 * u + 2 * kq;
#pragma unroll
                for (int h = 0; h < NA; ++h) a[u][h] = load_pair_end(ra[h], k, n);
#pragma unroll
                for (int g = 0; g < NB; ++g) b[u][g] = zero_past(load_pair_end(rb[g], k, n), k, n);
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int h = 0; h < NA; ++h)
#pragma unroll
                    for (int g = 0; g < NB; ++g) acc[h][g] = dmfma(a[u][h][x], b[u][g][x], acc[h][g]);
    }
}

constexpr int kDW = 16;      // columns per group (the MFMA tile's 16 columns)
constexpr int kNW = 16;      // waves per workgroup, one per column
constexpr int kDT = kWave * kNW;
constexpr int kBMax = 64;    // rows per block at most (one lane each)
// rows of V whose gradients and coefficients fit LDS (double: 96 KB); the
// same memory holds the residuals E of the data source's full gradient
constexpr int kVLds = 384;
template <typename T> constexpr size_t dense_lds_bytes() { return 2 * (size_t)kVLds * kDW * sizeof(T); }
static_assert(kDenseELds * kDW * sizeof(double) <= dense_lds_bytes<double>() && kDenseELds % 16 == 0, "E in LDS");

enum : int { kDSweep = 0, kDDone = 1, kDFail = 2 };

template <typename T>
struct DenseSm {
    T sjj[kBMax][kBMax + 1];  // S[J, J] of the current block
    T db[kDW][kBMax + 4];     // minus the block's changes, column by column
    int ck[kDW];              // the group's columns
    T sig[kDW], lam[kDW];
    int state[kDW], status[kDW];
    int outer[kDW], sweeps[kDW], lsweeps[kDW], updates[kDW], checks[kDW], added[kDW];
    int have[kDW];            // secant step: the last update was a fresh one ...
    T sp[kDW], hp[kDW];       // ... at sigma sp, giving h(sp) = hp (B then in Bp)
    int viol;                 // bit c: column c has a violator
    int scan[kNW];
    int refresh;              // some column updated sigma: recompute R
    int v[kVLds];             // V (its first kVLds rows)
};

// Block-wide compaction of the rows marked in `mark` (in ascending order)
// into V; every marked row becomes 1.  Returns |V|, of which at most `cap`
// entries are written.
template <typename T>
__device__ __forceinline__ int compact_v(const DenseArgs<T> &A, DenseSm<T> &sm, int64_t cap)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    int base = 0;
    for (int64_t j0 = 0; j0 < A.p; j0 += kDT) {
        const int64_t j = j0 + tid;
        const bool f = j < A.p && A.mark[j] != 0;
        const unsigned long long m = __ballot(f);
        if (lane == 0) sm.scan[wv] = __popcll(m);
        __syncthreads();
        int off = base, tot = 0;
        for (int w = 0; w < kNW; ++w) {
            off += w < wv ? sm.scan[w] : 0;
            tot += sm.scan[w];
        }
        if (f) {
            const int at = off + lanes_below(m);
            if (at < cap) A.V[at] = (int)j;
            A.mark[j] = 1;
        }
        base += tot;
        __syncthreads();
    }
    return base;
}

// V from the marks; when it covers 15/16 of the predictors (j < pv: a scaled
// lasso's responses follow them and never enter V) and all of them fit `cap`
// rows, the others are taken as well.  A row that a full gradient adds later
// costs the group a new S on V and all its sweeps again, where a row too many
// costs at most 1/8 more per sweep; and with every predictor in V, no result
// depends on which columns the queue's order puts into a group.
template <typename T>
__device__ __forceinline__ int build_v(const DenseArgs<T> &A, DenseSm<T> &sm, int64_t cap)
{
    const int nv = compact_v(A, sm, cap);
    if (nv >= A.pv || A.pv > cap || 16 * (int64_t)nv < 15 * A.pv) return nv;
    for (int64_t j = threadIdx.x; j < A.pv; j += kDT) A.mark[j] = 1;
    __syncthreads();
    return compact_v(A, sm, cap);
}

// position of row j in V[0 .. nv) (j is in V)
__device__ __forceinline__ int v_pos(const int *V, int nv, int j)
{
    int lo = 0, hi = nv;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (V[mid] < j) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// For the data source: S[V, V] and s = S[V, K] of the current V on the
// matrix cores (from Xt), unit diagonal; each wave forms 32 x 32 blocks of
// the upper triangle and stores them both ways.  For S itself: s gathered.
template <typename T, bool DATA>
__device__ __forceinline__ void form_s(const DenseArgs<T> &A, DenseSm<T> &sm, int nv, int m)
{
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    const int64_t n = A.n;
    if constexpr (DATA) {
        const double invn = 1.0 / (double)n;
        const double *Xt = A.Xt;
        const int tb = (nv + 31) / 32;
        const int nblk = tb * (tb + 1) / 2;
        auto vrow = [&](int a) { return Xt + (int64_t)(a < nv ? A.V[a] : 0) * n; };
        for (int t = wv; t < nblk; t += kNW) {
            int bi = 0, q = t;
            while (q >= tb - bi) q -= tb - bi, ++bi;
            const int a0 = 32 * bi, b0 = 32 * (bi + q);
            const double *const ra[2] = {vrow(a0 + (lane & 15)), vrow(a0 + 16 + (lane & 15))};
            const double *const rb[2] = {vrow(b0 + (lane & 15)), vrow(b0 + 16 + (lane & 15))};
            d4 acc[2][2] = {{{0, 0, 0, 0}, {0, 0, 0, 0}}, {{0, 0, 0, 0}, {0, 0, 0, 0}}};
            rows_mma<2, 2>(acc, ra, rb, n);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < 2; ++g)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int a = a0 + 16 * h + drow<double>(lane, r), b = b0 + 16 * g + (lane & 15);
                        if (a < nv && b < nv && a <= b) {
                            const double v = a == b ? 1.0 : acc[h][g][r] * invn;
                            A.Svv[(int64_t)a * nv + b] = v;
                            A.Svv[(int64_t)b * nv + a] = v;
                        }
                    }
        }
        const double *xc = Xt + (int64_t)((lane & 15) < m ? sm.ck[lane & 15] : 0) * n;
        for (int t = wv; t < tb; t += kNW) {
            const int a0 = t * 32;
            const double *const ra[2] = {vrow(a0 + (lane & 15)), vrow(a0 + 16 + (lane & 15))};
            const double *const rc[1] = {xc};
            d4 acc[2][1] = {{{0, 0, 0, 0}}, {{0, 0, 0, 0}}};
            rows_mma<2, 1>(acc, ra, rc, n);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int a = a0 + 16 * h + drow<double>(lane, r), c = lane & 15;
                    if (a < nv)
                        A.sk[(int64_t)a * kDW + c] = (T)(c < m ? (A.V[a] == sm.ck[c] ? 1.0 : acc[h][0][r] * invn) : 0.0);
                }
        }
    } else {
        for (int64_t e = threadIdx.x; e < (int64_t)nv * kDW; e += kDT) {
            const int a = (int)(e / kDW), c = (int)(e % kDW);
            A.sk[e] = c < m ? A.S[(int64_t)A.V[a] * A.p + sm.ck[c]] : T(0);
        }
    }
}

// Row a of S[V, V] at column position b.
template <typename T, bool DATA>
__device__ __forceinline__ const T *vv_row(const DenseArgs<T> &A, const int *V, int nv, int64_t a)
{
    if constexpr (DATA) return (const T *)A.Svv + a * nv;
    else return A.S + (int64_t)V[a] * A.p;
}
template <typename T, bool DATA>
__device__ __forceinline__ T vv_at(const T *row, const int *V, int64_t b)
{
    if constexpr (DATA) return row[b];
    else return row[V[b]];
}

// Place of (row v of V, column c) in the gradients and coefficients while the
// columns iterate: in LDS the columns of a row are rotated by the row, so a
// wave that reads one column over consecutive rows meets all banks.
template <bool LR> __device__ __forceinline__ int64_t rix(int64_t v, int c)
{
    return LR ? v * kDW + ((c + v) & (kDW - 1)) : v * kDW + c;
}

// ... NT tiles of a wave at a time
template <typename T, bool DATA, bool LR, int NT>
__device__ __forceinline__ void fresh_tiles(const DenseArgs<T> &A, const int *V, int nv, int tv, T *R, const T *B)
{
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    for (int t0 = wv; t0 < tv; t0 += NT * kNW) {
        typename DAcc<T>::type acc[NT];
        const T *row[NT];
        T s[NT][4];
#pragma unroll
        for (int h = 0; h < NT; ++h) {
            const int a0 = 16 * (t0 + h * kNW), ra = a0 + (lane & 15);
            row[h] = vv_row<T, DATA>(A, V, nv, ra < nv ? ra : nv - 1);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int a = a0 + drow<T>(lane, r);
                s[h][r] = A.sk[(int64_t)(a < nv ? a : nv - 1) * kDW + (lane & 15)];
                acc[h][r] = T(0);
            }
        }
        tiles_mma<T, NT, NT == 1 ? 6 : 4>(acc, nv, [&](int h, int64_t k) { return vv_at<T, DATA>(row[h], V, k); },
                            [&](int64_t k) { return B[rix<LR>(k, lane & 15)]; });
#pragma unroll
        for (int h = 0; h < NT; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int a = 16 * (t0 + h * kNW) + drow<T>(lane, r);
                if (a < nv) R[rix<LR>(a, lane & 15)] = s[h][r] - acc[h][r];
            }
    }
}

// R = s - S[V, V] B[V, K] for all rows of V (fresh, no accumulated rounding)
template <typename T, bool DATA, bool LR>
__device__ __forceinline__ void fresh_r(const DenseArgs<T> &A, const int *V, int nv, T *R, const T *B)
{
    const int tv = (nv + 15) / 16;
    if (tv <= kNW) fresh_tiles<T, DATA, LR, 1>(A, V, nv, tv, R, B);
    else fresh_tiles<T, DATA, LR, 2>(A, V, nv, tv, R, B);
}

// The full gradient over all p rows for the group's columns; every j outside
// V with |g_j| > lambda_c + kkt_tol is marked 2 and sets bit c of sm.viol.
// lds: dense_lds_bytes of scratch.
template <typename T, bool DATA>
__device__ __forceinline__ void kkt_all(const DenseArgs<T> &A, DenseSm<T> &sm, int nv, int m, T *lds)
{
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    const int64_t p = A.p;
    const int tp = (int)((p + 31) / 32);
    const int c = lane & 15;
    const T thr = sm.lam[c] + A.kkt_tol;
    const int ck = sm.ck[c];
    // (few gradients pass the threshold: the mark is read for those alone)
    auto flag = [&](int64_t j, T g) {
        if ((g < T(0) ? -g : g) > thr && j < A.pv && c < m && j != ck && A.mark[j] == 0) {
            A.mark[j] = 2;
            atomicOr(&sm.viol, 1 << c);
        }
    };
    if constexpr (DATA) {
        // E = x_K - X_V B[V, K] (n x 16, sample by sample; in LDS where it
        // fits), then g = Xt E / n
        const int64_t n = A.n;
        const double *Xt = A.Xt;
        const int tn = (int)((n + 15) / 16);
        const int nch = (int)((n + 15) / 16);  // chunks of 16 samples
        const bool in_lds = dense_e_rows(n) == 0;
        // within 8 samples the even ones come first: the order the pairs of
        // a row of the data are multiplied in
        auto epos = [](int64_t k) { return (k & ~(int64_t)7) | ((k & 1) << 2) | ((k >> 1) & 3); };
        auto full_gradient = [&](double *E) {
            for (int t = wv; t < tn; t += kNW) {
                const int64_t i0 = (int64_t)t * 16;
                d4 acc[1] = {{0, 0, 0, 0}};
                // rows of A: the samples of the tile; B: the coefficients
                const int64_t ii = i0 + c < n ? i0 + c : n - 1;
                tiles_mma<double, 1, 4>(acc, nv, [&](int, int64_t k) { return Xt[(int64_t)A.V[k] * n + ii]; },
                                        [&](int64_t k) { return (double)A.Bd[k * kDW + c]; });
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t i = i0 + drow<double>(lane, r);
                    if (i < n) E[epos(i) * kDW + c] = c < m ? Xt[(int64_t)ck * n + i] - acc[0][r] : 0.0;
                }
            }
            // samples past n in the last chunk multiply zeros
            for (int64_t e = n * kDW + threadIdx.x; e < (int64_t)nch * 16 * kDW; e += kDT)
                E[epos(e / kDW) * kDW + e % kDW] = 0.0;
            __syncthreads();
            const double invn = 1.0 / (double)n;
            for (int t = wv; t < tp; t += kNW) {
                const int64_t j0 = (int64_t)t * 32;
                const double *row[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int64_t j = j0 + 16 * h + c;
                    row[h] = Xt + (j < p ? j : p - 1) * n;
                }
                d4 acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
                const int kq = lane >> 4;
                // whole chunks: the next two chunks' loads are in flight behind
                // this one's products (past the last it is loaded again)
                const int nfull = (int)(n / 16);
                dpair a[3][2][2];
                const double *const r0 = row[0] + 2 * kq, *const r1 = row[1] + 2 * kq;
                auto load = [&](int ch, int d) {
                    const int64_t k = 16 * (int64_t)(ch < nfull ? ch : nfull - 1);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        a[d][u][0] = load_pair(r0 + k, 8 * u);
                        a[d][u][1] = load_pair(r1 + k, 8 * u);
                    }
                };
                auto mul = [&](int ch, int d) {
                    const double *e = E + (16 * (int64_t)ch + kq) * kDW + c;
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int x = 0; x < 2; ++x) {
                            const double y = e[(8 * u + 4 * x) * kDW];
                            acc[0] = dmfma(a[d][u][0][x], y, acc[0]);
                            acc[1] = dmfma(a[d][u][1][x], y, acc[1]);
                        }
                };
                if (nfull > 0) {
                    load(0, 0);
                    load(1, 1);
                    for (int ch = 0; ch < nfull; ch += 3) {
#pragma unroll
                        for (int d = 0; d < 3; ++d) {
                            load(ch + d + 2, (d + 2) % 3);
                            if (ch + d < nfull) mul(ch + d, d);
                        }
                    }
                }
                if (nfull < nch) {
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int h = 0; h < 2; ++h)
                            a[0][u][h] = load_pair_end(row[h], 16 * (int64_t)nfull + 8 * u + 2 * kq, n);
                    mul(nfull, 0);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) flag(j0 + 16 * h + drow<double>(lane, r), (T)(acc[h][r] * invn));
            }
        };
        if (in_lds) full_gradient((double *)lds);
        else full_gradient(A.E);
    } else {
        const int *V = A.V;
        for (int t = wv; t < tp; t += kNW) {
            const int64_t j0 = (int64_t)t * 32;
            const T *row[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int64_t j = j0 + 16 * h + c;
                row[h] = A.S + (j < p ? j : p - 1) * p;
            }
            typename DAcc<T>::type acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
            tiles_mma<T, 2, 4>(acc, nv, [&](int h, int64_t k) { return row[h][V[k]]; },
                               [&](int64_t k) { return A.Bd[k * kDW + c]; });
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t j = j0 + 16 * h + drow<T>(lane, r);
                    if (j < p) flag(j, A.S[j * p + ck] - acc[h][r]);
                }
        }
    }
}

// What follows a column's lasso solve at sigma `so` whose noise update is
// sqrt(s2) (Algorithm 1), with the secant step of the LDS tiers: two fresh
// updates on one support and one sign pattern (`same`; the previous one at
// sigma sp gave hp) give the fixed point of the affine model h(sigma)^2 = C0 +
// C2 sigma^2, and B moves along its affine path to it, by f times its change
// since the previous update (the stopping test stays the plain one).
template <typename T> struct NoiseStep {
    int state, status;
    T sig, f;
    bool next;  // a new lasso at sigma `sig` follows
};
template <typename T>
__device__ __forceinline__ NoiseStep<T> noise_step(const DenseArgs<T> &A, T so, T s2, int outer, bool have, bool same,
                                                   T sp, T hp)
{
    NoiseStep<T> o{kDSweep, kColOk, so, T(0), false};
    if (!(s2 > DegenerateFloor<T>::v)) {
        o.sig = s2 > T(0) ? sqrt(s2) : T(0);
        o.status = kColDegenerate;
        o.state = kDFail;
        return o;
    }
    const T sn = sqrt(s2);
    T ds = sn - so;
    ds = ds < T(0) ? -ds : ds;
    o.sig = sn;
    if (ds < A.tol) {
        o.state = kDDone;
    } else if (outer >= A.max_outer) {
        o.status = kColNoconv;
        o.state = kDFail;
    } else {
        o.next = true;
        if (have && same) {
            const T c2 = (sn * sn - hp * hp) / (so * so - sp * sp);
            const T c0 = sn * sn - c2 * so * so;
            T dsp = so - sp;
            dsp = dsp < T(0) ? -dsp : dsp;
            if (dsp > T(64) * Eps<T>::v * so && c2 >= T(0) && c2 < T(1) && c0 > T(0)) {
                const T ss = sqrt(c0 / (T(1) - c2));
                T jump = ss - sn;
                jump = jump < T(0) ? -jump : jump;
                if (jump <= T(16) * ds) {
                    o.f = (ss - so) / (so - sp);
                    o.sig = ss;
                }
            }
        }
    }
    return o;
}

// V of up to kBMax rows: one block, so every column's whole iteration runs in
// its own wave (one lane per row of V, S[V, V] in LDS), with no barrier until
// all are done.  A.Bd holds the coefficients before and after.
template <typename T, bool DATA>
__device__ __forceinline__ void run_small(const DenseArgs<T> &A, DenseSm<T> &sm, int nv, int m)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), c = tid / kWave;
    for (int e = tid; e < kBMax * kBMax; e += kDT) {
        const int i = e >> 6, j = e & 63;
        T x = T(0);
        if (i < nv && j < nv) x = vv_at<T, DATA>(vv_row<T, DATA>(A, A.V, nv, i), A.V, j);
        sm.sjj[i][j] = x;
    }
    __syncthreads();
    if (c < m && sm.state[c] == kDSweep) {
        const bool act = lane < nv && A.V[lane < nv ? lane : 0] != sm.ck[c];
        const int64_t e = (int64_t)lane * kDW + c;
        const unsigned long long lanes = __ballot(act);
        const T s = act ? A.sk[e] : T(0);
        T beta = act ? A.Bd[e] : T(0), bp = T(0);
        T sig = sm.sig[c], lam = sm.lam[c], sp = sm.sp[c], hp = sm.hp[c];
        bool have = false;
        int outer = sm.outer[c], sweeps = sm.sweeps[c], ls = sm.lsweeps[c], updates = sm.updates[c];
        int state = kDSweep, status = kColOk;
        while (state == kDSweep) {
            // the gradient from scratch at every new lambda
            T r = s;
            for (unsigned long long nz = __ballot(beta != T(0)); nz; nz &= nz - 1) {
                const int q = __builtin_ctzll(nz);
                r -= sm.sjj[q][lane] * bcast(beta, q);
            }
            for (;;) {
                const T beta0 = beta;
                sweep_lanes(lam, lanes, r, beta, [&](int j, T d) { r -= sm.sjj[j][lane] * d; });
                const T dl = beta - beta0;  // each coordinate changes at most once
                updates += __popcll(__ballot(dl != T(0)));
                ++sweeps;
                ++ls;
                if (!__ballot((dl < T(0) ? -dl : dl) >= A.tol)) break;
                if (ls >= A.max_sweeps) {
                    status = kColNoconv;
                    state = kDFail;
                    break;
                }
            }
            if (state != kDSweep) break;
            ++outer;
            const T s2 = T(1) - wave_sum(beta * (s + r));
            const bool same =
                !__ballot((beta > T(0)) != (bp > T(0)) || (beta < T(0)) != (bp < T(0)));
            const NoiseStep<T> o = noise_step(A, sig, s2, outer, have, same, sp, hp);
            ls = 0;
            if (o.next) {
                if (o.f != T(0)) beta += o.f * (beta - bp);
                bp = beta;
                have = o.f == T(0);
                sp = sig;
                hp = sqrt(s2);
                lam = o.sig * A.lambda0;
            }
            sig = o.sig;
            state = o.state;
            status = o.status;
        }
        if (act) A.Bd[e] = beta;
        if (lane == 0) {
            sm.sig[c] = sig;
            sm.lam[c] = lam;
            sm.outer[c] = outer;
            sm.sweeps[c] = sweeps;
            sm.lsweeps[c] = ls;
            sm.updates[c] = updates;
            sm.state[c] = state;
            sm.status[c] = status;
            sm.have[c] = 0;
        }
    }
}

// The columns' iterations on a larger V, until every column is done.  R and B
// (LR: in LDS, else in global memory) hold the gradients and the
// coefficients; V its rows.
template <typename T, bool DATA, bool LR>
__device__ __forceinline__ void run_sweeps(const DenseArgs<T> &A, DenseSm<T> &sm, const int *V, int nv, int m, int b,
                                           T *R, T *B)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int c = wv;  // this wave's column
    const int tv = (nv + 15) / 16;
    constexpr int NX = kBMax * kBMax / kDT;  // entries of a block's S[J, J] per thread
    constexpr int PT = 2, PU = 8;            // tiles and steps of the delayed update loaded ahead
    const int lb = b <= 16 ? 4 : (b <= 32 ? 5 : 6);
    // this lane's rows of S[V, V] in the wave's first PT tiles (rows past V
    // repeat its last: their results go nowhere).  Here and below no load is
    // under a condition of its own: each would wait for itself.
    const T *prow[PT];
#pragma unroll
    for (int h = 0; h < PT; ++h) {
        const int ra = 16 * (wv + h * kNW) + (lane & 15);
        prow[h] = vv_row<T, DATA>(A, V, nv, ra < nv ? ra : nv - 1);
    }
    // entry e of a block's S[J, J] (rows of b places; those past V repeat its
    // last row and are never used)
    auto at = [&](int v0, int e) {
        const int i = v0 + (e >> lb), j = v0 + (e & (b - 1));
        return vv_at<T, DATA>(vv_row<T, DATA>(A, V, nv, i < nv ? i : nv - 1), V, j < nv ? j : nv - 1);
    };
    for (int e = tid; e < b * b; e += kDT) sm.sjj[e >> lb][e & (b - 1)] = at(0, e);
    __syncthreads();
    for (;;) {
        bool any = false;
        for (int q = 0; q < kDW; ++q) any |= sm.state[q] == kDSweep;
        if (!any) break;
        bool over = false;  // a change of the sweep reached tol
        const bool live_col = c < m && sm.state[c] == kDSweep;
        const T lam = sm.lam[c];
        const int ck = sm.ck[c];
        int nupd = 0;
        for (int v0 = 0; v0 < nv; v0 += b) {
            const int bb = nv - v0 < b ? nv - v0 : b;
            // the next block's S[J, J] (after the last the first one's
            // again) and the operands of the delayed update, S[V, J] (the
            // places past the block meet zero changes), in flight during
            // this sweep
            T nx[NX], pa[PT][PU];
            const int vn = v0 + b < nv ? v0 + b : 0;
#pragma unroll
            for (int q = 0; q < NX; ++q)
                if (q * kDT < b * b) nx[q] = at(vn, (tid + q * kDT) & (b * b - 1));
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                const int k = v0 + 4 * u + (lane >> 4);
                const int kc = k < nv ? k : nv - 1;
                const int64_t col = DATA ? kc : V[kc];
#pragma unroll
                for (int h = 0; h < PT; ++h) pa[h][u] = prow[h][col];
            }
            // --- the column's sweep of the block ----------------------------
            T dl = T(0);  // this lane's change
            if (live_col) {
                const int v = v0 + (lane < bb ? lane : 0);
                const bool act = lane < bb && V[v] != ck;
                const int64_t e = rix<LR>(v, c);
                T r = R[e];
                const T beta0 = act ? B[e] : T(0);
                T beta = beta0;
                sweep_lanes(lam, __ballot(act), r, beta, [&](int j, T d) { r -= sm.sjj[j][lane] * d; });
                dl = act ? beta - beta0 : T(0);  // each coordinate changes at most once
                nupd += __popcll(__ballot(dl != T(0)));
                over |= __ballot((dl < T(0) ? -dl : dl) >= A.tol) != 0ull;
                if (dl != T(0)) B[e] = beta;
            }
            sm.db[c][lane] = -dl;
            __syncthreads();
            // --- delayed rank-b update of every row of V ---------------------
            // (PT tiles of a wave at a time, their products interleaved)
            for (int t0 = wv; t0 < tv; t0 += PT * kNW) {
                typename DAcc<T>::type acc[PT];
#pragma unroll
                for (int h = 0; h < PT; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // (LDS holds every row of the tiles)
                        const int a = 16 * (t0 + h * kNW) + drow<T>(lane, r);
                        acc[h][r] = R[rix<LR>(a < (LR ? kVLds : nv) ? a : nv - 1, lane & 15)];
                    }
                auto change = [&](int64_t k) { return sm.db[lane & 15][k]; };
                const T *row[PT];
#pragma unroll
                for (int h = 0; h < PT; ++h) {
                    const int ra = 16 * (t0 + h * kNW) + (lane & 15);
                    row[h] = t0 == wv ? prow[h] : vv_row<T, DATA>(A, V, nv, ra < nv ? ra : nv - 1);
                }
                int k0 = 0;  // the steps done from the operands loaded ahead
                if (t0 == wv) {
#pragma unroll
                    for (int u = 0; u < PU; ++u)
                        if (4 * u < bb) {
                            const T x = change(4 * u + (lane >> 4));
#pragma unroll
                            for (int h = 0; h < PT; ++h)
                                if (t0 + h * kNW < tv) acc[h] = dmfma(pa[h][u], x, acc[h]);
                        }
                    k0 = bb < 4 * PU ? bb : 4 * PU;
                }
                if (k0 < bb)
                    tiles_mma<T, PT, 4>(
                        acc, bb - k0, [&](int h, int64_t k) { return vv_at<T, DATA>(row[h], V, v0 + k0 + k); },
                        [&](int64_t k) { return change(k0 + k); });
#pragma unroll
                for (int h = 0; h < PT; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int a = 16 * (t0 + h * kNW) + drow<T>(lane, r);
                        if (a < nv) R[rix<LR>(a, lane & 15)] = acc[h][r];
                    }
            }
#pragma unroll
            for (int q = 0; q < NX; ++q)
                if (q * kDT < b * b) {
                    const int e = (tid + q * kDT) & (b * b - 1);  // (b 16: the same values several times)
                    sm.sjj[e >> lb][e & (b - 1)] = nx[q];
                }
            __syncthreads();
        }
        // --- per column: inner stop, noise update, outer stop ---------------
        // (every lane of the column's wave takes the same decisions; lane 0
        // records them)
        if (tid == 0) sm.refresh = 0;
        __syncthreads();
        if (live_col) {
            const int ls = sm.lsweeps[c] + 1;
            const T so = sm.sig[c];
            if (over) {
                if (lane == 0) {
                    sm.lsweeps[c] = ls;
                    if (ls >= A.max_sweeps) {
                        sm.status[c] = kColNoconv;
                        sm.state[c] = kDFail;
                    }
                }
            } else {
                T part = T(0);
                bool diff = false;
                for (int v = lane; v < nv; v += kWave) {
                    const int64_t e = (int64_t)v * kDW + c, q = rix<LR>(v, c);
                    const T bv = B[q], pv = A.Bp[e];
                    part += bv * (A.sk[e] + R[q]);
                    diff |= (bv > T(0)) != (pv > T(0)) || (bv < T(0)) != (pv < T(0));
                }
                const T s2 = T(1) - wave_sum(part);
                const int outer = sm.outer[c] + 1;
                const NoiseStep<T> o =
                    noise_step(A, so, s2, outer, sm.have[c] != 0, __ballot(diff) == 0ull, sm.sp[c], sm.hp[c]);
                if (o.next) {
                    // the step (when taken), then B is the next update's Bp
                    for (int v = lane; v < nv; v += kWave) {
                        const int64_t e = (int64_t)v * kDW + c, q = rix<LR>(v, c);
                        T bv = B[q];
                        if (o.f != T(0)) {
                            bv += o.f * (bv - A.Bp[e]);
                            B[q] = bv;
                        }
                        A.Bp[e] = bv;
                    }
                }
                if (lane == 0) {
                    sm.lsweeps[c] = 0;
                    sm.outer[c] = outer;
                    sm.sig[c] = o.sig;
                    sm.state[c] = o.state;
                    sm.status[c] = o.status;
                    if (o.next) {
                        sm.lam[c] = o.sig * A.lambda0;
                        sm.have[c] = o.f == T(0);
                        sm.sp[c] = so;
                        sm.hp[c] = sqrt(s2);
                        sm.refresh = 1;
                    }
                }
            }
            if (lane == 0) {
                ++sm.sweeps[c];
                sm.updates[c] += nupd;
            }
        }
        __syncthreads();
        // new lambdas: gradients recomputed from scratch (no drift)
        if (sm.refresh) {
            fresh_r<T, DATA, LR>(A, V, nv, R, B);
            __syncthreads();
        }
    }
}

// The iterations of a group: V of up to kBMax rows column by column; else the
// gradients and coefficients in LDS while they last where V fits (A.Bd holds
// the coefficients before and after), else in the workspace.
template <typename T, bool DATA>
__device__ __forceinline__ void iterate(const DenseArgs<T> &A, DenseSm<T> &sm, int nv, int m, int b, T *lds)
{
    const int tid = threadIdx.x;
    if (nv <= kBMax) {
        run_small<T, DATA>(A, sm, nv, m);
    } else if (nv <= kVLds) {
        T *R = lds, *B = lds + (size_t)kVLds * kDW;
        for (int v = tid; v < nv; v += kDT) sm.v[v] = A.V[v];
        for (int e = tid; e < nv * kDW; e += kDT) B[rix<true>(e / kDW, e % kDW)] = A.Bd[e];
        __syncthreads();
        fresh_r<T, DATA, true>(A, sm.v, nv, R, B);
        __syncthreads();
        run_sweeps<T, DATA, true>(A, sm, sm.v, nv, m, b, R, B);
        for (int e = tid; e < nv * kDW; e += kDT) A.Bd[e] = B[rix<true>(e / kDW, e % kDW)];
    } else {
        fresh_r<T, DATA, false>(A, A.V, nv, A.R, A.Bd);
        __syncthreads();
        run_sweeps<T, DATA, false>(A, sm, A.V, nv, m, b, A.R, A.Bd);
    }
    __syncthreads();
}

// Workgroup bi of nb takes the groups bi, bi + nb, .. of the queue (or of
// po.take).
template <typename T, typename TS, bool DATA>
__device__ __forceinline__ void dense_groups(const DenseArgs<T> &A0, const DenseSrc<TS> &src, DenseSm<T> &sm, T *lds,
                                             int64_t bi, int64_t nb, const DensePutOff &po)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    if (po.take && bi >= *po.ntake) return;  // (as a rule nothing was put off)
    if (*A0.flags) return;
    const int64_t p = A0.p;
    // the queue, or (no queue) the columns 0 .. ncols - 1
    const int q = A0.queue ? *A0.qcnt : (int)A0.ncols;
    const int ng = po.take ? *po.ntake : (q + kDW - 1) / kDW;
    if (bi >= ng) return;
    // this workgroup's slice of the workspace
    DenseArgs<T> A = A0;
    {
        const int64_t vc = A0.vcap;
        A.mark += bi * p;
        A.V += bi * vc;
        A.Vold += bi * vc;
        A.R += bi * vc * kDW;
        A.Bd += bi * vc * kDW;
        A.Bp += bi * vc * kDW;
        A.sk += bi * vc * kDW;
        if (DATA) {
            A.Svv += bi * A0.svv_cap * A0.svv_cap;
            A.E += bi * kDW * dense_e_rows(A0.n);
        }
    }
    // V may hold vcap rows (and, from the data, svv_cap)
    const int64_t vlim = DATA && A.svv_cap < A.vcap ? A.svv_cap : A.vcap;
    for (int64_t j = tid; j < p; j += kDT) A.mark[j] = 0;
    __syncthreads();
    const int b = A.block <= 16 ? 16 : (A.block <= 32 ? 32 : kBMax);
    for (int gi = (int)bi; gi < ng; gi += (int)nb) {
        const int g0 = (po.take ? po.take[gi] : gi) * kDW;
        const int m = q - g0 < kDW ? q - g0 : kDW;
        // --- the group's columns and their start --------------------------
        if (tid < kDW) {
            const int c = tid;
            sm.ck[c] = c < m ? (A.queue ? A.queue[g0 + c] : g0 + c) : 0;
            const int64_t k = sm.ck[c];
            double sg = c < m && src.sigma ? src.sigma[k] : 1.0;
            sg = sg > 0.0 && sg < 1e300 ? sg : 1.0;
            sm.sig[c] = (T)sg;
            sm.lam[c] = (T)sg * A.lambda0;
            sm.state[c] = c < m ? kDSweep : kDDone;
            sm.status[c] = kColOk;
            sm.outer[c] = sm.sweeps[c] = sm.lsweeps[c] = sm.updates[c] = sm.checks[c] = sm.added[c] = 0;
            sm.have[c] = 0;
            sm.sp[c] = sm.hp[c] = T(0);
        }
        if (tid == 0) sm.viol = 0;
        __syncthreads();
        // mark the start lists (and pending candidates) of the group's columns
        for (int c = wv; c < m; c += kNW) {
            const int64_t k = sm.ck[c];
            int cnt = src.cnt ? src.cnt[k] : 0;
            cnt = cnt < 0 ? 0 : cnt;
            const int64_t base = cnt > kWMax ? p * (int64_t)kWMax + src.off[k] : k * (int64_t)kWMax;
            for (int i = lane; i < cnt; i += kWave) {
                const int j = src.idx[base + i];
                if (j >= 0 && j < p && j != k) A.mark[j] = 1;
            }
            if (src.pend_cnt) {
                int np = src.pend_cnt[k];
                np = np < 0 ? 0 : (np > kPendMax ? kPendMax : np);
                for (int i = lane; i < np; i += kWave) {
                    const int j = src.pend_idx[k * kPendMax + i];
                    if (j >= 0 && j < p && j != k) A.mark[j] = 1;
                }
            }
        }
        __syncthreads();
        int nv = build_v(A, sm, vlim);
        bool gfail = false;
        if ((int64_t)nv > vlim) {
            // V does not fit this workgroup's buffers: the group fails, or is
            // put off (rare)
            if (tid < m) sm.status[tid] = kColWorkset, sm.state[tid] = kDFail;
            gfail = true;
            nv = 0;
        }
        for (int64_t e = tid; e < (int64_t)nv * kDW; e += kDT) A.Bd[e] = T(0);
        __syncthreads();
        for (int c = wv; c < m && nv > 0; c += kNW) {
            const int64_t k = sm.ck[c];
            int cnt = src.cnt ? src.cnt[k] : 0;
            cnt = cnt < 0 ? 0 : cnt;
            const int64_t base = cnt > kWMax ? p * (int64_t)kWMax + src.off[k] : k * (int64_t)kWMax;
            for (int i = lane; i < cnt; i += kWave) {
                const int j = src.idx[base + i];
                if (j >= 0 && j < p && j != k) A.Bd[(int64_t)v_pos(A.V, nv, j) * kDW + c] = (T)src.beta[base + i];
            }
        }
        __syncthreads();
        int rounds = 0;
        for (;;) {
            // --- S on V, then sweeps until every column is done -------------
            form_s<T, DATA>(A, sm, nv, m);
            __syncthreads();
            iterate<T, DATA>(A, sm, nv, m, b, lds);
            // --- KKT over all p rows -----------------------------------------
            bool any_done = false;
            for (int c = 0; c < m; ++c) any_done |= sm.state[c] == kDDone;
            if (!any_done || gfail) break;
            if (tid == 0) sm.viol = 0;
            __syncthreads();
            kkt_all<T, DATA>(A, sm, nv, m, lds);
            __syncthreads();
            const int viol = sm.viol;
            if (tid < m && sm.state[tid] == kDDone) {
                ++sm.checks[tid];
                if (viol & (1 << tid)) {
                    if (rounds >= A.max_rounds) {
                        sm.status[tid] = kColNoconv;
                        sm.state[tid] = kDFail;
                    } else {
                        sm.state[tid] = kDSweep;
                    }
                }
            }
            __syncthreads();
            if (!viol || rounds >= A.max_rounds) {
                // rows marked 2 were not taken: clear them
                for (int64_t j = tid; j < p; j += kDT)
                    if (A.mark[j] == 2) A.mark[j] = 0;
                __syncthreads();
                break;
            }
            ++rounds;
            // --- V grows: move B to the new row positions ---------------------
            // (R, rebuilt below, holds the old B meanwhile; Vold the old V)
            const int nv_old = nv;
            for (int64_t e = tid; e < (int64_t)nv_old * kDW; e += kDT) A.R[e] = A.Bd[e];
            for (int64_t e = tid; e < (int64_t)nv_old; e += kDT) A.Vold[e] = A.V[e];
            __syncthreads();
            nv = build_v(A, sm, vlim);
            if (tid < m) {
                sm.added[tid] += nv - nv_old;
                sm.have[tid] = 0;  // B moved: the secant needs two fresh updates again
            }
            if ((int64_t)nv > vlim) {
                if (tid < m) sm.status[tid] = kColWorkset, sm.state[tid] = kDFail;
                gfail = true;
                nv = 0;
            }
            for (int64_t e = tid; e < (int64_t)nv * kDW; e += kDT) A.Bd[e] = T(0);
            __syncthreads();
            for (int64_t e = tid; e < (int64_t)nv_old * kDW && nv > 0; e += kDT) {
                const int a = (int)(e / kDW), c = (int)(e % kDW);
                const T v = A.R[e];
                if (v != T(0)) A.Bd[(int64_t)v_pos(A.V, nv, A.Vold[a]) * kDW + c] = v;
            }
            __syncthreads();
            if (gfail) break;
        }
        if (gfail) {  // (V does not hold every mark)
            if (tid == 0 && po.put) po.put[atomicAdd(po.nput, 1)] = g0 / kDW;
            for (int64_t j = tid; j < p; j += kDT) A.mark[j] = 0;
            __syncthreads();
        }
        // --- results: the nonzeros of each column, ascending ---------------
        for (int c = wv; c < m && !(gfail && po.put); c += kNW) {
            const int64_t k = sm.ck[c];
            int cnt = 0;
            for (int v0 = 0; v0 < nv; v0 += kWave) {
                const int v = v0 + lane;
                const bool nz = v < nv && A.Bd[(int64_t)v * kDW + c] != T(0);
                cnt += __popcll(__ballot(nz));
            }
            int status = sm.status[c];
            int64_t base = k * (int64_t)kWMax;
            if (cnt > kWMax) {
                int off = 0;
                if (lane == 0) off = atomicAdd(A.pool_cnt, cnt);
                off = __shfl(off, 0);
                if ((int64_t)off + cnt > A.pool_cap) {
                    status = kColWorkset;
                    cnt = kWMax;
                } else {
                    base = p * (int64_t)kWMax + off;
                    if (lane == 0) A.w_off[k] = off;
                }
            }
            int pos = 0;
            for (int v0 = 0; v0 < nv && pos < cnt; v0 += kWave) {
                const int v = v0 + lane;
                const T bv = v < nv ? A.Bd[(int64_t)v * kDW + c] : T(0);
                const bool nz = bv != T(0);
                const unsigned long long mk = __ballot(nz);
                const int at = pos + lanes_below(mk);
                if (nz && at < cnt) {
                    A.w_idx[base + at] = A.V[v];
                    A.w_beta[base + at] = bv;
                }
                pos += __popcll(mk);
            }
            if (lane == 0) {
                A.w_cnt[k] = cnt;
                A.sigma[k] = (double)sm.sig[c];
                A.lam_used[k] = (double)sm.lam[c];
                A.col_status[k] = status;
                if (A.band_cnt) A.band_cnt[k] = kBandMax + 1;
                int *ci = A.info + k * A.info_stride;
                if (A.info_stride == 4) {
                    ci[0] += sm.outer[c];
                    ci[1] += sm.sweeps[c];
                    ci[2] += sm.updates[c];
                    ci[3] += sm.checks[c];
                } else {
                    ci[0] += sm.outer[c];
                    ci[1] += sm.sweeps[c];
                    ci[2] += sm.updates[c];
                    ci[3] += sm.checks[c];
                    ci[4] += sm.added[c];
                }
                atomicAdd(&A.counters[kCntDense], 1ull);
            }
        }
        // clear the marks of V for the next group
        for (int64_t e = tid; e < (int64_t)nv; e += kDT) A.mark[A.V[e]] = 0;
        __syncthreads();
    }
}

template <typename T, typename TS, bool DATA>
__global__ __launch_bounds__(kDT) void k_dense(DenseArgs<T> A0, DenseSrc<TS> src, DensePutOff po)
{
    __shared__ DenseSm<T> sm;
    extern __shared__ __align__(16) unsigned char dense_lds[];
    dense_groups<T, TS, DATA>(A0, src, sm, reinterpret_cast<T *>(dense_lds), blockIdx.x, gridDim.x, po);
}

// block b is workgroup b - off[d] of problem d
template <typename T, typename TS, bool DATA>
__global__ __launch_bounds__(kDT) void k_dense_grouped(const DenseJob<T, TS> *__restrict__ tab,
                                                       const int64_t *__restrict__ off, int nd)
{
    __shared__ DenseSm<T> sm;
    extern __shared__ __align__(16) unsigned char dense_lds[];
    const int64_t b = blockIdx.x;
    const int d = group_of(off, nd, b);
    dense_groups<T, TS, DATA>(tab[d].a, tab[d].src, sm, reinterpret_cast<T *>(dense_lds), b - off[d],
                              off[d + 1] - off[d], DensePutOff{});
}

} // namespace

template <typename T, typename TS>
void launch_dense(const DenseArgs<T> &a, const DenseSrc<TS> &src, hipStream_t s, int blocks, const DensePutOff &po)
{
    if constexpr (sizeof(T) == 8) {
        if (a.Xt) {
            hipLaunchKernelGGL((k_dense<T, TS, true>), dim3(blocks), dim3(kDT), dense_lds_bytes<T>(), s, a, src, po);
            return;
        }
    }
    hipLaunchKernelGGL((k_dense<T, TS, false>), dim3(blocks), dim3(kDT), dense_lds_bytes<T>(), s, a, src, po);
}

template <typename T, typename TS>
void launch_dense_grouped(const DenseJob<T, TS> *tab, const int64_t *off, int nd, int64_t blocks, hipStream_t s)
{
    // (from the data: the mixed form's polish; from S: the other forms)
    constexpr bool DATA = !std::is_same<T, TS>::value;
    hipLaunchKernelGGL((k_dense_grouped<T, TS, DATA>), dim3((unsigned)blocks), dim3(kDT), dense_lds_bytes<T>(), s, tab,
                       off, nd);
}

template void launch_dense_grouped<double, double>(const DenseJob<double, double> *, const int64_t *, int, int64_t,
                                                   hipStream_t);
template void launch_dense_grouped<float, float>(const DenseJob<float, float> *, const int64_t *, int, int64_t,
                                                 hipStream_t);
template void launch_dense_grouped<double, float>(const DenseJob<double, float> *, const int64_t *, int, int64_t,
                                                  hipStream_t);
template void launch_dense<double, double>(const DenseArgs<double> &, const DenseSrc<double> &, hipStream_t, int,
                                          const DensePutOff &);
template void launch_dense<float, float>(const DenseArgs<float> &, const DenseSrc<float> &, hipStream_t, int,
                                          const DensePutOff &);
template void launch_dense<double, float>(const DenseArgs<double> &, const DenseSrc<float> &, hipStream_t, int,
                                          const DensePutOff &);

} // namespace spmesl
