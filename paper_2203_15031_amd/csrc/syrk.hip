// syrk.hip -- the sample covariance S = Xs^T Xs / n on the matrix cores.
//
// S is the only dense contraction of the method (n p^2 multiply-adds).  Only
// the upper triangle of square tiles is computed; each tile is
// written twice, once as is and once transposed, so S is stored full and
// every row of S is a contiguous read for the solver.  The diagonal is set
// to exactly 1 (s_jj = 1 for standardised columns, Section 2.2), which the
// coordinate update relies on.
//
// Three forms:
//   * double: v_mfma_f64_16x16x4f64, Xs row-major n x p;
//   * float : v_mfma_f32_16x16x4f32, same layout;
//   * mixed : two-term bfloat16 split x = hi + lo of float(x), products
//             hi*hi + hi*lo + lo*hi accumulated in float by
//             v_mfma_f32_16x16x32_bf16 (the split in operand order).
//
// Operand layout of the 16x16xK MFMAs used here (wave64): lane l supplies
// row l%16 of A and column l%16 of B, at k-block l/16.  Accumulator element r
// of lane l is D[4*(l/16) + r][l%16] for the float-output MFMAs and
// D[4*r + l/16][l%16] for the double one (checked on the device).
#include "common.hpp"

namespace spmesl {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ d4 mfma16x16x4(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma16x16x4(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <typename T> struct Acc;
template <> struct Acc<double> { typedef d4 type; };
template <> struct Acc<float> { typedef f4 type; };

// row of accumulator element r of `lane` within a 16x16 block
template <typename T> __device__ __forceinline__ int acc_row(int lane, int r);
template <> __device__ __forceinline__ int acc_row<double>(int lane, int r) { return 4 * r + (lane >> 4); }
template <> __device__ __forceinline__ int acc_row<float>(int lane, int r) { return 4 * (lane >> 4) + r; }

// The screen (see Screen): entry s_jk = s_kj = v of a symmetric pair (j != k)
// makes j a candidate of column k and k one of column j (those below pv);
// v = 0 records nothing.  Candidates of a tile are collected in LDS and
// flushed with one round of global atomics per tile, so no wave waits on a
// global atomic inside the store loops.
// Per-wave candidate lists (no atomics): wave w appends to its own segment
// and keeps the count in a wave-uniform register.
template <int NW, int N>
struct ScreenWaves {
    static constexpr int kCap = N;  // entries per wave
    int n[NW];
    int jk[NW][2 * N];
};

// PV: only variables below pv are candidates (else every variable is).
template <bool PV, typename L, typename T>
__device__ __forceinline__ void screen_pair_wave(L &lst, int wv, int &count, int *cnt, int *idx, T thr, int64_t pv,
                                                 int64_t j, int64_t k, T v)
{
    const bool hit = cnt && j != k && (v < T(0) ? -v : v) > thr;
    const unsigned long long mask = __ballot(hit);
    if (!mask) return;
    const int q = count + 2 * lanes_below(mask);
    count += 2 * __popcll(mask);
    if (!hit) return;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        int a = (int)(d ? k : j);        // a joins column b
        const int b = (int)(d ? j : k);
        if (PV && a >= pv) a = -1;       // no candidate: an empty slot
        if (q + d < L::kCap) {
            lst.jk[wv][2 * (q + d)] = a;
            lst.jk[wv][2 * (q + d) + 1] = b;
        } else if (!PV || a >= 0) {
            const int pos = atomicAdd(&cnt[b], 1);
            if (pos < kPendMax) idx[(int64_t)b * kPendMax + pos] = a;
        }
    }
}

template <int NW, int N>
__device__ __forceinline__ void screen_flush_waves(ScreenWaves<NW, N> &lst, int *cnt, int *idx)
{
    if (!cnt) return;
    for (int w = 0; w < NW; ++w) {
        const int m = lst.n[w] < N ? lst.n[w] : N;
        for (int q0 = threadIdx.x; q0 < m; q0 += 8 * (int)blockDim.x) {
            int jj[8], pos[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int q = q0 + u * (int)blockDim.x;
                pos[u] = kPendMax;
                jj[u] = 0;
                if (q < m) {
                    jj[u] = lst.jk[w][2 * q];
                    if (jj[u] >= 0) pos[u] = atomicAdd(&cnt[lst.jk[w][2 * q + 1]], 1);
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int q = q0 + u * (int)blockDim.x;
                if (q < m && pos[u] < kPendMax) idx[(int64_t)lst.jk[w][2 * q + 1] * kPendMax + pos[u]] = jj[u];
            }
        }
    }
}

// Blocks that share a row panel are kept on the same XCD (blocks are
// dispatched to the 8 XCDs round-robin): the position of block bid of nb in
// an order that gives each XCD a contiguous run.
__device__ __forceinline__ int64_t xcd_order(int64_t nb, int64_t bid)
{
    const int64_t x = bid & 7, q = nb >> 3, r = nb & 7;
    return x * q + (x < r ? x : r) + (bid >> 3);
}

// Upper-triangle tile t (bj <= bk) of a T x T tiling, in strips of kStrip
// tile rows taken column by column: the tiles an XCD runs at a time (64 at
// two blocks per CU) then share 8 row and 8 column panels in its L2, where
// row by row they shared one row panel and streamed 64 column panels.
constexpr int kStrip = 8;
__device__ __forceinline__ void tri_tile(int T, int64_t t, int *bj, int *bk)
{
    int r0 = 0;
    for (;;) {
        const int h = T - r0 < kStrip ? T - r0 : kStrip;  // rows of the strip
        const int64_t cnt = (int64_t)h * (T - r0) - (int64_t)h * (h - 1) / 2;
        if (t < cnt || r0 + h >= T) {
            // the first h columns of the strip hold 1, 2, .., h tiles
            int c = 0;
            while (c < h - 1 && t > c) {
                t -= c + 1;
                ++c;
            }
            if (c == h - 1) {
                *bk = r0 + c + (int)(t / h);
                *bj = r0 + (int)(t % h);
            } else {
                *bk = r0 + c;
                *bj = r0 + (int)t;
            }
            return;
        }
        t -= cnt;
        r0 += h;
    }
}

// Map a linear block id to an upper-triangle tile, XCD-aware.
__device__ __forceinline__ void tile_of_block(int T, int *bj, int *bk)
{
    tri_tile(T, xcd_order(gridDim.x, blockIdx.x), bj, bk);
}

template <bool NT, typename V> __device__ __forceinline__ void store_s(V *at, V v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, at);
    else *at = v;
}

// A wave's NA x NB accumulator blocks (from variable j0 / k0 of S) to S and
// the screen (PV: candidates j < pv), straight from the accumulators: element
// r of lane l is row acc_row(l, r), column l % 16 of its 16 x 16 block.
// Direct: 16 lanes store consecutive entries of a row of S; mirrored: in the
// float layout the lane's four rows are four consecutive columns of row kk,
// one 16-byte store.  A diagonal tile stores its upper triangle both ways, so
// S is symmetric bit for bit.  NT: nontemporal stores.  Returns the wave's
// count of screen entries.
template <typename T, int NA, int NB, bool NT, bool PV, typename SCR>
__device__ __forceinline__ int store_tile(const typename Acc<T>::type (&acc)[NA][NB], T *__restrict__ S, int64_t p,
                                          int64_t j0, int64_t k0, bool diag, T invn, T thr, int64_t pv,
                                          int *__restrict__ scnt, int *__restrict__ sidx, SCR &scr, int w)
{
    const int lane = threadIdx.x & 63;
    const int c16 = lane & 15;
    const bool vec_ok = sizeof(T) == 4 && (p & 3) == 0;  // rows of S 16-byte aligned
    const int jl = acc_row<T>(lane, 0);
    constexpr int JS = sizeof(T) == 4 ? 1 : 4;           // row step per element
    int nscr = 0;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int64_t kk = k0 + 16 * b + c16;
            const int64_t jb = j0 + 16 * a + jl;
            T v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = jb + JS * r == kk ? T(1) : acc[a][b][r] * invn;
            // screen: a pair above the threshold is a candidate of both
            // columns (every lane takes part in the ballots)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool mine = jb + JS * r < p && kk < p && (!diag || jb + JS * r < kk);
                screen_pair_wave<PV>(scr, w, nscr, scnt, sidx, thr, pv, jb + JS * r, kk, mine ? v[r] : T(0));
            }
            if (kk >= p) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (jb + JS * r < p && (!diag || jb + JS * r <= kk)) store_s<NT>(&S[(jb + JS * r) * p + kk], v[r]);
            if (vec_ok && jb + 3 < p && (!diag || kk > jb + 3)) {
                if constexpr (sizeof(T) == 4)
                    store_s<NT>(reinterpret_cast<f4 *>(&S[kk * p + jb]), f4{v[0], v[1], v[2], v[3]});
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (jb + JS * r < p && (!diag || kk > jb + JS * r)) store_s<NT>(&S[kk * p + jb + JS * r], v[r]);
            }
        }
    return nscr;
}

// ---------------------------------------------------------------------------
// double and float forms: operands straight from Xs into registers
//
// A block of four waves computes one EDGE x EDGE tile, each wave its own
// quarter, with no LDS staging and no barrier: the 16 x 4 operands of the
// matrix instructions are 16 consecutive variables of 4 samples, which Xs
// (samples x variables) holds as full 128-byte (double) or 64-byte (float)
// rows, and a wave keeps the loads of the next D - 1 steps in flight behind
// the NB x NB operations of the current one.  Each entry takes its products
// in sample order whatever the edge, so S is the same to the bit.
// ---------------------------------------------------------------------------
template <typename T, int EDGE> struct SyrkShape {
    static constexpr int NB = EDGE / 32;  // 16 x 16 blocks per wave and dimension
    // sample steps of operands held: a step is NB x NB operations of 64
    // (double) or 32 cycles; 128 (double): as many as leave two waves per SIMD
    static constexpr int D = EDGE >= 128 ? (sizeof(T) == 8 ? 2 : 4) : (EDGE >= 64 ? 8 : 24);
    typedef ScreenWaves<4, 448> Scr;
};

template <typename T, int EDGE>
__device__ __forceinline__ void syrk_tile(const T *__restrict__ Xs, int64_t n, int64_t p, T *__restrict__ S, int bj,
                                          int bk, T invn, T thr, int64_t pv, int *__restrict__ scnt,
                                          int *__restrict__ sidx, typename SyrkShape<T, EDGE>::Scr &scr)
{
    constexpr int NB = SyrkShape<T, EDGE>::NB, D = SyrkShape<T, EDGE>::D;
    typedef typename Acc<T>::type AccT;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w & 1, wn = w >> 1;
    const int64_t j0 = (int64_t)bj * EDGE + 16 * NB * wm, k0 = (int64_t)bk * EDGE + 16 * NB * wn;
    const bool diag = bj == bk;
    int nscr = 0;
    // the wave below the diagonal of a diagonal tile has nothing to store,
    // nor has one past the last variable
    if (j0 < p && k0 < p && !(diag && wm > wn)) {
        const int kq = lane >> 4, c16 = lane & 15;
        // variables past the last load that one (never stored)
        unsigned ca[NB], cb[NB];  // p is below 2^30
#pragma unroll
        for (int a = 0; a < NB; ++a) {
            const int64_t ja = j0 + 16 * a + c16, kb = k0 + 16 * a + c16;
            ca[a] = (unsigned)(kq * p + (ja < p ? ja : p - 1));
            cb[a] = (unsigned)(kq * p + (kb < p ? kb : p - 1));
        }
        AccT acc[NB][NB];
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[a][b] = AccT{0, 0, 0, 0};
        const int64_t full = n / 4;  // whole steps of 4 samples
        T av[D][NB], bv[D][NB];
        const T *src = Xs;  // the next step to load
        auto load = [&](int d) {
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                av[d][a] = src[ca[a]];
                bv[d][a] = src[cb[a]];
            }
            src += 4 * p;
        };
        auto mul = [&](int d) {
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[a][b] = mfma16x16x4(av[d][a], bv[d][b], acc[a][b]);
        };
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (d < full) load(d);
        int64_t s0 = 0;
        for (; s0 + 2 * D - 1 <= full; s0 += D) {  // every load of the round is a whole step
#pragma unroll
            for (int d = 0; d < D; ++d) {
                load((d + D - 1) % D);
                mul(d);
            }
        }
        for (; s0 < full; s0 += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (s0 + d + D - 1 < full) load((d + D - 1) % D);
                if (s0 + d < full) mul(d);
            }
        }
        if (n % 4) {
            const bool in = 4 * full + kq < n;
            src = Xs + 4 * full * p;
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                av[0][a] = in ? src[ca[a]] : T(0);
                bv[0][a] = in ? src[cb[a]] : T(0);
            }
            mul(0);
        }
        nscr = store_tile<T, NB, NB, false, true>(acc, S, p, j0, k0, diag, invn, thr, pv, scnt, sidx, scr, w);
    }
    if (lane == 0) scr.n[w] = nscr;
    __syncthreads();
    screen_flush_waves(scr, scnt, sidx);
}

template <typename T, int EDGE>
__global__ __launch_bounds__(256, 2) void k_syrk(const T *__restrict__ Xs, int64_t n, int64_t p, T *__restrict__ S,
                                              int Tt, T invn, T thr, int64_t pv, int *__restrict__ scnt,
                                              int *__restrict__ sidx)
{
    __shared__ typename SyrkShape<T, EDGE>::Scr scr;
    int bj, bk;
    tile_of_block(Tt, &bj, &bk);
    syrk_tile<T, EDGE>(Xs, n, p, S, bj, bk, invn, thr, pv, scnt, sidx, scr);
}

// The tiles of many problems in one launch, one tile per block: block b
// (in the XCD-aware order) is tile b - off[d] of problem d.
template <typename T, int EDGE>
__global__ __launch_bounds__(256, 2) void k_syrk_grouped(const SyrkJobT<T> *__restrict__ tab,
                                                      const int64_t *__restrict__ off, int nd)
{
    __shared__ typename SyrkShape<T, EDGE>::Scr scr;
    const int64_t t = xcd_order(gridDim.x, blockIdx.x);
    const int d = group_of(off, nd, t);
    const SyrkJobT<T> &J = tab[d];
    int bj, bk;
    tri_tile(J.Tt, t - off[d], &bj, &bk);
    syrk_tile<T, EDGE>(J.Xs, J.n, J.p, J.S, bj, bk, J.invn, J.thr, J.pv, J.scnt, J.sidx, scr);
}

// Tile edge of the double (dbl) and float forms from the launch's numbers of
// 64 x 64 and 128 x 128 tiles (every edge gives the same bits).  Measured, in
// us, edges 32 / 64 / 128 (n x p, no screen), and the LDS-staged kernels these
// replaced (64 below 256 tiles of 128, then 128; float 64):
//   double 100 x 200      7.5 /  9.6 /  24             (start 9.9)
//   double 1500 x 300     30 /   62 / 197               (105)
//   double 250 x 756      15 /   17 /  44               (25)
//   double 200 x 1000     18 /   16 /  38               (23)
//   double 400 x 5000    326 /  234 / 235               (283)
//   double 1000 x 5000   738 /  491 / 531               (625)
//   double 1000 x 10000 2756 / 1835 / 1707              (2010)
//   float 1500 x 300      20 /   46 / 136               (70)
//   float 200 x 1000      13 /   13 /  29               (18)
//   float 333 x 2047      39 /   37 /  45               (45)
//   float 400 x 5000     197 /  162 / 158               (191)
//   float 1000 x 10000  1635 / 1348 / 1142              (1508)
// Few tiles leave SIMDs idle behind a serial chain of n / 4 steps, so they are
// cut smaller; many are bound by the operands' traffic from L2 (64: about
// 16 bytes per cycle and CU beside the matrix cores), so they are cut larger.
int syrk_edge(int64_t tiles64, int64_t tiles128, bool dbl)
{
    if (tiles64 < 120) return 32;
    return tiles128 >= (dbl ? 2000 : 800) ? 128 : 64;
}

template <typename T>
SyrkJobT<T> syrk_job_mfma(const T *Xs, int64_t n, int64_t p, T *S, const Screen &sc, int edge, int64_t *tiles)
{
    SyrkJobT<T> j{};
    j.Xs = Xs;
    j.n = n;
    j.p = p;
    j.S = S;
    j.Tt = (int)((p + edge - 1) / edge);
    j.invn = (T)(1.0 / (double)n);
    if constexpr (sizeof(T) == 8)
        j.thr = (T)sc.thr64;
    else
        j.thr = (T)sc.thr32;
    j.pv = sc.pv > 0 ? sc.pv : p;
    j.scnt = sc.cnt;
    j.sidx = sc.idx;
    *tiles = (int64_t)j.Tt * (j.Tt + 1) / 2;
    return j;
}

template <typename T>
void launch_syrk_mfma_grouped(const SyrkJobT<T> *tab, const int64_t *tile_off, int nd, int64_t tiles, int edge,
                              hipStream_t s)
{
    if (tiles <= 0) return;
    if (edge == 128)
        hipLaunchKernelGGL((k_syrk_grouped<T, 128>), dim3((unsigned)tiles), dim3(256), 0, s, tab, tile_off, nd);
    else if (edge == 32)
        hipLaunchKernelGGL((k_syrk_grouped<T, 32>), dim3((unsigned)tiles), dim3(256), 0, s, tab, tile_off, nd);
    else
        hipLaunchKernelGGL((k_syrk_grouped<T, 64>), dim3((unsigned)tiles), dim3(256), 0, s, tab, tile_off, nd);
}

template SyrkJobT<double> syrk_job_mfma<double>(const double *, int64_t, int64_t, double *, const Screen &, int,
                                                int64_t *);
template SyrkJobT<float> syrk_job_mfma<float>(const float *, int64_t, int64_t, float *, const Screen &, int,
                                              int64_t *);
template void launch_syrk_mfma_grouped<double>(const SyrkJobT<double> *, const int64_t *, int, int64_t, int,
                                               hipStream_t);
template void launch_syrk_mfma_grouped<float>(const SyrkJobT<float> *, const int64_t *, int, int64_t, int,
                                              hipStream_t);

template <typename T>
static void launch_syrk_t(const T *Xs, int64_t n, int64_t p, T *S, T thr, const Screen &sc, hipStream_t s)
{
    const int64_t t64 = (p + 63) / 64, t128 = (p + 127) / 128;
    const int edge = syrk_edge(t64 * (t64 + 1) / 2, t128 * (t128 + 1) / 2, sizeof(T) == 8);
    const int Tt = (int)((p + edge - 1) / edge);
    const dim3 grid((unsigned)((int64_t)Tt * (Tt + 1) / 2));
    const T invn = (T)(1.0 / (double)n);
    const int64_t pv = sc.pv > 0 ? sc.pv : p;
    if (edge == 128)
        hipLaunchKernelGGL((k_syrk<T, 128>), grid, dim3(256), 0, s, Xs, n, p, S, Tt, invn, thr, pv, sc.cnt, sc.idx);
    else if (edge == 32)
        hipLaunchKernelGGL((k_syrk<T, 32>), grid, dim3(256), 0, s, Xs, n, p, S, Tt, invn, thr, pv, sc.cnt, sc.idx);
    else
        hipLaunchKernelGGL((k_syrk<T, 64>), grid, dim3(256), 0, s, Xs, n, p, S, Tt, invn, thr, pv, sc.cnt, sc.idx);
}

void launch_syrk_f64(const double *Xs, int64_t n, int64_t p, double *S, const Screen &sc, hipStream_t s)
{
    launch_syrk_t<double>(Xs, n, p, S, sc.thr64, sc, s);
}
void launch_syrk_f32(const float *Xs, int64_t n, int64_t p, float *S, const Screen &sc, hipStream_t s)
{
    launch_syrk_t<float>(Xs, n, p, S, sc.thr32, sc, s);
}

// ---------------------------------------------------------------------------
// mixed form: bf16 split, operands in the order of split_offset (the 64 lanes
// of a wave read one 16 x 32 operand of hi or lo as 1 KB of consecutive
// memory or LDS, 16 bytes per lane, without bank conflicts)
//
// Both kernels give every entry its products in the same order (per 32
// samples lo hi, hi lo, hi hi), so S is the same to the bit whichever runs.
// ---------------------------------------------------------------------------
constexpr int kBfKC = 32;  // samples per step (one MFMA k-step)

__device__ __forceinline__ f4 bf_mma(bf8 ha, bf8 la, bf8 hb, bf8 lb, f4 c)
{
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(la, hb, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ha, lb, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(ha, hb, c, 0, 0, 0);
}

// --- 64 x 64 tiles: operands straight into registers ----------------------
// A block of four waves, each its own 32 x 32 quarter, with no LDS staging
// and no barrier: a wave keeps the loads of the next three steps (8 operands
// each) in flight behind the 12 matrix-core operations of the current one.
// Small p is bound by the latency of one tile: 25 -> 5.3 us at n = 100,
// p = 200, 37 -> 6.6 at n = 250, p = 500 and 98 -> 33 at n = 1000, p = 2000
// against 256 x 256 tiles (1, 3 and 36 of them).
constexpr int kBfSmall = 64;
typedef ScreenWaves<4, 448> BfScreen64;

__device__ __forceinline__ void bf_tile64(const uint16_t *__restrict__ split, int64_t npad, int64_t p,
                                          float *__restrict__ S, float invn, float thr, int *__restrict__ scnt,
                                          int *__restrict__ sidx, int bj, int bk, BfScreen64 &scr)
{
    constexpr int NB = 2, D = 4;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w & 1, wn = w >> 1;
    const int ks = (int)(npad / kBfKC);
    const int64_t j0 = (int64_t)bj * kBfSmall + 32 * wm, k0 = (int64_t)bk * kBfSmall + 32 * wn;
    const bool diag = bj == bk;
    int nscr = 0;
    // the wave below the diagonal of a diagonal tile has nothing to store,
    // nor has one past the last variable
    if (j0 < p && k0 < p && !(diag && wm > wn)) {
        const int64_t rbs = (p + 15) / 16;
        const bf8 *pa[NB], *pb[NB];
#pragma unroll
        for (int a = 0; a < NB; ++a) {
            // row blocks past the last load that one (never stored)
            const int64_t ra = j0 / 16 + a, rb = k0 / 16 + a;
            pa[a] = reinterpret_cast<const bf8 *>(split) + (ra < rbs ? ra : rbs - 1) * ks * 128;
            pb[a] = reinterpret_cast<const bf8 *>(split) + (rb < rbs ? rb : rbs - 1) * ks * 128;
        }
        f4 acc[NB][NB];
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[a][b] = f4{0, 0, 0, 0};
        bf8 ha[D][NB], la[D][NB], hb[D][NB], lb[D][NB];
        auto load = [&](int st, int d) {
            const int64_t o = (int64_t)(st < ks ? st : ks - 1) * 128;
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                ha[d][a] = (pa[a] + o)[lane];
                la[d][a] = (pa[a] + o + 64)[lane];
                hb[d][a] = (pb[a] + o)[lane];
                lb[d][a] = (pb[a] + o + 64)[lane];
            }
        };
#pragma unroll
        for (int d = 0; d < D - 1; ++d) load(d, d);
        for (int s0 = 0; s0 < ks; s0 += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                load(s0 + d + D - 1, (d + D - 1) % D);
                if (s0 + d < ks) {
#pragma unroll
                    for (int a = 0; a < NB; ++a)
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            acc[a][b] = bf_mma(ha[d][a], la[d][a], hb[d][b], lb[d][b], acc[a][b]);
                }
            }
        }
        nscr = store_tile<float, NB, NB, false, false>(acc, S, p, j0, k0, diag, invn, thr, p, scnt, sidx, scr, w);
    }
    if (lane == 0) scr.n[w] = nscr;
    __syncthreads();
    screen_flush_waves(scr, scnt, sidx);
}

__global__ __launch_bounds__(256) void k_syrk_bf16x3_64(const uint16_t *__restrict__ split, int64_t npad, int64_t p,
                                                        float *__restrict__ S, int Tt, float invn, float thr,
                                                        int *__restrict__ scnt, int *__restrict__ sidx)
{
    __shared__ BfScreen64 scr;
    int bj, bk;
    tile_of_block(Tt, &bj, &bk);
    bf_tile64(split, npad, p, S, invn, thr, scnt, sidx, bj, bk, scr);
}

// The tiles of many problems in one launch: block b (in the XCD-aware order)
// is tile b - off[d] of problem d.
__global__ __launch_bounds__(256) void k_syrk_bf16x3_64_grouped(const SyrkJob *__restrict__ tab,
                                                                const int64_t *__restrict__ off, int nd)
{
    __shared__ BfScreen64 scr;
    const int64_t g = xcd_order(gridDim.x, blockIdx.x);
    const int d = group_of(off, nd, g);
    const SyrkJob &J = tab[d];
    int bj, bk;
    tri_tile(J.Tt, g - off[d], &bj, &bk);
    bf_tile64(J.split, J.npad, J.p, J.S, J.invn, J.thr, J.scnt, J.sidx, bj, bk, scr);
}

// --- 256 x 256 tiles: two LDS stages, operands one block ahead -------------
// A block of 8 waves (64 x 128 each); a stage holds the operands of 32
// samples of the tile's 256 row and 256 column variables (64 KB, copied by
// the direct global-to-LDS path).  Within a stage a wave keeps the operands
// of the next column block in flight behind the 12 matrix-core operations of
// the current one.  The one barrier of a stage stands before its last two
// column blocks, whose operands are already in registers: past it every wave
// is done with the stage's LDS, the next stage's copies (issued a whole
// stage earlier) have landed, the copies after that are issued into the
// freed buffer, and the first operands of the next stage are read behind the
// remaining 24 operations.  Reading all operands of a stage behind its
// barrier took 61 us at n = 400, p = 5000 and 1462 at n = 1000, p = 20000
// (no screen); this order takes 53.5 and 1310 (3 n p^2 bf16 operations in
// the latter: 0.92 PFLOP/s), the stores of S being about a third of it.
constexpr int kBfTile = 256;
constexpr int kBfPanel = kBfTile * kBfKC * 4;  // 32 KB: 16 blocks of 16 variables, hi and lo
constexpr int kBfStage = 2 * kBfPanel;
typedef ScreenWaves<8, 448> BfScreen;          // fills the LDS left by the two stages
constexpr int kBfLds = 2 * kBfStage + (int)sizeof(BfScreen);
static_assert(kBfLds <= 160 * 1024, "LDS of one block");

// Issue the copies of one stage.  A diagonal tile copies its one panel only.
// Row blocks past the last load that one (those results are never stored).
__device__ __forceinline__ void bf_issue(const uint16_t *__restrict__ split, int ks, int64_t rbs, int64_t rj,
                                         int64_t rk, int st, bool diag, unsigned char *stage)
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // wave wv copies row blocks wv and wv + 8 of each panel, hi and lo
    const int npan = diag ? 1 : 2;
    for (int pnl = 0; pnl < npan; ++pnl)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int g = wv + 8 * h;
            int64_t rb = (pnl ? rk : rj) + g;
            rb = rb < rbs ? rb : rbs - 1;
            const uint16_t *src = split + (rb * ks + st) * 1024 + lane * 8;
#pragma unroll
            for (int part = 0; part < 2; ++part)
                __builtin_amdgcn_global_load_lds(
                    src + part * 512,
                    (__attribute__((address_space(3))) void *)(stage + pnl * kBfPanel + g * 2048 + part * 1024), 16,
                    0, 0);
        }
}

// One 256 x 256 tile (bj, bk) of one problem's S, by the whole block.
template <bool NT>
__device__ __forceinline__ void bf_tile256(const uint16_t *__restrict__ split, int64_t npad, int64_t p,
                                           float *__restrict__ S, float invn, float thr, int *__restrict__ scnt,
                                           int *__restrict__ sidx, int bj, int bk, unsigned char *bf_lds)
{
    BfScreen &scr = *reinterpret_cast<BfScreen *>(bf_lds + 2 * kBfStage);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w & 3, wn = w >> 2;
    const int ks = (int)(npad / kBfKC);  // even
    const int64_t rbs = (p + 15) / 16;
    const int64_t j0 = (int64_t)bj * kBfTile, k0 = (int64_t)bk * kBfTile;
    const bool diag = bj == bk;
    f4 acc[4][8];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[a][b] = f4{0, 0, 0, 0};
    const unsigned char *const la0 = bf_lds + wm * 8192 + lane * 16;
    const unsigned char *const lb0 = bf_lds + (diag ? 0 : kBfPanel) + wn * 16384 + lane * 16;
    bf8 ha[2][4], la[2][4], hb[4], lb[4];
    auto read_a = [&](int buf) {
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            ha[buf][a] = *reinterpret_cast<const bf8 *>(la0 + buf * kBfStage + a * 2048);
            la[buf][a] = *reinterpret_cast<const bf8 *>(la0 + buf * kBfStage + a * 2048 + 1024);
        }
    };
    auto read_b = [&](int buf, int b, int slot) {
        hb[slot] = *reinterpret_cast<const bf8 *>(lb0 + buf * kBfStage + b * 2048);
        lb[slot] = *reinterpret_cast<const bf8 *>(lb0 + buf * kBfStage + b * 2048 + 1024);
    };
    auto mul = [&](int buf, int b, int slot) {
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[a][b] = bf_mma(ha[buf][a], la[buf][a], hb[slot], lb[slot], acc[a][b]);
    };
    __syncthreads();  // the previous tile's flush is done with the LDS
    bf_issue(split, ks, rbs, j0 / 16, k0 / 16, 0, diag, bf_lds);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    bf_issue(split, ks, rbs, j0 / 16, k0 / 16, 1, diag, bf_lds + kBfStage);
    read_a(0);
    read_b(0, 0, 0);
    for (int s0 = 0; s0 < ks; s0 += 2) {
#pragma unroll
        for (int cur = 0; cur < 2; ++cur) {
            // blocks b = 0 .. 5 in slots 0 and 1, 6 and 7 in slots 2 and 3
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                if (b < 5) {
                    read_b(cur, b + 1, (b + 1) & 1);
                } else {
                    read_b(cur, 6, 2);
                    read_b(cur, 7, 3);
                }
                __builtin_amdgcn_sched_barrier(0);
                mul(cur, b, b & 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (s0 + cur + 1 < ks) {
                // this wave's reads of the stage are done and its copies of
                // the next have landed; past the barrier every wave's are
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                if (s0 + cur + 2 < ks)
                    bf_issue(split, ks, rbs, j0 / 16, k0 / 16, s0 + cur + 2, diag, bf_lds + cur * kBfStage);
                read_a(cur ^ 1);
                read_b(cur ^ 1, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            mul(cur, 6, 2);
            mul(cur, 7, 3);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const int nscr = store_tile<float, 4, 8, NT, false>(acc, S, p, j0 + 64 * wm, k0 + 128 * wn, diag, invn, thr, p, scnt,
                                                 sidx, scr, w);
    if (lane == 0) scr.n[w] = nscr;
    __syncthreads();
    screen_flush_waves(scr, scnt, sidx);
}

template <bool NT>
__global__ __launch_bounds__(512) void k_syrk_bf16x3_256(const uint16_t *__restrict__ split, int64_t npad, int64_t p,
                                                         float *__restrict__ S, int Tt, float invn, float thr,
                                                         int *__restrict__ scnt, int *__restrict__ sidx)
{
    extern __shared__ __align__(16) unsigned char bf_lds[];
    const int64_t ntiles = (int64_t)Tt * (Tt + 1) / 2;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        int bj, bk;
        tri_tile(Tt, t, &bj, &bk);
        bf_tile256<NT>(split, npad, p, S, invn, thr, scnt, sidx, bj, bk, bf_lds);
    }
}

__global__ __launch_bounds__(512) void k_syrk_bf16x3_256_grouped(const SyrkJob *__restrict__ tab,
                                                                 const int64_t *__restrict__ off, int nd)
{
    extern __shared__ __align__(16) unsigned char bf_lds[];
    const int64_t total = off[nd];
    for (int64_t g = blockIdx.x; g < total; g += gridDim.x) {
        const int d = group_of(off, nd, g);
        const SyrkJob &J = tab[d];
        int bj, bk;
        tri_tile(J.Tt, g - off[d], &bj, &bk);
        bf_tile256<false>(J.split, J.npad, J.p, J.S, J.invn, J.thr, J.scnt, J.sidx, bj, bk, bf_lds);
    }
}

// Tile edge from the number of 256 x 256 tiles of the launch: both kernels
// take 84 us at n = 1000, p = 4000 (136 of them); with 120 the 64 x 64 tiles
// take 43 us against 49 (n = 400, p = 3700), with 210 they take 73 against
// 54 (n = 400, p = 5000).  A batch's tiles are of many sizes (most of a small
// problem's large tile is padding, and the launch ends on the longest), so
// its large tiles have to come to two rounds of the chip.
int syrk_bf16x3_edge(int64_t tiles256, bool grouped)
{
    return tiles256 >= (grouped ? 512 : 144) ? kBfTile : kBfSmall;
}

SyrkJob syrk_job_bf16x3(const uint16_t *split, int64_t n, int64_t npad, int64_t p, float *S, const Screen &sc,
                        int edge, int64_t *tiles)
{
    SyrkJob j{};
    j.split = split;
    j.npad = npad;
    j.p = p;
    j.S = S;
    j.Tt = (int)((p + edge - 1) / edge);
    j.invn = (float)(1.0 / (double)n);
    j.thr = sc.thr32;
    j.scnt = sc.cnt;
    j.sidx = sc.idx;
    *tiles = (int64_t)j.Tt * (j.Tt + 1) / 2;
    return j;
}

// 256 x 256 tiles: one block per CU (LDS and registers), at most one per tile
static unsigned bf_grid256(int64_t tiles) { return (unsigned)(tiles < 256 ? tiles : 256); }

void launch_syrk_bf16x3_grouped(const SyrkJob *tab, const int64_t *tile_off, int nd, int64_t tiles, int edge,
                                hipStream_t s)
{
    if (tiles <= 0) return;
    if (edge == kBfTile)
        hipLaunchKernelGGL(k_syrk_bf16x3_256_grouped, dim3(bf_grid256(tiles)), dim3(512), kBfLds, s, tab, tile_off,
                           nd);
    else
        hipLaunchKernelGGL(k_syrk_bf16x3_64_grouped, dim3((unsigned)tiles), dim3(256), 0, s, tab, tile_off, nd);
}

void launch_syrk_bf16x3(const uint16_t *split, int64_t n, int64_t npad, int64_t p, float *S, const Screen &sc,
                        hipStream_t s)
{
    const int64_t t256 = (p + kBfTile - 1) / kBfTile;
    const int edge = syrk_bf16x3_edge(t256 * (t256 + 1) / 2, false);
    const int Tt = (int)((p + edge - 1) / edge);
    const int64_t tiles = (int64_t)Tt * (Tt + 1) / 2;
    const float invn = (float)(1.0 / (double)n);
    // an S larger than the 256 MB memory-side cache is stored past it (with
    // ordinary stores p = 20000 takes 2% longer, and the pass that reads S
    // next 5%; a smaller S is better left in the cache)
    const bool nt = 4 * p * p > (int64_t)256 << 20;
    if (edge == kBfTile && nt)
        hipLaunchKernelGGL(k_syrk_bf16x3_256<true>, dim3(bf_grid256(tiles)), dim3(512), kBfLds, s, split, npad, p, S,
                           Tt, invn, sc.thr32, sc.cnt, sc.idx);
    else if (edge == kBfTile)
        hipLaunchKernelGGL(k_syrk_bf16x3_256<false>, dim3(bf_grid256(tiles)), dim3(512), kBfLds, s, split, npad, p, S,
                           Tt, invn, sc.thr32, sc.cnt, sc.idx);
    else
        hipLaunchKernelGGL(k_syrk_bf16x3_64, dim3((unsigned)tiles), dim3(256), 0, s, split, npad, p, S, Tt, invn,
                           sc.thr32, sc.cnt, sc.idx);
}

} // namespace spmesl
