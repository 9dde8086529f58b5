// lbfgs.hip -- limited-memory BFGS helpers of the outer inversion loop
// (include/seisgrad.h: lbfgs_push, lbfgs_direction).
//
// The paper's inversions use L-BFGS-B (Applications, FWI); here the bounds
// are kept by clipping the model after each step and the direction is the
// two-loop recursion (Nocedal & Wright, Algorithm 7.4).  Models of a batch
// keep separate histories; every inner product is an FP64 reduction in a
// fixed order, so the direction is bitwise reproducible.
#include "../../include/seisgrad.h"
#include "sg_error.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <initializer_list>
#include <type_traits>

using sg::fail;

namespace {

constexpr int LB_THREADS = 1024;
constexpr int LB_MAXMEM = 64;
constexpr int LB_CHUNKS = 256;   // workgroups per model of the partial sums, at most
constexpr int PUSH_ONE = 24 * LB_THREADS;   // elements up to which one workgroup forms a pair
constexpr long long MAX_THREADS = (1ll << 32) - 1;   // of a launch's grid
static_assert(LB_CHUNKS <= LB_THREADS && 4 * LB_CHUNKS <= PUSH_ONE, "partial sums fit");

// v of another lane of the wavefront (DPP control CTRL), 0 where there is none
// or the row of 16 lanes is not in the mask ROWS.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double v)
{
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xf, true);
    return __longlong_as_double((long long)(unsigned)lo | (long long)hi << 32);
}
__device__ __forceinline__ double lane_of(double v, int l)
{
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)u, l), hi = __builtin_amdgcn_readlane((int)(u >> 32), l);
    return __longlong_as_double((long long)(unsigned)lo | (long long)hi << 32);
}
// Sum over a row of 16 lanes, in its last lane.
__device__ __forceinline__ double row_sum(double v)
{
    v += dpp<0x111, 0xf>(v);               // row_shr 1, 2, 4, 8
    v += dpp<0x112, 0xf>(v);
    v += dpp<0x114, 0xf>(v);
    return v + dpp<0x118, 0xf>(v);
}

// Sums of N doubles per thread of a workgroup of LB_THREADS in a fixed order;
// every thread gets them.  One barrier: another must follow before red is used
// again.  (Lanes are added by DPP, off the LDS pipe: with a shuffle per step
// and every thread adding up the 16 wavefronts, 2000 models of 500 elements
// took 94 us for a direction of 5 pairs, with a tree in LDS 80, now 56.)
template <int N>
__device__ __forceinline__ void block_sums(double (&v)[N], double (*red)[LB_THREADS / 64])
{
    static_assert(LB_THREADS / 64 == 16 && N <= 4, "a row of lanes holds the wavefronts' sums");
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        double t = row_sum(v[k]);
        t += dpp<0x142, 0xa>(t);           // row_bcast 15: row 0 into 1, 2 into 3
        t += dpp<0x143, 0xc>(t);           // row_bcast 31: rows 0 and 1 into 2 and 3
        if (lane == 63) red[k][threadIdx.x >> 6] = t;
    }
    __syncthreads();
    const double t = row_sum(lane < 16 * N ? red[lane >> 4][lane & 15] : 0.0);
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = lane_of(t, 16 * k + 15);
}

// A model's vectors are only 4-byte aligned (n may be odd): doubles in two words.
__device__ __forceinline__ void put_f64(float *p, double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    p[0] = __uint_as_float((unsigned)u);
    p[1] = __uint_as_float((unsigned)(u >> 32));
}
__device__ __forceinline__ double get_f64(const float *p)
{
    return __longlong_as_double((long long)(__float_as_uint(p[0]) | (unsigned long long)__float_as_uint(p[1]) << 32));
}

// s, y of the models that store a pair, and their sums (y.s, y.y).  Elements
// are loaded NL at a time, the last ones as far as there are any (with ten loads
// per thread whatever n is, clamped to the last element, 2000 models of 500 elements
// took 24 us, one element at a time 12, now 7.6; 20 of 10201, from memory, 9.5 / 9.8 / 8.4).  ONE: one workgroup per model, which
// writes the sums.  Otherwise nb workgroups per model leave their two partial
// sums in the first 4 nb elements of the stored y, which lbfgs_pair_kernel
// adds up and then replaces by the elements (so the inputs may not lie in S or Y).
template <bool ONE>
__global__ __launch_bounds__(LB_THREADS) void lbfgs_push_kernel(int nmodels, long long n, int mem, int nb,
                                                                const int *slot, const float *m_new,
                                                                const float *m_old, const float *g_new,
                                                                const float *g_old, float *S, float *Y, double *ysyy)
{
    constexpr int NL = 4;
    __shared__ double red[2][LB_THREADS / 64];
    const int b = ONE ? blockIdx.x : blockIdx.x / nb, blk = ONE ? 0 : blockIdx.x - b * nb;
    const int k = slot[b];
    if (k < 0 || k >= mem) return;                 // this model keeps its history unchanged
    const long long o = (long long)b * n, step = (ONE ? 1 : nb) * (long long)(NL * LB_THREADS);
    float *s = S + ((long long)k * nmodels + b) * n, *y = Y + ((long long)k * nmodels + b) * n;
    double sum[2] = {0.0, 0.0};
    // NL elements from i0 on, or (TAIL) those of them below n
    auto run = [&](long long i0, auto TAIL) {
        constexpr bool tail = decltype(TAIL)::value;
        float mn[NL], mo[NL], gn[NL], go[NL];
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const long long i = i0 + j * LB_THREADS;
            if (!tail || i < n) {
                mn[j] = m_new[o + i]; mo[j] = m_old[o + i]; gn[j] = g_new[o + i]; go[j] = g_old[o + i];
            }
        }
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const long long i = i0 + j * LB_THREADS;
            if (!tail || i < n) {
                const float si = mn[j] - mo[j], yi = gn[j] - go[j];
                s[i] = si;
                if (ONE || i >= 4 * nb) y[i] = yi;
                sum[0] += (double)yi * si;
                sum[1] += (double)yi * yi;
            }
        }
    };
    long long i0 = blk * (long long)(NL * LB_THREADS) + threadIdx.x;
    for (; i0 + (NL - 1) * LB_THREADS < n; i0 += step) run(i0, std::false_type());
    if (i0 < n) run(i0, std::true_type());
    block_sums(sum, red);
    if (threadIdx.x == 0) {
        if constexpr (ONE) {
            ysyy[2 * ((long long)k * nmodels + b)] = sum[0];
            ysyy[2 * ((long long)k * nmodels + b) + 1] = sum[1];
        } else {
            put_f64(y + 4 * blk, sum[0]);
            put_f64(y + 4 * blk + 2, sum[1]);
        }
    }
}

// The sums of the pairs just formed from their nb <= LB_THREADS partial sums,
// then the elements of y that held them; one workgroup per model.
__global__ __launch_bounds__(LB_THREADS) void lbfgs_pair_kernel(int nmodels, long long n, int mem, int nb,
                                                                const int *slot, const float *g_new,
                                                                const float *g_old, float *Y, double *ysyy)
{
    __shared__ double red[2][LB_THREADS / 64];
    const int b = blockIdx.x;
    const int k = slot[b];
    if (k < 0 || k >= mem) return;
    const long long o = (long long)b * n;
    float *y = Y + ((long long)k * nmodels + b) * n;
    const int t = threadIdx.x;
    double sum[2] = {t < nb ? get_f64(y + 4 * t) : 0.0, t < nb ? get_f64(y + 4 * t + 2) : 0.0};
    block_sums(sum, red);                 // its barrier: every partial sum has been read
    for (int i = t; i < 4 * nb; i += LB_THREADS) y[i] = g_new[o + i] - g_old[o + i];
    if (t == 0) {
        ysyy[2 * ((long long)k * nmodels + b)] = sum[0];
        ysyy[2 * ((long long)k * nmodels + b) + 1] = sum[1];
    }
}

// ---------------------------------------------------- direction over the chip
// The two-loop recursion needs q only in inner products with the stored
// vectors, so with the products of the vectors among themselves and with g
// in hand it runs on scalars (FP64):
//   s_i.q_i = s_i.g - sum_{j newer} alpha_j s_i.y_j
//   y_i.r_i = gamma (y_i.g - sum_j alpha_j y_i.y_j) + sum_{j older} (alpha_j - beta_j) y_i.s_j
// and p = -(gamma (g - sum alpha_j y_j) + sum (alpha_j - beta_j) s_j).  The
// vectors are read twice, by every CU, instead of once per loop step by one
// workgroup whose every step waits for the reduction before it (push +
// direction, 8 pairs: 20 models of 10201 elements 77 -> 25 us, 200 models 129 ->
// 78 us, one model of 500000 4.82 ms -> 68 us).
// The products are summed per chunk of elements and then over the chunks in
// order.  The partial sums and then the coefficients live in p, which is
// written last: the coefficients in its first LB_HEAD floats, whose elements
// the workgroup forms that reads them last (a count of those that have read
// them lies behind them; as a launch of its own 3.7 us).
constexpr int LB_CMAX = 15;      // pairs: the columns (y of each, g) fill one matrix tile, the rows two
constexpr int LB_SUB = 512;      // chunks are multiples of this many elements
constexpr int LB_GT = 256;
constexpr int LB_HEAD = 64;      // floats
static_assert(2 * (2 * LB_CMAX + 1) < LB_HEAD, "the coefficients and the count fit the head");

// Products of c pairs, newest first: s_i.g, y_i.g, then for j < i (j newer) s_i.y_j and y_i.y_j.
__host__ __device__ constexpr int lb_dots(int c) { return c * c + c; }
__device__ __forceinline__ int lb_sg(int i) { return 2 * i; }
__device__ __forceinline__ int lb_yg(int i) { return 2 * i + 1; }
__device__ __forceinline__ int lb_sy(int c, int i, int j) { return 2 * c + i * (i - 1) + 2 * j; }
__device__ __forceinline__ int lb_yy(int c, int i, int j) { return lb_sy(c, i, j) + 1; }

struct LbHist {
    int newest, count;
    __device__ LbHist(const int *hist, int b, int mem)
    {
        newest = hist[2 * b + 1];
        count = (newest < 0 || newest >= mem) ? 0 : max(0, min(hist[2 * b], mem));
    }
    __device__ int slot(int j, int mem) const { return (newest - j + mem) % mem; }   // j = 0: newest
};

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // a vector's elements are 4-byte aligned

// One chunk of one model: its share of every product, on the FP64 matrix
// cores: rows (s, y by pair, 16 per tile) times columns (y by pair, then g),
// K = elements.  A wavefront takes every fourth run of 16 LB_U elements; lane
// (row or column l mod 16, l / 16) loads four neighbouring elements of each 16
// and gives them to four instructions (both operands the same elements, so
// their order within K is free).  The four wavefronts' sums are added in
// turn.  (Products formed one after another on staged vectors: 20 us against
// the 3 us of the loads for 20 models of 10201, 8 pairs.)
constexpr int LB_U = 4;
template <int TILES>
__global__ __launch_bounds__(LB_GT) void lbfgs_products_kernel(int nmodels, long long n, int mem, int nchunks,
                                                               long long chunk, const int *hist, const float *S,
                                                               const float *Y, const float *g, float *p)
{
    constexpr int WAVES = LB_GT / 64;
    __shared__ double part[WAVES][TILES * 16][17];
    const int b = blockIdx.x / nchunks, ch = blockIdx.x - b * nchunks;
    const LbHist h(hist, b, mem);
    const int c = h.count;
    const long long o = (long long)b * n;
    const long long lo = ch * chunk, hi = min(n, lo + chunk);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int rc = lane & 15, kk = lane >> 4;
    // vector q of the products (2 pair: s, 2 pair + 1: y, 2 c: g); g for an unused row or column
    auto vec = [&](int q) {
        return q >= 2 * c ? g + o : (q & 1 ? Y : S) + ((long long)h.slot(q >> 1, mem) * nmodels + b) * n;
    };
    const float *A[TILES], *B = vec(min(2 * rc + 1, 2 * c));
    f64x4 acc[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        A[t] = vec(16 * t + rc);
        acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    }
    for (long long e0 = lo + wv * 16 * LB_U; e0 < hi; e0 += WAVES * 16 * LB_U) {
        f32x4u xa[TILES][LB_U], xb[LB_U];
        if (e0 + 16 * LB_U <= hi) {
#pragma unroll
            for (int u = 0; u < LB_U; ++u) {
                const long long e = e0 + 16 * u + 4 * kk;
                xb[u] = *reinterpret_cast<const f32x4u *>(B + e);
#pragma unroll
                for (int t = 0; t < TILES; ++t) xa[t][u] = *reinterpret_cast<const f32x4u *>(A[t] + e);
            }
        } else {                          // the end of the chunk: elements past it are zero
#pragma unroll
            for (int u = 0; u < LB_U; ++u)
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const long long e = e0 + 16 * u + 4 * kk + m, ec = min(e, hi - 1);
                    const float bv = B[ec];
                    xb[u][m] = e < hi ? bv : 0.f;
#pragma unroll
                    for (int t = 0; t < TILES; ++t) {
                        const float av = A[t][ec];
                        xa[t][u][m] = e < hi ? av : 0.f;
                    }
                }
        }
#pragma unroll
        for (int u = 0; u < LB_U; ++u)
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int t = 0; t < TILES; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)xa[t][u][m], (double)xb[u][m], acc[t], 0, 0, 0);
    }
    // register m of lane (column rc, kk) holds row 4 m + kk
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int m = 0; m < 4; ++m) part[wv][16 * t + 4 * m + kk][rc] = acc[t][m];
    __syncthreads();
    float *out = p + o + LB_HEAD + 2ll * ch * lb_dots(mem);
    auto put = [&](int d, int row, int col) {
        double t = 0.0;
        for (int w = 0; w < WAVES; ++w) t += part[w][row][col];
        put_f64(out + 2 * d, t);
    };
    for (int q = threadIdx.x; q < 2 * c * (c + 1); q += LB_GT) {
        const int row = q / (c + 1), j = q - row * (c + 1), i = row >> 1;
        if (j == c) put(row & 1 ? lb_yg(i) : lb_sg(i), row, c);
        else if (j < i) put(row & 1 ? lb_yy(c, i, j) : lb_sy(c, i, j), row, j);
    }
}

// The scalar recursion of one model; coefficients of g, then of (s, y) by
// pair.  Eight lanes add up a product's chunks (l, l + 8, ..), then the
// lanes in turn; in the recursion lane i carries pair i.
__global__ __launch_bounds__(LB_THREADS) void lbfgs_scalars_kernel(int nmodels, long long n, int mem, int nchunks,
                                                                   const int *hist, const double *ysyy, float *p)
{
    constexpr int NL = 8;
    __shared__ double dot[lb_dots(LB_CMAX)];
    const int b = blockIdx.x;
    const LbHist h(hist, b, mem);
    const int c = h.count, nd = lb_dots(c);
    float *pm = p + (long long)b * n;
    for (int d0 = 0; d0 < nd; d0 += LB_THREADS / 8) {
        const int d = d0 + (int)(threadIdx.x >> 3), l = threadIdx.x & 7;
        const float *src = pm + LB_HEAD + 2ll * min(d, nd - 1);
        double t = 0.0;
        for (int q0 = l; q0 < nchunks; q0 += 8 * NL) {
            double x[NL];
#pragma unroll
            for (int q = 0; q < NL; ++q)
                x[q] = q0 + 8 * q < nchunks ? get_f64(src + 2ll * (q0 + 8 * q) * lb_dots(mem)) : 0.0;
#pragma unroll
            for (int q = 0; q < NL; ++q) t += x[q];
        }
        double sum = 0.0;
        for (int q = 0; q < 8; ++q) sum += __shfl(t, q, 8);
        if (l == 0 && d < nd) dot[d] = sum;
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int i = threadIdx.x, ic = min(i, max(c - 1, 0));
    double ys = 1.0, yy = 1.0;
    if (i < c) {
        const long long k = (long long)h.slot(i, mem) * nmodels + b;
        ys = ysyy[2 * k];
        yy = ysyy[2 * k + 1];
    }
    const double gamma = c > 0 ? __shfl(ys, 0, 64) / __shfl(yy, 0, 64) : 1.0;
    double t = c > 0 ? dot[lb_sg(ic)] : 0.0, al = 0.0, u = c > 0 ? dot[lb_yg(ic)] : 0.0, cs = 0.0;
    for (int j = 0; j < c; ++j) {
        if (i == j) al = t / ys;
        const double aj = __shfl(al, j, 64);
        if (i > j && i < c) t -= aj * dot[lb_sy(c, ic, j)];
        if (i < c) u -= aj * (i == j ? yy : i > j ? dot[lb_yy(c, ic, j)] : dot[lb_yy(c, j, ic)]);
    }
    u *= gamma;
    for (int j = c - 1; j >= 0; --j) {
        if (i == j) cs = al - u / ys;
        const double cj = __shfl(cs, j, 64);
        if (i < j) u += cj * dot[lb_sy(c, j, ic)];
    }
    if (i == 0) {
        put_f64(pm, -gamma);
        pm[LB_HEAD - 1] = __uint_as_float(0u);
    }
    if (i < c) {
        put_f64(pm + 2 + 4 * i, -cs);
        put_f64(pm + 4 + 4 * i, gamma * al);
    }
}

// p: nb workgroups per model the elements after the head, the last of them to
// have read the coefficients then the head.  (Which one that is does not
// change a value.)
__global__ __launch_bounds__(LB_GT) void lbfgs_combine_kernel(int nmodels, long long n, int mem, int nb,
                                                              const int *hist, const float *S, const float *Y,
                                                              const float *g, float *p)
{
    __shared__ double co[2 * LB_CMAX + 1];
    __shared__ unsigned before;
    const int b = blockIdx.x / nb;
    const LbHist h(hist, b, mem);
    const int c = h.count;
    const long long o = (long long)b * n;
    float *pm = p + o;
    if ((int)threadIdx.x < 2 * c + 1) co[threadIdx.x] = get_f64(pm + 2 * threadIdx.x);
    __syncthreads();                      // the coefficients have been read
    if (threadIdx.x == 0)
        before = __hip_atomic_fetch_add(reinterpret_cast<unsigned *>(pm + LB_HEAD - 1), 1u, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
    auto element = [&](long long i) {
        double t = co[0] * g[o + i];
#pragma unroll 4
        for (int j = 0; j < c; ++j) {
            const long long k = ((long long)h.slot(j, mem) * nmodels + b) * n + i;
            t += co[1 + 2 * j] * S[k];
            t += co[2 + 2 * j] * Y[k];
        }
        pm[i] = (float)t;
    };
    for (long long i = LB_HEAD + (blockIdx.x - b * nb) * (long long)LB_GT + threadIdx.x; i < n; i += nb * (long long)LB_GT)
        element(i);
    __syncthreads();
    if (before == (unsigned)nb - 1 && threadIdx.x < LB_HEAD) element(threadIdx.x);
}

// p = -H g for model b over hist[2b] pairs ending at ring slot hist[2b+1];
// p holds q, then r, in place.
__global__ __launch_bounds__(LB_THREADS) void lbfgs_direction_kernel(int nmodels, long long n, int mem,
                                                                     const int *hist, const float *S,
                                                                     const float *Y, const double *ysyy,
                                                                     const float *g, float *p)
{
    __shared__ double red[1][LB_THREADS / 64];
    __shared__ double alpha[LB_MAXMEM];
    const int b = blockIdx.x;
    const int newest = hist[2 * b + 1];
    const int count = (newest < 0 || newest >= mem) ? 0 : max(0, min(hist[2 * b], mem));
    const long long o = (long long)b * n;
    float *q = p + o;
    for (long long i = threadIdx.x; i < n; i += LB_THREADS) q[i] = g[o + i];
    __syncthreads();
    auto slot_of = [&](int j) { return (newest - j + mem) % mem; };   // j = 0: newest
    for (int j = 0; j < count; ++j) {
        const int k = slot_of(j);
        const float *s = S + ((long long)k * nmodels + b) * n, *y = Y + ((long long)k * nmodels + b) * n;
        double sq[1] = {0.0};
        for (long long i = threadIdx.x; i < n; i += LB_THREADS) sq[0] += (double)s[i] * q[i];
        block_sums(sq, red);
        const double a = sq[0] / ysyy[2 * ((long long)k * nmodels + b)];
        if (threadIdx.x == 0) alpha[j] = a;
        const float af = (float)a;
        for (long long i = threadIdx.x; i < n; i += LB_THREADS) q[i] -= af * y[i];
        __syncthreads();
    }
    float gamma = 1.f;
    if (count > 0) {
        const long long k = slot_of(0);
        gamma = (float)(ysyy[2 * (k * nmodels + b)] / ysyy[2 * (k * nmodels + b) + 1]);
    }
    for (long long i = threadIdx.x; i < n; i += LB_THREADS) q[i] *= gamma;
    __syncthreads();
    for (int j = count - 1; j >= 0; --j) {
        const int k = slot_of(j);
        const float *s = S + ((long long)k * nmodels + b) * n, *y = Y + ((long long)k * nmodels + b) * n;
        double yr[1] = {0.0};
        for (long long i = threadIdx.x; i < n; i += LB_THREADS) yr[0] += (double)y[i] * q[i];
        block_sums(yr, red);
        const double beta = yr[0] / ysyy[2 * ((long long)k * nmodels + b)];
        const float c = (float)(alpha[j] - beta);
        for (long long i = threadIdx.x; i < n; i += LB_THREADS) q[i] += c * s[i];
        __syncthreads();
    }
    for (long long i = threadIdx.x; i < n; i += LB_THREADS) q[i] = -q[i];
}

// Is the direction of c pairs faster by products over the whole chip than by
// one workgroup per model?  Estimates in us fitted to 1 .. 4000 models of 600 ..
// 500000 elements.  The loop: a chain of reductions per pair and model, about
// 400 models at a time, and its traffic, from memory once the vectors of the
// models at work exceed the last-level cache.  The products: three launches, and the
// FP64 matrix cores' rate, which has one of few pairs pay for 16 columns.
// Measured, loop / products, by models x elements and pairs: 1 x 2000, 3 10.4 / 12.3,
// 5 14.6 / 12.9; 20 x 10201, 8 47 / 15; 200 x 10000, 2 30.5 / 44.9; 100 x 20000, 1 30 / 43,
// 5 117 / 53; 1000 x 40000, 1 392 / 620; 1000 x 6000, 5 145 / 149; 1000 x 2000, 8 80 / 77;
// 400 x 20000, 5 292 / 192; 1000 x 3000, 15 241 / 198; 1 x 500000, 1 729 / 41.
bool products_faster(int nmodels, long long n, int c)
{
    const double e = 1e-5 * nmodels * n;
    const bool cached = (2.0 * c + 2.0) * 4.0 * std::min(nmodels, 512) * n <= 128e6;
    const double per_element = 0.6e-3 * std::min(2.4, 1.0 + n / 60000.0);
    const double loop = 1.06 * (3.0 + c * (1.0 + per_element * n)) * std::max(1.0, nmodels / 400.0) +
                        e * (cached ? 0.3 + 0.13 * c : 0.5 + 0.45 * c);
    const double products = 12.0 + 6e-3 * nmodels + (c > 8 ? 6.0 + e * (1.0 + 0.33 * c) : e * (1.25 + 0.2 * c));
    return products < loop;
}

// Do n floats at a and m at b share memory?
bool overlap(const float *a, long long n, const float *b, long long m)
{
    return (uintptr_t)a < (uintptr_t)(b + m) && (uintptr_t)b < (uintptr_t)(a + n);
}

} // namespace

extern "C" {

int lbfgs_push(int32_t nmodels, int64_t n, int32_t mem, const int32_t *slot, const float *m_new,
               const float *m_old, const float *g_new, const float *g_old, float *S, float *Y, double *ysyy,
               sg_stream_t stream)
{
    if (nmodels < 1 || n < 1 || mem < 1 || mem > LB_MAXMEM)
        return fail(SG_EINVAL, "need nmodels, n >= 1 and 1 <= mem <= %d", LB_MAXMEM);
    if (!slot || !m_new || !m_old || !g_new || !g_old || !S || !Y || !ysyy)
        return fail(SG_EINVAL, "NULL pointer argument");
    hipStream_t st = (hipStream_t)stream;
    // Up to PUSH_ONE elements one workgroup per model forms the pair and its sums
    // (models x elements, inputs in the L2 / in memory, us, one workgroup / several:
    // 1 x 20000 6.2 / 8.4, 7.4 / 7.7; 200 x 20000 16.2 / 19.3, 23.3 / 25.7; 20 x 40000
    // 11.3 / 8.6, 21.7 / 9.7; 200 x 40000 30.5 / 32.0, 43.9 / 43.2; 2 x 500000 128 / 8.6,
    // 215 / 10.6).  So do pairs formed in place, in an S or Y that holds one of the
    // inputs: the partial sums of several workgroups and their replacement would read
    // what they have overwritten.
    bool in_place = false;
    for (const float *in : {m_new, m_old, g_new, g_old})
        for (const float *out : {S, Y})
            in_place |= overlap(in, (long long)nmodels * n, out, (long long)mem * nmodels * n);
    const int nb = (int)std::min<long long>((n + 4 * LB_THREADS - 1) / (4 * LB_THREADS), LB_CHUNKS);
    if (n <= PUSH_ONE || (long long)nmodels * nb * LB_THREADS > MAX_THREADS || in_place) {
        lbfgs_push_kernel<true><<<nmodels, LB_THREADS, 0, st>>>(nmodels, n, mem, 1, slot, m_new, m_old, g_new, g_old,
                                                                S, Y, ysyy);
    } else {
        lbfgs_push_kernel<false><<<nmodels * nb, LB_THREADS, 0, st>>>(nmodels, n, mem, nb, slot, m_new, m_old, g_new,
                                                                      g_old, S, Y, ysyy);
        lbfgs_pair_kernel<<<nmodels, LB_THREADS, 0, st>>>(nmodels, n, mem, nb, slot, g_new, g_old, Y, ysyy);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(SG_EDEVICE, "lbfgs_push launch: %s", hipGetErrorString(e));
    return SG_OK;
}

int lbfgs_direction(int32_t nmodels, int64_t n, int32_t mem, const int32_t *hist, const float *S, const float *Y,
                    const double *ysyy, const float *g, float *p, sg_stream_t stream)
{
    if (nmodels < 1 || n < 1 || mem < 1 || mem > LB_MAXMEM)
        return fail(SG_EINVAL, "need nmodels, n >= 1 and 1 <= mem <= %d", LB_MAXMEM);
    if (!hist || !S || !Y || !ysyy || !g || !p) return fail(SG_EINVAL, "NULL pointer argument");
    if (p == g) return fail(SG_EINVAL, "p must not alias g");
    hipStream_t st = (hipStream_t)stream;
    // The products where they are faster and p has room for two chunks' partial
    // sums; longer histories keep one workgroup per model.
    const int per = 2 * lb_dots(std::min<int>(mem, LB_CMAX));     // floats of a chunk's partial sums
    const bool room = mem <= LB_CMAX && n >= LB_HEAD + 2 * per && products_faster(nmodels, n, mem);
    const long long want = room ? std::min<long long>({(n + LB_SUB - 1) / LB_SUB, (n - LB_HEAD) / per, LB_CHUNKS}) : 1;
    const long long chunk = ((n + want - 1) / want + LB_SUB - 1) / LB_SUB * LB_SUB;
    const int nchunks = (int)((n + chunk - 1) / chunk);
    if (room && (long long)nmodels * std::max(nchunks * LB_GT, LB_THREADS) <= MAX_THREADS) {
        if (mem <= 8)
            lbfgs_products_kernel<1><<<nmodels * nchunks, LB_GT, 0, st>>>(nmodels, n, mem, nchunks, chunk, hist, S, Y, g, p);
        else
            lbfgs_products_kernel<2><<<nmodels * nchunks, LB_GT, 0, st>>>(nmodels, n, mem, nchunks, chunk, hist, S, Y, g, p);
        lbfgs_scalars_kernel<<<nmodels, LB_THREADS, 0, st>>>(nmodels, n, mem, nchunks, hist, ysyy, p);
        const int nb = (int)std::min<long long>((n - LB_HEAD + LB_GT - 1) / LB_GT, std::max(1, 16384 / nmodels));
        lbfgs_combine_kernel<<<nmodels * nb, LB_GT, 0, st>>>(nmodels, n, mem, nb, hist, S, Y, g, p);
    } else {
        lbfgs_direction_kernel<<<nmodels, LB_THREADS, 0, st>>>(nmodels, n, mem, hist, S, Y, ysyy, g, p);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(SG_EDEVICE, "lbfgs_direction launch: %s", hipGetErrorString(e));
    return SG_OK;
}

} // extern "C"
