// util.hip -- small kernels: fill, Ricker wavelet, FP64 misfit and dot
// reductions (fixed reduction order, so results are bitwise reproducible).
#include "sg_internal.h"

#include <mutex>

namespace sg {

__global__ void fill_kernel(float *p, long long n, float v)
{
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

void launch_fill(float *p, long long n, float v, hipStream_t s)
{
    if (n <= 0) return;
    const int blocks = (int)std::min<long long>((n + 255) / 256, 16384);
    fill_kernel<<<blocks, 256, 0, s>>>(p, n, v);
}

// The fields of a state to or from a checkpoint in one launch, U items of 16
// bytes in flight per thread (a copy per field: 2 us each at 101 x 101 with
// 20-cell layer, 12 us for six, now 3; 300 x 150 with 4 shots 23 -> 4.6 us; 128^3
// + 20 79 -> 55).  STREAM: more than the last-level cache holds, past it
// (400^3 + 24 952 us as copies per field, 1007 cached, 863 streamed; 128^3 + 20
// 55 cached, 64 streamed).
template <bool STREAM>
__global__ __launch_bounds__(256) void copy_fields_kernel(CopyFields c, long long n4)
{
    constexpr int U = 4;
    // pointers out of an array: their address space has to be said
    typedef float V4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(1))) V4 *Global;
    const Global src = (Global)c.src[blockIdx.y], dst = (Global)c.dst[blockIdx.y];
    const long long i0 = blockIdx.x * (256ll * U) + threadIdx.x;
    V4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const long long i = min(i0 + u * 256, n4 - 1);
        v[u] = STREAM ? __builtin_nontemporal_load(src + i) : src[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (i0 + u * 256 < n4) {
            if constexpr (STREAM) __builtin_nontemporal_store(v[u], dst + i0 + u * 256);
            else dst[i0 + u * 256] = v[u];
        }
}

void launch_copy_fields(const CopyFields &c, long long n, hipStream_t s)
{
    if (n <= 0 || c.count == 0) return;
    const long long n4 = n / 4;            // whole frame rows: a multiple of 32 floats
    const dim3 grid((unsigned)((n4 + 1023) / 1024), c.count);
    if (n4 * 16 * c.count > 256ll << 20) copy_fields_kernel<true><<<grid, 256, 0, s>>>(c, n4);
    else                                 copy_fields_kernel<false><<<grid, 256, 0, s>>>(c, n4);
}

// Fold the padded cells of 2-D models onto the physical cells that they
// replicate: each cell's sum over its padded cells in z, x order, times
// dchat/dc = 2 dt^2 c / dx^2 if cpad is given.  A workgroup per row and run of
// `cols` of the columns between the ends: all four wavefronts the columns, in the
// first run two of them, and one each end cell, whose P + 1
// (corner: (P + 1)^2) cells it loads 64 at a time and adds up lane by lane (a
// thread that loaded and added them one by one took 38 us for P = 20, 84 us
// for P = 32; now 14 and 30).  Long rows are cut so that a few of them fill the
// chip as well (16000 x 64, P = 20: a thread per cell 43 us, a workgroup per
// whole row 275, now 15).
// m0, iz0: model and row of the first workgroup.
__global__ __launch_bounds__(256) void fold2_kernel(Grid2 g, int m0, int iz0, int cols, const float *acc,
                                                    const float *cpad, double dt, double dx, float *out)
{
    constexpr int U = 8;                   // loads in flight
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const unsigned r = iz0 + blockIdx.x, dm = r / g.nz;
    const long long m = m0 + (int)dm;
    const int iz = (int)(r - dm * g.nz);
    const int zlo = iz == 0 ? 0 : iz + g.P, zhi = iz == g.nz - 1 ? g.NZ - 1 : iz + g.P;
    const float *am = acc + m * g.plane;
    auto at = [&](int pz, int px) { return (long long)(pz + OZ) * g.SX + px + OX; };
    auto store = [&](int ix, float v) {
        if (cpad) {
            const double c = cpad[m * g.plane + at(iz + g.P, ix + g.P)];
            v = (float)(2.0 * dt * dt * c / (dx * dx)) * v;
        }
        out[(m * g.nz + iz) * g.nx + ix] = v;
    };
    if (blockIdx.y > 0 || wv >= 2) {
        const int waves = blockIdx.y > 0 ? 4 : 2, x0 = 1 + blockIdx.y * cols, x1 = min(x0 + cols, g.nx - 1);
        for (int ix = x0 + (wv + waves - 4) * 64 + lane; ix < x1; ix += waves * 64) {
            float v = 0.f;
            if (zlo == zhi) v += am[at(zlo, ix + g.P)];
            else for (int p0 = zlo; p0 <= zhi; p0 += U) {
                float x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = am[at(min(p0 + u, zhi), ix + g.P)];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (p0 + u <= zhi) v += x[u];
            }
            store(ix, v);
        }
        return;
    }
    const int ix = wv ? g.nx - 1 : 0;
    if (wv && g.nx == 1) return;           // the one column is the first wavefront's
    const int xlo = ix == 0 ? 0 : ix + g.P, xhi = ix == g.nx - 1 ? g.NX - 1 : ix + g.P;
    const int nch = (xhi - xlo) / 64 + 1, items = (zhi - zlo + 1) * nch;   // runs of up to 64 cells, in order
    float v = 0.f;
    for (int q0 = 0; q0 < items; q0 += U) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = min(q0 + u, items - 1), r = q / nch, b = xlo + (q - r * nch) * 64;
            const float xv = am[at(zlo + r, min(b + lane, xhi))];
            x[u] = b + lane <= xhi ? xv : 0.f;             // (zeros added behind a run change nothing)
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u, b = xlo + (q % nch) * 64, cnt = q < items ? min(64, xhi - b + 1) : 0;
            for (int l = 0; l < cnt; l += 8) {
                float y[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[u]), l + e));
#pragma unroll
                for (int e = 0; e < 8; ++e) v += y[e];
            }
        }
    }
    if (lane == 0) store(ix, v);
}

void launch_fold2(const Grid2 &g, int nmodels, const float *acc, const float *cpad, double dt, double dx, float *out,
                  hipStream_t s)
{
    const long long rows = (long long)nmodels * g.nz;
    const int most = (int)std::max(1ll, std::min<long long>(g.nx / 128, 2048 / rows));
    const int cols = std::max(1, (g.nx - 2 + most - 1) / most), runs = std::max(1, (g.nx - 2 + cols - 1) / cols);
    constexpr long long R = 1 << 23;       // a launch holds fewer than 2^32 threads on an axis
    for (long long row0 = 0; row0 < rows; row0 += R)
        fold2_kernel<<<dim3((unsigned)std::min(R, rows - row0), runs), 256, 0, s>>>(g, (int)(row0 / g.nz), (int)(row0 % g.nz), cols,
                                                                                    acc, cpad, dt, dx, out);
}

// Ricker wavelet r(t) = (1 - 2 a) exp(-a), a = (pi f0 (t - t0))^2, in FP64.
__global__ void ricker_kernel(double f0, double t0, double dt, int nt, float *out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nt) return;
    double a = M_PI * f0 * (k * dt - t0);
    a *= a;
    out[k] = (float)((1.0 - 2.0 * a) * exp(-a));
}

void launch_ricker(double f0, double t0, double dt, int nt, float *out, hipStream_t s)
{
    ricker_kernel<<<(nt + 255) / 256, 256, 0, s>>>(f0, t0, dt, nt, out);
}

// Block-wide FP64 sum in a fixed tree order (wavefront shuffles, then LDS).
__device__ double block_sum(double v)
{
    __shared__ double part[16];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) part[wv] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0) {
        const int nw = blockDim.x >> 6;
        for (int i = 0; i < nw; ++i) r += part[i];
    }
    return r; // valid in thread 0
}

// Pass 1: block b handles [b*chunk, min(n, (b+1)*chunk)); resid = pred - obs,
// partial[b] = sum 1/2 resid^2 (FP64).
__global__ __launch_bounds__(256) void misfit_kernel(const float *pred, const float *obs, long long n,
                                                     long long chunk, float *resid, double *partial)
{
    const long long lo = (long long)blockIdx.x * chunk;
    const long long hi = min(n, lo + chunk);
    constexpr int U = 4;                   // elements in flight per thread, added in order
    double acc = 0.0;
    for (long long i0 = lo + threadIdx.x; i0 < hi; i0 += 256 * U) {
        float p[U], o[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long i = min(i0 + 256 * u, hi - 1);
            p[u] = pred[i];
            o[u] = obs[i];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long i = i0 + 256 * u;
            if (i >= hi) break;
            const float r = p[u] - o[u];
            if (resid) resid[i] = r;
            acc += 0.5 * (double)r * (double)r;
        }
    }
    const double s = block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// The final sum; a non-finite result also raises *flag (when given), which
// the host reads at its next synchronising status query.
__global__ __launch_bounds__(256) void sum_partials_kernel(const double *partial, int np, double *out, int *flag)
{
    double acc = 0.0;
    for (int i = threadIdx.x; i < np; i += blockDim.x) acc += partial[i];
    const double s = block_sum(acc);
    if (threadIdx.x == 0) {
        *out = s;
        if (flag && !isfinite(s)) *flag = 1;
    }
}

void launch_misfit(const float *pred, const float *obs, long long n, float *resid,
                   double *partials, int nparts, double *J, int *flag, hipStream_t s)
{
    if (nparts <= 1 || partials == nullptr) {
        misfit_kernel<<<1, 256, 0, s>>>(pred, obs, n, n > 0 ? n : 1, resid, J);
        return;
    }
    // a workgroup takes at least 1024 elements: 50500 in 3885 workgroups of 13
    // and as many partial sums took 4.9 + 5.6 us, so 3.3 + 2.1
    const long long chunk = std::max(1024ll, (n + nparts - 1) / nparts);
    const int nb = (int)((n + chunk - 1) / chunk);
    if (nb <= 0) {
        misfit_kernel<<<1, 256, 0, s>>>(pred, obs, 0, 1, resid, J);
        return;
    }
    misfit_kernel<<<nb, 256, 0, s>>>(pred, obs, n, chunk, resid, partials);
    sum_partials_kernel<<<1, 256, 0, s>>>(partials, nb, J, flag);
}

__global__ __launch_bounds__(1024) void dot_kernel(const float *x, const float *y, long long n, double *out)
{
    double acc = 0.0;
    for (long long i = threadIdx.x; i < n; i += blockDim.x) acc += (double)x[i] * (double)y[i];
    const double s = block_sum(acc);
    if (threadIdx.x == 0) *out = s;
}

void launch_dot(const float *x, const float *y, long long n, double *out, hipStream_t s)
{
    dot_kernel<<<1, 1024, 0, s>>>(x, y, n, out);
}

// Range check of a model's parameters on the device: the largest vp (as the
// bits of a positive float, whose order is that of the integers) and which
// checks fail.  Bound by the one read of the fields: 400^3 cells (256 MB) in
// 58 us, 128^3 in 16 (with two atomics per wavefront on the one result 158 and
// 97), where copying them to the host and looping over them took about 110 ms
// of every init_model and update_model.  A small model is one workgroup's, with
// nothing to clear before it (update_model of 16 x 16 cells, host loop / two launches /
// one: 27.5 / 32.1 / 30.0 us).
__global__ __launch_bounds__(256) void range_kernel(const float *vp, const float *vs, const float *rho, long long n,
                                                    ParamRange *out)
{
    float top = 0.f;
    unsigned bad = 0u;
    constexpr int U = 8;                   // cells in flight per thread
    const long long step = (long long)gridDim.x * 256;
    for (long long ib = blockIdx.x * 256ll + threadIdx.x; ib < n; ib += U * step) {
        float v[U], s[U], r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long i = min(ib + u * step, n - 1);
            v[u] = vp[i];
            s[u] = vs ? vs[i] : 0.f;
            r[u] = vs ? rho[i] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {      // (the last cell may be taken more than once)
            if (!(v[u] > 0.f) || !isfinite(v[u])) bad |= PARAM_BAD_VP;
            else top = fmaxf(top, v[u]);
            if (vs && (!(s[u] > 0.f) || !(s[u] < v[u]) || !(r[u] > 0.f) || !isfinite(r[u]))) bad |= PARAM_BAD_ELASTIC;
        }
    }
    __shared__ float st[256];
    __shared__ unsigned sb[256];
    st[threadIdx.x] = top;
    sb[threadIdx.x] = bad;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    for (int w = 64; w < 256; w += 64) {
        top = fmaxf(top, st[threadIdx.x + w]);
        bad |= sb[threadIdx.x + w];
    }
    for (int o = 32; o > 0; o >>= 1) {
        top = fmaxf(top, __shfl_down(top, o, 64));
        bad |= __shfl_down(bad, o, 64);
    }
    if (threadIdx.x == 0 && gridDim.x == 1) {
        *out = ParamRange{__float_as_uint(top), bad};
    } else if (threadIdx.x == 0) {
        atomicMax(&out->vmax_bits, __float_as_uint(top));
        if (bad) atomicOr(&out->bad, bad);
    }
}

void launch_param_range(const float *vp, const float *vs, const float *rho, long long n, ParamRange *out,
                        hipStream_t s)
{
    static_assert(sizeof(ParamRange) == 2 * sizeof(float), "cleared as floats");
    const int blocks = n <= 8192 ? 1 : (int)std::min<long long>((n + 2047) / 2048, 1024);
    if (blocks > 1) launch_fill(reinterpret_cast<float *>(out), 2, 0.f, s);
    range_kernel<<<blocks, 256, 0, s>>>(vp, vs, rho, n, out);
}

// Partial sums of the allocation-free misfit: a static device array, one per
// device, held until the process ends.  Host code never passes `scratch`
// itself (on the host it names a stand-in, not the device address): the
// address is taken once per device with hipGetSymbolAddress and kept.
static __device__ __align__(256) double scratch[NOALLOC_PARTS];

namespace {
std::mutex g_scratch_mu;
double *g_scratch_ptr[256] = {};
} // namespace

int noalloc_scratch(double **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 256) return -1;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return -1;
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return 0;
}

} // namespace sg
