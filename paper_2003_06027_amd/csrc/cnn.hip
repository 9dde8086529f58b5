// cnn.hip -- kernels and C ABI of the learned gradient preconditioner
// (include/sg_cnn.h).
//
// The 32 -> 32 channel 3x3 layers are implicit GEMMs on the matrix cores:
// v_mfma_f32_16x16x32_bf16 with one 3x3 tap (32 input channels) per
// K-block.  A workgroup of four wavefronts computes a 4 x 64 output tile,
// one row per wavefront; the 6 x 66 input tile (one-pixel zero halo) goes
// straight from global memory into LDS (direct 16-byte loads) in swizzled
// slots, which makes the 16-byte fragment reads of 16 consecutive pixels
// bank-conflict free.  The weight gradient uses the pixels as the K
// dimension and reduces per workgroup, then over workgroups in a fixed
// order.  The thin layers c1 (1 -> 32) and c6 (32 -> 1) are per-pixel FP32
// kernels: as GEMMs they would have K = 9 or N = 1, which matrix cores
// cannot fill.  Every reduction has a fixed order, so results are bitwise
// reproducible from call to call.
#include "../../include/seisgrad.h"
#include "../../include/sg_cnn.h"
#include "sg_error.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

using sg::fail;

namespace {

using u16 = unsigned short;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // where only floats are aligned
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

constexpr int CH = CNN_CHANNELS;
constexpr int TH = 4, TW = 64;           // output tile: 4 rows x 64 columns
constexpr int LH = TH + 2, LW = TW + 2;  // input tile with a one-pixel halo
constexpr int NT = 256;                  // threads per workgroup (4 wavefronts)
constexpr int WMID = CH * 9 * CH;        // weights of one 32 -> 32 layer
constexpr int PMID = WMID + CH;          // ... with its biases
constexpr int OFF_C1 = 0, OFF_C2 = 9 * CH + CH, OFF_C6 = OFF_C2 + 4 * PMID;
constexpr int MAX_WG_WGRAD = 512;        // workgroups (partials) of the MFMA weight gradient
constexpr int MAX_WG_THIN = 1024;        // ... of the thin-layer weight gradients
constexpr int THIN_STRIDE = 320;         // partial row of a thin layer (289 or 320 used)
constexpr int MAX_WG_LOSS = 1024;
static_assert(OFF_C6 + 9 * CH + 1 == CNN_NPARAMS, "parameter layout");

__device__ __forceinline__ float bf2f(u16 h) { return __uint_as_float((unsigned)h << 16); }

// BF16 of an FP32 value, to nearest with ties to even (the hardware's
// conversion; inf stays inf, NaN stays NaN).
__device__ __forceinline__ u16 f2bf(float f) { return __builtin_bit_cast(u16, (__bf16)f); }

__device__ __forceinline__ unsigned pack2(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, bf16x2{(__bf16)a, (__bf16)b});
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The 6 x COLS halo tile (pixels y0-1 .. y0+4, x0-1 .. x0+COLS-2 of image n) straight
// from global memory into LDS, 16 bytes (8 channels) per lane and load: item
// i = (pixel i / 4, slot i % 4) fills 16-byte slot i, which holds chunk
// (i % 4) ^ sw(pixel) of the pixel.  The swizzle sw(p) = (p / 4) % 4 puts the
// same chunk of 16 consecutive pixels on 16 distinct 16-byte bank groups.
// Pixels outside the image get zeros from a plain LDS store of their slots.
// The caller waits for the loads and synchronises.
__device__ __forceinline__ int halo_slot(int pix, int q) { return pix * 4 + (q ^ ((pix >> 2) & 3)); }

template <int COLS>
__device__ __forceinline__ void dma_halo_swizzled(const u16 *__restrict__ x, int n, int H, int W, int y0, int x0,
                                                  unsigned char *lds)
{
    constexpr int NV = LH * COLS * 4, K = (NV + NT - 1) / NT;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * NT;
        if (i >= NV) continue;
        const int pix = i >> 2, q = (i & 3) ^ ((pix >> 2) & 3);
        const int rr = pix / COLS, c = pix - rr * COLS;
        const int y = y0 - 1 + rr, xx = x0 - 1 + c;
        if (y >= 0 && y < H && xx >= 0 && xx < W)
            __builtin_amdgcn_global_load_lds((const void *)(x + (((long long)n * H + y) * W + xx) * CH + q * 8),
                                             (void __attribute__((address_space(3))) *)(lds + (k * NT + (threadIdx.x & ~63)) * 16),
                                             16, 0, 0);
        else
            *(u32x4 *)(lds + i * 16) = u32x4{0u, 0u, 0u, 0u};
    }
}

// out[i] = sum over b of part[b][i] in FP64, in a fixed order: lane l of
// output i sums rows b = l, l + 16, ... in ascending order, then the 16 lane
// sums are added in lane order.  256 threads = 16 outputs x 16 lanes.  A lane
// issues the loads of 16 of its rows before adding them, so that a chain of
// nb / 16 rows costs nb / 256 memory latencies.  The reduction of a layer's
// weight gradient rides in the first workgroups of the launch that forms its
// input gradient (4.6 to 7 us of each layer as a launch of its own).
struct Reduce {
    const float *part;
    int nb, stride, count;
    float *out;
    int blocks() const { return (count + 15) / 16; }
};
__device__ __forceinline__ void reduce_partials(const Reduce &a, int block, double (*red)[17])
{
    constexpr int U = 16;
    const int o = threadIdx.x & 15, l = threadIdx.x >> 4;
    const int i = block * 16 + o;
    double s = 0.0;
    if (i < a.count) {
        int b = l;
        for (; b + 16 * (U - 1) < a.nb; b += 16 * U) {
            float v[U];
#pragma unroll
            for (int k = 0; k < U; ++k) v[k] = a.part[(long long)(b + 16 * k) * a.stride + i];
#pragma unroll
            for (int k = 0; k < U; ++k) s += (double)v[k];
        }
        for (; b < a.nb; b += 16) s += (double)a.part[(long long)b * a.stride + i];
    }
    red[l][o] = s;
    __syncthreads();
    if (l == 0 && i < a.count) {
        double t = red[0][o];
        for (int k = 1; k < 16; ++k) t += red[k][o];
        a.out[i] = (float)t;
    }
}

// ------------------------------------------------------------ 32 -> 32 layer
struct ConvArgs {
    const u16 *x, *w;
    const float *bias;
    const u16 *res, *gate;
    u16 *y;
    float *y32;
    int N, H, W, relu;
    Reduce red;                            // of the first nred grid slices
    int nred;
};

// grid (ceil(W/(16 MB)), ceil(H/4), N).  Lane l of a wavefront: r = l % 16 is the
// fragment row (a pixel for A, an output channel for B), g = l / 16 selects
// the 8 channels 8g .. 8g+7 of the K-block; the accumulator holds output
// pixels 4g .. 4g+3 of each 16-pixel block for output channel r.  The
// accumulators go through LDS ([pixel][channel], FP32) so that the epilogue
// reads and writes 8 channels of a pixel per lane in 16- and 32-byte
// accesses instead of single 2- and 4-byte elements.
constexpr int OS = CH + 4;                 // FP32 stride of an output pixel in LDS
constexpr int conv_lds(int MB)
{
    const int in = LH * (16 * MB + 2) * 64, out = 4 * 16 * MB * OS * 4;
    return in > out ? in : out;
}

// FRAG: the weights are stored in fragment order, element ((tap * 2 + nb) *
// 64 + lane) * 8 + e, so that a fragment load is one contiguous KiB (the
// network's own copies); else as [co][tap][ci] (the single-layer entry
// point), where the 64 lanes' 16 bytes lie in 16 rows.  Those loads bounded
// the kernel: about 85 cache accesses for each of a wavefront's 18.  With
// them contiguous, the residual and gate loaded before the LDS pass and the
// hardware's BF16 conversion, a launch on 8 x 256^2 pixels went from 33.2 to
// 22.3 us (3.0 TB/s of activations read and written).
//
// MB: 16-pixel blocks per wavefront, a tile of 4 x 16 MB pixels.
template <bool FRAG, int MB>
__global__ __launch_bounds__(NT) void conv3x3_mfma_kernel(ConvArgs a)
{
    constexpr int TW = 16 * MB, LW = TW + 2;
    __shared__ __attribute__((aligned(16))) unsigned char lds_raw[conv_lds(MB)];
    u16 *lds = reinterpret_cast<u16 *>(lds_raw);
    if constexpr (FRAG) {
        if ((int)blockIdx.z < a.nred) {
            const int b = (int)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x);
            reduce_partials(a.red, b, reinterpret_cast<double (*)[17]>(lds_raw));   // (past the last output: nothing)
            return;
        }
    }
    const int n = (int)blockIdx.z - (FRAG ? a.nred : 0), y0 = blockIdx.y * TH, x0 = blockIdx.x * TW;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;

    bf16x8 bw[9][2];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
            bw[t][nb] = __builtin_bit_cast(bf16x8, *(const u32x4 *)(a.w + (FRAG ? ((t * 2 + nb) * 64 + lane) * 8
                                                                               : ((16 * nb + r) * 9 + t) * CH + 8 * g)));

    dma_halo_swizzled<LW>(a.x, n, a.H, a.W, y0, x0, lds_raw);
    __builtin_amdgcn_s_waitcnt(0);         // this thread's direct loads have landed in LDS
    __syncthreads();

    f32x4 acc[MB][2];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
        acc[mb][0] = acc[mb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int ky = t / 3, kx = t - 3 * (t / 3);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const u16 *p = lds + halo_slot((wv + ky) * LW + 16 * mb + r + kx, g) * 8;
            const bf16x8 av = __builtin_bit_cast(bf16x8, *(const u32x4 *)p);
            acc[mb][0] = mfma(av, bw[t][0], acc[mb][0]);
            acc[mb][1] = mfma(av, bw[t][1], acc[mb][1]);
        }
    }

    // the residual and the gate of this lane's output items, in flight while
    // the accumulators pass through LDS
    const int y = y0 + wv;
    const long long rowbase = ((long long)n * a.H + y) * a.W;
    constexpr int NIT = TW * 4 / 64;       // items (8 channels of a pixel) per lane
    u16x8 rv[NIT], gv[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int item = lane + 64 * it, px = item >> 2, q = item & 3;
        rv[it] = gv[it] = u16x8{0, 0, 0, 0, 0, 0, 0, 0};
        if (y >= a.H || x0 + px >= a.W) continue;
        const long long idx = (rowbase + x0 + px) * CH + 8 * q;
        if (a.res) rv[it] = *reinterpret_cast<const u16x8 *>(a.res + idx);
        if (a.gate) gv[it] = *reinterpret_cast<const u16x8 *>(a.gate + idx);
    }

    __syncthreads();                       // every wavefront is done with the input tile
    float *orow = reinterpret_cast<float *>(lds_raw) + wv * TW * OS;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int j = 0; j < 4; ++j) orow[(16 * mb + 4 * g + j) * OS + 16 * nb + r] = acc[mb][nb][j];
    __syncthreads();

    if (y >= a.H) return;
    const int q = lane & 3;                // every item of a lane: channels 8q .. 8q+7
    f32x4 blo = {0.f, 0.f, 0.f, 0.f}, bhi = blo;
    if (a.bias) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            blo[k] = a.bias[8 * q + k];
            bhi[k] = a.bias[8 * q + 4 + k];
        }
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int px = (lane + 64 * it) >> 2;
        if (x0 + px >= a.W) continue;
        const long long idx = (rowbase + x0 + px) * CH + 8 * q;
        const f32x4 lo = *reinterpret_cast<const f32x4 *>(orow + px * OS + 8 * q);
        const f32x4 hi = *reinterpret_cast<const f32x4 *>(orow + px * OS + 8 * q + 4);
        float v[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = lo[k] + blo[k];
            v[4 + k] = hi[k] + bhi[k];
        }
        if (a.res)
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] += bf2f(rv[it][k]);
        if (a.relu)
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = fmaxf(v[k], 0.f);
        if (a.gate)
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = bf2f(gv[it][k]) > 0.f ? v[k] : 0.f;
        *reinterpret_cast<u32x4 *>(a.y + idx) = u32x4{pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]),
                                                      pack2(v[6], v[7])};
        if (a.y32) {
            *reinterpret_cast<f32x4 *>(a.y32 + idx) = f32x4{v[0], v[1], v[2], v[3]};
            *reinterpret_cast<f32x4 *>(a.y32 + idx + 4) = f32x4{v[4], v[5], v[6], v[7]};
        }
    }
}

// Stage an image tile of ROWS x COLS pixels starting at (y0 - HALO, x0 - HALO)
// straight from global memory into LDS: 16 bytes (8 channels) per lane and
// load into consecutive 16-byte slots, slot i = chunk i % 4 of tile pixel
// i / 4 (a 64-byte pixel stride); pixels outside the image get zeros from
// plain LDS stores.  The caller waits for the loads and synchronises.
template <int ROWS, int COLS, int HALO>
__device__ __forceinline__ void dma_tile(const u16 *__restrict__ x, int n, int H, int W, int y0, int x0,
                                         unsigned char *lds)
{
    constexpr int NV = ROWS * COLS * 4, K = (NV + NT - 1) / NT;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * NT;
        if (i >= NV) continue;
        const int pix = i >> 2, q = i & 3;
        const int rr = pix / COLS, c = pix - rr * COLS;
        const int y = y0 - HALO + rr, xx = x0 - HALO + c;
        if (y >= 0 && y < H && xx >= 0 && xx < W)
            __builtin_amdgcn_global_load_lds((const void *)(x + (((long long)n * H + y) * W + xx) * CH + q * 8),
                                             (void __attribute__((address_space(3))) *)(lds + (k * NT + (threadIdx.x & ~63)) * 16),
                                             16, 0, 0);
        else
            *(u32x4 *)(lds + i * 16) = u32x4{0u, 0u, 0u, 0u};
    }
}

// Weight gradient, K = pixels.  Each wavefront owns one tile row (two
// K-blocks of 32 pixels); K index 8g + e of a lane maps to pixel 4e + g of
// the block, the same for both operands.  The fragments, eight pixels of one
// channel per lane from tiles stored by pixel, come from two transposing LDS
// reads each: of 16 lanes, lane 4e + c addresses channels 4c .. 4c+3 of row e
// (here pixel 4e + g), and lane j receives channel j of rows 0 .. 3.  Pixel p
// sits in pixel slot rot_slot(p), odd pixels with their channel halves
// exchanged, so that the rows that 32 lanes read at once (pixels 0, 4, 8, 12
// and 1, 5, 9, 13) cover all banks once.
//
// While a tile is multiplied, the next one is on its way: x alternates
// between two LDS buffers; dy, whose row only its own wavefront loads and
// reads, is taken into fragments first and its buffer refilled at once.
// Registers (152 of accumulators) hold a CU to two workgroups, whose loads,
// LDS reads and MFMAs ran in sequence before: 8 x 256^2 pixels 45.4 us (with
// eight 2-byte reads per fragment), 43.7 (transposing reads alone), 24.2 now.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int rot_slot(int p) { return (p & ~3) | ((p + (p >> 2)) & 3); }
__device__ __forceinline__ int rot_pixel(int slot) { return (slot & ~3) | ((slot - (slot >> 2)) & 3); }
constexpr int PXW = CH;                    // u16 stride of a pixel slot

// A fragment at byte `at` of the LDS array (pixels 16 further on: 16 slots on).
typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ bf16x8 tr_frag(lds_char *at)
{
    typedef __attribute__((address_space(3))) s16x4 lds4;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)at);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)(at + 16 * PXW * 2));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}
// Byte of pixel pix, channel ch of its lower half; the upper half: ^ HALF.
constexpr unsigned HALF = 32;
__device__ __forceinline__ unsigned tr_at(int pix, int ch)
{
    return (unsigned)(rot_slot(pix) * PXW * 2 + ((2 * ch) ^ ((pix & 1) << 5)));
}

struct WgradArgs {
    const u16 *dy, *x;
    float *part;  // [gridDim.x][PMID]
    int N, H, W, tx, ty, ntiles;
};

// Pixel slots [0, NV / 4) of a rows x COLS tile at (y0, x0), NV / 4 pixels,
// by lanes first, first + step, ..: 16-byte direct loads, zeros outside the image.
template <int COLS, int NV, int STEP>
__device__ __forceinline__ void dma_rot(const u16 *__restrict__ x, int n, int H, int W, int y0, int x0, int first,
                                        unsigned char *lds)
{
#pragma unroll
    for (int k = 0; k < (NV + STEP - 1) / STEP; ++k) {
        const int i = first + k * STEP;
        if (i >= NV) continue;
        const int pix = rot_pixel(i >> 2), q = (i & 3) ^ ((pix & 1) << 1);
        const int rr = pix / COLS, c = pix - rr * COLS;
        const int y = y0 + rr, xx = x0 + c;
        if (y >= 0 && y < H && xx >= 0 && xx < W)
            __builtin_amdgcn_global_load_lds((const void *)(x + (((long long)n * H + y) * W + xx) * CH + q * 8),
                                             (void __attribute__((address_space(3))) *)(lds + __builtin_amdgcn_readfirstlane(i & ~63) * 16),
                                             16, 0, 0);
        else
            *(u32x4 *)(lds + i * 16) = u32x4{0u, 0u, 0u, 0u};
    }
}

constexpr int XTILE = LH * LW * PXW, YTILE = TH * TW * PXW;   // u16 of the two tiles
constexpr int RS = CH + 4;                 // FP32 row stride of a tap in the reduction (distinct banks per lane group)
static_assert(LH * LW % 4 == 0 && TW % 4 == 0, "whole groups of four pixels");
static_assert((2 * XTILE + YTILE) * 2 >= 4 * 3 * CH * RS * 4 + 4 * CH * 4, "the reduction reuses the staging space");

__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void wgrad3x3_mfma_kernel(WgradArgs a)
{
    __shared__ __attribute__((aligned(16))) u16 smem[2 * XTILE + YTILE];
    u16 *lg = smem + 2 * XTILE;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int tp = 4 * (r >> 2) + g, tc = 4 * (r & 3);   // pixel and channel a lane addresses
    const bf16x8 ones = __builtin_bit_cast(bf16x8, u16x8{0x3f80, 0x3f80, 0x3f80, 0x3f80,
                                                         0x3f80, 0x3f80, 0x3f80, 0x3f80});
    f32x4 acc[9][2][2];
    f32x4 accb[2];
#pragma unroll
    for (int t = 0; t < 9; ++t)
        acc[t][0][0] = acc[t][0][1] = acc[t][1][0] = acc[t][1][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    accb[0] = accb[1] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto load = [&](int tile, u16 *lx) {
        const int per = a.tx * a.ty;
        const int n = tile / per, rem = tile - n * per;
        const int y0 = (rem / a.tx) * TH, x0 = (rem - (rem / a.tx) * a.tx) * TW;
        // an opaque copy of the thread id: the pixels of its items are worked
        // out again for each tile rather than kept in (spilled) registers
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        dma_rot<LW, LH * LW * 4, NT>(a.x, n, a.H, a.W, y0 - 1, x0 - 1, tid, (unsigned char *)lx);
        dma_rot<TW, TW * 4, 64>(a.dy, n, a.H, a.W, y0 + wv, x0, lane, (unsigned char *)(lg + wv * TW * PXW));
    };
    // Bytes of this lane's rows.  A tap's pixel is 66 ky + kx on: the slot of
    // 66 ky is 64 ky slots and 2 ky pixels, and 32 pixels are 32 slots, so
    // seven addresses and constants serve the 36 fragments of a tile row.
    static_assert(LW == 66, "the slot of a row below");
    lds_char *sm = (lds_char *)(void *)smem;
    unsigned xo[7];
#pragma unroll
    for (int d = 0; d < 7; ++d) xo[d] = tr_at(wv * LW + tp + d, tc);
    const unsigned yo = (2 * XTILE + wv * TW * PXW) * 2 + tr_at(tp, tc);

    auto step = [&](int tile, auto CUR) {
        constexpr int cur = decltype(CUR)::value;
        __builtin_amdgcn_s_waitcnt(0);     // this wavefront's loads have landed
        __syncthreads();                   // all have; the other x buffer is free
        bf16x8 A[2][2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            A[kb][0] = tr_frag(sm + yo + kb * 32 * PXW * 2);
            A[kb][1] = tr_frag(sm + (yo ^ HALF) + kb * 32 * PXW * 2);
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);                // lgkmcnt(0): the fragments are in registers
        __builtin_amdgcn_sched_barrier(0);
        if (tile + (int)gridDim.x < a.ntiles) load(tile + gridDim.x, smem + (cur ^ 1) * XTILE);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            accb[0] = mfma(A[kb][0], ones, accb[0]);
            accb[1] = mfma(A[kb][1], ones, accb[1]);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int ky = t / 3, kx = t - 3 * (t / 3);
                const int on = (cur * XTILE + (ky * 64 + kb * 32) * PXW) * 2;
                const bf16x8 B0 = tr_frag(sm + xo[2 * ky + kx] + on), B1 = tr_frag(sm + (xo[2 * ky + kx] ^ HALF) + on);
                acc[t][0][0] = mfma(A[kb][0], B0, acc[t][0][0]);
                acc[t][1][0] = mfma(A[kb][1], B0, acc[t][1][0]);
                acc[t][0][1] = mfma(A[kb][0], B1, acc[t][0][1]);
                acc[t][1][1] = mfma(A[kb][1], B1, acc[t][1][1]);
            }
        }
    };
    load(blockIdx.x, smem);
    for (int tile = blockIdx.x; tile < a.ntiles; tile += 2 * gridDim.x) {
        step(tile, std::integral_constant<int, 0>{});
        if (tile + (int)gridDim.x < a.ntiles) step(tile + gridDim.x, std::integral_constant<int, 1>{});
    }

    // fixed-order sum over the four wavefronts, three taps at a time through
    // LDS ([wavefront][tap][co][ci]), into one partial row
    float *red = reinterpret_cast<float *>(smem), *redb = red + 4 * 3 * CH * RS;
    float *out = a.part + (long long)blockIdx.x * PMID;
#pragma unroll
    for (int t0 = 0; t0 < 9; t0 += 3) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int ib = 0; ib < 2; ++ib)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        red[((wv * 3 + t) * CH + 16 * cb + 4 * g + j) * RS + 16 * ib + r] = acc[t0 + t][cb][ib][j];
        if (t0 == 0 && r == 0)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int j = 0; j < 4; ++j) redb[wv * CH + 16 * cb + 4 * g + j] = accb[cb][j];
        __syncthreads();
        for (int i = threadIdx.x; i < 3 * CH * CH / 4; i += NT) {
            const int ci = 4 * (i % (CH / 4)), co = i / (CH / 4) % CH, t = i / (CH * CH / 4);
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) v += *(const f32x4 *)(red + ((w * 3 + t) * CH + co) * RS + ci);
            *(f32x4u *)(out + (co * 9 + t0 + t) * CH + ci) = v;
        }
        if (t0 == 0 && threadIdx.x < CH) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) v += redb[w * CH + threadIdx.x];
            out[WMID + threadIdx.x] = v;
        }
    }
}

__global__ __launch_bounds__(256) void reduce_partials_kernel(Reduce r)
{
    __shared__ double red[16][17];
    reduce_partials(r, (int)blockIdx.x, red);
}

// Element of the weight (out, tap, in) in fragment order (see conv3x3_mfma_kernel).
__device__ __forceinline__ int frag_at(int out, int tap, int in)
{
    return ((tap * 2 + (out >> 4)) * 64 + (in >> 3) * 16 + (out & 15)) * 8 + (in & 7);
}

// BF16 copies of c2..c5 in fragment order: wf[L] as they are and wt[L]
// flipped and transposed, the weights of the input gradient.
// (Weight i of the 4 WMID.)
__device__ __forceinline__ void prep_weight(int i, const float *__restrict__ params, u16 *__restrict__ wf,
                                            u16 *__restrict__ wt)
{
    const int L = i / WMID, k = i - L * WMID;
    const int co = k / (9 * CH), t = (k / CH) % 9, ci = k % CH;
    const u16 b = f2bf(params[OFF_C2 + L * PMID + k]);
    wf[L * WMID + frag_at(co, t, ci)] = b;
    wt[L * WMID + frag_at(ci, 8 - t, co)] = b;
}

// ------------------------------------------------------------- thin layers
// The image row and column of flat pixel p (fewer than 2^29: 32-bit
// divisions; with 64-bit ones c1 took 15.1 instead of 12.8 us on 8 x 256^2).
__device__ __forceinline__ void pixel_of(unsigned p, int H, int W, int &y, int &x)
{
    const unsigned q = p / (unsigned)W;
    x = (int)(p - q * (unsigned)W);
    y = (int)(q % (unsigned)H);
}

// c1: x1 = relu(b + sum_t w[co][t] g[pix + off_t]) in FP32, stored BF16.
// The thin layers c1 and c6's input gradient work on runs of NT consecutive
// pixels (flat n, y, x order), whose 32 channels are NT x 64 contiguous
// bytes: a thread computes one pixel (the weights are then the same for every
// lane), and the 64-byte pixels pass through LDS in the swizzled slots of
// halo_slot, so that global memory sees whole 1 KiB runs per instruction.
__device__ __forceinline__ void store_pixels(const unsigned char *lds, long long p0, long long total, u16 *dst)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int j = threadIdx.x + k * NT, pix = j >> 2, q = j & 3;
        if (p0 + pix < total)
            *(u32x4 *)(dst + (p0 + pix) * CH + q * 8) = *(const u32x4 *)(lds + halo_slot(pix, q) * 16);
    }
}

// The first PREP_WG workgroups form the weight copies that the following
// launches read (as a launch of its own 2.5 us).
constexpr int PREP_WG = 4 * WMID / NT;
static_assert(4 * WMID % NT == 0, "whole workgroups");
__global__ __launch_bounds__(NT) void conv_in_kernel(const float *__restrict__ g, const float *__restrict__ params,
                                                     u16 *__restrict__ x1, int N, int H, int W,
                                                     u16 *__restrict__ wf, u16 *__restrict__ wt)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[NT * 64];
    if (blockIdx.x < PREP_WG) {
        prep_weight((int)(blockIdx.x * NT + threadIdx.x), params, wf, wt);
        return;
    }
    const long long total = (long long)N * H * W, p0 = (long long)(blockIdx.x - PREP_WG) * NT, p = p0 + threadIdx.x;
    if (p < total) {
        int y, x;
        pixel_of((unsigned)p, H, W, y, x);
        float v[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int dy = t / 3 - 1, dx = t % 3 - 1;
            v[t] = (y + dy >= 0 && y + dy < H && x + dx >= 0 && x + dx < W) ? g[(int)p + dy * W + dx] : 0.f;
        }
        const float *w = params + OFF_C1, *b = params + OFF_C1 + 9 * CH;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int co = 8 * q + e;
                float s = b[co];
#pragma unroll
                for (int t = 0; t < 9; ++t) s = fmaf(w[co * 9 + t], v[t], s);
                o[e] = fmaxf(s, 0.f);
            }
            *(u32x4 *)(lds + halo_slot(threadIdx.x, q) * 16) =
                u32x4{pack2(o[0], o[1]), pack2(o[2], o[3]), pack2(o[4], o[5]), pack2(o[6], o[7])};
        }
    }
    __syncthreads();
    store_pixels(lds, p0, total, x1);
}

// c6 and the global residual: p = -g + b + sum_t sum_ci w[t][ci] x3[pix + off_t][ci].
// On the 4 x 64 tiles of the 32 -> 32 layers, x3 with its halo staged in LDS
// as for those layers; one thread per pixel, the sum in tap, channel order.
__global__ __launch_bounds__(NT) void conv_out_kernel(const u16 *__restrict__ x3, const float *__restrict__ g,
                                                      const float *__restrict__ params, float *__restrict__ p,
                                                      int N, int H, int W)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[LH * LW * 64];
    const int n = blockIdx.z, y0 = blockIdx.y * TH, x0 = blockIdx.x * TW;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    dma_halo_swizzled<LW>(x3, n, H, W, y0, x0, lds);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const int y = y0 + wv, x = x0 + lane;
    if (y >= H || x >= W) return;
    const float *w = params + OFF_C6;
    float s = params[OFF_C6 + 9 * CH];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int yy = y + t / 3 - 1, xx = x + t % 3 - 1;
        if (yy < 0 || yy >= H || xx < 0 || xx >= W) continue;
        const int pix = (wv + t / 3) * LW + lane + t % 3;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x4 u = *(const u32x4 *)(lds + halo_slot(pix, q) * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s = fmaf(w[t * CH + 8 * q + 2 * e], __uint_as_float(u[e] << 16), s);
                s = fmaf(w[t * CH + 8 * q + 2 * e + 1], __uint_as_float(u[e] & 0xffff0000u), s);
            }
        }
    }
    const long long i = ((long long)n * H + y) * W + x;
    p[i] = s - g[i];
}

// Input gradient of c6 gated by x3 > 0: G[pix][ci] = [x3 > 0] sum_t w[t][ci] dp[pix - off_t].
// The first nred workgroups reduce c6's weight gradient.
__global__ __launch_bounds__(NT) void dgrad_out_kernel(const float *__restrict__ dp, const u16 *__restrict__ x3,
                                                       const float *__restrict__ params, u16 *__restrict__ G,
                                                       int N, int H, int W, Reduce red, int nred)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[NT * 64];
    if ((int)blockIdx.x < nred) {
        reduce_partials(red, (int)blockIdx.x, reinterpret_cast<double (*)[17]>(lds));
        return;
    }
    const long long total = (long long)N * H * W, p0 = (long long)(blockIdx.x - nred) * NT, p = p0 + threadIdx.x;
    // the gates x3 of the run, straight into the swizzled slots (16 bytes per lane and load)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int j = threadIdx.x + k * NT, pix = j >> 2, q = (j & 3) ^ ((pix >> 2) & 3);
        if (p0 + pix < total)
            __builtin_amdgcn_global_load_lds((const void *)(x3 + (p0 + pix) * CH + q * 8),
                                             (void __attribute__((address_space(3))) *)(lds + (k * NT + (threadIdx.x & ~63)) * 16),
                                             16, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (p < total) {
        int y, x;
        pixel_of((unsigned)p, H, W, y, x);
        float d[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int dy = 1 - t / 3, dx = 1 - t % 3;
            d[t] = (y + dy >= 0 && y + dy < H && x + dx >= 0 && x + dx < W) ? dp[(int)p + dy * W + dx] : 0.f;
        }
        const float *w = params + OFF_C6;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32x4 *slot = (u32x4 *)(lds + halo_slot(threadIdx.x, q) * 16);
            const u32x4 gt = *slot;
            float o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int ci = 8 * q + e;
                float s = 0.f;
#pragma unroll
                for (int t = 0; t < 9; ++t) s = fmaf(w[t * CH + ci], d[t], s);
                const unsigned gv = (e & 1) ? (gt[e >> 1] & 0xffff0000u) : (gt[e >> 1] << 16);
                o[e] = __uint_as_float(gv) > 0.f ? s : 0.f;
            }
            *slot = u32x4{pack2(o[0], o[1]), pack2(o[2], o[3]), pack2(o[4], o[5]), pack2(o[6], o[7])};
        }
    }
    __syncthreads();
    store_pixels(lds, p0, total, G);
}

// Weight gradients of the thin layers, on the 4 x 64 pixel tiles of the
// 32 -> 32 layers (grid-stride over tiles, per-thread register sums, one
// partial row per workgroup; the rows are reduced in a fixed order after).
// c6: out[t * 32 + ci] = sum_p dp[p] x3[p + off_t][ci] (t < 9), out[288] = sum dp.
// c1: out[co * 9 + t] = sum_p G[p][co] g[p + off_t], out[288 + co] = sum_p G[p][co].
// Bound by LDS reads and instruction issue, since each output is one FP32
// chain over the tile's pixels in order.  128 threads take a tile: 96 of them
// one channel and the three taps of a kernel row, so that a pixel costs one
// read of the activation and one of the image (broadcast) for three chains,
// 32 the bias sums; a workgroup works on two tiles at once, whose sums are
// added in tile order.  (With a thread per output, two reads per term and a
// second pass for outputs 256 .. 320: 37.9 us for c1, 25.6 us for c6 on
// 8 x 256^2 pixels, against 19.5 and 23.8.)
template <bool OUT>
__global__ __launch_bounds__(NT) void wgrad_thin_kernel(const float *__restrict__ img, const u16 *__restrict__ act,
                                                        float *__restrict__ part, int H, int W, int tx, int ty,
                                                        int ntiles)
{
    constexpr int PW = 32;                 // u16 stride of a staged pixel (the slots of dma_tile)
    constexpr int NA = (OUT ? LH * LW : TH * TW) * PW, NI = OUT ? TH * TW : LH * LW;
    __shared__ __attribute__((aligned(16))) u16 la2[2][NA];
    __shared__ __attribute__((aligned(16))) float li2[2][NI];
    __shared__ float xs[3][128];
    const int half = threadIdx.x >> 7, j = threadIdx.x & 127;
    const bool taps = j < 96;
    const int ky = taps ? j >> 5 : 0, ch = j & 31;
    float acc[3] = {0.f, 0.f, 0.f};
    for (int tile0 = blockIdx.x; tile0 < ntiles; tile0 += 2 * gridDim.x) {
        __syncthreads();
        for (int q = 0; q < 2; ++q) {      // both tiles staged by the whole workgroup
            const int tile = tile0 + q * (int)gridDim.x;
            if (tile >= ntiles) break;
            const int per = tx * ty;
            const int n = tile / per, rem = tile - n * per;
            const int y0 = (rem / tx) * TH, x0 = (rem - (rem / tx) * tx) * TW;
            float *li = li2[q];
            if (OUT) {
                dma_tile<LH, LW, 1>(act, n, H, W, y0, x0, reinterpret_cast<unsigned char *>(la2[q]));
                for (int i = threadIdx.x; i < TH * TW; i += NT) {
                    const int y = y0 + i / TW, x = x0 + i % TW;
                    li[i] = (y < H && x < W) ? img[((long long)n * H + y) * W + x] : 0.f;
                }
            } else {
                dma_tile<TH, TW, 0>(act, n, H, W, y0, x0, reinterpret_cast<unsigned char *>(la2[q]));
                for (int i = threadIdx.x; i < LH * LW; i += NT) {
                    const int y = y0 - 1 + i / LW, x = x0 - 1 + i % LW;
                    li[i] = (y >= 0 && y < H && x >= 0 && x < W) ? img[((long long)n * H + y) * W + x] : 0.f;
                }
            }
        }
        __builtin_amdgcn_s_waitcnt(0);     // this thread's direct loads have landed in LDS
        __syncthreads();
        const bool mine = tile0 + half * (int)gridDim.x < ntiles;
        const u16 *la = la2[half];
        const float *li = li2[half];
        float s[3] = {0.f, 0.f, 0.f};
        if (mine && taps) {
            for (int r = 0; r < TH; ++r) {
                if (OUT) {
                    const u16 *ap = la + (r + ky) * LW * PW + ch;
                    float w0 = bf2f(ap[0]), w1 = bf2f(ap[PW]);
#pragma unroll 8
                    for (int c = 0; c < TW; ++c) {
                        const float w2 = bf2f(ap[(c + 2) * PW]), d = li[r * TW + c];
                        s[0] = fmaf(d, w0, s[0]);
                        s[1] = fmaf(d, w1, s[1]);
                        s[2] = fmaf(d, w2, s[2]);
                        w0 = w1;
                        w1 = w2;
                    }
                } else {
                    const float *ip = li + (r + ky) * LW;
                    const u16 *ap = la + r * TW * PW + ch;
                    float v0 = ip[0], v1 = ip[1];
#pragma unroll 8
                    for (int c = 0; c < TW; ++c) {
                        const float v2 = ip[c + 2], d = bf2f(ap[c * PW]);
                        s[0] = fmaf(d, v0, s[0]);
                        s[1] = fmaf(d, v1, s[1]);
                        s[2] = fmaf(d, v2, s[2]);
                        v0 = v1;
                        v1 = v2;
                    }
                }
            }
        } else if (mine && (!OUT || ch == 0)) {
#pragma unroll 8
            for (int i = 0; i < TH * TW; ++i) s[0] += OUT ? li[i] : bf2f(la[i * PW + ch]);
        }
        if (half == 1)
#pragma unroll
            for (int k = 0; k < 3; ++k) xs[k][j] = s[k];
        __syncthreads();
        if (half == 0) {
            const bool both = tile0 + (int)gridDim.x < ntiles;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                acc[k] += s[k];
                if (both) acc[k] += xs[k][j];
            }
        }
    }
    if (half) return;
    float *out = part + (long long)blockIdx.x * THIN_STRIDE;
    if (taps) {
#pragma unroll
        for (int k = 0; k < 3; ++k) out[OUT ? (ky * 3 + k) * CH + ch : ch * 9 + ky * 3 + k] = acc[k];
    } else if (!OUT || ch == 0) {
        out[9 * CH + ch] = acc[0];
    }
}

// --------------------------------------------------------- loss and Adam
__device__ void block_sum2(double &a, double &b)
{
    __shared__ double sa[256], sb[256];
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            sa[threadIdx.x] += sa[threadIdx.x + s];
            sb[threadIdx.x] += sb[threadIdx.x + s];
        }
        __syncthreads();
    }
    a = sa[0];
    b = sb[0];
}

__global__ __launch_bounds__(256) void loss_partial_kernel(const float *__restrict__ p, const float *__restrict__ t,
                                                           const float *__restrict__ m, long long n, long long per_wg,
                                                           double *__restrict__ part)
{
    const long long i0 = blockIdx.x * per_wg, i1 = i0 + per_wg < n ? i0 + per_wg : n;
    constexpr int U = 4;                   // loads of U elements in flight, added in order
    double s = 0.0, c = 0.0;
    for (long long ib = i0 + threadIdx.x; ib < i1; ib += 256 * U) {
        float pv[U], tv[U], mv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long i = min(ib + 256 * u, i1 - 1);
            pv[u] = p[i]; tv[u] = t[i]; mv[u] = m[i];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (ib + 256 * u >= i1) break;
            const double r = (double)pv[u] - (double)tv[u];
            s += (double)mv[u] * r * r;
            c += (double)mv[u];
        }
    }
    block_sum2(s, c);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = s;
        part[2 * blockIdx.x + 1] = c;
    }
}

__global__ __launch_bounds__(256) void loss_final_kernel(const double *__restrict__ part, int nb, double *L,
                                                         double *count)
{
    double s = 0.0, c = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) {
        s += part[2 * b];
        c += part[2 * b + 1];
    }
    block_sum2(s, c);
    if (threadIdx.x == 0) {
        *L = c > 0 ? s / c : 0.0;
        *count = c;
    }
}

__global__ void loss_grad_kernel(const float *__restrict__ p, const float *__restrict__ t, const float *__restrict__ m,
                                 long long n, const double *__restrict__ count, float *__restrict__ dp)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double c = *count;
    dp[i] = c > 0 ? (float)(2.0 * (double)m[i] * ((double)p[i] - (double)t[i]) / c) : 0.f;
}

__global__ void adam_kernel(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, long long n, float lr, float b1, float b2, float eps,
                            float c1, float c2)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// ----------------------------------------------------------------- packing
__global__ __launch_bounds__(256) void field_inv_rms_kernel(const float *__restrict__ a, const float *__restrict__ b,
                                                            int nsrc, const int *__restrict__ order, int fh, int fw,
                                                            double *__restrict__ inv)
{
    const int s = blockIdx.x;
    const int f = order ? order[s] : s;
    const bool valid = f >= 0 && f < nsrc;
    const long long n = (long long)fh * fw, base = (long long)f * n;
    double acc = 0.0, dummy = 0.0;
    constexpr int U = 16;                  // loads of U elements in flight, added in order
    for (long long ib = threadIdx.x; valid && ib < n; ib += 256 * U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long i = base + min(ib + 256 * u, n - 1);
            v[u] = b ? a[i] - b[i] : a[i];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (ib + 256 * u >= n) break;
            acc += (double)v[u] * (double)v[u];
        }
    }
    block_sum2(acc, dummy);
    if (threadIdx.x == 0) inv[s] = acc > 0 ? 1.0 / sqrt(acc / (double)n) : 0.0;
}

// I: an unsigned index type that holds `total` (32-bit divisions where they do:
// 4.0 and 5.0 us for 20 fields of 101^2 with 64-bit ones, 3.5 and 2.7 so).
template <class I>
__global__ void pack_kernel(const float *__restrict__ a, const float *__restrict__ b, int nsrc,
                            const int *__restrict__ order, int nfields, int fh, int fw, int frame, const double *__restrict__ inv,
                            float *__restrict__ patches, float *__restrict__ mask, long long total)
{
    const I i = (I)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (I)total) return;
    const I P = 2 * (I)frame, r = i / P;
    const int xx = (int)(i - r * P), yy = (int)(r % P);
    const long long q = (long long)(r / P);
    const int by = yy >= frame, bx = xx >= frame;
    const long long s = q * 4 + by * 2 + bx;
    const int ly = yy - by * frame, lx = xx - bx * frame;
    const long long f = s < nfields ? (order ? order[s] : s) : -1;
    const bool inside = f >= 0 && f < nsrc && ly < fh && lx < fw;
    float v = 0.f;
    if (inside) {
        const long long k = (f * fh + ly) * fw + lx;
        v = b ? a[k] - b[k] : a[k];
        if (inv) v *= (float)inv[s];
    }
    patches[i] = v;
    if (mask) mask[i] = inside ? 1.f : 0.f;
}

template <class I>
__global__ void unpack_kernel(const float *__restrict__ patches, int nfields, int fh, int fw, int frame,
                              float *__restrict__ fields)
{
    const I i = (I)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (I)((long long)nfields * fh * fw)) return;
    const I row = i / (I)fw;
    const int lx = (int)(i - row * (I)fw), ly = (int)(row % (I)fh);
    const long long s = (long long)(row / (I)fh), P = 2ll * frame;
    const int k = (int)(s % 4);
    const long long src = ((s / 4) * P + (k / 2) * frame + ly) * P + (k % 2) * frame + lx;
    fields[i] = patches[src];
}

// --------------------------------------------------------------- host side
#define HIPCHECK(x)                                                                  \
    do {                                                                             \
        hipError_t e_ = (x);                                                         \
        if (e_ != hipSuccess)                                                        \
            return fail(SG_EDEVICE, "%s failed: %s", #x, hipGetErrorString(e_));     \
    } while (0)

constexpr size_t ALIGN = 256;
size_t up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

struct CnnLayout {
    size_t wf, wt, act[5], gbuf[3], part, loss, total;
};

CnnLayout cnn_layout(int n, int h, int w)
{
    CnnLayout L;
    const size_t A = up((size_t)n * h * w * CH * sizeof(u16));
    size_t o = 0;
    L.wf = o; o += up(4 * WMID * sizeof(u16));
    L.wt = o; o += up(4 * WMID * sizeof(u16));
    for (auto &x : L.act) { x = o; o += A; }
    for (auto &x : L.gbuf) { x = o; o += A; }
    L.part = o;
    const size_t pm = (size_t)MAX_WG_WGRAD * PMID, pt = (size_t)MAX_WG_THIN * THIN_STRIDE;
    o += up((pm > pt ? pm : pt) * sizeof(float));
    L.loss = o; o += up((2 * MAX_WG_LOSS + 2) * sizeof(double));
    L.total = o;
    return L;
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

int check_dims(int n, int h, int w)
{
    if (n < 1 || h < 1 || w < 1) return fail(SG_EINVAL, "image extents must be positive (n=%d h=%d w=%d)", n, h, w);
    if ((long long)n * h * w >= (1LL << 29)) return fail(SG_EINVAL, "images too large (n h w >= 2^29 pixels)");
    return SG_OK;
}

// Tiles 32 instead of 64 pixels wide up to one wide tile per compute unit: there a
// layer lasts as long as one wavefront's instruction stream, which is half as long.
// On fuller grids the wider tile's smaller halo counts.  Forward + backward of the network,
// 64 / 32 wide, us: 1 x 64^2 (16 tiles) 35.5 + 80.3 / 29.5 + 73.3; 1 x 200^2 (200) 40.5 +
// 99.5 / 38.0 + 98.6; 1 x 256^2 (256) 42.4 + 102.0 / 37.8 + 100.2; 4 x 142^2 (432) 45.6 + 117.0 /
// 41.3 + 122.7; 3 x 256^2 (768) 59.3 + 152.1 / 61.8 + 151.1; 8 x 256^2 (2048) 112.8 + 259.4 /
// 123.1 + 262.3.
bool conv_half(int n, int h, int w)
{
    return (long long)((w + TW - 1) / TW) * ((h + TH - 1) / TH) * n <= 256;
}

template <bool FRAG>
int launch_conv(const u16 *x, int n, int h, int w, const u16 *wgt, const float *bias, const u16 *res,
                const u16 *gate, int relu, u16 *y, float *y32, hipStream_t s, const Reduce *red = nullptr)
{
    ConvArgs a{x, wgt, bias, res, gate, y, y32, n, h, w, relu, {}, 0};
    const bool half = conv_half(n, h, w);
    const int tw = half ? TW / 2 : TW;
    dim3 grid((w + tw - 1) / tw, (h + TH - 1) / TH, n);
    if (grid.y > 65535u || grid.z > 65535u) return fail(SG_EINVAL, "image batch too large for one launch");
    if (red) {
        const long long slice = (long long)grid.x * grid.y, slices = (red->blocks() + slice - 1) / slice;
        if (n + slices <= 65535) {
            a.red = *red;
            a.nred = (int)slices;
            grid.z += a.nred;
        } else {                           // no room in the grid
            reduce_partials_kernel<<<red->blocks(), 256, 0, s>>>(*red);
            HIPCHECK(hipGetLastError());
        }
    }
    if (half) conv3x3_mfma_kernel<FRAG, 2><<<grid, NT, 0, s>>>(a);
    else      conv3x3_mfma_kernel<FRAG, 4><<<grid, NT, 0, s>>>(a);
    HIPCHECK(hipGetLastError());
    return SG_OK;
}

// The partial sums of a weight gradient; red: their reduction, still to be launched.
int launch_wgrad(const u16 *dy, const u16 *x, int n, int h, int w, float *part, float *out, Reduce &red, hipStream_t s)
{
    WgradArgs a;
    a.dy = dy;
    a.x = x;
    a.part = part;
    a.N = n;
    a.H = h;
    a.W = w;
    a.tx = (w + TW - 1) / TW;
    a.ty = (h + TH - 1) / TH;
    const long long nt = (long long)a.tx * a.ty * n;
    if (nt > (1LL << 31) - 1) return fail(SG_EINVAL, "too many tiles");
    a.ntiles = (int)nt;
    const int nwg = a.ntiles < MAX_WG_WGRAD ? a.ntiles : MAX_WG_WGRAD;
    wgrad3x3_mfma_kernel<<<nwg, NT, 0, s>>>(a);
    HIPCHECK(hipGetLastError());
    red = Reduce{part, nwg, PMID, PMID, out};
    return SG_OK;
}

int launch_reduce(const Reduce &red, hipStream_t s)
{
    reduce_partials_kernel<<<red.blocks(), 256, 0, s>>>(red);
    HIPCHECK(hipGetLastError());
    return SG_OK;
}

template <bool OUT>
int launch_wgrad_thin(const float *img, const u16 *act, int n, int h, int w, float *part, float *out, Reduce &red,
                      hipStream_t s)
{
    const int tx = (w + TW - 1) / TW, ty = (h + TH - 1) / TH;
    const long long nt = (long long)tx * ty * n;
    if (nt > (1LL << 31) - 1) return fail(SG_EINVAL, "too many tiles");
    const int nwg = nt < MAX_WG_THIN ? (int)nt : MAX_WG_THIN;
    wgrad_thin_kernel<OUT><<<nwg, NT, 0, s>>>(img, act, part, h, w, tx, ty, (int)nt);
    HIPCHECK(hipGetLastError());
    red = Reduce{part, nwg, THIN_STRIDE, OUT ? 9 * CH + 1 : 9 * CH + CH, out};
    return SG_OK;
}

unsigned blocks(long long n, int t = 256) { return (unsigned)((n + t - 1) / t); }

} // namespace

extern "C" {

size_t cnn_workspace_bytes(int32_t n, int32_t h, int32_t w)
{
    if (n < 1 || h < 1 || w < 1) return 0;
    return cnn_layout(n, h, w).total;
}

int cnn_forward(const float *params, const float *g, int32_t n, int32_t h, int32_t w, float *p, void *ws,
                size_t ws_bytes, sg_stream_t stream)
{
    if (int e = check_dims(n, h, w)) return e;
    if (!params || !g || !p || !ws) return fail(SG_EINVAL, "NULL pointer argument");
    const CnnLayout L = cnn_layout(n, h, w);
    if (ws_bytes < L.total || !aligned16(ws))
        return fail(SG_EINVAL, "workspace too small or misaligned (%zu < %zu bytes)", ws_bytes, L.total);
    hipStream_t s = (hipStream_t)stream;
    char *base = (char *)ws;
    u16 *wf = (u16 *)(base + L.wf), *wt = (u16 *)(base + L.wt);
    u16 *x1 = (u16 *)(base + L.act[0]), *a2 = (u16 *)(base + L.act[1]), *x2 = (u16 *)(base + L.act[2]);
    u16 *a4 = (u16 *)(base + L.act[3]), *x3 = (u16 *)(base + L.act[4]);
    const long long pix = (long long)n * h * w;
    conv_in_kernel<<<PREP_WG + blocks(pix, NT), NT, 0, s>>>(g, params, x1, n, h, w, wf, wt);
    HIPCHECK(hipGetLastError());
    const float *bias = params + OFF_C2 + WMID;
    if (int e = launch_conv<true>(x1, n, h, w, wf + 0 * WMID, bias + 0 * PMID, nullptr, nullptr, 1, a2, nullptr, s)) return e;
    if (int e = launch_conv<true>(a2, n, h, w, wf + 1 * WMID, bias + 1 * PMID, x1, nullptr, 1, x2, nullptr, s)) return e;
    if (int e = launch_conv<true>(x2, n, h, w, wf + 2 * WMID, bias + 2 * PMID, nullptr, nullptr, 1, a4, nullptr, s)) return e;
    if (int e = launch_conv<true>(a4, n, h, w, wf + 3 * WMID, bias + 3 * PMID, x2, nullptr, 1, x3, nullptr, s)) return e;
    conv_out_kernel<<<dim3((w + TW - 1) / TW, (h + TH - 1) / TH, n), NT, 0, s>>>(x3, g, params, p, n, h, w);
    HIPCHECK(hipGetLastError());
    return SG_OK;
}

int cnn_backward(const float *params, const float *g, const float *dp, int32_t n, int32_t h, int32_t w, float *grad,
                 void *ws, size_t ws_bytes, sg_stream_t stream)
{
    if (int e = check_dims(n, h, w)) return e;
    if (!params || !g || !dp || !grad || !ws) return fail(SG_EINVAL, "NULL pointer argument");
    const CnnLayout L = cnn_layout(n, h, w);
    if (ws_bytes < L.total || !aligned16(ws))
        return fail(SG_EINVAL, "workspace too small or misaligned (%zu < %zu bytes)", ws_bytes, L.total);
    hipStream_t s = (hipStream_t)stream;
    char *base = (char *)ws;
    const u16 *wt = (const u16 *)(base + L.wt);
    const u16 *x1 = (u16 *)(base + L.act[0]), *a2 = (u16 *)(base + L.act[1]), *x2 = (u16 *)(base + L.act[2]);
    const u16 *a4 = (u16 *)(base + L.act[3]), *x3 = (u16 *)(base + L.act[4]);
    u16 *G0 = (u16 *)(base + L.gbuf[0]), *G1 = (u16 *)(base + L.gbuf[1]), *G2 = (u16 *)(base + L.gbuf[2]);
    float *part = (float *)(base + L.part);
    const long long pix = (long long)n * h * w;

    Reduce red;
    if (int e = launch_wgrad_thin<true>(dp, x3, n, h, w, part, grad + OFF_C6, red, s)) return e;
    dgrad_out_kernel<<<red.blocks() + blocks(pix, NT), NT, 0, s>>>(dp, x3, params, G0, n, h, w, red, red.blocks()); // G0 = d pre(x3)
    HIPCHECK(hipGetLastError());
    float *gm = grad + OFF_C2;
    // layer L: its weight gradient's partial sums, then its input gradient with their reduction
    auto layer = [&](int L, const u16 *dy, const u16 *x, const u16 *res, u16 *dx) -> int {
        if (int e = launch_wgrad(dy, x, n, h, w, part, gm + L * PMID, red, s)) return e;
        return launch_conv<true>(dy, n, h, w, wt + L * WMID, nullptr, res, x, 0, dx, nullptr, s, &red);
    };
    if (int e = layer(3, G0, a4, nullptr, G1)) return e;   // d pre(a4)
    if (int e = layer(2, G1, x2, G0, G2)) return e;        // d pre(x2)
    if (int e = layer(1, G2, a2, nullptr, G0)) return e;   // d pre(a2)
    if (int e = layer(0, G0, x1, G2, G1)) return e;        // d pre(x1)
    if (int e = launch_wgrad_thin<false>(g, G1, n, h, w, part, grad + OFF_C1, red, s)) return e;
    return launch_reduce(red, s);
}

int cnn_loss(const float *p, const float *t, const float *mask, int64_t count, double *L_dev, float *dp, void *ws,
             size_t ws_bytes, sg_stream_t stream)
{
    if (!p || !t || !mask || !L_dev || !ws) return fail(SG_EINVAL, "NULL pointer argument");
    if (count < 1) return fail(SG_EINVAL, "count must be positive");
    const CnnLayout L = cnn_layout(1, 1, 1);
    if (ws_bytes < L.total) return fail(SG_EINVAL, "workspace too small (%zu < %zu bytes)", ws_bytes, L.total);
    // the reduction area sits at the end of every layout; use the last bytes
    double *part = (double *)((char *)ws + ws_bytes / ALIGN * ALIGN - up((2 * MAX_WG_LOSS + 2) * sizeof(double)));
    hipStream_t s = (hipStream_t)stream;
    long long nwg = (count + 1023) / 1024;  // 4 elements per thread (16 left half the CUs without work on 8 x 256^2)
    if (nwg > MAX_WG_LOSS) nwg = MAX_WG_LOSS;
    const long long per = (count + nwg - 1) / nwg;
    nwg = (count + per - 1) / per;
    loss_partial_kernel<<<(unsigned)nwg, 256, 0, s>>>(p, t, mask, count, per, part);
    HIPCHECK(hipGetLastError());
    double *cnt = part + 2 * MAX_WG_LOSS;
    loss_final_kernel<<<1, 256, 0, s>>>(part, (int)nwg, L_dev, cnt);
    HIPCHECK(hipGetLastError());
    if (dp) {
        loss_grad_kernel<<<blocks(count), 256, 0, s>>>(p, t, mask, count, cnt, dp);
        HIPCHECK(hipGetLastError());
    }
    return SG_OK;
}

int cnn_adam(float *params, const float *grad, float *m, float *v, int64_t n, float lr, float beta1, float beta2,
             float eps, int32_t step, sg_stream_t stream)
{
    if (!params || !grad || !m || !v) return fail(SG_EINVAL, "NULL pointer argument");
    if (n < 1 || step < 1) return fail(SG_EINVAL, "n and step must be positive");
    if (!(beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f && eps > 0.f))
        return fail(SG_EINVAL, "Adam needs 0 <= beta < 1 and eps > 0");
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, step)));
    adam_kernel<<<blocks(n), 256, 0, (hipStream_t)stream>>>(params, grad, m, v, n, lr, beta1, beta2, eps, c1, c2);
    HIPCHECK(hipGetLastError());
    return SG_OK;
}

int cnn_pack(const float *a, const float *b, int32_t nsrc, const int32_t *order, int32_t nfields, int32_t fh,
             int32_t fw, int32_t frame, int32_t normalise, double *inv_rms, float *patches, float *mask,
             sg_stream_t stream)
{
    if (!a || !patches) return fail(SG_EINVAL, "NULL pointer argument");
    if (nfields < 1 || nsrc < 1 || fh < 1 || fw < 1 || frame < fh || frame < fw)
        return fail(SG_EINVAL, "need nfields, nsrc, fh, fw >= 1 and fh, fw <= frame");
    if (normalise && !inv_rms) return fail(SG_EINVAL, "normalise needs inv_rms");
    hipStream_t s = (hipStream_t)stream;
    if (normalise) {
        field_inv_rms_kernel<<<nfields, 256, 0, s>>>(a, b, nsrc, order, fh, fw, inv_rms);
        HIPCHECK(hipGetLastError());
    }
    const long long total = (long long)((nfields + 3) / 4) * 4 * frame * frame;
    auto pack = total < (1ll << 31) ? pack_kernel<unsigned> : pack_kernel<unsigned long long>;
    pack<<<blocks(total), 256, 0, s>>>(a, b, nsrc, order, nfields, fh, fw, frame, normalise ? inv_rms : nullptr, patches,
                                       mask, total);
    HIPCHECK(hipGetLastError());
    return SG_OK;
}

int cnn_unpack(const float *patches, int32_t nfields, int32_t fh, int32_t fw, int32_t frame, float *fields,
               sg_stream_t stream)
{
    if (!patches || !fields) return fail(SG_EINVAL, "NULL pointer argument");
    if (nfields < 1 || fh < 1 || fw < 1 || frame < fh || frame < fw)
        return fail(SG_EINVAL, "need nfields, fh, fw >= 1 and fh, fw <= frame");
    const long long total = (long long)nfields * fh * fw;
    auto unpack = total < (1ll << 31) ? unpack_kernel<unsigned> : unpack_kernel<unsigned long long>;
    unpack<<<blocks(total), 256, 0, (hipStream_t)stream>>>(patches, nfields, fh, fw, frame, fields);
    HIPCHECK(hipGetLastError());
    return SG_OK;
}

int cnn_conv3x3(const uint16_t *x, int32_t n, int32_t h, int32_t w, const uint16_t *wgt, const float *bias,
                const uint16_t *res, const uint16_t *gate, int32_t relu, uint16_t *y, float *y32, sg_stream_t stream)
{
    if (int e = check_dims(n, h, w)) return e;
    if (!x || !wgt || !y) return fail(SG_EINVAL, "NULL pointer argument");
    if (!aligned16(x) || !aligned16(wgt) || !aligned16(res) || !aligned16(gate) || !aligned16(y) || !aligned16(y32))
        return fail(SG_EINVAL, "x, wgt, res, gate, y and y32 must be 16-byte aligned");
    return launch_conv<false>(x, n, h, w, wgt, bias, res, gate, relu, y, y32, (hipStream_t)stream);
}

int cnn_conv3x3_wgrad(const uint16_t *dy, const uint16_t *x, int32_t n, int32_t h, int32_t w, float *dw, void *ws,
                      size_t ws_bytes, sg_stream_t stream)
{
    if (int e = check_dims(n, h, w)) return e;
    if (!dy || !x || !dw || !ws) return fail(SG_EINVAL, "NULL pointer argument");
    if (!aligned16(dy) || !aligned16(x)) return fail(SG_EINVAL, "dy and x must be 16-byte aligned");
    const CnnLayout L = cnn_layout(1, 1, 1);
    if (ws_bytes < L.total) return fail(SG_EINVAL, "workspace too small (%zu < %zu bytes)", ws_bytes, L.total);
    Reduce red;
    if (int e = launch_wgrad(dy, x, n, h, w, (float *)((char *)ws + L.part), dw, red, (hipStream_t)stream)) return e;
    return launch_reduce(red, (hipStream_t)stream);
}

} // extern "C"
