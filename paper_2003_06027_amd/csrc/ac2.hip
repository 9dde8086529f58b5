// ac2.hip -- gfx950 kernels of the 2-D acoustic recursion and its adjoint.
//
// Forward step k (paper: U_{k+1} = A(theta) U_k + F_k, Eq. (1); PDE Eq. (12)
// in the constant-density form u_tt = c^2 lap(u) + f with an auxiliary-field
// absorbing layer).  In scaled variables (chat = dt^2 c^2/dx^2, phi~ = dx*phi,
// h = zeta dt/2, L~ and D~ the 8th-order stencils without the 1/dx factors):
//   pass A (layer cells only):
//     phi~_j^k = p_j phi~_j^{k-1} + q_j D~_j u^k,   p_j = (1-h_j)/(1+h_j),
//                                                  q_j = 2(h_other - h_j)/(1+h_j)
//   pass B (every cell):
//     w~^k    = L~ u^k + D~_x phi~_x^k + D~_z phi~_z^k
//     u^{k+1} = alpha (beta u^k - gamma u^{k-1} + chat w~^k + dt^2 f^k)
// with alpha = 1/(1+h_x+h_z), beta = 2 - 4 h_x h_z, gamma = 1 - h_x - h_z
// (1, 2, 1 in the interior).  The stored state after step k is
// (u^{k+1}, u^k, phi~^k); outside the layer phi~ stays exactly zero.
// Tiles more than 4 cells from the layer ("interior" tiles) skip the phi
// terms and the damping coefficients.  The others ("near" tiles) run pass A
// themselves on the tile + 4, from u^k on the tile + 8 in LDS, then pass B
// from LDS: phi~^k of a cell is then computed by its own tile and by the
// neighbours whose ring covers it (the same expression, the same value),
// and written by its own tile only, into the other buffer of a pair
// (phi~^{k-1} and phi~^k live in different buffers, so a neighbour that
// still reads phi~^{k-1} of the cell is not disturbed).
//
// Adjoint step k (Eq. (4): lambda_k = A^T lambda_{k+1} + residual; Eq. (5)
// for the gradient), in the alpha-scaled variable s = alpha * dJ/du and the
// q-scaled layer adjoint c_j = q_j * dJ/dphi~_j (q is constant in time, so
// c obeys the same recursion as dJ/dphi~ multiplied by q):
//   pass A (layer cells):
//     c_j^{k+1} = p_j c_j^{k+2} - q_j D~_j(chat s^{k+2})
//   pass B (every cell):
//     a^{k+1} = R^T dJ/dd^{k+1} - D~_x c_x^{k+1} - D~_z c_z^{k+1}
//               + beta s^{k+2} + L~(chat s^{k+2}) - gamma s^{k+3}
//     s^{k+1} = alpha a^{k+1};   dJ/dchat += s^{k+1} w~^k
// using L~^T = L~ and D~^T = -D~ (zero cells beyond the grid).  Near tiles
// fold pass A in as in the forward step (chat s^{k+2} on the tile + 8 in
// LDS; c^{k+2} and c^{k+1} in the two buffers of a pair).
//
// Cache policy: an operand that only its own cell reads or writes in a step
// (u^{k-1} and s^{k+3} in the one-step kernels, the new wavefields, the
// snapshots, the gradient accumulators) is loaded and stored non-temporally,
// so that it does not displace what neighbouring tiles share (u^k, chat s,
// chat, the layer auxiliaries).  A load that the ring of a neighbouring tile
// repeats (u^{k-1}, s^{k+3} in the blocked kernels) stays cached: streaming
// it made the blocked adjoint 2 % slower.
#include "sg_internal.h"

#include <type_traits>

namespace sg {

// 8th-order centred weights: second derivative (a_1..a_4; the centre weight
// -205/72 = -2 sum a_m is folded into the difference form below) and first
// derivative.
constexpr float A1 = (float)(8.0 / 5.0);
constexpr float A2 = (float)(-1.0 / 5.0);
constexpr float A3 = (float)(8.0 / 315.0);
constexpr float A4 = (float)(-1.0 / 560.0);
constexpr float D1 = (float)(4.0 / 5.0);
constexpr float D2 = (float)(-1.0 / 5.0);
constexpr float D3 = (float)(4.0 / 105.0);
constexpr float D4 = (float)(-1.0 / 280.0);

__device__ __forceinline__ long long fidx(const Grid2 &g, int iz, int ix)
{
    return (long long)(iz + OZ) * g.SX + (ix + OX);
}

// 8th-order Laplacian (x + z) of an LDS tile with row stride W.  The weights
// sum to zero, so L~u = sum_m a_m ((u_{+m} - u_0) + (u_{-m} - u_0)) along each
// axis: neighbour differences of a smooth field are exact or nearly so in
// FP32, which keeps the rounding error proportional to L~u instead of u.
// The multiply-adds are explicit so that every kernel evaluating the
// stencil rounds identically (the one- and two-step paths agree bitwise).
__device__ __forceinline__ float lap8(const float *c, int W)
{
    const float c0 = c[0];
    auto pair = [&](int o) { return (c[o] - c0) + (c[-o] - c0); };
    float t = A4 * (pair(4) + pair(4 * W));
    t = fmaf(A3, pair(3) + pair(3 * W), t);
    t = fmaf(A2, pair(2) + pair(2 * W), t);
    return fmaf(A1, pair(1) + pair(W), t);
}

template <class T>
__device__ __forceinline__ float d8(const T *c, long long s)
{
    return D1 * (c[s] - c[-s]) + D2 * (c[2 * s] - c[-2 * s])
         + D3 * (c[3 * s] - c[-3 * s]) + D4 * (c[4 * s] - c[-4 * s]);
}

// Work id of this workgroup with consecutive ids on one XCD: the hardware
// hands workgroups to the 8 XCDs round-robin, so id b runs on XCD b % 8; the
// remap gives each XCD a contiguous range of (tile, shot) work, which keeps
// neighbouring tiles -- and their shared halos -- in the same L2.
__device__ __forceinline__ int xcd_work_id(int nblocks)
{
    const int b = blockIdx.x;
    const int per = nblocks / NXCD, rem = nblocks % NXCD;
    const int x = b % NXCD, j = b / NXCD;
    return x * per + min(x, rem) + j;
}

// Is a tile within 4 cells of the absorbing layer (its cells need the phi
// terms or damping coefficients)?
__device__ __forceinline__ bool near_layer(const Grid2 &g, int x0, int z0)
{
    return g.P > 0 && (x0 - 4 < g.P || x0 + TX + 4 > g.P + g.nx ||
                       z0 - 4 < g.P || z0 + TZ + 4 > g.P + g.nz);
}

// Rows of a tile per workgroup.  A launch of few tiles is bound by the
// instruction stream of one wavefront, not by the chip: at 32 rows a thread
// of a tile by the layer works through 4 rows of about 200 VALU instructions
// each, 7 us for a launch that leaves most CUs idle.  Tiles are then split
// into 2 or 4 workgroups of 16 or 8 rows (the halo rows loaded and, by the
// layer, their phi terms formed by both neighbours).  Every value is formed
// by the same expression, so results do not depend on the split.
struct TileItem {
    int tile, shot;
    int sub;              // which RW rows of the tile
};

// Item w of a launch over (shot, tile, rows), rows fastest.
template <int RW>
__device__ __forceinline__ TileItem tile_item(const int *tiles, int ntl, int w)
{
    constexpr int NS = TZ / RW;
    const int t = w / NS, shot = t / ntl;
    return TileItem{tiles[t - shot * ntl], shot, w - t * NS};
}

// Fill the (RW+8) x (TX+8) LDS tile: own cells by the caller, the 4-cell
// halo here (value f(frame index)).
template <int RW, int NT, class Fn>
__device__ __forceinline__ void load_halo(const Grid2 &g, float *lds, int x0, int z0, Fn f)
{
    constexpr int H = 4, W = TX + 2 * H;
    constexpr int NH = 2 * H * W + 2 * RW * H;
    for (int i = threadIdx.x; i < NH; i += NT) {
        int r, c;
        if (i < 2 * H * W) {
            const int s = i / W;
            c = i - s * W;
            r = s < H ? s : s + RW;
        } else {
            const int j = i - 2 * H * W;
            const int rr = j / (2 * H), cc = j - rr * (2 * H);
            r = H + rr;
            c = cc < H ? cc : cc + TX;
        }
        lds[r * W + c] = f(fidx(g, z0 - H + r, x0 - H + c));
    }
}

// The source term dt^2 f^k of one node: a separately rounded product, so
// that no kernel fuses it into the addition that injects it (whether the
// compiler would fuse depends on the kernel's shape; every kernel injecting
// a source must round identically for the one- and two-step paths to agree).
__device__ __forceinline__ float src_value(float scale, float w)
{
    float v = scale * w;
    asm("" : "+v"(v));                    // __fmul_rn is fused all the same (8-row tiles by the layer)
    return v;
}

// A layer cell of the padded grid.
__device__ __forceinline__ bool layer_cell_at(const Grid2 &g, int iz, int ix)
{
    return iz < g.P || iz >= g.P + g.nz || ix < g.P || ix >= g.P + g.nx;
}

// Several source nodes per shot: the sum of dt^2/(dx dz) r_j(t_k) over the
// nodes j at each cell of these RW rows, in the LDS array sadd (dynamic, only
// when nsrc > 1).  The entries of a tile are sorted by cell, so one thread
// adds up a cell's run of entries, in entry order; the cells without one hold
// zero.  (Every cell stepping through all entries of its tile, one dependent
// load after another, took 25 us of a 32 us launch at 49 nodes.)  begin()
// reads the tile's range and clears the array before the barrier that
// publishes the tile; fill() runs after it and ends with a barrier.
template <int RW, int NT>
struct NodeSources {
    int b, e;
    __device__ __forceinline__ bool any() const { return b < e; }
    __device__ __forceinline__ void begin(const Ac2FwdArgs &a, const TileItem &it, float *sadd)
    {
        b = e = 0;
        if (a.nsrc <= 1) return;
        const int *off = a.src_off + (long long)it.shot * (a.g.ntx * a.g.ntz + 1);
        b = off[it.tile];
        e = off[it.tile + 1];
        if (!any()) return;
        for (int i = threadIdx.x; i < RW * TX; i += NT) sadd[i] = 0.f;
    }
    __device__ __forceinline__ void fill(const Ac2FwdArgs &a, const TileItem &it, float *sadd) const
    {
        if (!any()) return;               // uniform over the block
        for (int i = b + threadIdx.x; i < e; i += NT) {
            const int cell = src_cell(a.src_ent[i]);
            if (i > b && src_cell(a.src_ent[i - 1]) == cell) continue;    // not first of its cell
            const int own = cell - it.sub * RW * TX;
            if (own < 0 || own >= RW * TX) continue;
            float v = 0.f;
            for (int m = i; m < e && src_cell(a.src_ent[m]) == cell; ++m)
                v += a.src_scale * a.wav[((long long)it.shot * a.nsrc + src_node(a.src_ent[m])) * a.nt + a.k];
            sadd[own] = v;
        }
        __syncthreads();
    }
};

// The receivers of a tile: its entry range and this thread's first entry,
// loaded with the tile's operands so that the dependent loads overlap them.
struct TileRecs {
    int b, e, ent;
    template <class Args>
    __device__ __forceinline__ void begin(const Args &a, const TileItem &it)
    {
        const int *off = a.rec_off + (long long)it.shot * (a.g.ntx * a.g.ntz + 1);
        b = off[it.tile];
        e = off[it.tile + 1];
        ent = 0;
        if (b + (int)threadIdx.x < e) ent = a.rec_ent[b + threadIdx.x];
    }
    __device__ __forceinline__ bool any() const { return b < e; }
};

// Record u^{k+1} of the receivers on these RW rows; val(row, column) reads it
// from LDS.
template <int RW, int NT, class Fn>
__device__ __forceinline__ void record_tile(const Ac2FwdArgs &a, const TileItem &it, const TileRecs &rc, Fn val)
{
    for (int i = rc.b + threadIdx.x; i < rc.e; i += NT) {
        const int ent = i == rc.b + (int)threadIdx.x ? rc.ent : a.rec_ent[i];
        const int own = rec_cell(ent) - it.sub * RW * TX;
        if (own < 0 || own >= RW * TX) continue;
        const int r = own / TX, c = own - r * TX;
        a.seis[((long long)it.shot * a.nt + a.k) * a.nrec + rec_id(ent)] = val(r, c);
    }
}

// Add R^T dJ/dd^{k+1} to the cells of these RW rows (at(row, column) is the
// LDS cell), deterministic per cell: the thread of a cell's first entry adds
// up the run.  d0: the sample of this thread's first entry, loaded early.
template <int RW, int NT, class Fn>
__device__ __forceinline__ void inject_tile(const Ac2AdjArgs &a, const TileItem &it, const TileRecs &rc, float d0,
                                            Fn at)
{
    const float *d = a.dJdd + ((long long)it.shot * a.nt + a.k) * a.nrec;
    for (int i = rc.b + threadIdx.x; i < rc.e; i += NT) {
        const bool pre = i == rc.b + (int)threadIdx.x;
        const int ent = pre ? rc.ent : a.rec_ent[i];
        const int cell = rec_cell(ent), own = cell - it.sub * RW * TX;
        if (own < 0 || own >= RW * TX) continue;
        if (i > rc.b && rec_cell(a.rec_ent[i - 1]) == cell) continue;  // not first of its cell
        float sum = 0.f;
        sum += pre ? d0 : d[rec_id(ent)];
        for (int m = i + 1; m < rc.e && rec_cell(a.rec_ent[m]) == cell; ++m) sum += d[rec_id(a.rec_ent[m])];
        const int r = own / TX, c = own - r * TX;
        at(r, c) += sum;
    }
}

__device__ __forceinline__ float first_sample(const Ac2AdjArgs &a, const TileItem &it, const TileRecs &rc)
{
    return rc.b + (int)threadIdx.x < rc.e
               ? a.dJdd[((long long)it.shot * a.nt + a.k) * a.nrec + rec_id(rc.ent)] : 0.f;
}

// Several source nodes per shot: the wavelet gradient of the nodes on these
// RW rows, scale * s^{k+1}; own(row offset j) is this thread's s^{k+1}, put
// into LDS at at(row, column).  (As a launch of its own: 1.4 us of every step.)
template <int RW, int NT, class Fo, class Fn>
__device__ __forceinline__ void gather_nodes(const Ac2AdjArgs &a, const TileItem &it, Fo own, Fn at)
{
    if (a.nsrc <= 1 || !a.gwav) return;
    const int *off = a.src_off + (long long)it.shot * (a.g.ntx * a.g.ntz + 1);
    const int b = off[it.tile], e = off[it.tile + 1];
    if (b >= e) return;                   // uniform over the block
    constexpr int RPT = RW * TX / NT;
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < RPT; ++j) at(ly * RPT + j, lx) = own(j);
    __syncthreads();
    for (int i = b + threadIdx.x; i < e; i += NT) {
        const int ent = a.src_ent[i], cell = src_cell(ent) - it.sub * RW * TX;
        if (cell < 0 || cell >= RW * TX) continue;
        a.gwav[((long long)it.shot * a.nsrc + src_node(ent)) * a.nt + a.k] = a.src_scale * at(cell / TX, cell % TX);
    }
}

__global__ void ac2_src_gather_kernel(int nshots, int nsrc, long long plane, const long long *node_f,
                                      const float *s1, float *gw, int nt, int k, float scale)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nshots * nsrc) return;
    const int shot = i / nsrc;
    gw[(long long)i * nt + k] = scale * s1[(long long)shot * plane + node_f[i]];
}

void launch_ac2_src_gather(int nshots, int nsrc, long long plane, const long long *node_f, const float *s1,
                           float *gw, int nt, int k, float scale, hipStream_t s)
{
    const int n = nshots * nsrc;
    ac2_src_gather_kernel<<<(n + 255) / 256, 256, 0, s>>>(nshots, nsrc, plane, node_f, s1, gw, nt, k, scale);
}

// ------------------------------------------------------------ forward pass B
// RW rows of a tile away from the layer (the interior update), u^k with a
// 4-cell halo in LDS.
template <int RW, int NT, bool SNAP, bool REC>
__device__ __forceinline__ void fwd_tile(const Ac2FwdArgs &a, float *su, float *sadd, const TileItem &it)
{
    constexpr int H = 4, W = TX + 2 * H, RPT = RW * TX / NT;
    const Grid2 &g = a.g;
    const int shot = it.shot;
    const int tz = it.tile / g.ntx, tx = it.tile - tz * g.ntx;
    const int x0 = tx * TX, z0 = tz * TZ + it.sub * RW;
    if (z0 >= g.NZ) return;
    const long long so = (long long)shot * g.plane;
    const float *u = a.u + so;
    const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX;
    const int ix = x0 + lx;

    NodeSources<RW, NT> ns;
    ns.begin(a, it, sadd);
    TileRecs rc{};
    if constexpr (REC) rc.begin(a, it);
    float uc[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int r = ly * RPT + j;
        uc[j] = u[fidx(g, z0 + r, ix)];
        su[(r + H) * W + lx + H] = uc[j];
    }
    load_halo<RW, NT>(g, su, x0, z0, [&](long long f) { return u[f]; });
    __syncthreads();
    ns.fill(a, it, sadd);

    const float *chat = a.chat + (long long)(shot / a.shots_per_model) * g.plane;
    const float *um = a.um + so;
    float *uo = a.un + so;
    const long long src = a.src_f[shot];
    const float sval = src_value(a.src_scale, a.wav[(long long)shot * a.nt + a.k]);
    float un[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int r = ly * RPT + j, iz = z0 + r;
        const long long f = fidx(g, iz, ix);
        float w = lap8(su + (r + H) * W + lx + H, W);
        un[j] = 0.f;
        if (iz < g.NZ && ix < g.NX) {
            // 2u - um + chat w = u + ((u - um) + chat w)
            float inc = fmaf(chat[f], w, uc[j] - __builtin_nontemporal_load(um + f));
            if (f == src) inc += sval;
            if (ns.any()) inc += sadd[r * TX + lx];
            const float v = uc[j] + inc;
            __builtin_nontemporal_store(v, uo + f);
            un[j] = v;
            if constexpr (SNAP) __builtin_nontemporal_store(w, a.snap + so + f);
        }
    }

    if constexpr (REC) {
        if (rc.any()) {                   // uniform over the block
            __syncthreads();
#pragma unroll
            for (int j = 0; j < RPT; ++j) su[(ly * RPT + j + H) * W + lx + H] = un[j];
            __syncthreads();
            record_tile<RW, NT>(a, it, rc, [&](int r, int c) { return su[(r + H) * W + c + H]; });
        }
    }
}

// One forward step on a list of tiles away from the layer.
template <int RW, bool SNAP, bool REC>
__global__ __launch_bounds__(NTH) void ac2_fwd_kernel(Ac2FwdArgs a)
{
    __shared__ float su[(RW + 8) * (TX + 8)];
    extern __shared__ float sadd[];
    const int w = xcd_work_id(a.ntl * a.nshots * (TZ / RW));
    fwd_tile<RW, NTH, SNAP, REC>(a, su, sadd, tile_item<RW>(a.tiles, a.ntl, w));
}

// ------------------------------------------------------------ adjoint pass B
// RW rows of a tile away from the layer, chat s^{k+2} with a 4-cell halo in LDS.
template <int RW, int NT>
__device__ __forceinline__ void adj_tile(const Ac2AdjArgs &a, float *sc, const TileItem &it)
{
    constexpr int H = 4, W = TX + 2 * H, RPT = RW * TX / NT;
    const Grid2 &g = a.g;
    const int shot = it.shot;
    const int tz = it.tile / g.ntx, tx = it.tile - tz * g.ntx;
    const int x0 = tx * TX, z0 = tz * TZ + it.sub * RW;
    if (z0 >= g.NZ) return;
    const long long so = (long long)shot * g.plane;
    const float *s2 = a.s2 + so;
    const float *chat = a.chat + (long long)(shot / a.shots_per_model) * g.plane;
    const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX;
    const int ix = x0 + lx;

    TileRecs rc{};
    rc.begin(a, it);
    float sc2[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int r = ly * RPT + j;
        const long long f = fidx(g, z0 + r, ix);
        sc2[j] = s2[f];
        sc[(r + H) * W + lx + H] = chat[f] * sc2[j];
    }
    load_halo<RW, NT>(g, sc, x0, z0, [&](long long f) { return chat[f] * s2[f]; });
    __syncthreads();
    const float d0 = first_sample(a, it, rc);

    const float *s3 = a.s3 + so;
    float *s1o = a.s1 + so;
    float av[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int r = ly * RPT + j, iz = z0 + r;
        float v = lap8(sc + (r + H) * W + lx + H, W);
        if (iz < g.NZ && ix < g.NX) {
            const long long f = fidx(g, iz, ix);
            v += sc2[j] + (sc2[j] - __builtin_nontemporal_load(s3 + f));
        }
        av[j] = v;
    }

    if (rc.any()) {   // receiver residual injection, uniform over the block
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RPT; ++j) sc[(ly * RPT + j + H) * W + lx + H] = av[j];
        __syncthreads();
        inject_tile<RW, NT>(a, it, rc, d0, [&](int r, int c) -> float & { return sc[(r + H) * W + c + H]; });
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RPT; ++j) av[j] = sc[(ly * RPT + j + H) * W + lx + H];
    }

    const long long src = a.src_f[shot];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int r = ly * RPT + j, iz = z0 + r;
        if (iz < g.NZ && ix < g.NX) {
            const long long f = fidx(g, iz, ix);
            const float s1 = av[j];
            __builtin_nontemporal_store(s1, s1o + f);
            __builtin_nontemporal_store(fmaf(s1, __builtin_nontemporal_load(a.snap + so + f), __builtin_nontemporal_load(a.grad + so + f)), a.grad + so + f);
            if (a.gwav && f == src) a.gwav[(long long)shot * a.nt + a.k] = s1 * a.src_scale;
        }
    }
    gather_nodes<RW, NT>(a, it, [&](int j) { return av[j]; },
                         [&](int r, int c) -> float & { return sc[(r + H) * W + c + H]; });
}

// (8 waves per SIMD: 64 VGPRs, no spill; measured 2 % faster than the
// compiler's choice of 70.  The forward's one-step variants are slower at 8.)
template <int RW>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(8))) void ac2_adj_kernel(Ac2AdjArgs a)
{
    __shared__ float sc[(RW + 8) * (TX + 8)];
    const int w = xcd_work_id(a.ntl * a.nshots * (TZ / RW));
    adj_tile<RW, NTH>(a, sc, tile_item<RW>(a.tiles, a.ntl, w));
}

// ---------------------------------------------------------- two-step kernels
// Blocked tiles: the tile and its 8-cell halo are physical cells, so pass A
// and every layer term vanish there and the forward update reduces to
// u^{k+1} = u^k + ((u^k - u^{k-1}) + chat w~^k) (+ source).  One launch
// forms u^{k+1} on the tile + 4 in LDS from u^k on the tile + 8, then
// u^{k+2} on the tile: two steps for one read of u^k, u^{k-1} and chat and
// one write of u^{k+1}, u^{k+2}.  Each value is computed with exactly the
// operations of the single-step kernel, so results agree bit for bit.
constexpr int H2 = 8;                       // u^k halo of a blocked tile
constexpr int W0 = TX + 2 * H2, W1 = TX + 8;
// of RW rows of a tile: rows of the tile + 8 and + 4, cells of the 4-cell ring around them
constexpr int rows0(int RW) { return RW + 2 * H2; }
constexpr int rows1(int RW) { return RW + 8; }
constexpr int nring(int RW) { return rows1(RW) * W1 - RW * TX; }
// The forward blocked tiles take NTB threads (RB rows each): 8 waves per
// SIMD in 55 VGPRs against 5 at 256 threads (C2: 141 -> 136 us per launch).
// The blocked adjoint takes 256 threads in a launch of its own (512 ran 2 %
// slower: 195 -> 199 us) and the step's 512 in one grid with the tiles by the layer,
// where what the shared grid saves is more (64 shots, whole pass: 454 us per step
// apart, 451 so).
constexpr int NTB = 512;
static_assert(8 * TX % NTB == 0 && NTB % TX == 0, "whole rows per thread");

// The tile + 8 of a field (rows start 32-byte aligned: x0 - 8 + OX is a
// multiple of 8) straight from global memory into LDS:
// 16 bytes per lane and load, item q into the 16-byte slot q (the LDS rows
// of W0 floats have no padding, so item order is slot order).  Every cell
// lies inside the zero frame.  The caller waits for the loads
// (s_waitcnt) before the barrier that publishes the tile.
template <int RW, int NT>
__device__ __forceinline__ void dma_tile8(const Grid2 &g, const float *u, float *lds, int x0, int z0)
{
    constexpr int Q = W0 / 4, N4 = rows0(RW) * Q;
#pragma unroll
    for (int it = 0; it < (N4 + NT - 1) / NT; ++it) {
        const int q = threadIdx.x + it * NT;
        if (q < N4) {
            const int r = q / Q, c = (q - r * Q) * 4;
            __builtin_amdgcn_global_load_lds((const void *)(u + fidx(g, z0 - H2 + r, x0 - H2 + c)),
                                             (void __attribute__((address_space(3))) *)(lds + (it * NT + (threadIdx.x & ~63)) * 4),
                                             16, 0, 0);
        }
    }
}

// The product chat * s on the tile + 8 in two phases: dma_product_load puts
// s straight into LDS (as dma_tile8) and chat of the same 16-byte items into
// registers; after the caller's wait and barrier, product_in_place multiplies
// each thread's items in LDS (one FP32 product per cell, chat times s).  The
// caller synchronises again before the tile is read.
template <int RW, int NT>
__device__ __forceinline__ void dma_product_load(const Grid2 &g, const float *s, const float *mul, float *lds,
                                                 int x0, int z0, float4 (&m)[(rows0(RW) * (W0 / 4) + NT - 1) / NT])
{
    constexpr int Q = W0 / 4, N4 = rows0(RW) * Q;
#pragma unroll
    for (int it = 0; it < (N4 + NT - 1) / NT; ++it) {
        const int q = threadIdx.x + it * NT;
        if (q < N4) {
            const int r = q / Q, c = (q - r * Q) * 4;
            const long long f = fidx(g, z0 - H2 + r, x0 - H2 + c);
            __builtin_amdgcn_global_load_lds((const void *)(s + f),
                                             (void __attribute__((address_space(3))) *)(lds + (it * NT + (threadIdx.x & ~63)) * 4),
                                             16, 0, 0);
            m[it] = *reinterpret_cast<const float4 *>(mul + f);
        }
    }
}

template <int RW, int NT>
__device__ __forceinline__ void product_in_place(float *lds, const float4 (&m)[(rows0(RW) * (W0 / 4) + NT - 1) / NT])
{
    constexpr int N4 = rows0(RW) * (W0 / 4);
#pragma unroll
    for (int it = 0; it < (N4 + NT - 1) / NT; ++it) {
        const int q = threadIdx.x + it * NT;
        if (q < N4) {
            float4 v = *reinterpret_cast<const float4 *>(lds + 4 * q);
            v.x = m[it].x * v.x; v.y = m[it].y * v.y; v.z = m[it].z * v.z; v.w = m[it].w * v.w;
            *reinterpret_cast<float4 *>(lds + 4 * q) = v;
        }
    }
}

// Cell i of the ring (the first and last 4 rows of the rows + 4, then columns
// 0-3 and 68-71 of the rows between), as (row, column) of the rows + 4.
template <int RW>
__device__ __forceinline__ void ring_cell(int i, int &r, int &c)
{
    if (i < 8 * W1) {
        const int rr = i / W1;
        r = rr < 4 ? rr : rr + RW;
        c = i - rr * W1;
    } else {
        const int j = i - 8 * W1, cc = j & 7;
        r = 4 + (j >> 3);
        c = cc < 4 ? cc : cc + TX;
    }
}

// s0: u^k on the rows + 8 (rows0 x W0), s1: u^{k+1} on the rows + 4 (rows1 x W1)
template <int RW>
__device__ __forceinline__ void fwd2_tile(const Ac2Fwd2Args &a, float *s0, float *s1, const TileItem &it)
{
    constexpr int RB = RW * TX / NTB, NRING = nring(RW), RING_ITB = (NRING + NTB - 1) / NTB;
    const Grid2 &g = a.g;
    const int shot = it.shot;
    const int tz = it.tile / g.ntx, tx = it.tile - tz * g.ntx;
    const int x0 = tx * TX, z0 = tz * TZ + it.sub * RW;
    const long long so = (long long)shot * g.plane;
    const float *um = a.um + so;
    const float *chat = a.chat + (long long)(shot / a.shots_per_model) * g.plane;
    const long long src = a.src_f[shot];
    const float sv0 = src_value(a.src_scale, a.wav[(long long)shot * a.nt + a.k]);
    const float sv1 = src_value(a.src_scale, a.wav[(long long)shot * a.nt + a.k + 1]);
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;

    // own cells: column lx, rows ly*RB .. +RB-1; their chat and u^{k-1} first
    float ch[RB], pm[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const long long f = fidx(g, z0 + ly * RB + j, x0 + lx);
        ch[j] = chat[f];
        pm[j] = um[f];
    }
    // ring cells of the tile + 4
    float rch[RING_ITB], rpm[RING_ITB];
    long long rf[RING_ITB];
#pragma unroll
    for (int q = 0; q < RING_ITB; ++q) {
        const int i = threadIdx.x + q * NTB;
        rf[q] = -1;
        if (i < NRING) {
            int r, c;
            ring_cell<RW>(i, r, c);
            rf[q] = fidx(g, z0 - 4 + r, x0 - 4 + c);
            rch[q] = chat[rf[q]];
            rpm[q] = um[rf[q]];
        }
    }
    dma_tile8<RW, NTB>(g, a.u0 + so, s0, x0, z0);
    __builtin_amdgcn_s_waitcnt(0);       // the tile's direct loads have landed in LDS
    __syncthreads();

    // step k: u^{k+1} on the tile + 4 (own cells, then the ring)
    float uk[RB], u1[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const int r = ly * RB + j;
        const long long f = fidx(g, z0 + r, x0 + lx);
        const float *cc = s0 + (r + H2) * W0 + lx + H2;
        const float wk = lap8(cc, W0);
        uk[j] = cc[0];
        float inc = fmaf(ch[j], wk, uk[j] - pm[j]);
        if (f == src) inc += sv0;
        u1[j] = uk[j] + inc;
        s1[(r + 4) * W1 + lx + 4] = u1[j];
        __builtin_nontemporal_store(u1[j], a.u1 + so + f);
        if (a.snap0) __builtin_nontemporal_store(wk, a.snap0 + so + f);
    }
#pragma unroll
    for (int q = 0; q < RING_ITB; ++q) {
        const int i = threadIdx.x + q * NTB;
        if (i < NRING) {
            int r, c;
            ring_cell<RW>(i, r, c);
            const float *cc = s0 + (r + 4) * W0 + c + 4;
            const float wk = lap8(cc, W0);
            const float u = cc[0];
            float inc = fmaf(rch[q], wk, u - rpm[q]);
            if (rf[q] == src) inc += sv0;
            s1[r * W1 + c] = u + inc;
        }
    }
    __syncthreads();

    // step k+1 on the tile
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const int r = ly * RB + j;
        const long long f = fidx(g, z0 + r, x0 + lx);
        const float wk = lap8(s1 + (r + 4) * W1 + lx + 4, W1);
        float inc = fmaf(ch[j], wk, u1[j] - uk[j]);
        if (f == src) inc += sv1;
        __builtin_nontemporal_store(u1[j] + inc, a.u2 + so + f);
        if (a.snap1) __builtin_nontemporal_store(wk, a.snap1 + so + f);
    }
}

template <int RW>
__global__ __launch_bounds__(NTB) void ac2_fwd2_kernel(Ac2Fwd2Args a)
{
    __shared__ __attribute__((aligned(16))) float s0[rows0(RW) * W0];
    __shared__ float s1[rows1(RW) * W1];
    const int w = xcd_work_id(a.ntl * a.nshots * (TZ / RW));
    fwd2_tile<RW>(a, s0, s1, tile_item<RW>(a.tiles, a.ntl, w));
}

// Adjoint steps k and k-1 on blocked tiles (no receivers within 4 cells):
// s^{k+1} on the tile + 4 from chat s^{k+2} on the tile + 8, then s^k on
// the tile; the gradient gets s^{k+1} w~^k, then s^k w~^{k-1}, as in two
// single steps.
// p0: chat s^{k+2} on the rows + 8 (rows0 x W0), p1: chat s^{k+1} on the rows + 4 (rows1 x W1)
template <int RW, int NT>
__device__ __forceinline__ void adj2_tile(const Ac2Adj2Args &a, float *p0, float *p1, const TileItem &item)
{
    constexpr int RPT = RW * TX / NT, NRING = nring(RW), RING_IT = (NRING + NT - 1) / NT;
    const Grid2 &g = a.g;
    const int shot = item.shot, tz = item.tile / g.ntx, tx = item.tile - tz * g.ntx;
    const int x0 = tx * TX, z0 = tz * TZ + item.sub * RW;
    const long long so = (long long)shot * g.plane;
    const float *s2 = a.s2 + so, *s3 = a.s3 + so;
    const float *chat = a.chat + (long long)(shot / a.shots_per_model) * g.plane;
    const long long src = a.src_f[shot];
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;

    float ch[RPT], q2[RPT], q3[RPT], gr[RPT], w1[RPT], w0[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const long long f = fidx(g, z0 + ly * RPT + j, x0 + lx);
        ch[j] = chat[f];
        q2[j] = s2[f];
        q3[j] = s3[f];
        gr[j] = __builtin_nontemporal_load(a.grad + so + f);
        w1[j] = __builtin_nontemporal_load(a.snap1 + so + f);
        w0[j] = __builtin_nontemporal_load(a.snap0 + so + f);
    }
    float rch[RING_IT], rq2[RING_IT], rq3[RING_IT];
#pragma unroll
    for (int it = 0; it < RING_IT; ++it) {
        const int i = threadIdx.x + it * NT;
        if (i < NRING) {
            int r, c;
            ring_cell<RW>(i, r, c);
            const long long f = fidx(g, z0 - 4 + r, x0 - 4 + c);
            rch[it] = chat[f];
            rq2[it] = s2[f];
            rq3[it] = s3[f];
        }
    }
    float4 cm[(rows0(RW) * (W0 / 4) + NT - 1) / NT];
    dma_product_load<RW, NT>(g, s2, chat, p0, x0, z0, cm);
    __builtin_amdgcn_s_waitcnt(0);       // the tile's direct loads have landed in LDS
    __syncthreads();
    product_in_place<RW, NT>(p0, cm);
    __syncthreads();

    // step k: s^{k+1} on the tile + 4
    float v1[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int r = ly * RPT + j;
        const long long f = fidx(g, z0 + r, x0 + lx);
        float v = lap8(p0 + (r + H2) * W0 + lx + H2, W0);
        v += q2[j] + (q2[j] - q3[j]);
        v1[j] = v;
        p1[(r + 4) * W1 + lx + 4] = ch[j] * v;
        __builtin_nontemporal_store(v, a.o1 + so + f);
        if (a.gwav && f == src) a.gwav[(long long)shot * a.nt + a.k] = v * a.src_scale;
    }
#pragma unroll
    for (int it = 0; it < RING_IT; ++it) {
        const int i = threadIdx.x + it * NT;
        if (i < NRING) {
            int r, c;
            ring_cell<RW>(i, r, c);
            float v = lap8(p0 + (r + 4) * W0 + c + 4, W0);
            v += rq2[it] + (rq2[it] - rq3[it]);
            p1[r * W1 + c] = rch[it] * v;
        }
    }
    __syncthreads();

    // step k-1 on the tile
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int r = ly * RPT + j;
        const long long f = fidx(g, z0 + r, x0 + lx);
        float v = lap8(p1 + (r + 4) * W1 + lx + 4, W1);
        v += v1[j] + (v1[j] - q2[j]);
        __builtin_nontemporal_store(v, a.o0 + so + f);
        float t = fmaf(v1[j], w1[j], gr[j]);
        __builtin_nontemporal_store(fmaf(v, w0[j], t), a.grad + so + f);
        if (a.gwav && f == src) a.gwav[(long long)shot * a.nt + a.k - 1] = v * a.src_scale;
    }
}

template <int RW>
__global__ __launch_bounds__(NTH) void ac2_adj2_kernel(Ac2Adj2Args a)
{
    __shared__ __attribute__((aligned(16))) float p0[rows0(RW) * W0];
    __shared__ float p1[rows1(RW) * W1];
    const int w = xcd_work_id(a.ntl * a.nshots * (TZ / RW));
    adj2_tile<RW, NTH>(a, p0, p1, tile_item<RW>(a.tiles, a.ntl, w));
}

// ---------------------------------------------------------------- near tiles
// The tiles within 4 cells of the layer, with pass A folded in.  LDS: the stepped field on
// the tile + 8 (as the blocked kernels stage it), the x auxiliary on the
// tile's rows x the tile + 4 columns, the z auxiliary on the tile + 4 rows x
// the tile's columns.
// Every value is formed by the same expression as in separate passes, so
// results do not depend on which tile computes a ring cell.  NTN threads per
// tile (RN rows each): the LDS arrays cap the workgroups per CU, so a
// larger workgroup keeps more waves resident.
constexpr int WPX = TX + 8;      // x auxiliary: columns x0 - 4 .. x0 + TX + 3
constexpr int NTN = 512;         // threads of a near tile
static_assert(8 * TX % NTN == 0 && NTN % TX == 0, "whole rows per thread");
constexpr int nu8(int RW) { return rows0(RW) * W0; }      // the field on the rows + 8
constexpr int npx(int RW) { return RW * WPX; }            // x auxiliary
constexpr int npz(int RW) { return (RW + 8) * TX; }       // z auxiliary: rows z0 - 4 .. z0 + RW + 3

// Halo cells of the auxiliaries' LDS arrays: the 4 + 4 columns of the x
// array beside the tile (RW x 8, at most one per thread) and the 4 + 4 rows
// of the z array above and below it (8 x TX, one per thread).
constexpr int NHZ = 8 * TX;
static_assert(TZ * 8 <= NTN && NHZ <= NTN, "one halo cell of each array per thread");

__device__ __forceinline__ void halo_x_cell(int i, int &r, int &c)
{
    r = i >> 3;
    const int cc = i & 7;
    c = cc < 4 ? cc : cc + TX;           // column of the x array (x0 - 4 + c)
}

template <int RW>
__device__ __forceinline__ void halo_z_cell(int i, int &r, int &c)
{
    const int rr = i / TX;
    c = i - rr * TX;
    r = rr < 4 ? rr : rr + RW;           // row of the z array (z0 - 4 + r)
}

template <int RW, bool SNAP, bool REC>
__device__ __forceinline__ void fwd_near_tile(const Ac2FwdArgs &a, float *su, float *sx, float *sz, float *sadd,
                                              const TileItem &it)
{
    constexpr int RN = RW * TX / NTN, NHX = RW * 8;
    const Grid2 &g = a.g;
    const int shot = it.shot;
    const int tz = it.tile / g.ntx, tx = it.tile - tz * g.ntx;
    const int x0 = tx * TX, z0 = tz * TZ + it.sub * RW;
    if (z0 >= g.NZ) return;
    const long long so = (long long)shot * g.plane;
    // ly is uniform over a wavefront (TX lanes): rows and their tables in scalar registers
    const int tid = threadIdx.x, lx = tid % TX, ly = __builtin_amdgcn_readfirstlane(tid / TX);
    const int ix = x0 + lx;
    const bool inx = ix < g.NX;
    const float *__restrict__ chat = a.chat + (long long)(shot / a.shots_per_model) * g.plane;
    const float *__restrict__ um = a.um + so;
    const float *__restrict__ phx0 = a.phx0 + so;
    const float *__restrict__ phz0 = a.phz0 + so;
    float *__restrict__ phx = a.phx + so;
    float *__restrict__ phz = a.phz + so;

    NodeSources<RW, NTN> ns;
    ns.begin(a, it, sadd);
    TileRecs rc{};
    if constexpr (REC && RW < TZ) rc.begin(a, it);
    // operands of the own cells and of the halo cells first (none depends on LDS)
    const float hxc = inx ? a.hx[ix] : 0.f, pxc = inx ? a.px[ix] : 0.f, ihxc = inx ? a.ihx[ix] : 0.f;
    float ch[RN], pm[RN], hzr[RN], fx[RN], fz[RN], pzr[RN], ihzr[RN];
    unsigned lay = 0u;
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int iz = z0 + ly * RN + j;
        const long long f = fidx(g, iz, ix);
        ch[j] = pm[j] = hzr[j] = fx[j] = fz[j] = 0.f;
        pzr[j] = iz < g.NZ ? a.pz[iz] : 0.f;
        ihzr[j] = iz < g.NZ ? a.ihz[iz] : 0.f;
        if (iz < g.NZ && inx) {
            ch[j] = chat[f];
            pm[j] = __builtin_nontemporal_load(um + f);
            hzr[j] = a.hz[iz];
            if (layer_cell_at(g, iz, ix)) {
                lay |= 1u << j;
                fx[j] = phx0[f];
                fz[j] = phz0[f];
            }
        }
    }
    // halo cells of the x and z arrays, one of each per thread
    float xhx = 0.f, xhz = 0.f, xp = 0.f, xih = 0.f, xf = 0.f;
    int xr, xc;
    halo_x_cell(tid < NHX ? tid : 0, xr, xc);
    const bool xl = tid < NHX && z0 + xr < g.NZ && x0 - 4 + xc >= 0 && x0 - 4 + xc < g.NX &&
                    layer_cell_at(g, z0 + xr, x0 - 4 + xc);
    if (xl) {
        const int iz = z0 + xr, jx = x0 - 4 + xc;
        xhx = a.hx[jx]; xhz = a.hz[iz]; xp = a.px[jx]; xih = a.ihx[jx];
        xf = phx0[fidx(g, iz, jx)];
    }
    float zhx = 0.f, zhz = 0.f, zp = 0.f, zih = 0.f, zf = 0.f;
    int zr, zc;
    halo_z_cell<RW>(tid, zr, zc);
    const bool zl = tid < NHZ && z0 - 4 + zr >= 0 && z0 - 4 + zr < g.NZ && x0 + zc < g.NX &&
                    layer_cell_at(g, z0 - 4 + zr, x0 + zc);
    if (zl) {
        const int iz = z0 - 4 + zr, jx = x0 + zc;
        zhx = a.hx[jx]; zhz = a.hz[iz]; zp = a.pz[iz]; zih = a.ihz[iz];
        zf = phz0[fidx(g, iz, jx)];
    }
    dma_tile8<RW, NTN>(g, a.u + so, su, x0, z0);           // u^k on the rows + 8
    const long long src = a.src_f[shot];
    const float sval = src_value(a.src_scale, a.wav[(long long)shot * a.nt + a.k]);
    __builtin_amdgcn_s_waitcnt(0);       // the tile's direct loads have landed in LDS
    __syncthreads();
    ns.fill(a, it, sadd);

    // pass A: phi~^k on the own layer cells (written out) and the halo cells
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int r = ly * RN + j;
        float vx = 0.f, vz = 0.f;
        if (lay >> j & 1u) {
            const int iz = z0 + r;
            const long long f = fidx(g, iz, ix);
            const float *cu = su + (r + H2) * W0 + lx + H2;
            const float qx = 2.f * (hzr[j] - hxc) * ihxc;
            const float qz = 2.f * (hxc - hzr[j]) * ihzr[j];
            vx = pxc * fx[j] + qx * d8(cu, 1);
            vz = pzr[j] * fz[j] + qz * d8(cu, (long long)W0);
            phx[f] = vx;
            phz[f] = vz;
        }
        sx[r * WPX + lx + 4] = vx;
        sz[(r + 4) * TX + lx] = vz;
    }
    if (tid < NHX) {
        float v = 0.f;
        if (xl) {
            const float qx = 2.f * (xhz - xhx) * xih;
            v = xp * xf + qx * d8(su + (xr + H2) * W0 + xc + 4, 1);
        }
        sx[xr * WPX + xc] = v;
    }
    if (tid < NHZ) {
        float v = 0.f;
        if (zl) {
            const float qz = 2.f * (zhx - zhz) * zih;
            v = zp * zf + qz * d8(su + (zr + 4) * W0 + zc + H2, (long long)W0);
        }
        sz[zr * TX + zc] = v;
    }
    __syncthreads();

    // pass B on the tile
    float *uo = a.un + so;
    float un[RN];
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int r = ly * RN + j, iz = z0 + r;
        const float *cu = su + (r + H2) * W0 + lx + H2;
        const float uc = cu[0];
        float w = lap8(cu, W0);
        un[j] = 0.f;
        if (iz < g.NZ && inx) {
            const long long f = fidx(g, iz, ix);
            w += d8(sx + r * WPX + lx + 4, 1) + d8(sz + (r + 4) * TX + lx, (long long)TX);
            const float hx = hxc, hz = hzr[j];
            // alpha (beta u - gamma um + chat w + src) with
            // beta u - gamma um = u + (u - um) + (hx + hz) um - 4 hx hz u
            const float alpha = 1.f / (1.f + hx + hz);
            const float umf = pm[j];
            float inc = (uc - umf) + ((hx + hz) * umf - 4.f * hx * hz * uc) + ch[j] * w;
            if (f == src) inc += sval;
            if (ns.any()) inc += sadd[r * TX + lx];
            const float v = alpha * (uc + inc);
            __builtin_nontemporal_store(v, uo + f);
            un[j] = v;
            if constexpr (SNAP) __builtin_nontemporal_store(w, a.snap + so + f);
        }
    }

    if constexpr (REC) {
        // whole tiles: loaded here, where full CUs hide the latency
        if constexpr (RW == TZ) rc.begin(a, it);
        if (rc.any()) {                   // uniform over the block
            __syncthreads();
#pragma unroll
            for (int j = 0; j < RN; ++j) su[(ly * RN + j + H2) * W0 + lx + H2] = un[j];
            __syncthreads();
            record_tile<RW, NTN>(a, it, rc, [&](int r, int c) { return su[(r + H2) * W0 + c + H2]; });
        }
    }
}

// 34.8 KB of LDS per tile allow 4 tiles per CU: 8 waves per SIMD at 512
// threads, which the forward reaches in 56 VGPRs without spills (256-thread
// tiles held 4 waves per SIMD and ran the C2 near tiles 16 % slower).  The
// adjoint keeps 66 VGPRs and 7 waves: limited to 64 it spills and runs 4 %
// slower.  Taking the row index through readfirstlane puts the rows' z
// tables in scalar registers (forward 62 -> 56, adjoint 78 -> 66 VGPRs).
template <int RW, bool SNAP, bool REC>
__global__ __launch_bounds__(NTN) __attribute__((amdgpu_waves_per_eu(8))) void ac2_near_kernel(Ac2FwdArgs a)
{
    __shared__ __attribute__((aligned(16))) float su[nu8(RW)];
    __shared__ float sx[npx(RW)];
    __shared__ float sz[npz(RW)];
    extern __shared__ float sadd[];
    const int w = xcd_work_id(a.ntl * a.nshots * (TZ / RW));
    fwd_near_tile<RW, SNAP, REC>(a, su, sx, sz, sadd, tile_item<RW>(a.tiles, a.ntl, w));
}

// Everything that a forward step k launches in one grid: the blocked tiles'
// steps k, k+1 (b), the tiles by the layer (a) and the other one-step tiles
// (o).  They read only u^k, u^{k-1} (and phi~^{k-1}) and write disjoint cells
// of u^{k+1} (and u^{k+2}, phi~^k, the seismograms), so they need no order.
// They share one LDS buffer.
constexpr int step_lds(int RW)
{
    const int near = nu8(RW) + npx(RW) + npz(RW), blk = rows0(RW) * W0 + rows1(RW) * W1;
    return near > blk ? near : blk;
}
static_assert(NTN == NTB, "one block size for the step");
template <int RW, bool SNAP, bool REC, bool OTHER>
__global__ __launch_bounds__(NTN) __attribute__((amdgpu_waves_per_eu(8)))
void ac2_step_kernel(Ac2FwdArgs a, Ac2FwdArgs o, Ac2Fwd2Args b)
{
    constexpr int NS = TZ / RW;
    __shared__ __attribute__((aligned(16))) float lds[step_lds(RW)];
    extern __shared__ float sadd[];
    const int nb = b.ntl * b.nshots * NS, na = a.ntl * a.nshots * NS, no = o.ntl * o.nshots * NS;
    const int w = xcd_work_id(nb + na + no);
    if (w < nb) {
        fwd2_tile<RW>(b, lds, lds + rows0(RW) * W0, tile_item<RW>(b.tiles, b.ntl, w));
    } else if (!OTHER || w < nb + na) {
        fwd_near_tile<RW, SNAP, REC>(a, lds, lds + nu8(RW), lds + nu8(RW) + npx(RW), sadd,
                                     tile_item<RW>(a.tiles, a.ntl, w - nb));
    } else if constexpr (OTHER) {
        fwd_tile<RW, NTN, SNAP, REC>(o, lds, sadd, tile_item<RW>(o.tiles, o.ntl, w - nb - na));
    }
}

template <int RW>
__device__ __forceinline__ void adj_near_tile(const Ac2AdjArgs &a, float *sc, float *sx, float *sz,
                                              const TileItem &it)
{
    constexpr int RN = RW * TX / NTN, NHX = RW * 8;
    const Grid2 &g = a.g;
    const int shot = it.shot;
    const int tz = it.tile / g.ntx, tx = it.tile - tz * g.ntx;
    const int x0 = tx * TX, z0 = tz * TZ + it.sub * RW;
    if (z0 >= g.NZ) return;
    const long long so = (long long)shot * g.plane;
    // ly is uniform over a wavefront (TX lanes): rows and their tables in scalar registers
    const int tid = threadIdx.x, lx = tid % TX, ly = __builtin_amdgcn_readfirstlane(tid / TX);
    const int ix = x0 + lx;
    const bool inx = ix < g.NX;
    const float *__restrict__ s2 = a.s2 + so;
    const float *__restrict__ s3 = a.s3 + so;
    const float *__restrict__ chat = a.chat + (long long)(shot / a.shots_per_model) * g.plane;
    const float *__restrict__ cx0 = a.cx0 + so;
    const float *__restrict__ cz0 = a.cz0 + so;
    float *__restrict__ cxo = a.cx + so;
    float *__restrict__ czo = a.cz + so;

    TileRecs rc{};
    rc.begin(a, it);
    const float hxc = inx ? a.hx[ix] : 0.f, pxc = inx ? a.px[ix] : 0.f, ihxc = inx ? a.ihx[ix] : 0.f;
    float sc2[RN], q3[RN], hzr[RN], fx[RN], fz[RN], pzr[RN], ihzr[RN];
    unsigned lay = 0u;
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int iz = z0 + ly * RN + j;
        const long long f = fidx(g, iz, ix);
        sc2[j] = s2[f];
        q3[j] = hzr[j] = fx[j] = fz[j] = 0.f;
        pzr[j] = iz < g.NZ ? a.pz[iz] : 0.f;
        ihzr[j] = iz < g.NZ ? a.ihz[iz] : 0.f;
        if (iz < g.NZ && inx) {
            q3[j] = __builtin_nontemporal_load(s3 + f);
            hzr[j] = a.hz[iz];
            if (layer_cell_at(g, iz, ix)) {
                lay |= 1u << j;
                fx[j] = cx0[f];
                fz[j] = cz0[f];
            }
        }
    }
    // halo cells of the x and z arrays, one of each per thread
    float xhx = 0.f, xhz = 0.f, xp = 0.f, xih = 0.f, xf = 0.f;
    int xr, xc;
    halo_x_cell(tid < NHX ? tid : 0, xr, xc);
    const bool xl = tid < NHX && z0 + xr < g.NZ && x0 - 4 + xc >= 0 && x0 - 4 + xc < g.NX &&
                    layer_cell_at(g, z0 + xr, x0 - 4 + xc);
    if (xl) {
        const int iz = z0 + xr, jx = x0 - 4 + xc;
        xhx = a.hx[jx]; xhz = a.hz[iz]; xp = a.px[jx]; xih = a.ihx[jx];
        xf = cx0[fidx(g, iz, jx)];
    }
    float zhx = 0.f, zhz = 0.f, zp = 0.f, zih = 0.f, zf = 0.f;
    int zr, zc;
    halo_z_cell<RW>(tid, zr, zc);
    const bool zl = tid < NHZ && z0 - 4 + zr >= 0 && z0 - 4 + zr < g.NZ && x0 + zc < g.NX &&
                    layer_cell_at(g, z0 - 4 + zr, x0 + zc);
    if (zl) {
        const int iz = z0 - 4 + zr, jx = x0 + zc;
        zhx = a.hx[jx]; zhz = a.hz[iz]; zp = a.pz[iz]; zih = a.ihz[iz];
        zf = cz0[fidx(g, iz, jx)];
    }
    float4 cm[(rows0(RW) * (W0 / 4) + NTN - 1) / NTN];
    dma_product_load<RW, NTN>(g, s2, chat, sc, x0, z0, cm); // chat s^{k+2} on the rows + 8
    __builtin_amdgcn_s_waitcnt(0);       // the tile's direct loads have landed in LDS
    __syncthreads();
    const float d0 = first_sample(a, it, rc);
    product_in_place<RW, NTN>(sc, cm);
    __syncthreads();

    // pass A: c^{k+1} on the own layer cells (written out) and the halo cells
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int r = ly * RN + j;
        float vx = 0.f, vz = 0.f;
        if (lay >> j & 1u) {
            const int iz = z0 + r;
            const long long f = fidx(g, iz, ix);
            const float *cc = sc + (r + H2) * W0 + lx + H2;
            const float qx = 2.f * (hzr[j] - hxc) * ihxc;
            const float qz = 2.f * (hxc - hzr[j]) * ihzr[j];
            vx = pxc * fx[j] - qx * d8(cc, 1);
            vz = pzr[j] * fz[j] - qz * d8(cc, (long long)W0);
            cxo[f] = vx;
            czo[f] = vz;
        }
        sx[r * WPX + lx + 4] = vx;
        sz[(r + 4) * TX + lx] = vz;
    }
    if (tid < NHX) {
        float v = 0.f;
        if (xl) {
            const float qx = 2.f * (xhz - xhx) * xih;
            v = xp * xf - qx * d8(sc + (xr + H2) * W0 + xc + 4, 1);
        }
        sx[xr * WPX + xc] = v;
    }
    if (tid < NHZ) {
        float v = 0.f;
        if (zl) {
            const float qz = 2.f * (zhx - zhz) * zih;
            v = zp * zf - qz * d8(sc + (zr + 4) * W0 + zc + H2, (long long)W0);
        }
        sz[zr * TX + zc] = v;
    }
    __syncthreads();

    // the snapshot and the gradient accumulator of the own cells, loaded
    // here so that their latency overlaps pass B (loaded with the other
    // operands before pass A, they would spill)
    float snv[RN], grv[RN];
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int iz = z0 + ly * RN + j;
        snv[j] = grv[j] = 0.f;
        if (iz < g.NZ && inx) {
            const long long f = fidx(g, iz, ix);
            snv[j] = __builtin_nontemporal_load(a.snap + so + f);
            grv[j] = __builtin_nontemporal_load(a.grad + so + f);
        }
    }

    // pass B on the tile
    float *s1o = a.s1 + so;
    float av[RN];
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int r = ly * RN + j, iz = z0 + r;
        float v = lap8(sc + (r + H2) * W0 + lx + H2, W0);
        if (iz < g.NZ && inx) {
            v -= d8(sx + r * WPX + lx + 4, 1) + d8(sz + (r + 4) * TX + lx, (long long)TX);
            const float hx = hxc, hz = hzr[j];
            const float s3f = q3[j];
            v += sc2[j] + ((sc2[j] - s3f) + ((hx + hz) * s3f - 4.f * hx * hz * sc2[j]));
        }
        av[j] = v;
    }

    if (rc.any()) {   // receiver residual injection, uniform over the block
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RN; ++j) sc[(ly * RN + j + H2) * W0 + lx + H2] = av[j];
        __syncthreads();
        inject_tile<RW, NTN>(a, it, rc, d0, [&](int r, int c) -> float & { return sc[(r + H2) * W0 + c + H2]; });
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RN; ++j) av[j] = sc[(ly * RN + j + H2) * W0 + lx + H2];
    }

    const long long src = a.src_f[shot];
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int r = ly * RN + j, iz = z0 + r;
        if (iz < g.NZ && inx) {
            const long long f = fidx(g, iz, ix);
            const float s1 = av[j] / (1.f + hxc + hzr[j]);
            __builtin_nontemporal_store(s1, s1o + f);
            __builtin_nontemporal_store(fmaf(s1, snv[j], grv[j]), a.grad + so + f);
            if (a.gwav && f == src) a.gwav[(long long)shot * a.nt + a.k] = s1 * a.src_scale;
            av[j] = s1;
        }
    }
    gather_nodes<RW, NTN>(a, it, [&](int j) { return av[j]; },
                          [&](int r, int c) -> float & { return sc[(r + H2) * W0 + c + H2]; });
}

template <int RW>
__global__ __launch_bounds__(NTN) __attribute__((amdgpu_waves_per_eu(6))) void ac2_adj_near_kernel(Ac2AdjArgs a)
{
    __shared__ __attribute__((aligned(16))) float sc[nu8(RW)];
    __shared__ float sx[npx(RW)];
    __shared__ float sz[npz(RW)];
    const int w = xcd_work_id(a.ntl * a.nshots * (TZ / RW));
    adj_near_tile<RW>(a, sc, sx, sz, tile_item<RW>(a.tiles, a.ntl, w));
}

// The adjoint's step in one grid, as the forward's: steps k, k-1 of the
// blocked tiles (b), step k of the tiles by the layer (a) and of the others (o).
template <int RW, bool OTHER>
__global__ __launch_bounds__(NTN) __attribute__((amdgpu_waves_per_eu(6)))
void ac2_adj_step_kernel(Ac2AdjArgs a, Ac2AdjArgs o, Ac2Adj2Args b)
{
    constexpr int NS = TZ / RW;
    __shared__ __attribute__((aligned(16))) float lds[step_lds(RW)];
    const int nb = b.ntl * b.nshots * NS, na = a.ntl * a.nshots * NS, no = o.ntl * o.nshots * NS;
    const int w = xcd_work_id(nb + na + no);
    if (w < nb) {
        adj2_tile<RW, NTN>(b, lds, lds + rows0(RW) * W0, tile_item<RW>(b.tiles, b.ntl, w));
    } else if (!OTHER || w < nb + na) {
        adj_near_tile<RW>(a, lds, lds + nu8(RW), lds + nu8(RW) + npx(RW), tile_item<RW>(a.tiles, a.ntl, w - nb));
    } else if constexpr (OTHER) {
        adj_tile<RW, NTN>(o, lds, tile_item<RW>(o.tiles, o.ntl, w - nb - na));
    }
}

// ------------------------------------------------------------------ launchers
// f(integral_constant<int, RW>) with the rows per workgroup of a launch of
// `tiles` tiles: whole tiles where they give every CU two workgroups, else
// half or quarter tiles.  Measured on forward + recompute + adjoint, us per
// step, 32 / 16 / 8 rows: 15 tiles 22.3 / - / 15.2; 300 tiles 21.0 / 18.8 /
// 21.2; 900 tiles 34.8 / 36.8 / 45.5; 192 tiles by the layer and 420 blocked
// ones, forward alone, 10.9 / 10.4 / 10.2; from 768 tiles the repeated halo work costs more than it fills.
constexpr int FILL2 = 512;
template <class F>
void with_rows(int tiles, F &&f)
{
    if (tiles <= 0) return;
    if (tiles >= FILL2) f(std::integral_constant<int, TZ>{});
    else if (2 * tiles >= FILL2) f(std::integral_constant<int, TZ / 2>{});
    else f(std::integral_constant<int, TZ / 4>{});
}

// Dynamic LDS of the forward step: the node sources of RW rows.
inline size_t node_lds(const Ac2FwdArgs &a, int RW)
{
    return a.nsrc > 1 ? sizeof(float) * RW * TX : 0;
}

// f(snapshot?, records?) of a forward launch as constants
template <class F>
void with_outputs(const Ac2FwdArgs &a, F &&f)
{
    const bool rec = a.seis != nullptr;
    if (a.snap) { if (rec) f(std::true_type(), std::true_type()); else f(std::true_type(), std::false_type()); }
    else        { if (rec) f(std::false_type(), std::true_type()); else f(std::false_type(), std::false_type()); }
}

// One grid or several.  A step of fewer than FILL2 tiles is bound by the
// latency of a launch, so its lists go out as one grid (260 x 160, 49 source
// nodes: 38 -> 17 us per forward + recompute + adjoint step; 1000 x 500, one
// shot: 31 -> 23).  From there on the other one-step tiles, few and in need of
// a kernel of more registers, go apart; the tiles by the layer and the blocked
// ones still share a grid, so that neither waits for the last workgroups of
// the other: 1000 x 500, recording forward of 8 and 24 shots 21.0 -> 19.6 and
// 47.8 -> 47.4 us per step (apart from STEP_REC tiles on: with 64 shots the whole
// pass went from 454 to 457); adjoint, whole pass of 4, 16 and 64 shots 50.3 -> 47.1,
// 133 -> 130 and 454 -> 451.
constexpr int STEP_REC = 8192;

void launch_ac2_step(const Ac2FwdArgs &a, const Ac2FwdArgs &o, const Ac2Fwd2Args &b, bool pair, hipStream_t s)
{
    const int na = a.ntl * a.nshots, no = o.ntl * o.nshots, nb = b.ntl * b.nshots, nt = na + no + nb;
    const bool all = pair && nt < FILL2;
    with_outputs(a, [&](auto snap, auto rec) {
        constexpr bool S = decltype(snap)::value, R = decltype(rec)::value;
        auto grid = [&](const Ac2FwdArgs &others) {
            const int n = na + nb + others.ntl * others.nshots;
            with_rows(n, [&](auto rows) {
                constexpr int RW = decltype(rows)::value;
                ac2_step_kernel<RW, S, R, (RW < TZ)><<<n * (TZ / RW), NTN, node_lds(a, RW), s>>>(a, others, b);
            });
        };
        if (all && (na > 0) + (no > 0) + (nb > 0) > 1) {
            grid(o);
            return;
        }
        with_rows(no, [&](auto rows) {
            constexpr int RW = decltype(rows)::value;
            ac2_fwd_kernel<RW, S, R><<<no * (TZ / RW), NTH, node_lds(o, RW), s>>>(o);
        });
        if (pair && na > 0 && nb > 0 && (!R || na + nb < STEP_REC)) {
            Ac2FwdArgs none = o;
            none.ntl = 0;
            grid(none);
            return;
        }
        with_rows(na, [&](auto rows) {
            constexpr int RW = decltype(rows)::value;
            ac2_near_kernel<RW, S, R><<<na * (TZ / RW), NTN, node_lds(a, RW), s>>>(a);
        });
        with_rows(nb, [&](auto rows) {
            constexpr int RW = decltype(rows)::value;
            ac2_fwd2_kernel<RW><<<nb * (TZ / RW), NTB, 0, s>>>(b);
        });
    });
}

void launch_ac2_adj_step(const Ac2AdjArgs &a, const Ac2AdjArgs &o, const Ac2Adj2Args &b, bool pair, hipStream_t s)
{
    const int na = a.ntl * a.nshots, no = o.ntl * o.nshots, nb = b.ntl * b.nshots, nt = na + no + nb;
    const bool all = pair && nt < FILL2;
    auto grid = [&](const Ac2AdjArgs &others) {
        const int n = na + nb + others.ntl * others.nshots;
        with_rows(n, [&](auto rows) {
            constexpr int RW = decltype(rows)::value;
            ac2_adj_step_kernel<RW, (RW < TZ)><<<n * (TZ / RW), NTN, 0, s>>>(a, others, b);
        });
    };
    if (all && (na > 0) + (no > 0) + (nb > 0) > 1) {
        grid(o);
        return;
    }
    with_rows(no, [&](auto rows) {
        constexpr int RW = decltype(rows)::value;
        ac2_adj_kernel<RW><<<no * (TZ / RW), NTH, 0, s>>>(o);
    });
    if (pair && na > 0 && nb > 0) {
        Ac2AdjArgs none = o;
        none.ntl = 0;
        grid(none);
        return;
    }
    with_rows(na, [&](auto rows) {
        constexpr int RW = decltype(rows)::value;
        ac2_adj_near_kernel<RW><<<na * (TZ / RW), NTN, 0, s>>>(a);
    });
    with_rows(nb, [&](auto rows) {
        constexpr int RW = decltype(rows)::value;
        ac2_adj2_kernel<RW><<<nb * (TZ / RW), NTH, 0, s>>>(b);
    });
}

__global__ void ac2_prep_kernel(Grid2 g, int nmodels, const float *vp, double dt, double dx,
                                float *chat, float *cpad)
{
    const long long n = (long long)nmodels * g.plane;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const long long m = i / g.plane, f = i - m * g.plane;
        const int fz = (int)(f / g.SX), fx = (int)(f - (long long)fz * g.SX);
        const int iz = fz - OZ, ix = fx - OX;
        float c = 0.f, ch = 0.f;
        if (iz >= 0 && iz < g.NZ && ix >= 0 && ix < g.NX) {
            const int pz = min(max(iz - g.P, 0), g.nz - 1), px = min(max(ix - g.P, 0), g.nx - 1);
            c = vp[(m * g.nz + pz) * g.nx + px];
            const double cd = c;
            ch = (float)(dt * dt * cd * cd / (dx * dx));
        }
        chat[i] = ch;
        cpad[i] = c;
    }
}

void launch_ac2_prep(const Grid2 &g, int nmodels, const float *vp, double dt, double dx,
                     float *chat, float *cpad, hipStream_t s)
{
    const long long n = (long long)nmodels * g.plane;
    const int blocks = (int)std::min<long long>((n + 255) / 256, 65536);
    ac2_prep_kernel<<<blocks, 256, 0, s>>>(g, nmodels, vp, dt, dx, chat, cpad);
}

// ------------------------------------------------------------ grad finalize
// Pass 1: per padded cell, sum dJ/dchat over the model's shots in shot order
// (coalesced over cells).  Pass 2: the fold with the chain rule.
__global__ void ac2_sum_shots_kernel(Grid2 g, int nmodels, int spm, const float *grad, float *acc)
{
    const long long n = (long long)nmodels * g.plane;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const long long m = i / g.plane, f = i - m * g.plane;
        float v = 0.f;
        for (int s = 0; s < spm; ++s) v += grad[(m * spm + s) * g.plane + f];
        acc[i] = v;
    }
}

void launch_ac2_finalize(const Grid2 &g, int nmodels, int spm, const float *grad, float *acc,
                         const float *cpad, double dt, double dx, float *g_vp, hipStream_t s)
{
    const float *sum = grad;               // one shot per model: its gradient is the sum
    if (spm > 1) {
        const long long n = (long long)nmodels * g.plane;
        const int blocks = (int)std::min<long long>((n + 255) / 256, 65536);
        ac2_sum_shots_kernel<<<blocks, 256, 0, s>>>(g, nmodels, spm, grad, acc);
        sum = acc;
    }
    launch_fold2(g, nmodels, sum, cpad, dt, dx, g_vp, s);
}

} // namespace sg
