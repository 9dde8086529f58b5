// ad2.hip -- gfx950 kernels of the 2-D acoustic equation in divergence form,
// u_tt = div(c^2 grad u) + f (Eq. (12) as printed), on a staggered grid with
// a convolutional PML, and its adjoint (Eqs. (4)-(5)).
//
// Scaled variables: chat = dt^2 c^2 / dx^2 at the nodes, khat = (chat_i +
// chat_{i+1}) / 2 at the half nodes (a neighbour beyond the padded grid takes
// the edge value, so chat is replicated one node beyond it), differences
// without the 1/dx factor,
//   Dp' u (i + 1/2) = 9/8 (u_{i+1} - u_i) - 1/24 (u_{i+2} - u_{i-1}),
//   Dm' q (i)       = 9/8 (q_i - q_{i-1}) - 1/24 (q_{i+1} - q_{i-2}),
// psi' = dx psi and xi' = dt^2 xi for the layer memories.  Forward step k,
// one launch over (tile, shot):
//   G' = Dp' u^k;   psi'^{k+1} = bh psi'^k + ah G';   S' = G' + psi'^{k+1}
//   q' = khat S';   H' = Dm' q';   xi'^{k+1} = b xi'^k + a H'
//   u^{k+1} = 2 u^k - u^{k-1} + H'x + xi'x + H'z + xi'z + dt^2/(dx dz) sum_j r_j(t_k)
// Half-node values exist on [0, NX) x [0, NZ) only (zero beyond), so that
// Dm'^T = -Dp'.  psi' is read in the halo and written by its owner, so it
// alternates between two buffers; xi' is read only at its own node and is
// updated in place.
//
// Adjoint launch k computes lambda^k = dJ/du^k.  The layer adjoints are
// kept multiplied by their constant coefficients, Y = a dJ/dxi' (nodes) and
// Z = ah dJ/dpsi' (half nodes), so they vanish outside the layer:
//   Y^{k+1} = a lambda^{k+1} + b Y^{k+2};   Hb = lambda^{k+1} + Y^{k+1}
//   qb = -Dp' Hb;  Sb = khat qb;  Z^{k+1} = ah Sb + bh Z^{k+2};  Gb = Sb + Z^{k+1}
//   lambda^k = 2 lambda^{k+1} - lambda^{k+2} - Dm' Gbx - Dm' Gbz + R^T dJ/dd_{k-1}
//   dJ/dchat_i += 1/2 (qb S' at the two half nodes beside node i, per axis),
//   S' of forward step k being a snapshot
// Y and Z alternate between two buffers like psi'.
// Cache policy: u^{k-1} (lambda^{k+2}) and its overwrite, the xi' memories,
// the snapshot stores and the gradient accumulator are streamed
// (non-temporal); the
// snapshot loads of the adjoint stay cached, since the half-node averages
// read each of them from two rows (streaming them cost 16 % of the adjoint).
#include <algorithm>
#include <type_traits>
#include "ad2_internal.h"

// Multiply-adds are fused only where written as fmaf: whether the compiler
// would fuse the others depends on the rows per workgroup, and a shot's
// values must not.  Which products are fused follows groups of four rows of a
// 32-row tile: a row's place in its group (0 .. 3) and a half row's (M = 0 .. 6,
// from two above the first row), whatever rows a thread takes.  The only reason
// for these places is that results stay what they were, bit for bit, with four
// rows per thread, where the compiler had fused these products: ahead of a
// wavefront values are differences of denormal numbers, which another rounding
// changes in their leading digits.  They have no meaning of their own, and one flux
// is rounded differently for its tile and for the neighbour's extra column.  Every
// product rounded would be as exact (errors against 64 bits within 2 % of each other)
// and faster: 1000x500, 64 shots, forward 247 against 251 us, recompute 272 / 274,
// adjoint 362 / 365.
#pragma clang fp contract(off)

namespace sg {
namespace {

// A workgroup takes 16 rows of a 64 x 32 tile, 512 threads of 2 rows each, or
// 8 rows in launches of few tiles; whole tiles (4 rows per thread) leave no
// registers to load the layer memories and snapshots before the first
// barrier.  A launch of few tiles is bound by the workgroups that one CU takes
// in turn: 8 rows where 16 would not fill the CUs, and where 16 would give a
// second workgroup to few of them (129 to 192 tiles: 3 of 8 rows per CU
// instead of 2 of 16).  Forward + recompute + adjoint, us per step, 16 / 8
// rows: 36 tiles 18.0 / 15.9; 72 tiles 18.4 / 17.4; 96 tiles 18.7 / 19.3; 128
// tiles 18.7 / 19.6; 144 tiles 23.3 / 22.7; 180 tiles 24.2 / 24.0; 216 tiles
// 25.0 / 28.0; 360 tiles 33.7 / 38.4; 32 rows: 108 tiles 39.1, 144 tiles 38.3.
//
// EARLY launches, of at most EARLY_AD2 16-row workgroups (two per CU) and those
// of 8 rows, have every load in flight before the first barrier, in registers
// that leave half the wavefronts; the others load chat beside the thread's
// nodes and the layer's tables at their use, and the adjoint steps through the
// nodes by the layer (a load behind the previous node's stores: 3 us of an
// 11 us launch).  300 x 150 + 20-cell layer, late -> early: 1 shot 20.7 -> 16.0 us
// per step, 4 shots 27.0 -> 22.7; 9 shots, 648 workgroups, 33.0 -> 34.2.
// 1000 x 500 + 32-cell layer, 64 shots (late): 890.
//
// A thread's rows are uniform over its wavefront (TX lanes); taken through
// readfirstlane, they put the z tables in scalar registers.
constexpr int FILL_AD2 = 96, EARLY_AD2 = 512;
constexpr int NTA = 512;
static_assert(8 * TX % NTA == 0 && NTA % TX == 0, "whole rows per thread");
constexpr int AH = 3;              // halo of the composite stencil Dm' khat Dp'
constexpr int AW = TX + 2 * AH;    // node tile with halo: RW + 2 AH rows of AW
constexpr int nodes(int RW) { return (RW + 2 * AH) * AW; }
constexpr int QXW = TX + 3;        // x half nodes x0-2 .. x0+TX on each row of the tile
constexpr float S1 = (float)(9.0 / 8.0);
constexpr float S2 = (float)(-1.0 / 24.0);

__device__ __forceinline__ long long fr(const Grid2 &g, int iz, int ix)
{
    return (long long)(iz + OZ) * g.SX + ix + OX;
}

// 9/8 (c - b) - 1/24 (d - a) of four consecutive values: Dp' at i + 1/2
// from (u_{i-1}, u_i, u_{i+1}, u_{i+2}), Dm' at i from (q_{i-2}, .., q_{i+1}).
__device__ __forceinline__ float d4(float a, float b, float c, float d)
{
    return fmaf(S1, c - b, S2 * (d - a));
}

// The same from the inner difference c - b and the outer one d - a.
__device__ __forceinline__ float d4(float inner, float outer)
{
    return fmaf(S1, inner, S2 * outer);
}

// Outer difference d - a of z fluxes, a = ka sa and d = kd sd: in a tile away from
// the layer, a group's first row (0) takes the product a unrounded and its last row (3) the
// product d.
__device__ __forceinline__ float outer(int row, float a, float ka, float sa, float d, float kd, float sd)
{
    float o = d - a;
    if (row == 0) o = fmaf(-ka, sa, d);
    if (row == 3) o = fmaf(kd, sd, -a);
    return o;
}

// Consecutive work ids on one XCD (workgroups are dealt to the 8 XCDs
// round-robin), so that neighbouring tiles share an L2.
__device__ __forceinline__ int xcd_id(int nblocks)
{
    const int b = blockIdx.x;
    const int per = nblocks / NXCD, rem = nblocks % NXCD;
    const int x = b % NXCD, j = b / NXCD;
    return x * per + min(x, rem) + j;
}

// Does the tile or its 3-node halo reach the absorbing layer or the edge of
// the grid (layer memories, masks of the half-node range)?
template <int RW>
__device__ __forceinline__ bool near_edge_z(const Grid2 &g, int z0)
{
    return z0 - AH < g.P || z0 + RW + AH > g.P + g.nz;
}
template <int RW>
__device__ __forceinline__ bool near_edge(const Grid2 &g, int x0, int z0)
{
    return x0 - AH < g.P || x0 + TX + AH > g.P + g.nx || near_edge_z<RW>(g, z0);
}

// RW rows (sub) of a tile.
struct Rows {
    int tile, shot, sub, x0, z0;
};
template <int RW>
__device__ __forceinline__ Rows rows_of(const Grid2 &g, int nshots)
{
    constexpr int NS = TZ / RW;
    const int ntl = g.ntx * g.ntz;
    const int w = xcd_id(ntl * nshots * NS), t = w / NS;
    Rows o;
    o.sub = w - t * NS;
    o.shot = t / ntl;
    o.tile = t - o.shot * ntl;
    const int tz = o.tile / g.ntx, tx = o.tile - tz * g.ntx;
    o.x0 = tx * TX;
    o.z0 = tz * TZ + o.sub * RW;
    return o;
}

// A tile's source or receiver entries: the range, and this thread's first
// entry with its value, loaded early.
struct Entries {
    int b, e, ent;
    float v;
    __device__ __forceinline__ void range(const int *off, const int *list, const Rows &o, int ntiles)
    {
        off += (long long)o.shot * (ntiles + 1);
        b = off[o.tile];
        e = off[o.tile + 1];
        ent = b + (int)threadIdx.x < e ? list[b + threadIdx.x] : 0;
        v = 0.f;
    }
    template <class F>
    __device__ __forceinline__ void first(F val_of)
    {
        if (b + (int)threadIdx.x < e) v = val_of(ent);
    }
    __device__ __forceinline__ bool any() const { return b < e; }
};

// acc[cell] = sum of add(sum, value) over the tile's entries of each cell of
// these RW rows (acc: TX*RW floats, zeroed here).  Entries are sorted by
// cell; the first entry of each cell sums its run in entry order, so
// duplicates add up deterministically.  Every thread of the block must call
// this.
template <int RW, class CellOf, class ValOf, class Add>
__device__ __forceinline__ void gather_entries(float *acc, const int *ent, const Entries &en, int sub, CellOf cell_of,
                                               ValOf val_of, Add add)
{
    for (int i = threadIdx.x; i < TX * RW; i += NTA) acc[i] = 0.f;
    __syncthreads();
    for (int i = en.b + (int)threadIdx.x; i < en.e; i += NTA) {
        const bool pre = i == en.b + (int)threadIdx.x;
        const int x = pre ? en.ent : ent[i], c = cell_of(x), own = c - sub * RW * TX;
        if (own < 0 || own >= RW * TX || (i > en.b && cell_of(ent[i - 1]) == c)) continue;
        float v = add(0.f, pre ? en.v : val_of(x));
        for (int j = i + 1; j < en.e && cell_of(ent[j]) == c; ++j) v = add(v, val_of(ent[j]));
        acc[own] = v;
    }
    __syncthreads();
}

// chat beside a thread's nodes (right of the last lane's, beside the extra
// column's half node) and the layer's tables at its half nodes and nodes.
// EARLY: loaded with the other operands before the first barrier, so that no
// load of the launch waits behind one; else, in fewer registers, at their use.
template <int RW, bool EARLY, bool NEAR>
struct Coefs {
    static constexpr int RPA = RW * TX / NTA, NZH = NEAR && EARLY ? RPA + 3 : 1, NZN = NEAR && EARLY ? RPA : 1;
    float cr[RPA], ce0, ce1, bx, ax, ebx, eax, b0, a0, bz[NZH], az[NZH], b0zr[NZN], a0zr[NZN];

    __device__ __forceinline__ void right(const Grid2 &g, const float *ch, int j, int iz, int ix, int lx)
    {
        cr[j] = 0.f;
        if (lx == TX - 1) cr[j] = ch[fr(g, iz, ix + 1)];
    }
    __device__ __forceinline__ void own_x(const Grid2 &g, const Ad2Cpml &t, int ix)
    {
        bx = ax = 0.f;
        if constexpr (NEAR) {
            const int i = min(ix, g.NX - 1);
            bx = t.bhx[i];
            ax = t.ahx[i];
        }
    }
    __device__ __forceinline__ void extra(const Grid2 &g, const Ad2Cpml &t, const float *ch, int x0, int z0, int er,
                                          int eh)
    {
        const long long f = fr(g, z0 + er, x0 - 2 + eh);
        ce0 = ch[f];
        ce1 = ch[f + 1];
        ebx = eax = 0.f;
        if constexpr (NEAR) {
            const int i = min(max(x0 - 2 + eh, 0), g.NX - 1);
            ebx = t.bhx[i];
            eax = t.ahx[i];
        }
    }
    __device__ __forceinline__ void load(const Grid2 &g, const Ad2Cpml &t, const float *ch, const Rows &o, int tid,
                                         int er, int eh)
    {
        const int lx = tid % TX, r0 = __builtin_amdgcn_readfirstlane(tid / TX) * RPA, ix = o.x0 + lx;
#pragma unroll
        for (int j = 0; j < RPA; ++j) right(g, ch, j, o.z0 + r0 + j, ix, lx);
        if (tid < 3 * RW) extra(g, t, ch, o.x0, o.z0, er, eh);
        own_x(g, t, ix);
        if constexpr (NEAR) {
            b0 = t.b0x[min(ix, g.NX - 1)];
            a0 = t.a0x[min(ix, g.NX - 1)];
#pragma unroll
            for (int m = 0; m < RPA + 3; ++m) {
                const int i = min(max(o.z0 + r0 - 2 + m, 0), g.NZ - 1);
                bz[m] = t.bhz[i];
                az[m] = t.ahz[i];
                if (m >= 2 && m < RPA + 2) {
                    b0zr[m - 2] = t.b0z[i];
                    a0zr[m - 2] = t.a0z[i];
                }
            }
        }
    }
    // of the half row m (iz) of this thread, of its node row j (iz), of its node column
    __device__ __forceinline__ float bhz(const Ad2Cpml &t, int m, int iz) const { return EARLY ? bz[EARLY ? m : 0] : t.bhz[iz]; }
    __device__ __forceinline__ float ahz(const Ad2Cpml &t, int m, int iz) const { return EARLY ? az[EARLY ? m : 0] : t.ahz[iz]; }
    __device__ __forceinline__ float b0z(const Ad2Cpml &t, int j, int iz) const { return EARLY ? b0zr[EARLY ? j : 0] : t.b0z[iz]; }
    __device__ __forceinline__ float a0z(const Ad2Cpml &t, int j, int iz) const { return EARLY ? a0zr[EARLY ? j : 0] : t.a0z[iz]; }
    __device__ __forceinline__ float b0x(const Ad2Cpml &t, int ix) const { return EARLY ? b0 : t.b0x[ix]; }
    __device__ __forceinline__ float a0x(const Ad2Cpml &t, int ix) const { return EARLY ? a0 : t.a0x[ix]; }
};

// ------------------------------------------------------------------ forward
// Work split of a tile: thread (lx, ly) owns column x0 + lx and rows
// r0 = ly*RPA .. r0+RPA-1.  The z fluxes of its column (its own half rows and
// the three around them that its Dm' needs) are computed in registers from
// its column of the u tile; the x fluxes go through LDS (own half column by
// every thread, the three extra columns x0-2, x0-1, x0+TX by the first 3*RW
// threads).  chat of the own column is read once per thread; the right
// neighbour's comes from the next lane (one wavefront = one tile row).  The
// z part runs first so that only Hz and u^k of the own rows stay live.
// psi: psi'x^k there.
template <bool NEAR, bool SNAP>
__device__ __forceinline__ float fwd_xflux(const Ad2FwdArgs &a, const float *su, long long so, int x0, int z0, int r,
                                           int h, float c0, float c1, float psi, float bh, float ah)
{
    const Grid2 &g = a.g;
    const int iz = z0 + r, ix = x0 - 2 + h;
    const float *s = su + (r + AH) * AW + h;
    const float G = d4(s[0], s[1], s[2], s[3]);
    float q = 0.f;
    if (!NEAR || (ix >= 0 && ix < g.NX)) {
        const long long f = fr(g, iz, ix);
        const bool own = h >= 2 && h < TX + 2 && iz < g.NZ;
        float S = G;
        if constexpr (NEAR) {
            const float p = fmaf(bh, psi, ah * G);
            S = G + p;
            if (own) a.psxn[so + f] = p;
        }
        if constexpr (SNAP) {
            if (own) __builtin_nontemporal_store(S, a.snx + so + f);
        }
        q = 0.5f * (c0 + c1) * S;
    }
    return q;
}

template <int RW, bool EARLY, bool NEAR, bool SNAP, bool REC>
__device__ __forceinline__ void fwd_tile(const Ad2FwdArgs &a, float *su, float *qx, const Rows &o)
{
    constexpr int RPA = RW * TX / NTA;
    const Grid2 &g = a.g;
    const int x0 = o.x0, z0 = o.z0, shot = o.shot;
    const long long so = (long long)shot * g.plane;
    const float *u = a.u + so;
    const float *ch = a.chat + (long long)(shot / a.shots_per_model) * g.plane;
    const int tid = threadIdx.x, lx = tid % TX, ly = __builtin_amdgcn_readfirstlane(tid / TX), r0 = ly * RPA, ix = x0 + lx;

    // u^k on the tile + 3 straight from global memory into LDS: 4 bytes per
    // lane and load into consecutive LDS words (item order is the row-major
    // order of su); every cell lies inside the zero frame
    {
        constexpr int NV = nodes(RW), K = (NV + NTA - 1) / NTA;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = tid + k * NTA;
            if (i < NV) {
                const int r = i / AW, c = i - r * AW;
                __builtin_amdgcn_global_load_lds((const void *)(u + fr(g, z0 - AH + r, x0 - AH + c)),
                                                 (void __attribute__((address_space(3))) *)(su + k * NTA + (tid & ~63)),
                                                 4, 0, 0);
            }
        }
    }
    float cz[RPA + 4];                    // chat of rows z0+r0-2 .. z0+r0+RPA+1
#pragma unroll
    for (int m = 0; m < RPA + 4; ++m) cz[m] = ch[fr(g, z0 + r0 - 2 + m, ix)];
    float um[RPA];                        // u^{k-1} of the own rows, loaded early
#pragma unroll
    for (int j = 0; j < RPA; ++j) um[j] = __builtin_nontemporal_load(a.um + so + fr(g, z0 + r0 + j, ix));
    const int ntiles = g.ntx * g.ntz;
    Entries src{}, rec{};
    src.range(a.src_off, a.src_ent, o, ntiles);
    if constexpr (REC) rec.range(a.rec_off, a.rec_ent, o, ntiles);
    const float *w = a.wav + (long long)shot * a.nsrc * a.nt + a.k;
    auto sample = [&](int e) { return w[(long long)src_node(e) * a.nt]; };
    // layer memories: psi'z of the own column's half rows, psi'x of
    // the own half nodes and of this thread's extra column, xi' of the own rows
    float pz0[RPA + 3], px0[RPA], pxe = 0.f, xx0[RPA], xz0[RPA];
    const int er = tid / 3, ee = tid - 3 * er, eh = ee == 2 ? TX + 2 : ee;   // extra column: row, half node
    Coefs<RW, EARLY, NEAR> co;
    if constexpr (EARLY) co.load(g, a.t, ch, o, tid, er, eh);
    if constexpr (NEAR) {
#pragma unroll
        for (int m = 0; m < RPA + 3; ++m) pz0[m] = a.psz[so + fr(g, z0 + r0 - 2 + m, ix)];
#pragma unroll
        for (int j = 0; j < RPA; ++j) {
            const long long f = so + fr(g, z0 + r0 + j, ix);
            px0[j] = a.psx[f];
            xx0[j] = __builtin_nontemporal_load(a.xix + f);
            xz0[j] = __builtin_nontemporal_load(a.xiz + f);
        }
        if (tid < 3 * RW) pxe = a.psx[so + fr(g, z0 + er, x0 - 2 + eh)];
    }
    src.first(sample);
    __builtin_amdgcn_s_waitcnt(0);       // the tile's direct loads have landed in LDS
    __syncthreads();

    // place in its group of the thread's first row; none (8) in a tile that the layer reaches elsewhere
    // (found here, not at the top: 1000x500, 64 shots, forward 251 against 262 us, adjoint 365 against 367)
    const bool whole = !NEAR && !near_edge_z<TZ>(g, z0 - o.sub * RW);
    const int quad = __builtin_amdgcn_readfirstlane(whole || NEAR ? r0 & 3 : 8);
    // z fluxes of the own column at half rows z0+r0-2+m, m = 0 .. RPA+2
    float uc[RPA], hz[RPA];
    {
        float uz[RPA + 6];
#pragma unroll
        for (int m = 0; m < RPA + 6; ++m) uz[m] = su[(r0 + m) * AW + lx + AH];
        float qz[RPA + 3], kz[RPA + 3], sz[RPA + 3];      // the fluxes and their factors
#pragma unroll
        for (int m = 0; m < RPA + 3; ++m) {
            const int iz = z0 + r0 - 2 + m;
            const float G = d4(uz[m], uz[m + 1], uz[m + 2], uz[m + 3]);
            float q = 0.f;
            if (!NEAR || (iz >= 0 && iz < g.NZ)) {
                const long long f = fr(g, iz, ix);
                const bool own = m >= 2 && m < RPA + 2 && ix < g.NX;
                float S = G;
                if constexpr (NEAR) {
                    const float p = fmaf(co.bhz(a.t, m, iz), pz0[m], co.ahz(a.t, m, iz) * G);
                    S = G + p;
                    if (own) a.pszn[so + f] = p;
                }
                if constexpr (SNAP) {
                    if (own) __builtin_nontemporal_store(S, a.snz + so + f);
                }
                kz[m] = 0.5f * (cz[m] + cz[m + 1]);
                sz[m] = S;
                q = kz[m] * S;
            }
            qz[m] = q;
        }
#pragma unroll
        for (int j = 0; j < RPA; ++j) {
            uc[j] = uz[j + 3];
            if constexpr (NEAR) hz[j] = d4(qz[j], qz[j + 1], qz[j + 2], qz[j + 3]);
            else hz[j] = d4(qz[j + 2] - qz[j + 1], outer(quad + j, qz[j], kz[j], sz[j], qz[j + 3],
                                                         kz[j + 3], sz[j + 3]));
        }
    }
#pragma unroll
    for (int j = 0; j < RPA; ++j) {
        const float c0 = cz[j + 2];
        float c1 = __shfl_down(c0, 1, TX);
        if constexpr (!EARLY) co.right(g, ch, j, z0 + r0 + j, ix, lx);
        if (lx == TX - 1) c1 = co.cr[j];
        if constexpr (!EARLY) co.own_x(g, a.t, ix);
        qx[(r0 + j) * QXW + lx + 2] = fwd_xflux<NEAR, SNAP>(a, su, so, x0, z0, r0 + j, lx + 2, c0, c1, px0[j], co.bx,
                                                            co.ax);
    }
    if (tid < 3 * RW) {
        if constexpr (!EARLY) co.extra(g, a.t, ch, x0, z0, er, eh);
        qx[er * QXW + eh] = fwd_xflux<NEAR, SNAP>(a, su, so, x0, z0, er, eh, co.ce0, co.ce1, pxe, co.ebx, co.eax);
    }
    __syncthreads();                      // qx complete; su no longer read

    if (src.any()) {                      // uniform over the block
        gather_entries<RW>(su, a.src_ent, src, o.sub, [](int e) { return src_cell(e); }, sample,
                           [&](float v, float x) { return fmaf(a.src_scale, x, v); });
    }
    float un[RPA];
#pragma unroll
    for (int j = 0; j < RPA; ++j) {
        const int r = r0 + j, iz = z0 + r;
        const float *qa = qx + r * QXW + lx;
        const float Hx = d4(qa[0], qa[1], qa[2], qa[3]);
        un[j] = 0.f;
        if (iz < g.NZ && ix < g.NX) {
            const long long f = fr(g, iz, ix);
            float inc = Hx + hz[j];
            if constexpr (NEAR) {
                const float xx = fmaf(co.b0x(a.t, ix), xx0[j], co.a0x(a.t, ix) * Hx);
                const float xz = fmaf(co.b0z(a.t, j, iz), xz0[j], co.a0z(a.t, j, iz) * hz[j]);
                __builtin_nontemporal_store(xx, a.xix + so + f);
                __builtin_nontemporal_store(xz, a.xiz + so + f);
                inc += xx + xz;
            }
            inc += uc[j] - um[j];
            if (src.any()) inc += su[r * TX + lx];
            const float v = uc[j] + inc;
            __builtin_nontemporal_store(v, a.un + so + f);
            un[j] = v;
        }
    }
    if constexpr (REC) {
        if (rec.any()) {                  // uniform over the block
            __syncthreads();
#pragma unroll
            for (int j = 0; j < RPA; ++j) su[(r0 + j) * TX + lx] = un[j];
            __syncthreads();
            for (int i = rec.b + tid; i < rec.e; i += NTA) {
                const int ent = i == rec.b + tid ? rec.ent : a.rec_ent[i];
                const int own = rec_cell(ent) - o.sub * RW * TX;
                if (own < 0 || own >= RW * TX) continue;
                a.seis[((long long)shot * a.nt + a.k) * a.nrec + rec_id(ent)] = su[own];
            }
        }
    }
}

template <int RW, bool EARLY, bool SNAP, bool REC>
__global__ __launch_bounds__(NTA) __attribute__((amdgpu_waves_per_eu(EARLY ? 4 : 8)))
void ad2_fwd_kernel(Ad2FwdArgs a)
{
    __shared__ float su[nodes(RW)];
    __shared__ float qx[RW * QXW];
    const Rows o = rows_of<RW>(a.g, a.nshots);
    if (o.z0 >= a.g.NZ) return;
    if (near_edge<RW>(a.g, o.x0, o.z0)) fwd_tile<RW, EARLY, true, SNAP, REC>(a, su, qx, o);
    else                                fwd_tile<RW, EARLY, false, SNAP, REC>(a, su, qx, o);
}

// ------------------------------------------------------------------ adjoint
// Gradient per node: khat at a half node feeds its two nodes with weight
// 1/2 each, so dJ/dchat_i = 1/2 (p at i-1/2 + p at i+1/2) per axis, with
// p = qb S' the half-node product; the node at the far edge of each axis
// also takes the other half of its right half node (the chat beyond the
// grid is its replica).  The x product of the half node left of a thread's
// node comes from the neighbouring lane (lane 0: from the extra column).
// z0v: Z_x^{k+2} there; sn: S'x there.
template <bool NEAR, bool GRAD>
__device__ __forceinline__ float adj_xflux(const Ad2AdjArgs &a, const float *hx, long long so, int x0, int z0, int r,
                                           int h, float c0, float c1, bool want_p, float &p, float z0v, float sn,
                                           float ah, float bh)
{
    const Grid2 &g = a.g;
    const int iz = z0 + r, ix = x0 - 2 + h;
    const float *s = hx + (r + AH) * AW + h;
    const float qb = -d4(s[0], s[1], s[2], s[3]);
    float Gb = 0.f;
    p = 0.f;
    if (!NEAR || (ix >= 0 && ix < g.NX)) {
        const long long f = fr(g, iz, ix);
        const bool own = h >= 2 && h < TX + 2 && iz < g.NZ;
        const float Sb = 0.5f * (c0 + c1) * qb;
        Gb = Sb;
        if constexpr (NEAR) {
            const float z = fmaf(ah, Sb, bh * z0v);
            Gb = !GRAD || (h >= 2 && h < TX + 2) ? fmaf(0.5f * (c0 + c1), qb, z) : Sb + z;
            if (own) a.zxn[so + f] = z;
        }
        if constexpr (GRAD) {
            if (want_p && iz < g.NZ) p = qb * sn;
        }
    }
    return Gb;
}

template <int RW, bool EARLY, bool NEAR, bool GRAD>
__device__ __forceinline__ void adj_tile(const Ad2AdjArgs &a, float *hx, float *hz, float *qx, float *pl,
                                         const Rows &o)
{
    constexpr int RPA = RW * TX / NTA;
    const Grid2 &g = a.g;
    const int x0 = o.x0, z0 = o.z0, shot = o.shot;
    const long long so = (long long)shot * g.plane;
    const float *l1 = a.l1 + so;
    const float *ch = a.chat + (long long)(shot / a.shots_per_model) * g.plane;
    const int tid = threadIdx.x, lx = tid % TX, ly = __builtin_amdgcn_readfirstlane(tid / TX), r0 = ly * RPA, ix = x0 + lx;

    // Hb = lambda^{k+1} + Y^{k+1} per axis on the tile and its halo
    if constexpr (!NEAR) {
        // away from the layer the x and z arrays are both lambda^{k+1} itself:
        // straight from global memory into LDS (4 bytes per lane and load,
        // item order = the row-major order of hx; every cell inside the frame)
        constexpr int NV = nodes(RW), K = (NV + NTA - 1) / NTA;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = tid + k * NTA;
            if (i < NV) {
                const int r = i / AW, c = i - r * AW;
                __builtin_amdgcn_global_load_lds((const void *)(l1 + fr(g, z0 - AH + r, x0 - AH + c)),
                                                 (void __attribute__((address_space(3))) *)(hx + k * NTA + (tid & ~63)),
                                                 4, 0, 0);
            }
        }
    }
    // near the layer: y of one node from its operands, stored if it is its tile's
    auto stage = [&](int i, float l, float yx0, float yz0, float ax, float bx, float az, float bz) {
        const int r = i / AW, c = i - r * AW, iz = z0 - AH + r, jx = x0 - AH + c;
        float vx = l, vz = l;
        if (iz >= 0 && iz < g.NZ && jx >= 0 && jx < g.NX) {
            const float yx = fmaf(ax, l, bx * yx0);
            const float yz = fmaf(az, l, bz * yz0);
            if (r >= AH && r < AH + RW && c >= AH && c < AH + TX) {
                const long long f = fr(g, iz, jx);
                a.yxn[so + f] = yx;
                a.yzn[so + f] = yz;
            }
            vx = l + yx;
            vz = l + yz;
        }
        hx[i] = vx;
        hz[i] = vz;
    };
    auto node = [&](int i, long long &f, int &tz, int &tx) {       // its place and table rows
        const int r = i / AW, c = i - r * AW, iz = z0 - AH + r, jx = x0 - AH + c;
        f = fr(g, iz, jx);
        tz = min(max(iz, 0), g.NZ - 1);
        tx = min(max(jx, 0), g.NX - 1);
    };
    constexpr int KN = NEAR && EARLY ? (nodes(RW) + NTA - 1) / NTA : 1;
    float ln[KN], yx0[KN], yz0[KN], ax[KN], bx[KN], az[KN], bz[KN];
    float lc[RPA];                        // lambda^{k+1} of the own rows
    if constexpr (NEAR && EARLY) {
#pragma unroll
        for (int k = 0; k < KN; ++k) {
            long long f;
            int tz, tx;
            node(min(tid + k * NTA, nodes(RW) - 1), f, tz, tx);
            ln[k] = l1[f];
            yx0[k] = a.yx[so + f];
            yz0[k] = a.yz[so + f];
            ax[k] = a.t.a0x[tx];
            bx[k] = a.t.b0x[tx];
            az[k] = a.t.a0z[tz];
            bz[k] = a.t.b0z[tz];
        }
#pragma unroll
        for (int j = 0; j < RPA; ++j) lc[j] = l1[fr(g, z0 + r0 + j, ix)];
    } else if constexpr (NEAR) {
        for (int i = tid; i < nodes(RW); i += NTA) {
            long long f;
            int tz, tx;
            node(i, f, tz, tx);
            stage(i, l1[f], a.yx[so + f], a.yz[so + f], a.t.a0x[tx], a.t.b0x[tx], a.t.a0z[tz], a.t.b0z[tz]);
        }
    }
    float cz[RPA + 4];
#pragma unroll
    for (int m = 0; m < RPA + 4; ++m) cz[m] = ch[fr(g, z0 + r0 - 2 + m, ix)];
    float l2[RPA];                        // lambda^{k+2} of the own rows, loaded early
#pragma unroll
    for (int j = 0; j < RPA; ++j) l2[j] = __builtin_nontemporal_load(a.l2 + so + fr(g, z0 + r0 + j, ix));
    float gacc[RPA];                      // the gradient accumulator of the own rows, loaded early
    if constexpr (GRAD) {
#pragma unroll
        for (int j = 0; j < RPA; ++j) {
            const int iz = z0 + r0 + j;
            gacc[j] = iz < g.NZ && ix < g.NX ? __builtin_nontemporal_load(a.gn + so + fr(g, iz, ix)) : 0.f;
        }
    }
    Entries rec{};
    rec.range(a.rec_off, a.rec_ent, o, g.ntx * g.ntz);
    const float *d = a.dJdd + ((long long)shot * a.nt + (a.k - 1)) * a.nrec;   // read for k >= 1 only
    auto sample = [&](int en) { return d[rec_id(en)]; };
    // Z and the snapshots of the own column's half rows, of the own x
    // half nodes and of this thread's extra column
    float zz0[RPA + 3], sz0[RPA + 3], zx0[RPA], sx0[RPA], zxe = 0.f, sxe = 0.f;
    const int er = tid / 3, ee = tid - 3 * er, eh = ee == 2 ? TX + 2 : ee;   // extra column: row, half node
#pragma unroll
    for (int m = 0; m < RPA + 3; ++m) {
        const long long f = so + fr(g, z0 + r0 - 2 + m, ix);
        if constexpr (NEAR) zz0[m] = a.zz[f];
        if constexpr (GRAD) sz0[m] = a.snz[f];
    }
#pragma unroll
    for (int j = 0; j < RPA; ++j) {
        const long long f = so + fr(g, z0 + r0 + j, ix);
        zx0[j] = NEAR ? a.zx[f] : 0.f;
        sx0[j] = GRAD ? a.snx[f] : 0.f;
    }
    if (tid < 3 * RW) {
        const long long f = so + fr(g, z0 + er, x0 - 2 + eh);
        if constexpr (NEAR) zxe = a.zx[f];
        if constexpr (GRAD) sxe = a.snx[f];
    }
    Coefs<RW, EARLY, NEAR> co;
    if constexpr (EARLY) co.load(g, a.t, ch, o, tid, er, eh);
    if (a.k >= 1) rec.first(sample);
    if constexpr (NEAR && EARLY) {
#pragma unroll
        for (int k = 0; k < KN; ++k)
            if (tid + k * NTA < nodes(RW)) stage(tid + k * NTA, ln[k], yx0[k], yz0[k], ax[k], bx[k], az[k], bz[k]);
    }
    if constexpr (!NEAR) __builtin_amdgcn_s_waitcnt(0);   // the tile's direct loads have landed in LDS
    __syncthreads();
    const float *hzz = NEAR ? hz : hx;

    // place in its group of the thread's first row; none (8) in a tile that the layer reaches elsewhere
    const bool whole = !NEAR && !near_edge_z<TZ>(g, z0 - o.sub * RW);
    const int quad = __builtin_amdgcn_readfirstlane(whole || NEAR ? r0 & 3 : 8);
    float dz[RPA], gnz[RPA];              // Dm' Gb_z and the z gradient of the own rows
    {
        float hc[RPA + 6];
#pragma unroll
        for (int m = 0; m < RPA + 6; ++m) hc[m] = hzz[(r0 + m) * AW + lx + AH];
        float gz[RPA + 3], pz[RPA + 3], kz[RPA + 3], qz[RPA + 3];
#pragma unroll
        for (int m = 0; m < RPA + 3; ++m) {
            const int iz = z0 + r0 - 2 + m;
            const float qb = -d4(hc[m], hc[m + 1], hc[m + 2], hc[m + 3]);
            float Gb = 0.f;
            pz[m] = 0.f;
            if (!NEAR || (iz >= 0 && iz < g.NZ)) {
                const long long f = fr(g, iz, ix);
                const bool own = m >= 2 && m < RPA + 2 && ix < g.NX;
                kz[m] = 0.5f * (cz[m] + cz[m + 1]);
                qz[m] = qb;
                const float Sb = kz[m] * qb;
                Gb = Sb;
                if constexpr (NEAR) {
                    const float z = fmaf(co.ahz(a.t, m, iz), Sb, co.bhz(a.t, m, iz) * zz0[m]);
                    const int M = quad + m;
                    Gb = !GRAD || M < 2 || M == 6 ? fmaf(kz[m], qb, z) : Sb + z;
                    if (own) a.zzn[so + f] = z;
                }
                if constexpr (GRAD) {
                    if (m >= 1 && m < RPA + 2) pz[m] = qb * sz0[m];
                }
            }
            gz[m] = Gb;
        }
#pragma unroll
        for (int j = 0; j < RPA; ++j) {
            const int iz = z0 + r0 + j;
            if constexpr (!NEAR) lc[j] = hc[j + 3];
            if constexpr (NEAR) dz[j] = d4(gz[j], gz[j + 1], gz[j + 2], gz[j + 3]);
            else dz[j] = d4(gz[j + 2] - gz[j + 1], outer(quad + j, gz[j], kz[j], qz[j], gz[j + 3],
                                                         kz[j + 3], qz[j + 3]));
            float pp = pz[j + 1] + pz[j + 2];
            if constexpr (!NEAR && GRAD) {
                if (quad + j == 0) pp = fmaf(qz[j + 1], sz0[j + 1], pz[j + 2]);
                if (quad + j == 3) pp = fmaf(qz[j + 2], sz0[j + 2], pz[j + 1]);
            }
            gnz[j] = 0.5f * pp;
            if (iz == g.NZ - 1) gnz[j] = fmaf(0.5f, pz[j + 2], gnz[j]);
        }
    }
    float px[RPA];                        // x products at the own half column
#pragma unroll
    for (int j = 0; j < RPA; ++j) {
        const float c0 = cz[j + 2];
        float c1 = __shfl_down(c0, 1, TX);
        if constexpr (!EARLY) co.right(g, ch, j, z0 + r0 + j, ix, lx);
        if (lx == TX - 1) c1 = co.cr[j];
        if constexpr (!EARLY) co.own_x(g, a.t, ix);
        float pj;
        qx[(r0 + j) * QXW + lx + 2] = adj_xflux<NEAR, GRAD>(a, hx, so, x0, z0, r0 + j, lx + 2, c0, c1, true, pj,
                                                                   zx0[j], sx0[j], co.ax, co.bx);
        px[j] = pj;
    }
    if (tid < 3 * RW) {
        float p = 0.f;
        if constexpr (!EARLY) co.extra(g, a.t, ch, x0, z0, er, eh);
        qx[er * QXW + eh] = adj_xflux<NEAR, GRAD>(a, hx, so, x0, z0, er, eh, co.ce0, co.ce1, eh == 1, p, zxe, sxe,
                                                  co.eax, co.ebx);
        if (GRAD && eh == 1) pl[er] = p;  // the half node left of the tile's first column
    }
    __syncthreads();                      // qx, pl complete; hx, hz no longer read

    const bool inj = a.k >= 1 && rec.any();   // uniform over the block
    if (inj) {
        gather_entries<RW>(hx, a.rec_ent, rec, o.sub, [](int en) { return rec_cell(en); }, sample,
                           [](float v, float x) { return v + x; });
    }
#pragma unroll
    for (int j = 0; j < RPA; ++j) {
        const int r = r0 + j, iz = z0 + r;
        const float *ga = qx + r * QXW + lx;
        const float Dx = d4(ga[0], ga[1], ga[2], ga[3]);
        float gn = 0.f;
        if constexpr (GRAD) {
            float left = __shfl_up(px[j], 1, TX);
            if (lx == 0) left = pl[r];
            gn = fmaf(0.5f, left + px[j], gnz[j]);
            if (ix == g.NX - 1) gn = fmaf(0.5f, px[j], gn);
        }
        if (iz < g.NZ && ix < g.NX) {
            const long long f = fr(g, iz, ix);
            if constexpr (NEAR && !EARLY) lc[j] = l1[f];
            float v = lc[j] + ((lc[j] - l2[j]) - (Dx + dz[j]));
            if (inj) v += hx[r * TX + lx];
            __builtin_nontemporal_store(v, a.l0 + so + f);
            if constexpr (GRAD) __builtin_nontemporal_store(gacc[j] + gn, a.gn + so + f);
        }
    }
}

template <int RW, bool EARLY, bool GRAD>
__global__ __launch_bounds__(NTA) __attribute__((amdgpu_waves_per_eu(EARLY ? 4 : 8)))
void ad2_adj_kernel(Ad2AdjArgs a)
{
    __shared__ float hx[nodes(RW)];
    __shared__ float hz[nodes(RW)];
    __shared__ float qx[RW * QXW];
    __shared__ float pl[RW];
    const Rows o = rows_of<RW>(a.g, a.nshots);
    if (o.z0 >= a.g.NZ) return;
    if (near_edge<RW>(a.g, o.x0, o.z0)) adj_tile<RW, EARLY, true, GRAD>(a, hx, hz, qx, pl, o);
    else                                adj_tile<RW, EARLY, false, GRAD>(a, hx, hz, qx, pl, o);
}

// ------------------------------------------------------------------ model and gradient
__global__ void ad2_prep_kernel(Grid2 g, int nmodels, const float *vp, double dt, double dx, float *chat, float *cpad)
{
    const long long n = (long long)nmodels * g.plane;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const long long m = i / g.plane, f = i - m * g.plane;
        const int iz = (int)(f / g.SX) - OZ, ix = (int)(f - (f / g.SX) * g.SX) - OX;
        const bool in = iz >= 0 && iz < g.NZ && ix >= 0 && ix < g.NX;
        const bool rep = (ix == g.NX && iz >= 0 && iz < g.NZ) || (iz == g.NZ && ix >= 0 && ix < g.NX);
        float c = 0.f, ch = 0.f;
        if (in || rep) {
            const int pz = min(max(min(iz, g.NZ - 1) - g.P, 0), g.nz - 1);
            const int px = min(max(min(ix, g.NX - 1) - g.P, 0), g.nx - 1);
            c = vp[(m * g.nz + pz) * g.nx + px];
            const double cd = c;
            ch = (float)(dt * dt * cd * cd / (dx * dx));
        }
        chat[i] = ch;
        cpad[i] = in ? c : 0.f;
    }
}

// dJ/dchat per padded node, summed over the model's shots in shot order.
__global__ void ad2_sum_shots_kernel(Grid2 g, int nmodels, int spm, const float *gn, float *acc)
{
    const long long n = (long long)nmodels * g.plane;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const long long m = i / g.plane, f = i - m * g.plane;
        float v = 0.f;
        for (int s = 0; s < spm; ++s) v += gn[(m * spm + s) * g.plane + f];
        acc[i] = v;
    }
}

int blocks_for(long long n) { return (int)std::min<long long>((n + 255) / 256, 65536); }

} // namespace

// f(integral_constant<int, RW>, early?, workgroups) with the rows per
// workgroup of a launch over `tiles` tiles.
template <class F>
static void with_rows(int tiles, F &&f)
{
    constexpr std::integral_constant<int, 16> r16{};
    constexpr std::integral_constant<int, 8> r8{};
    if (tiles <= 0) return;
    const int n16 = tiles * (TZ / 16);
    if (tiles < FILL_AD2 || (tiles > 128 && tiles <= 192)) f(r8, std::true_type(), tiles * (TZ / 8));
    else if (n16 <= EARLY_AD2) f(r16, std::true_type(), n16);
    else f(r16, std::false_type(), n16);
}

void launch_ad2_fwd(const Ad2FwdArgs &a, hipStream_t s)
{
    const bool rec = a.seis && a.nrec > 0;
    with_rows(a.g.ntx * a.g.ntz * a.nshots, [&](auto R, auto early, int n) {
        constexpr int RW = decltype(R)::value;
        constexpr bool E = decltype(early)::value;
        if (a.snx) {
            if (rec) ad2_fwd_kernel<RW, E, true, true><<<n, NTA, 0, s>>>(a);
            else     ad2_fwd_kernel<RW, E, true, false><<<n, NTA, 0, s>>>(a);
        } else {
            if (rec) ad2_fwd_kernel<RW, E, false, true><<<n, NTA, 0, s>>>(a);
            else     ad2_fwd_kernel<RW, E, false, false><<<n, NTA, 0, s>>>(a);
        }
    });
}

void launch_ad2_adj(const Ad2AdjArgs &a, hipStream_t s)
{
    with_rows(a.g.ntx * a.g.ntz * a.nshots, [&](auto R, auto early, int n) {
        constexpr int RW = decltype(R)::value;
        constexpr bool E = decltype(early)::value;
        if (a.snx) ad2_adj_kernel<RW, E, true><<<n, NTA, 0, s>>>(a);
        else       ad2_adj_kernel<RW, E, false><<<n, NTA, 0, s>>>(a);
    });
}

void launch_ad2_prep(const Grid2 &g, int nmodels, const float *vp, double dt, double dx, float *chat, float *cpad,
                     hipStream_t s)
{
    ad2_prep_kernel<<<blocks_for((long long)nmodels * g.plane), 256, 0, s>>>(g, nmodels, vp, dt, dx, chat, cpad);
}

void launch_ad2_finalize(const Grid2 &g, int nmodels, int spm, const float *gn, float *acc, const float *cpad,
                         double dt, double dx, float *g_vp, hipStream_t s)
{
    if (spm > 1) ad2_sum_shots_kernel<<<blocks_for((long long)nmodels * g.plane), 256, 0, s>>>(g, nmodels, spm, gn, acc);
    launch_fold2(g, nmodels, spm > 1 ? acc : gn, cpad, dt, dx, g_vp, s);   // one shot per model is its own sum
}

} // namespace sg
