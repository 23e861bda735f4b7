// Near field and far-field evaluation at the cell centres of 4^3-cell leaves,
// and the near field's transpose, by reflection parity.
//
// Targets and Gauss points both sit on the lattice, and reflecting the axes
// about a leaf's centre maps its cells, and the 12^3 cells of its 27
// neighbour leaves, to themselves, so the map from the neighbourhood's
// densities to the field at the leaf's centres is block-diagonal in the eight
// parities chi of the reflection group (as the octet M2L, octet.hpp).  With s
// one of the 216 cells of the positive octant and t one of the leaf's 8,
//   H_chi[s] = sum_r (-1)^(chi.r) rho[r s],
//   G_chi[t, c] = sum_s F_chi[t, c][s] H_chi[s] + sum_{k of class chi} L[t, c][k] LE[k],
//   g_c[r t] = (-1)^(class(c).r) sum_chi (-1)^(chi.r) G_chi[t, c],
//   F_chi[t, c][s] = 1/8 sum_r (-1)^(chi.r) A[t, c][r s],
// A the direct sum's pair terms and L the far-field evaluation at the base
// centres (class(c): the reflections that flip component c).  Eight products of
// 8 C x 216 instead of one of 64 C x 1728: an eighth of the operations, and an
// operator that stays in the L2.  Rounding is relative to the largest pair term
// among a cell's images: in norm as with dense matrices, but the coincident pair
// leaves the rounding of its images' terms where those held a zero, and the FP32
// field of a lone cell is good to 2.5e-7 (dense: 4e-8) five cells away.
//
// What bounds it: the passes around the products, which themselves would take
// 0.18 ms at 256^3 cells and C = 3 in FP32: the neighbourhood's densities into
// LDS, the parity tiles, the exchange of the parities and the output.
// Measured there against the 27 dense leaf-to-leaf products (with their
// regathered densities): forward 1.91 -> 0.49 ms in FP32, 3.38 -> 0.96 in FP64;
// transposed 2.13 -> 0.90 in FP32; 64^3 cells forward 0.055 -> 0.017 ms.
#include <algorithm>

#include "octet.hpp"
#include "resolve.hpp"

// The FP32 transposed near field takes blocks of 4 x 4 x 2 leaves from this many
// (leaf, model) pairs on: three passes over the neighbourhood make the halo (4.5
// instead of 6 neighbours per leaf) count there (256^3, g: 0.90 ms against 1.07
// with blocks of 4 x 2 x 2; 16384 pairs of 64^3 cells x 4 0.064 against 0.076),
// smaller plans need the workgroups (8192 pairs 0.040 against 0.039, 4096 0.036
// against 0.028), and so do meshes that fill them worse (8^3 cells x 2048, 2^3
// leaves: 0.177 against 0.139).  Everywhere else 16 leaves are as fast or faster:
// the smaller tiles leave room for more workgroups per CU (256^3 forward, FP32
// 0.49 against 0.51 ms, FP64 0.96 against 1.18).
#ifndef GRAV_NEAR_WIDE_LEAVES
#define GRAV_NEAR_WIDE_LEAVES 16384
#endif

namespace grav {

namespace {

constexpr int kOctant = 216;  // base cells of a leaf's neighbourhood

// A workgroup's leaves: 4 x LY x LZ = 16 NC columns, the cells around them.
template <int NC>
struct NearBlock {
    static constexpr int LX = 4, LY = NC == 1 ? 2 : 4, LZ = 2;
    static constexpr int DX = 4 * (LX + 2), DY = 4 * (LY + 2), DZ = 4 * (LZ + 2);
    static constexpr int NCOL = 16 * NC;
};

struct NearGrid {
    int nx, ny, n;  // blocks along x and y, blocks per model
};

// Reflections that flip output component c of C.
__host__ __device__ inline int comp_class(int C, int c) { return C == 1 ? 4 : C == 3 ? 1 << c : c == 0 ? 0 : 1 << (c - 1); }

template <typename T>
__device__ __forceinline__ void walsh8(T (&v)[8])
{
#pragma unroll
    for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if ((r & bit) == 0) {
                const T x = v[r], y = v[r | bit];
                v[r] = x + y;
                v[r | bit] = x - y;
            }
}

// Staging of the parity tiles: thread (column, one of 12 base cells sx, sy of
// a chunk).  Chunk 3 jz + jy holds the base cells sz = jz, sy in {2 jy, 2 jy +
// 1}, so a thread's eight images sit at constant offsets from four addresses
// (the x and y images), and all address arithmetic is in the instructions.
template <typename T, int NC>
struct NearStage {
    using NB = NearBlock<NC>;
    static constexpr int CS = 4 * kNearChunk, TILE = 8 * NC * CS * 17;
    static constexpr int NT = NB::NCOL * CS;  // staging threads
    static_assert(CS == 12 && NT <= 512, "a chunk is two rows of six base cells, one per thread");
    const T *base[4];
    T *dst;
    bool on;
    __device__ __forceinline__ NearStage(const T *dens, T *hs, int tid, int flip)
    {
        on = tid < NT;
        const int sl = tid % CS, col = min(tid / CS, NB::NCOL - 1);
        const int sx = sl % 6, sy = sl / 6;
        const int x = 4 * (col % 4), y = 4 * (col / 4 % NB::LY), z = 4 * (col / (4 * NB::LY));
#pragma unroll
        for (int r = 0; r < 4; ++r)
            base[r] = dens + (z * NB::DY + (r & 2 ? y + 1 - sy : y + 6 + sy)) * NB::DX + (r & 1 ? x + 5 - sx : x + 6 + sx);
        dst = hs + (col / 16) * (CS * 17) + sl * 17 + col % 16;
        this->flip = flip;
    }
    int flip;
    // the tile of chunk (jz, jy): H_chi as B operands, [chi][column block][cell]
    // [column] with a stride of 17 (cells of a column and columns of a cell both
    // spread over the banks)
    __device__ __forceinline__ void put(int jz, int jy, int buf) const
    {
        if (!on)
            return;
        T v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r)
            v[r] = base[r & 3][((r & 4 ? 5 - jz : 6 + jz) * NB::DY + (r & 2 ? 4 - 2 * jy : 2 * jy)) * NB::DX];
        walsh8(v);
#pragma unroll
        for (int x = 0; x < 8; ++x)
            dst[buf * TILE + (x ^ flip) * (NC * CS * 17)] = v[x];
    }
};

// The values of the block's neighbourhood (at(cell) inside the mesh, zero
// outside) into LDS: rows of DX = 24 cells, 21 rows at a time; U loads in
// flight per thread, none under a branch.
template <typename T, int NC, class At>
__device__ __forceinline__ void near_fill(const DevGeom &g, int cx, int cy, int cz, int tid, T *dens, At &&at)
{
    using NB = NearBlock<NC>;
    constexpr int DX = NB::DX, RN = 512 / DX, ROWS = NB::DY * NB::DZ, U = 7;
    const int x = tid % DX, r0 = tid / DX, ix = cx + x;
    const bool xin = (r0 < RN) & ((uint32_t)ix < (uint32_t)g.n[0]);
    for (int b = 0; b < ROWS; b += U * RN) {
        double v[U];
        bool in[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = b + u * RN + r0;
            const int iy = cy + row % NB::DY, iz = cz + row / NB::DY;
            in[u] = xin & (row < ROWS) & ((uint32_t)iy < (uint32_t)g.n[1]) & ((uint32_t)iz < (uint32_t)g.n[2]);
            v[u] = at(in[u] ? ((int64_t)iz * g.n[1] + iy) * g.n[0] + ix : 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (r0 < RN && b + u * RN + r0 < ROWS)
                dens[(b + u * RN + r0) * DX + x] = in[u] ? (T)v[u] : (T)0;
    }
}

// The block's outputs from LDS to the mesh, VC values a cell: val(r, t, col, c)
// for the image r of base cell t of the leaf in column col.  Threads take
// (cell, value) pairs of a row of 16 cells, so that a wave stores contiguous
// runs.
template <int NC, int VC, class Put>
__device__ __forceinline__ void near_store(const DevGeom &g, int lx0, int ly0, int lz0, int tid, Put &&put)
{
    using NB = NearBlock<NC>;
    constexpr int W = 16 * VC, RN = 512 / W, ROWS = 16 * NB::LY * NB::LZ;
    const int x = tid % W / VC, c = tid % VC, r0 = tid / W;
    const int px = x & 3, tx = px >> 1 ? px - 2 : 1 - px, rx = px >> 1 ? 0 : 1;
    const int ix = 4 * lx0 + x;
    if (r0 >= RN || ix >= g.n[0])
        return;
    for (int row = r0; row < ROWS; row += RN) {
        const int y = row % (4 * NB::LY), z = row / (4 * NB::LY);
        const int iy = 4 * ly0 + y, iz = 4 * lz0 + z;
        if (iy >= g.n[1] || iz >= g.n[2])
            continue;
        const int py = y & 3, pz = z & 3;
        const int t = tx + 2 * (py >> 1 ? py - 2 : 1 - py) + 4 * (pz >> 1 ? pz - 2 : 1 - pz);
        const int r = rx | (py >> 1 ? 0 : 2) | (pz >> 1 ? 0 : 4);
        put(((int64_t)iz * g.n[1] + iy) * g.n[0] + ix, r, t, x / 4 + 4 * (y / 4 + NB::LY * (z / 4)), c);
    }
}

// Products over the 216 base cells: wave chi multiplies its parity's tile by
// its operator ([chunk][frag_at set]), chunk by chunk; the next chunk's tile is
// built between this one's instructions.  RB16 blocks of 16 rows, and RB4
// groups of four as 4x4x1 instructions (FP32: row lane % 4, each sub-row of
// lanes summing its own cells).
template <typename T, int NC, int RB16, int RB4, class Acc>
__device__ __forceinline__ void near_products(const NearStage<T, NC> &st, const T *hs, const T *A, int tid, int chi,
                                              Acc &acc)
{
    using ST = NearStage<T, NC>;
    constexpr int CK = kNearChunk, RB = RB16 + RB4, E = CK * RB, CS = ST::CS;
    const int lane = tid & 63, kr = lane >> 4;
    T an[2][E];
    load_set<T, E>(A, lane, an[0]);
    st.put(0, 0, 0);
    __syncthreads();
    const T *bs = hs + chi * (NC * CS * 17) + kr * 17 + (lane & 15);
#pragma unroll
    for (int j = 0; j < 18; ++j) {
        if (j + 1 < 18)
            load_set<T, E>(A + (j + 1) * E * 64, lane, an[(j + 1) & 1]);
        T b[CK][NC];
#pragma unroll
        for (int u = 0; u < CK; ++u)
#pragma unroll
            for (int c = 0; c < NC; ++c)
                b[u][c] = bs[(j & 1) * ST::TILE + c * (CS * 17) + u * 4 * 17];
        if (j + 1 < 18)
            st.put((j + 1) / 3, (j + 1) % 3, (j + 1) & 1);
#pragma unroll
        for (int u = 0; u < CK; ++u)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const T a = an[j & 1][u * RB + rb];
                    if constexpr (sizeof(T) == 8)
                        acc[c][rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[u][c], acc[c][rb], 0, 0, 0);
                    else if (rb >= RB16)
                        acc[c][rb] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, b[u][c], acc[c][rb], 0, 0, 0);
                    else
                        acc[c][rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b[u][c], acc[c][rb], 0, 0, 0);
                }
        __syncthreads();
    }
}

// Forward.  Row R = 8 c + t of the product is component c at base centre t.
// The far field runs in FP64 in both precisions; next to an FP32 near field
// its operator's rows are permuted (row i holds row 4 (i % 4) + i / 4) so that
// both instructions' output elements line up.
template <typename T, int NC, int C>
__global__ void __launch_bounds__(512)
k_near_par(DevGeom g, NearGrid ng, const double *rho, const T *A, const double *Lm, const int32_t *coef, int KC,
           const int32_t *tmap, const double *le, int64_t npts, double *out)
{
    using NB = NearBlock<NC>;
    using vec4 = __attribute__((__vector_size__(4 * sizeof(T)))) T;
    using dvec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int CS = 4 * kNearChunk, NCOL = NB::NCOL, RBN = (8 * C + 15) / 16, RR = 16 * RBN, EP = NCOL + 1;
    constexpr size_t kTiles = sizeof(T) * (NB::DX * NB::DY * NB::DZ + 2 * 8 * NC * CS * 17);
    constexpr size_t kExch = sizeof(double) * 8 * RR * EP;
    __shared__ __align__(16) char smem[kTiles > kExch ? kTiles : kExch];
    T *dens = reinterpret_cast<T *>(smem), *hs = dens + NB::DX * NB::DY * NB::DZ;
    double *ex = reinterpret_cast<double *>(smem);
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int chi = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t id = block_id();
    if (id >= (int64_t)ng.n * g.B)
        return;
    const int bm = (int)((uint32_t)id / (uint32_t)ng.n), blk = (int)((uint32_t)id - (uint32_t)bm * (uint32_t)ng.n);
    const int bx = blk % ng.nx, by = blk / ng.nx % ng.ny, bz = blk / (ng.nx * ng.ny);
    const int lx0 = bx * NB::LX, ly0 = by * NB::LY, lz0 = bz * NB::LZ;  // the block's first leaf
    const int64_t ncell = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const double *rb0 = rho + bm * ncell;
    // the far field's operands: the leaves' local expansions of this wave's
    // class, the first FK k steps already in flight during the near field
    constexpr int FK = 4;
    const DevLev &lv = g.lev[g.L];
    const double *lp[NC];
    bool have[NC];
    double fb[FK][NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int col = c * 16 + (lane & 15);
        const int lx = lx0 + col % 4, ly = ly0 + col / 4 % NB::LY, lz = lz0 + col / (4 * NB::LY);
        const int64_t tl = KC > 0 && lx < lv.ns[0] && ly < lv.ns[1] && lz < lv.ns[2]
                               ? tmap_lookup(lv, tmap, 3, lv.s0[0] + lx, lv.s0[1] + ly, lv.s0[2] + lz)
                               : -1;
        have[c] = tl >= 0;
        lp[c] = le + ((lv.tgt_off + (have[c] ? tl : 0)) * g.B + bm) * g.PS;
    }
    if (KC > 0) {
#pragma unroll
        for (int q = 0; q < FK; ++q) {
            const int k = coef[(chi * KC + min(q, KC - 1)) * 4 + kr];
#pragma unroll
            for (int c = 0; c < NC; ++c)
                fb[q][c] = lp[c][k];
        }
    }
    near_fill<T, NC>(g, 4 * (lx0 - 1), 4 * (ly0 - 1), 4 * (lz0 - 1), tid, dens, [&](int64_t cell) { return rb0[cell]; });
    __syncthreads();
    vec4 acc[NC][RBN];
    dvec4 far[NC][RBN];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int rb = 0; rb < RBN; ++rb) {
            acc[c][rb] = vec4{0, 0, 0, 0};
            far[c][rb] = dvec4{0, 0, 0, 0};
        }
    const NearStage<T, NC> st(dens, hs, tid, 0);
    near_products<T, NC, RBN, 0>(st, hs, A + (int64_t)chi * (kOctant / 4) * RBN * 64, tid, chi, acc);
    auto far_step = [&](int q, const double (&b)[NC]) {
        double a[RBN];
#pragma unroll
        for (int rb = 0; rb < RBN; ++rb)
            a[rb] = Lm[((int64_t)(chi * KC + q) * RBN + rb) * 64 + lane];
#pragma unroll
        for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
            for (int c = 0; c < NC; ++c)
                far[c][rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[rb], have[c] ? b[c] : 0.0, far[c][rb], 0, 0, 0);
    };
#pragma unroll
    for (int q = 0; q < FK; ++q)
        if (q < KC)
            far_step(q, fb[q]);
    for (int q = FK; q < KC; ++q) {
        const int k = coef[(chi * KC + q) * 4 + kr];
        double b[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
            b[c] = lp[c][k];
        far_step(q, b);
    }
    // G_chi through LDS (the tiles are done with), where the eight parities of
    // a (row, column) meet
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                ex[(chi * RR + 16 * rb + (sizeof(T) == 8 ? kr + 4 * r : 4 * kr + r)) * EP + c * 16 + (lane & 15)] =
                    (double)acc[c][rb][r] + far[c][rb][r];
    __syncthreads();
    const double sg = g.G * g.h, sp = g.G * g.h * g.h;
    for (int i = tid; i < 8 * C * NCOL; i += 512) {
        const int R = i / NCOL, col = i % NCOL;
        double v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x)
            v[x] = ex[(x * RR + R) * EP + col];
        walsh8(v);
        const int cls = comp_class(C, R / 8);
        const double sc = cls == 0 ? sp : sg;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            ex[(r * RR + R) * EP + col] = odd_parity(cls & r) ? -sc * v[r] : sc * v[r];
    }
    __syncthreads();
    double *o = out + ((int64_t)bm * g.M + npts) * C;
    near_store<NC, C>(g, lx0, ly0, lz0, tid, [&](int64_t cell, int r, int t, int col, int c) {
        o[cell * C + c] = ex[(r * RR + 8 * c + t) * EP + col];
    });
}

// Transposed: drho[r t] = sum_chi (-1)^(chi.r) sum_{c, s} F^T_chi[t][c, s]
// H_chi[c, s], with H of component c's weights at the 216 base centres (signs of
// class(c) included) and F^T from the pair terms of the centres around a source
// cell.  One pass over the neighbourhood per component.
template <typename T, int NC>
__global__ void __launch_bounds__(512)
k_t_near_par(DevGeom g, NearGrid ng, const double *resid, int64_t npts, const T *A, int add, double *drho)
{
    using NB = NearBlock<NC>;
    using vec4 = __attribute__((__vector_size__(4 * sizeof(T)))) T;
    constexpr int CS = 4 * kNearChunk, NCOL = NB::NCOL, EP = NCOL + 1;
    constexpr size_t kTiles = sizeof(T) * (NB::DX * NB::DY * NB::DZ + 2 * 8 * NC * CS * 17);
    constexpr size_t kExch = sizeof(double) * 8 * 8 * EP;
    __shared__ __align__(16) char smem[kTiles > kExch ? kTiles : kExch];
    T *dens = reinterpret_cast<T *>(smem), *hs = dens + NB::DX * NB::DY * NB::DZ;
    double *ex = reinterpret_cast<double *>(smem);
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int chi = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t id = block_id();
    if (id >= (int64_t)ng.n * g.B)
        return;
    const int bm = (int)((uint32_t)id / (uint32_t)ng.n), blk = (int)((uint32_t)id - (uint32_t)bm * (uint32_t)ng.n);
    const int bx = blk % ng.nx, by = blk / ng.nx % ng.ny, bz = blk / (ng.nx * ng.ny);
    const int lx0 = bx * NB::LX, ly0 = by * NB::LY, lz0 = bz * NB::LZ;
    const double *r0 = resid + ((int64_t)bm * g.M + npts) * g.C;
    // rows t = 0..7: two groups of four (FP32), or half a block of 16
    constexpr int RB4 = sizeof(T) == 4 ? 2 : 0, RB = sizeof(T) == 4 ? 2 : 1;
    vec4 acc[NC][RB];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            acc[c][rb] = vec4{0, 0, 0, 0};
    for (int comp = 0; comp < g.C; ++comp) {
        const int cls = comp_class(g.C, comp);
        const double sc = cls == 0 ? g.G * g.h * g.h : g.G * g.h;
        near_fill<T, NC>(g, 4 * (lx0 - 1), 4 * (ly0 - 1), 4 * (lz0 - 1), tid, dens,
                         [&](int64_t cell) { return sc * r0[cell * g.C + comp]; });
        __syncthreads();
        const NearStage<T, NC> st(dens, hs, tid, cls);
        near_products<T, NC, RB - RB4, RB4>(st, hs, A + (int64_t)(comp * 8 + chi) * (kOctant / 4) * RB * 64, tid, chi, acc);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (sizeof(T) == 8) {
                if (r < 2)
                    ex[(chi * 8 + kr + 4 * r) * EP + c * 16 + (lane & 15)] = acc[c][0][r];
            } else {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    // the four sub-rows' sums, in a fixed order
                    T v = acc[c][rb][r];
                    v += __shfl_xor(v, 16);
                    v += __shfl_xor(v, 32);
                    if (lane < 16)
                        ex[(chi * 8 + 4 * rb + r) * EP + c * 16 + lane] = (double)v;
                }
            }
        }
    __syncthreads();
    for (int i = tid; i < 8 * NCOL; i += 512) {
        const int t = i / NCOL, col = i % NCOL;
        double v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x)
            v[x] = ex[(x * 8 + t) * EP + col];
        walsh8(v);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            ex[(r * 8 + t) * EP + col] = v[r];
    }
    __syncthreads();
    double *o = drho + (int64_t)bm * g.n[0] * g.n[1] * g.n[2];
    near_store<NC, 1>(g, lx0, ly0, lz0, tid, [&](int64_t cell, int r, int t, int col, int) {
        const double v = ex[(r * 8 + t) * EP + col];
        o[cell] = add ? o[cell] + v : v;
    });
}

// Transposed far-field evaluation at the centres (FP64 in both precisions): the
// adjoint LE of a leaf by coefficient class,
//   LE[k of class chi] = sum_{t, c} L[t, c][k] H_chi[t, c],
// H_chi the parity sums of the leaf's own weights (signs of class(c) included).
// A workgroup takes 4 x 2 x 2 leaves; the weights pass through LDS once as rows
// of the mesh, once as parity tiles, and the expansions leave as whole rows.
// With `add`, the LE of a leaf that also holds user points is added to, every
// other one set.  What bounds it: memory (0.40 GB of residuals and 0.24 GB of
// expansions at 256^3 cells, C = 3, p = 10); measured there against one product
// per leaf of all its centres, 0.44 -> 0.23 ms.
template <int RBC, int C>
__global__ void __launch_bounds__(512)
k_t_l2p_par(DevGeom g, NearGrid ng, const double *resid, int64_t npts, const double *A, const int32_t *coef,
            const int32_t *tmap, int add, const int64_t *leaf_start, const int64_t *pend, double *le)
{
    using NB = NearBlock<1>;
    using dvec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int W = 16 * C, RN = 512 / W, NR = (64 + RN - 1) / RN, R8 = 8 * C, kRaw = 64 * W, kOut = 16 * 257;
    __shared__ double sm[kRaw > kOut ? kRaw : kOut], tile[8 * R8 * 17];
    __shared__ int32_t srow[16], sadd[16];
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int chi = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t id = block_id();
    if (id >= (int64_t)ng.n * g.B)
        return;
    const int bm = (int)((uint32_t)id / (uint32_t)ng.n), blk = (int)((uint32_t)id - (uint32_t)bm * (uint32_t)ng.n);
    const int bx = blk % ng.nx, by = blk / ng.nx % ng.ny, bz = blk / (ng.nx * ng.ny);
    const int lx0 = bx * NB::LX, ly0 = by * NB::LY, lz0 = bz * NB::LZ;
    const DevLev &lv = g.lev[g.L];
    if (tid < 16) {
        const int lx = lx0 + tid % 4, ly = ly0 + tid / 4 % 2, lz = lz0 + tid / 8;
        const int64_t tl = lx < lv.ns[0] && ly < lv.ns[1] && lz < lv.ns[2]
                               ? tmap_lookup(lv, tmap, 3, lv.s0[0] + lx, lv.s0[1] + ly, lv.s0[2] + lz)
                               : -1;
        srow[tid] = tl >= 0 && tl < lv.n_tgt ? (int32_t)(lv.tgt_off + tl) : -1;
        sadd[tid] = add && srow[tid] >= 0 && pend[tl] > max(leaf_start[tl], (int64_t)0);
    }
    {
        const double *r0 = resid + ((int64_t)bm * g.M + npts) * C;
        const int x = tid % W / C, c = tid % C, q = tid / W, ix = 4 * lx0 + x;
        const double sc = comp_class(C, c) == 0 ? g.G * g.h * g.h : g.G * g.h;
        double v[NR];
        int in[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int row = q + RN * i, iy = 4 * ly0 + (row & 7), iz = 4 * lz0 + (row >> 3);
            in[i] = (int)(q < RN) & (int)(row < 64) & (int)(ix < g.n[0]) & (int)(iy < g.n[1]) & (int)(iz < g.n[2]);
            v[i] = r0[in[i] ? (((int64_t)iz * g.n[1] + iy) * g.n[0] + ix) * C + c : 0];
        }
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (q < RN && q + RN * i < 64)
                sm[(q + RN * i) * W + x * C + c] = in[i] ? sc * v[i] : 0.0;
    }
    __syncthreads();
    if (tid < R8 * 16) {
        const int col = tid & 15, R = tid >> 4, c = R >> 3, cls = comp_class(C, c);
        const double *q = sm + 4 * (col & 3) * C + c;
        const int y = 4 * (col >> 2 & 1), z = 4 * (col >> 3);
        double v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int tx = r & 1 ? 1 - (R & 1) : 2 + (R & 1), ty = r & 2 ? 1 - (R >> 1 & 1) : 2 + (R >> 1 & 1),
                      tz = r & 4 ? 1 - (R >> 2 & 1) : 2 + (R >> 2 & 1);
            v[r] = q[((z + tz) * 8 + y + ty) * W + tx * C];
        }
        walsh8(v);
#pragma unroll
        for (int x = 0; x < 8; ++x)
            tile[((x ^ cls) * R8 + R) * 17 + col] = v[x];
    }
    __syncthreads();
    dvec4 acc[RBC];
#pragma unroll
    for (int rb = 0; rb < RBC; ++rb)
        acc[rb] = dvec4{0, 0, 0, 0};
    double a[2 * C][RBC];
#pragma unroll
    for (int ks = 0; ks < 2 * C; ++ks)
#pragma unroll
        for (int rb = 0; rb < RBC; ++rb)
            a[ks][rb] = A[((chi * 2 * C + ks) * RBC + rb) * 64 + lane];
#pragma unroll
    for (int ks = 0; ks < 2 * C; ++ks) {
        const double b = tile[(chi * R8 + 4 * ks + kr) * 17 + (lane & 15)];
#pragma unroll
        for (int rb = 0; rb < RBC; ++rb)
            acc[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks][rb], b, acc[rb], 0, 0, 0);
    }
    const int OP = g.PS + 1;
#pragma unroll
    for (int rb = 0; rb < RBC; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = coef[chi * 16 * RBC + 16 * rb + kr + 4 * i];
            sm[(lane & 15) * OP + (k >= 0 ? k : g.PS)] = acc[rb][i];  // (PS: a spare place)
        }
    for (int i = tid; i < 16 * (g.PS - g.P2); i += 512)
        sm[i / (g.PS - g.P2) * OP + g.P2 + i % (g.PS - g.P2)] = 0.0;
    __syncthreads();
    // two columns per wave
    for (int c = 2 * chi; c < 2 * chi + 2; ++c) {
        if (srow[c] < 0)
            continue;
        double *o = le + ((int64_t)srow[c] * g.B + bm) * g.PS;
        for (int k = lane; k < g.PS; k += 64)
            o[k] = sadd[c] ? o[k] + sm[c * OP + k] : sm[c * OP + k];
    }
}

template <int NC>
grav_status near_grid(const Plan *p, NearGrid &ng, dim3 &grid)
{
    using NB = NearBlock<NC>;
    const LevelInfo &lv = p->lev[p->L];
    ng.nx = (lv.ns[0] + NB::LX - 1) / NB::LX;
    ng.ny = (lv.ns[1] + NB::LY - 1) / NB::LY;
    ng.n = ng.nx * ng.ny * ((lv.ns[2] + NB::LZ - 1) / NB::LZ);
    if ((int64_t)ng.n * p->B > 0x7fffffffll)
        return GRAV_EUNSUPPORTED;
    grid = block_grid((int64_t)ng.n * p->B);
    return GRAV_OK;
}

template <typename T, int NC>
grav_status near_forward(const Plan *p, const DevGeom &g, const double *rho, double *out, hipStream_t s)
{
    NearGrid ng{};
    dim3 grid;
    GRAV_CHECK(near_grid<NC>(p, ng, grid));
#define NEAR_CASE(C)                                                                                              \
    case C:                                                                                                       \
        hipLaunchKernelGGL((k_near_par<T, NC, C>), grid, dim3(512), 0, s, g, ng, rho,                             \
                           reinterpret_cast<const T *>(p->d_near_op), (const double *)p->d_near_far,              \
                           (const int32_t *)p->d_near_coef, p->near_KC, (const int32_t *)p->d_tmap,               \
                           (const double *)p->d_le, p->d.n_points, out);                                          \
        break;
    switch (p->C) {
        NEAR_CASE(1)
        NEAR_CASE(3)
        NEAR_CASE(4)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef NEAR_CASE
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

template <typename T, int NC>
grav_status near_transposed(const Plan *p, const DevGeom &g, const double *resid, int add, double *drho, hipStream_t s)
{
    NearGrid ng{};
    dim3 grid;
    GRAV_CHECK(near_grid<NC>(p, ng, grid));
    hipLaunchKernelGGL((k_t_near_par<T, NC>), grid, dim3(512), 0, s, g, ng, resid, p->d.n_points,
                       reinterpret_cast<const T *>(p->d_near_opt), add, drho);
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

}  // namespace

grav_status launch_near_par(const Plan *p, const DevGeom &g, const double *rho, double *out, hipStream_t s)
{
    return p->d.precision == GRAV_FP64 ? near_forward<double, 1>(p, g, rho, out, s) : near_forward<float, 1>(p, g, rho, out, s);
}

grav_status launch_t_l2p_par(const Plan *p, const DevGeom &g, const double *resid, int add, hipStream_t s)
{
    NearGrid ng{};
    dim3 grid;
    GRAV_CHECK(near_grid<1>(p, ng, grid));
    const int h = (p->P + 1) / 2, RBC = (h * (h + 1) / 2 + 15) / 16;
#define TL2P(RBC, C)                                                                                              \
    hipLaunchKernelGGL((k_t_l2p_par<RBC, C>), grid, dim3(512), 0, s, g, ng, resid, p->d.n_points,                 \
                       (const double *)p->d_near_fart, (const int32_t *)p->d_class_coef, (const int32_t *)p->d_tmap, add, \
                       (const int64_t *)p->d_leaf_start, (const int64_t *)p->d_leaf_pend, p->d_le)
#define TL2P_CASE(C)                                                                                              \
    case C:                                                                                                       \
        if (RBC == 1)                                                                                             \
            TL2P(1, C);                                                                                           \
        else if (RBC == 2)                                                                                        \
            TL2P(2, C);                                                                                           \
        else                                                                                                      \
            TL2P(3, C);                                                                                           \
        break;
    switch (p->C) {
        TL2P_CASE(1)
        TL2P_CASE(3)
        TL2P_CASE(4)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef TL2P_CASE
#undef TL2P
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

grav_status launch_t_near_par(const Plan *p, const DevGeom &g, const double *resid, int add, double *drho, hipStream_t s)
{
    if (p->d.precision == GRAV_FP64)
        return near_transposed<double, 1>(p, g, resid, add, drho, s);
    NearGrid n1{}, n2{};
    dim3 grid;
    GRAV_CHECK(near_grid<1>(p, n1, grid));
    GRAV_CHECK(near_grid<2>(p, n2, grid));
    const bool wide = p->lev[p->L].n_src * p->B >= GRAV_NEAR_WIDE_LEAVES && 20 * (int64_t)n2.n <= 11 * (int64_t)n1.n;
    return wide ? near_transposed<float, 2>(p, g, resid, add, drho, s) : near_transposed<float, 1>(p, g, resid, add, drho, s);
}

}  // namespace grav
