// P2M of lattice sources and its transpose over sibling octets (octet.hpp).
//
// With rho_r[v] the density of child r's cell v, its axes mirrored into the
// (+,+,+) child's frame, and H_chi[v] = sum_r (-1)^(chi.r) rho_r[v]:
//   leaf    X_r[k] = (-1)^(class(k).r) sum_v Pm[v][k] rho_r[v],
//   parent  Y[i]   = sum_v T[i][v] H_{class(i)}[v],   T = M2M of that child times Pm,
// so the parents of the leaves need an eighth of the products and no leaf
// expansions, and those are formed only where the M2L reads them (under
// surface stations: the top of the mesh), in the M2L's element type.  The
// transpose takes the leaf level's M2L slots as they are, by parity:
//   drho_r[v] = sum_chi (-1)^(chi.r) (sum_k Pm[v][k] G_chi[k] + sum_{i of class chi} T[i][v] Y[i]).
//
// What bounds them: far from the stations the densities (read or written once),
// a workgroup's phases one after the other; where the leaves count, also the
// FP64 matrix instructions of Pm.  p = 10, leaf 4^3, from
// the densities to the level above the leaves and back, M2M and FP32 rows
// included: 32 models of 128^3 cells under stations 0.85 -> 0.19 ms (2.8 TB/s
// of densities) and 0.79 -> 0.22 ms; 256^3 cells with all leaves 0.27 -> 0.14 ms
// and 0.29 -> 0.16 ms.
#include <algorithm>

#include "octet.hpp"

// Up to a block per CU the P2M runs all octets with the leaf part in one launch:
// a block's chunks are a chain (1.2 us each), and two launches are two of them.
// Calls with two launches against one, us, p = 4: 64^3 cells in leaves of 8^3
// under stations 109 / 77 (the per-leaf form before 87); p = 10: 64^3 in leaves of
// 4^3 103 / 97, 128^3 (256 blocks) 121 / 113, x 16 models of 128^3 in leaves of 8^3
// (512 blocks) 311 / 331; FP64 p = 14 (two parts) 128^3 (512 blocks) 216 / 225.
#ifndef GRAV_P2M_ONE_LAUNCH_BLOCKS
#define GRAV_P2M_ONE_LAUNCH_BLOCKS 256
#endif

// The transpose takes blocks across models from this many blocks of single
// models on; fewer leave CUs idle, and a block reads as many slots a lane again.
// Octets in one block, of a model against across models, us: 12^3 cells (8
// octets), p = 10, x 64 models 40 against 59, x 256 28 / 32, x 512 37 / 29, x 2048
// 91 / 54; FP64 p = 14 65 / 83, 39 / 47, 49 / 36, 162 / 94.  The P2M is as fast or
// faster across models from 4 models on (12^3 x 512 40 against 21, 83 / 43).
#ifndef GRAV_T_P2M_PACK_BLOCKS
#define GRAV_T_P2M_PACK_BLOCKS 384
#endif

namespace grav {

namespace {

constexpr int kMaxCells = kMaxLeafCells * kMaxLeafCells * kMaxLeafCells;

struct P2MArgs {
    const uint32_t *key;            // of the leaf level's octets
    const int32_t *child, *parent;  // (parent -1: leaves at level 2)
    // octets; (octet, model) columns, octets fastest, `per` to a model (noct, or
    // whole blocks); blocks of 16
    uint32_t noct, per, ncol, nblk;
    int part;                       // parts of a block's rows
    int64_t at;                     // first octet's index in its level
    // octet and model of a column (past the last: the last one), whether there is one
    __device__ bool column(uint32_t col, int64_t &oct, int &bm) const
    {
        const uint32_t c = min(col, ncol - 1);
        bm = ncol == per ? 0 : (int)(c / per);
        const uint32_t j = c - bm * per;
        oct = min(j, noct - 1);
        return c == col && j < noct;
    }
};

// Cells of the (+,+,+) child: offsets from the octet's centre along the axes,
// and coordinates (a byte each).  The mirrored cell lies at -offset - stride.
struct CellEntry {
    int o[3];
    uint32_t v;
};
__device__ __forceinline__ void cell_table(const DevGeom &g, CellEntry *cell, int tid)
{
    const int b = g.b;
    for (int v = tid; v < b * b * b; v += 512) {
        const int x = v % b, y = v / b % b, z = v / (b * b);
        cell[v] = CellEntry{{x, y * g.n[0], z * g.n[0] * g.n[1]}, (uint32_t)x | (uint32_t)y << 8 | (uint32_t)z << 16};
    }
}

// An octet's centre: its coordinates in the mesh, and its element index in the
// densities of model bm.
struct Centre {
    int x[3];
    int64_t at;
    __device__ void set(const DevGeom &g, uint32_t key, int bm)
    {
#pragma unroll
        for (int a = 0; a < 3; ++a)
            x[a] = (2 * (int)compact3(key >> a) + 1 - g.shift[a]) * g.b;
        at = (((int64_t)bm * g.n[2] + x[2]) * g.n[1] + x[1]) * g.n[0] + x[0];
    }
};

// The images of a cell along axis a: coordinate in the mesh, and offset.
__device__ __forceinline__ int image_in(const DevGeom &g, const Centre &c, const CellEntry &e, int a, int neg)
{
    const int v = (int)(e.v >> (8 * a) & 255u);
    return (uint32_t)(c.x[a] + (neg ? -1 - v : v)) < (uint32_t)g.n[a];
}
__device__ __forceinline__ int image_off(const DevGeom &g, const CellEntry &e, int a, int neg)
{
    const int stride = a == 0 ? 1 : a == 1 ? g.n[0] : g.n[0] * g.n[1];
    return neg ? -e.o[a] - stride : e.o[a];
}

// A workgroup takes 16 columns (octet, model), octets fastest (16 octets of one
// model left meshes of few octets mostly empty: 4096 models of 16 x 4 x 4 cells,
// p = 10, 0.20 against 0.05 ms); wave w forms child w's leaf expansions (LEAF) and
// the parents' rows of class w.  The cells pass through
// LDS 16 at a time, as they are and as parity sums; a lane loads the four
// children on one side of the x plane, its partner four lanes on the others
// (with leaf edge 4, eight lanes then read 64 consecutive bytes).
// Pm's fragments pass through LDS too: read by each wave for itself, the loads
// of eight waves took longer than their products.  Orders of more than 8 row
// blocks take the leaf rows in two parts (the parents with the first).
template <int P, typename T, bool LEAF>
__global__ void __launch_bounds__(512, !LEAF || P <= 10 ? 4 : 2)
k_p2m_octet(DevGeom g, P2MArgs ar, const double *rho, const double *A, const double *Ap, const int32_t *coef, T *leaf,
            double *me, float *me32)
{
    using C = ClassShape<P>;
    using vec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int PS = OctShape<P, T>::PS, RB = PS / 16, RBL = RB > 8 ? (RB + 1) / 2 : RB, OP = PS + 1;
    // k step u, sub-row kr and column c at US u + 18 kr + c: the staging's 32
    // lanes (16 cells, two tiles) and the products' reads spread over the banks
    constexpr int US = 72, TILE = 4 * US + 1, kTiles = (LEAF ? 2 : 1) * 8 * TILE, kOut = 16 * OP;
    constexpr int NA = (4 * RBL * 64 + 511) / 512;  // operator values per thread and chunk
    __shared__ double sm[kTiles > kOut ? kTiles : kOut];
    __shared__ double sa[LEAF ? NA * 512 : 1], sp[LEAF ? 8 * 4 * C::RBC * 64 : 1];
    __shared__ CellEntry cell[kMaxCells];
    __shared__ __align__(4) uint8_t scls[LEAF ? PS : 4];
    __shared__ int64_t srow[16];
    double *const par = sm, *const raw = sm + 8 * TILE;
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t blk = (uint32_t)block_id(), bi = __builtin_amdgcn_readfirstlane(blk / (uint32_t)ar.part);
    const int part = (int)(blk - bi * ar.part);
    if (bi >= ar.nblk)
        return;
    const uint32_t col0 = bi * 16;
    const int b3 = g.b * g.b * g.b, NCH = (b3 + 15) / 16;
    cell_table(g, cell, tid);
    int64_t oct;
    int bm;
    if (tid < 16) {
        const bool valid = ar.column(col0 + tid, oct, bm);
        srow[tid] = valid ? (int64_t)ar.parent[oct] * g.B + bm : -1;
    }
    if (LEAF && tid < PS)
        scls[tid] = (uint8_t)sign_class(tid);
    // staging: column, cell of the chunk, side of the x plane
    const int scol = 2 * w + (lane >> 5), sv = (lane & 3) | (lane >> 1 & 12), half = lane >> 2 & 1;
    Centre ctr;
    ar.column(col0 + scol, oct, bm);
    ctr.set(g, ar.key[oct], bm);
    const bool up = ar.parent[0] >= 0 && part == 0;
    vec4 acc[RBL], accp[C::RBC];
#pragma unroll
    for (int r = 0; r < RBL; ++r)
        acc[r] = vec4{0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < C::RBC; ++r)
        accp[r] = vec4{0, 0, 0, 0};
    // the next chunk's densities and operators
    double m[4], ra[NA], ap[4][C::RBC];
    uint32_t ok = 0;
    const double *Au = Ap + (int64_t)w * 4 * NCH * C::RBC * 64 + lane;
    auto load = [&](int q) {
        if constexpr (LEAF)
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int e = tid + 512 * i;
                ra[i] = A[(q * ar.part + part) * (4 * RBL * 64) + min(e, 4 * RBL * 64 - 1)];
            }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < C::RBC; ++r)
                ap[u][r] = Au[((4 * q + u) * C::RBC + r) * 64];
        const int v = 16 * q + sv;
        const CellEntry e = cell[min(v, b3 - 1)];
        const int ix = image_in(g, ctr, e, 0, half) & (int)(v < b3);
        const int64_t x = ctr.at + image_off(g, e, 0, half);
        ok = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int in = ix & image_in(g, ctr, e, 1, r & 1) & image_in(g, ctr, e, 2, r >> 1);
            ok |= in ? 1u << r : 0u;
            m[r] = rho[in ? x + (image_off(g, e, 1, r & 1) + image_off(g, e, 2, r >> 1)) : 0];
        }
    };
    __syncthreads();
    load(0);
    for (int q = 0; q < NCH; ++q) {
        double h[4];
        [[maybe_unused]] double ca[4][C::RBC];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            h[r] = (ok >> r) & 1u ? m[r] : 0.0;
        if (q > 0)
            __syncthreads();  // the previous chunk's products are done
        const int at = (sv >> 2) * US + 18 * (sv & 3) + scol;
        if constexpr (LEAF) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                raw[(2 * r + half) * TILE + at] = h[r];
#pragma unroll
            for (int i = 0; i < NA; ++i)
                sa[tid + 512 * i] = ra[i];
        }
#pragma unroll
        for (int bit = 1; bit < 4; bit <<= 1)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if ((r & bit) == 0) {
                    const double x = h[r], y = h[r | bit];
                    h[r] = x + y;
                    h[r | bit] = x - y;
                }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double o = __shfl_xor(h[r], 4);
            par[(2 * r + half) * TILE + at] = half ? o - h[r] : h[r] + o;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < C::RBC; ++r)
                if constexpr (LEAF)
                    sp[((w * 4 + u) * C::RBC + r) * 64 + lane] = ap[u][r];
                else
                    ca[u][r] = ap[u][r];
        load(min(q + 1, NCH - 1));
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int at2 = w * TILE + u * US + 18 * kr + (lane & 15);
            const double bp = par[at2];
#pragma unroll
            for (int r = 0; r < C::RBC; ++r)
                accp[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                    LEAF ? sp[LEAF ? ((w * 4 + u) * C::RBC + r) * 64 + lane : 0] : ca[u][r], bp, accp[r], 0, 0, 0);
            if constexpr (LEAF) {
                const double bl = raw[at2];
#pragma unroll
                for (int r = 0; r < RBL; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[(u * RBL + r) * 64 + lane], bl, acc[r], 0, 0, 0);
            }
        }
    }
    // this lane's leaf, if the M2L reads it: the fragments' rows are ordered so
    // that a lane holds four consecutive coefficients of a block
    int32_t row = -1;
    if constexpr (LEAF) {
        const DevLev &lv = g.lev[g.L];
        bool need = ar.column(col0 + (lane & 15), oct, bm);
        const uint32_t k = ar.key[oct];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int c = 2 * (int)compact3(k >> a) + (w >> a & 1 ? 0 : 1);
            need = need && c >= lv.need_lo[a] && c <= lv.need_hi[a];
        }
        row = ar.child[oct * 8 + (7 ^ w)];
        row = need ? row : -1;
    }
    if (row >= 0) {
        using t4 = __attribute__((__vector_size__(4 * sizeof(T)))) T;
#pragma unroll
        for (int r = 0; r < RBL; ++r) {
            const int k0 = 16 * (part * RBL + r) + 4 * kr;
            if (RB == RBL || part * RBL + r < RB) {
                const uint32_t c = *reinterpret_cast<const uint32_t *>(scls + k0);
                t4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[i] = (T)(0x96u >> (c >> (8 * i) & (uint32_t)w) & 1u ? -acc[r][i] : acc[r][i]);
                *reinterpret_cast<t4 *>(leaf + ((int64_t)row * g.B + bm) * PS + k0) = v;
            }
        }
    }
    if (!up)
        return;
    __syncthreads();
    int ck[C::RBC][4];
#pragma unroll
    for (int r = 0; r < C::RBC; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            ck[r][i] = coef[w * 16 * C::RBC + 16 * r + kr + 4 * i];
#pragma unroll
    for (int r = 0; r < C::RBC; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            sm[(lane & 15) * OP + (ck[r][i] >= 0 ? ck[r][i] : PS)] = accp[r][i];  // (PS: a spare place)
    if constexpr (PS > P * P)
        for (int i = tid; i < 16 * (PS - P * P); i += 512)
            sm[i / (PS - P * P) * OP + P * P + i % (PS - P * P)] = 0.0;
    __syncthreads();
    for (int i = tid; i < 16 * PS; i += 512) {
        const int c = i / PS, k = i % PS;
        if (srow[c] < 0)
            continue;
        const int64_t o = srow[c] * PS + k;
        const double v = sm[c * OP + k];
        me[o] = v;
        if (me32)
            me32[o] = (float)v;
    }
}

// The transpose.  A workgroup takes 16 columns (octet, model) and NRB blocks of
// 16 cells; wave chi the products of parity chi, its slots (U > 0: U at a time)
// straight from memory, Pm's fragments and the parents' rows through LDS, where
// the eight parities meet as well.
template <int P, typename T, int NRB, int U>
__global__ void __launch_bounds__(512)
k_t_p2m_octet(DevGeom g, P2MArgs ar, SlotArgs<T> sl, const double *A, const double *Ap, const int32_t *coef,
              const double *me, double *drho)
{
    using C = ClassShape<P>;
    using vec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int PS = OctShape<P, T>::PS, RB = PS / 16, XP = PS + 1, KC = C::KC, GP = 17, NV = 32;
    constexpr int NX = 8 / OctShape<P, T>::RS, RS = OctShape<P, T>::RS;
    constexpr int kX = 16 * XP, kG = 8 * NV * GP, kA = 4 * NRB * 64, NA = kA / 512;
    static_assert(2 * kA <= kG, "operator chunks do not fit");
    __shared__ double sm[kX > kG ? kX : kG];
    __shared__ CellEntry cell[kMaxCells];
    __shared__ Centre sctr[16];
    __shared__ int64_t srow[16];
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int chi = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t blk = (uint32_t)block_id(), bi = __builtin_amdgcn_readfirstlane(blk / (uint32_t)ar.part);
    const int part = (int)(blk - bi * ar.part);
    if (bi >= ar.nblk)
        return;
    const uint32_t col0 = bi * 16;
    const int b3 = g.b * g.b * g.b, RBT = NRB * ar.part;
    cell_table(g, cell, tid);
    int64_t oct;
    int bm;
    if (tid < 16) {
        const bool valid = ar.column(col0 + tid, oct, bm);
        srow[tid] = (int64_t)ar.parent[oct] * g.B + bm;
        sctr[tid].set(g, ar.key[oct], bm);
        if (!valid)
            sctr[tid].x[0] = g.n[0] + 2 * kMaxLeafCells;  // its cells lie outside the mesh
    }
    __syncthreads();
    const bool down = ar.parent[0] >= 0;
    vec4 acc[NRB];
#pragma unroll
    for (int r = 0; r < NRB; ++r)
        acc[r] = vec4{0, 0, 0, 0};
    // this lane's slots, four coefficients at a time, the first slot's one ahead
    constexpr int DS = U == 0 ? 0 : 1;
    [[maybe_unused]] T nx[DS + 1][4];
    [[maybe_unused]] const T *pc = nullptr;
    [[maybe_unused]] int jb = 0, je = 0;
    [[maybe_unused]] bool some = false;
    const int64_t xs = (int64_t)sl.ncol * PS;
    if constexpr (U > 0) {
        ar.column(col0 + (lane & 15), oct, bm);
        const int64_t col = (ar.at + oct) * g.B + bm;
        const int64_t un = (sl.g0 + col / sl.ncol) * RS + chi / NX;
        jb = sl.uslot[un];
        je = sl.uslot[un + 1];
        some = je > jb;
        if (!some)
            jb = je = 0;
        pc = sl.part + (col % sl.ncol) * PS + (int64_t)(chi % NX) * xs + 4 * kr;
#pragma unroll
        for (int q = 0; q < (DS < RB ? DS : RB); ++q)
            load4(pc + (int64_t)jb * NX * xs + 16 * q, nx[q]);
    }
    if (down) {
        double f[KC <= 4 ? KC : 1][NRB];  // (higher orders: loaded where they are used)
        const double *Ax = Ap + ((int64_t)chi * KC * RBT + part * NRB) * 64 + lane;
        if constexpr (KC <= 4)
#pragma unroll
            for (int q = 0; q < KC; ++q)
#pragma unroll
                for (int r = 0; r < NRB; ++r)
                    f[q][r] = Ax[(q * RBT + r) * 64];
        int k[KC];
#pragma unroll
        for (int q = 0; q < KC; ++q)
            k[q] = coef[chi * 16 * C::RBC + 4 * q + kr];
        constexpr int NI = (16 * PS + 511) / 512;
        double y[NI];
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int i = min(tid + 512 * n, 16 * PS - 1);
            y[n] = me[srow[i / PS] * PS + i % PS];
        }
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int i = min(tid + 512 * n, 16 * PS - 1);
            sm[i / PS * XP + i % PS] = y[n];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            const double b = k[q] >= 0 ? sm[(lane & 15) * XP + k[q]] : 0.0;
#pragma unroll
            for (int r = 0; r < NRB; ++r)
                acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(KC <= 4 ? f[KC <= 4 ? q : 0][r] : Ax[(q * RBT + r) * 64], b,
                                                              acc[r], 0, 0, 0);
        }
    }
    if constexpr (U > 0) {
        // operator chunk q: four k steps of this part's row blocks
        double ra[NA];
        auto fragments = [&](int q) {
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int e = tid + 512 * i;
                ra[i] = A[((int64_t)(4 * q + e / (NRB * 64)) * RBT + part * NRB) * 64 + e % (NRB * 64)];
            }
        };
        fragments(0);
        __syncthreads();  // the parents' rows have been read
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            double *sa = sm + (q & 1) * kA;
#pragma unroll
            for (int i = 0; i < NA; ++i)
                sa[tid + 512 * i] = ra[i];
            double b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                b[u] = some ? (double)nx[q % DS][u] : 0.0;
            for (int j = jb + 1; j < je; j += U) {
                T s[U][4];
#pragma unroll
                for (int n = 0; n < U; ++n)
                    load4(pc + (int64_t)min(j + n, je - 1) * NX * xs + 16 * q, s[n]);
#pragma unroll
                for (int n = 0; n < U; ++n)
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        b[u] += j + n < je ? (double)s[n][u] : 0.0;
            }
            if (q + 1 < RB)
                fragments(q + 1);
            if (q + DS < RB)
                load4(pc + (int64_t)jb * NX * xs + 16 * (q + DS), nx[q % DS]);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int r = 0; r < NRB; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[(u * NRB + r) * 64 + lane], b[u], acc[r], 0, 0, 0);
        }
    }
    // two row blocks at a time (35 KB: three workgroups per CU; all four at once
    // left room for two, and the stores, half of the time, waited: 0.225 ms against
    // 0.207 far from the stations); a thread takes the four images of a cell on
    // one side of the x plane
#pragma unroll
    for (int r0 = 0; r0 < NRB; r0 += 2) {
        __syncthreads();  // LDS has been read
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                sm[(chi * NV + 16 * r + kr + 4 * i) * GP + (lane & 15)] = acc[r0 + r][i];
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 32 * NV / 512; ++n) {
            const int e = tid + 512 * n, rx = e >> 2 & 1, f = (e & 3) | (e >> 1 & ~3), vi = f % NV, c = f / NV;
            const int v = part * 16 * NRB + 16 * r0 + vi;
            double h[4];
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                const double x0 = sm[(2 * y * NV + vi) * GP + c], x1 = sm[((2 * y + 1) * NV + vi) * GP + c];
                h[y] = rx ? x0 - x1 : x0 + x1;
            }
#pragma unroll
            for (int bit = 1; bit < 4; bit <<= 1)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if ((r & bit) == 0) {
                        const double x = h[r], y = h[r | bit];
                        h[r] = x + y;
                        h[r | bit] = x - y;
                    }
            const Centre ct = sctr[c];
            const CellEntry ce = cell[min(v, b3 - 1)];
            if (v < b3 && image_in(g, ct, ce, 0, rx)) {
                double *d = drho + ct.at + image_off(g, ce, 0, rx);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (image_in(g, ct, ce, 1, r & 1) & image_in(g, ct, ce, 2, r >> 1))
                        d[image_off(g, ce, 1, r & 1) + image_off(g, ce, 2, r >> 1)] = h[r];
            }
        }
    }
}

// The leaf level's octets: within reach of the M2L, the others, or all of them.
// Blocks across models where blocks of single ones would be more than `pack` and
// an eighth of their columns or more empty (blocks that start at an octet row of
// the mesh read and write it in longer runs: 18 models of 76^3 cells, 4% empty,
// 43.6 us against 44.5).
enum class Reach { near, far, all };
P2MArgs p2m_args(const Plan *p, Reach r, int part, int64_t pack)
{
    const OctPlan &o = p->m2lt;
    const int64_t mid = o.reach[p->L], o0 = r == Reach::far ? mid : o.first[p->L];
    const int64_t noct = (r == Reach::near ? mid : o.first[p->L + 1]) - o0;
    const int64_t whole = (noct + 15) / 16;
    const int64_t per = whole * p->B * part > pack && 8 * 16 * whole >= 9 * noct ? noct : 16 * whole, ncol = per * p->B;
    return P2MArgs{o.d_key + o0,  o.d_child + 8 * o0, o.d_parent + o0, (uint32_t)noct,
                   (uint32_t)per, (uint32_t)ncol,     (uint32_t)((ncol + 15) / 16), part, o0 - o.first[p->L]};
}

}  // namespace

#define GRAV_ORDERS(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

// Expansions of the parents of the leaves, and of the leaves that the M2L
// reads into its input rows.
template <typename T>
static grav_status p2m(const Plan *p, const DevGeom &g, const double *rho, T *leaf, float *rows, Reach r, hipStream_t s)
{
    const bool far = r == Reach::far;
    const P2MArgs ar = p2m_args(p, r, !far && p->PS > 128 ? 2 : 1, 0);
    const int64_t grid = (int64_t)ar.nblk * ar.part;
    if ((int64_t)ar.per * p->B + 16 * (1 << 22) > 0xffffffffll)
        return GRAV_EUNSUPPORTED;  // (half a terabyte of expansions)
    // with no level above (leaves at level 2) the others have nothing to set
    if (grid == 0 || (far && p->L < 3))
        return GRAV_OK;
#define P2M_LAUNCH(P, LEAF)                                                                                      \
    hipLaunchKernelGGL((k_p2m_octet<P, T, LEAF>), block_grid(grid), dim3(512), 0, s, g, ar, rho,             \
                       (const double *)p->d_pm, (const double *)p->d_pm_up, (const int32_t *)p->d_class_coef, leaf, \
                       p->d_me, rows)
#define P2M_CASE(P)                                                                                              \
    case P:                                                                                                      \
        if (far)                                                                                                 \
            P2M_LAUNCH(P, false);                                                                                \
        else                                                                                                     \
            P2M_LAUNCH(P, true);                                                                                 \
        break;
    switch (p->P) {
        GRAV_ORDERS(P2M_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef P2M_CASE
#undef P2M_LAUNCH
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

grav_status launch_p2m(const Plan *p, const DevGeom &g, const double *rho, hipStream_t s)
{
    float *rows = reinterpret_cast<float *>(p->d_rows);
    auto run = [&](Reach r) {
        return p->d.precision == GRAV_FP64 ? p2m<double>(p, g, rho, p->d_me, nullptr, r, s)
                                           : p2m<float>(p, g, rho, rows, rows, r, s);
    };
    const OctPlan &o = p->m2lt;
    if ((o.first[p->L + 1] - o.first[p->L]) * p->B * (p->PS > 128 ? 2 : 1) <= 16 * GRAV_P2M_ONE_LAUNCH_BLOCKS)
        return run(Reach::all);
    GRAV_CHECK(run(Reach::near));
    return run(Reach::far);
}

// drho from the parents' adjoint expansions and the leaf level's M2L slots.
template <typename T>
static grav_status t_p2m(const Plan *p, const DevGeom &g, double *drho, Reach r, hipStream_t s)
{
    const bool far = r == Reach::far;
    const int RBT = (p->b * p->b * p->b + 15) / 16, NRB = RBT <= 2 ? 2 : 4;
    const OctPlan &o = p->m2lt;
    const P2MArgs ar = p2m_args(p, r, (RBT <= 2 ? 2 : (RBT + 3) / 4 * 4) / NRB, GRAV_T_P2M_PACK_BLOCKS);
    const int64_t grid = (int64_t)ar.nblk * ar.part;
    if ((int64_t)ar.per * p->B + 16 * (1 << 22) > 0xffffffffll)
        return GRAV_EUNSUPPORTED;  // (half a terabyte of expansions)
    if (grid == 0)
        return GRAV_OK;
    const SlotArgs<T> sl{reinterpret_cast<const T *>(p->d_part), o.d_uslot, o.gfirst[p->L], 16 * o.nc};
    // plans whose units are cut into many slots have few columns: several
    // loads in flight there
    const bool many = o.nseg > 2 * (int64_t)o.nunit;
#define T_P2M_LAUNCH(P, NRB, U)                                                                                  \
    hipLaunchKernelGGL((k_t_p2m_octet<P, T, NRB, U>), block_grid(grid), dim3(512), 0, s, g, ar, sl,          \
                       (const double *)p->d_pmt, (const double *)p->d_pmt_down, (const int32_t *)p->d_class_coef, \
                       (const double *)p->d_me, drho)
#define T_P2M_CASE(P)                                                                                            \
    case P:                                                                                                      \
        if (NRB == 2 && far)                                                                                     \
            T_P2M_LAUNCH(P, 2, 0);                                                                               \
        else if (NRB == 2)                                                                                       \
            T_P2M_LAUNCH(P, 2, 4);                                                                               \
        else if (far)                                                                                            \
            T_P2M_LAUNCH(P, 4, 0);                                                                               \
        else if (many)                                                                                           \
            T_P2M_LAUNCH(P, 4, 4);                                                                               \
        else                                                                                                     \
            T_P2M_LAUNCH(P, 4, 1);                                                                               \
        break;
    switch (p->P) {
        GRAV_ORDERS(T_P2M_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef T_P2M_CASE
#undef T_P2M_LAUNCH
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

grav_status launch_t_p2m(const Plan *p, const DevGeom &g, double *drho, hipStream_t s)
{
    for (Reach r : {Reach::near, Reach::far})
        GRAV_CHECK(p->d.precision == GRAV_FP64 ? t_p2m<double>(p, g, drho, r, s) : t_p2m<float>(p, g, drho, r, s));
    return GRAV_OK;
}

}  // namespace grav
