// Forward evaluation: upward sweep (P2M, M2M), downward sweep (M2L, L2L),
// evaluation (L2P and the near-field direct sum), following the stages of
// the FMM in Sec. 2.3.  All geometry is in the lattice frame (cell units,
// mesh origin at 0); see plan.hip.
#include <algorithm>
#include <cmath>

#include "octet.hpp"
#include "resolve.hpp"

namespace grav {

// Explicit sources: the leaves' expansions in FP32 for the mixed M2L (the
// levels above are written by the M2M).  Leaves farther than 3 boxes from every target box (for
// surface stations, the deep part of the mesh) are skipped: no M2L reads them.
// One thread per four coefficients; src and dst at the level's first row.
__global__ void __launch_bounds__(256) k_leaf_f32(DevGeom g, const double *src, int64_t n4, float *dst)
{
    const int64_t i = block_id() * blockDim.x + threadIdx.x;
    if (i >= n4)
        return;
    const int64_t j = i / ((int64_t)(g.PS / 4) * g.B);
    const DevLev &lv = g.lev[g.L];
    const int x = lv.s0[0] + (int)(j % lv.ns[0]), y = lv.s0[1] + (int)((j / lv.ns[0]) % lv.ns[1]),
              z = lv.s0[2] + (int)(j / ((int64_t)lv.ns[0] * lv.ns[1]));
    if (x < lv.need_lo[0] || x > lv.need_hi[0] || y < lv.need_lo[1] || y > lv.need_hi[1] || z < lv.need_lo[2] ||
        z > lv.need_hi[2])
        return;
    const double2 a = reinterpret_cast<const double2 *>(src)[2 * i], b = reinterpret_cast<const double2 *>(src)[2 * i + 1];
    reinterpret_cast<float4 *>(dst)[i] = make_float4((float)a.x, (float)a.y, (float)b.x, (float)b.y);
}

// --------------------------------------------------------------------------
// Near field (P2P): direct sum over the quadrature points of the cells of the
// 27 leaves around a target leaf (the near term of Eq. (13)); coincident
// pairs are skipped.  One workgroup per target leaf; the mesh cells of the 27
// leaves are staged in LDS 1024 at a time (positions relative to the leaf's
// corner, and densities: four loads per thread in flight and two barriers, where
// leaf by leaf took 27 round trips to memory); targets are spread over lanes
// and, when a leaf holds fewer than 256 targets, the sources over several lane
// groups whose partial sums are reduced through LDS.  Output in the lattice
// frame: near[i][model] = (sum m/r, sum m d/r^3).  FP64, 1024 stations over 16^3
// cells: 0.049 -> 0.021 ms.
// --------------------------------------------------------------------------
constexpr int kP2PChunk = 1024;

// Adds one source's terms (1/r, d/r^3) times its mass.
template <typename T>
__device__ __forceinline__ void add_pair(T cx, T cy, T cz, T mass, T (&acc)[4])
{
    const T r2 = cx * cx + cy * cy + cz * cz;
    if (r2 > coincident2<T>()) {
        const T ri = rsqrt_t(r2);
        const T m = mass * ri;
        const T m3 = m * ri * ri;
        acc[0] += m;
        acc[1] += m3 * cx;
        acc[2] += m3 * cy;
        acc[3] += m3 * cz;
    }
}

template <typename T>
__global__ void __launch_bounds__(256)
k_p2p(DevGeom g, const double *rho, const double *tpos, const int64_t *leaf_start,
      const int64_t *leaf_end, const uint32_t *tkey, const int32_t *leaves, int64_t n_leaves, double *near)
{
    __shared__ __align__(16) T sp[kP2PChunk][4];
    __shared__ double red[256][4];
    const DevLev &lv = g.lev[g.L];
    // a target leaf holding user points (past the last: the first without any)
    const bool in = block_id() < n_leaves;
    const int64_t leaf = leaves[in ? block_id() : 0];
    const int64_t ts = leaf_start[leaf], te = in ? leaf_end[leaf] : ts;
    const int64_t nt = te - ts;
    if (nt <= 0)
        return;  // no explicit points in this leaf (uniform over the workgroup)
    const uint32_t key = tkey[lv.tbox_off + leaf];
    const int lc[3] = {(int)compact3(key), (int)compact3(key >> 1), (int)compact3(key >> 2)};
    // the mesh cells of the 27 leaves, relative to the leaf's corner
    int corner[3], c0[3], cn[3];
    for (int a = 0; a < 3; ++a) {
        corner[a] = (lc[a] - g.shift[a]) * g.b;
        c0[a] = max(-g.b, -corner[a]);
        cn[a] = max(0, min(2 * g.b, g.n[a] - corner[a]) - c0[a]);
    }
    const int ncl = cn[0] * cn[1] * cn[2];
    // none (e.g. stations far above the mesh): the near field is zero
    if (ncl == 0) {
        for (int64_t e = threadIdx.x; e < nt * g.B * 4; e += blockDim.x)
            near[ts * g.B * 4 + e] = 0.0;
        return;
    }
    int TC = 1;
    while (TC < nt && TC < 256)
        TC <<= 1;
    const int S = 256 / TC;
    const int t = threadIdx.x;
    const int ti = t % TC, si = t / TC;
    const int64_t ncell = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const T go = (T)(0.5 / 1.7320508075688772);  // Gauss point offset, cell units
    for (int bm = 0; bm < g.B; ++bm) {
        for (int64_t t0 = 0; t0 < nt; t0 += TC) {
            const int64_t j = ts + t0 + ti;
            const bool valid = (t0 + ti) < nt;
            T tl[3] = {0, 0, 0};
            if (valid)
                for (int a = 0; a < 3; ++a)
                    tl[a] = (T)(tpos[3 * j + a] - (double)corner[a]);
            T acc[4] = {0, 0, 0, 0};
            for (int v0 = 0; v0 < ncl; v0 += kP2PChunk) {
                const int nv = min(kP2PChunk, ncl - v0);
                double r[kP2PChunk / 256];
                int c[kP2PChunk / 256][3];
#pragma unroll
                for (int i = 0; i < kP2PChunk / 256; ++i) {
                    const int v = min(v0 + t + 256 * i, ncl - 1);
                    const int yz = v / cn[0];
                    c[i][0] = c0[0] + v - yz * cn[0];
                    c[i][2] = yz / cn[1];
                    c[i][1] = c0[1] + yz - c[i][2] * cn[1];
                    c[i][2] += c0[2];
                    r[i] = rho[bm * ncell + ((int64_t)(corner[2] + c[i][2]) * g.n[1] + corner[1] + c[i][1]) * g.n[0] +
                               corner[0] + c[i][0]];
                }
                __syncthreads();  // the previous chunk has been read
#pragma unroll
                for (int i = 0; i < kP2PChunk / 256; ++i) {
                    T *q = sp[t + 256 * i];
                    q[0] = (T)c[i][0] + (T)0.5;
                    q[1] = (T)c[i][1] + (T)0.5;
                    q[2] = (T)c[i][2] + (T)0.5;
                    q[3] = (T)r[i];
                }
                __syncthreads();
                if (!valid)
                    continue;
                for (int v = si; v < nv; v += S) {
                    const T rv = sp[v][3];
                    if (rv == (T)0)
                        continue;
                    const T cx = tl[0] - sp[v][0], cy = tl[1] - sp[v][1], cz = tl[2] - sp[v][2];
                    if (g.q == 1) {
                        add_pair(cx, cy, cz, rv, acc);
                    } else {
#pragma unroll
                        for (int gp = 0; gp < 8; ++gp)
                            add_pair(cx - ((gp & 1) ? go : -go), cy - ((gp & 2) ? go : -go), cz - ((gp & 4) ? go : -go),
                                     rv * (T)0.125, acc);
                    }
                }
            }
            // reduce the S source groups
            __syncthreads();
            for (int c = 0; c < 4; ++c)
                red[t][c] = (double)acc[c];
            __syncthreads();
            if (si == 0 && valid) {
                double s4[4] = {0, 0, 0, 0};
                for (int k = 0; k < S; ++k)
                    for (int c = 0; c < 4; ++c)
                        s4[c] += red[k * TC + ti][c];
                double *o = near + (j * g.B + bm) * 4;
                for (int c = 0; c < 4; ++c)
                    o[c] = s4[c];
            }
        }
    }
}

// Explicit sources: masses in sorted order, mass[model][i].
__global__ void __launch_bounds__(256)
k_src_mass(const double *rho, const double *sw, const uint32_t *sperm, int64_t nsrc, int64_t n, double *mass)
{
    const int64_t t = block_id() * blockDim.x + threadIdx.x;
    if (t >= n)
        return;
    const int64_t i = t % nsrc;
    mass[t] = rho[t - i + sperm[i]] * sw[i];
}

// The nine runs of sources around a target leaf.
struct SourceRuns {
    const int64_t *start, *end;
};

// The sums of TG targets j0, j0 + 1, ... (those from te on repeat the last one,
// unused) over the runs, a thread per source: near[(j, model bm)].
template <typename T, int TG>
__device__ __forceinline__ void p2p_few(const SourceRuns &run, const double *spos, const double *mass, const double *tpos,
                                        const double (&corner)[3], int64_t j0, int64_t te, double *red, int bm, int B,
                                        double *near)
{
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    T tl[TG][3], acc[TG][4];
#pragma unroll
    for (int k = 0; k < TG; ++k)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            if (a < 3)
                tl[k][a] = (T)(tpos[3 * min(j0 + k, te - 1) + a] - corner[a]);
            acc[k][a] = 0;
        }
    struct Source {
        double x, y, z, m;
    };
    auto load = [&](int64_t i) { return Source{spos[3 * i + 0], spos[3 * i + 1], spos[3 * i + 2], mass[i]}; };
    auto add = [&](const Source &q) {
        const T sx = (T)(q.x - corner[0]), sy = (T)(q.y - corner[1]), sz = (T)(q.z - corner[2]), m = (T)q.m;
#pragma unroll
        for (int u = 0; u < TG; ++u)
            add_pair(tl[u][0] - sx, tl[u][1] - sy, tl[u][2] - sz, m, acc[u]);
    };
    // three runs at a time (each mostly shorter than the workgroup: the idle
    // wave changes from run to run)
#pragma unroll 1
    for (int k = 0; k < 9; k += 3) {
        int64_t i[3], e[3];
        Source q[3];
#pragma unroll
        for (int n = 0; n < 3; ++n) {
            i[n] = run.start[k + n] + ((t + 64 * n) & 255);
            e[n] = run.end[k + n];
            q[n] = load(max(min(i[n], e[n] - 1), (int64_t)0));
        }
#pragma unroll
        for (int n = 0; n < 3; ++n)
            if (i[n] < e[n])
                add(q[n]);
#pragma unroll
        for (int n = 0; n < 3; ++n)
            for (int64_t v = i[n] + 256; v < e[n]; v += 256)
                add(load(v));
    }
    // four sums over 64 lanes, target by target: two steps hand half of them on
    constexpr int N = 4 * TG;
#pragma unroll
    for (int u = 0; u < TG; ++u) {
        const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0;
        const double x = (double)(b0 ? acc[u][2] : acc[u][0]) + __shfl_xor((double)(b0 ? acc[u][0] : acc[u][2]), 1);
        const double y = (double)(b0 ? acc[u][3] : acc[u][1]) + __shfl_xor((double)(b0 ? acc[u][1] : acc[u][3]), 1);
        double v = (b1 ? y : x) + __shfl_xor(b1 ? x : y, 2);
#pragma unroll
        for (int bit = 4; bit < 64; bit <<= 1)
            v += __shfl_xor(v, bit);
        if (lane < 4)
            red[w * N + 4 * u + (b0 ? 2 : 0) + (b1 ? 1 : 0)] = v;
    }
    __syncthreads();
    if (t < N && j0 + t / 4 < te)
        near[((j0 + t / 4) * B + bm) * 4 + t % 4] = (red[t] + red[N + t]) + (red[2 * N + t] + red[3 * N + t]);
    __syncthreads();
}

// Near field with explicit sources: direct sum over the sources of the 27
// leaves around a target leaf (the near term of Eq. (13)), coincident pairs
// skipped; the sources of three leaves in a row along x are consecutive: nine
// runs.  Leaves of up to 16 targets: a thread per source, up to four targets at
// a time, sums reduced at the end (no barrier per leaf of sources, every lane
// busy: 65536 random points, two a leaf, 2.1 M sources 0.83 -> 0.22 ms, and 0.04 for the masses).  Others:
// targets over lanes, the sources staged in LDS in chunks of 256 and, when a
// leaf holds fewer than 256 targets, spread over several lane groups reduced
// through LDS in a fixed order.  Output as k_p2p, lattice frame.
template <typename T>
__global__ void __launch_bounds__(256)
k_p2p_src(DevGeom g, const double *mass, const double *spos, const int64_t *sstart, int64_t nsrc, const double *tpos,
          const int64_t *leaf_start, const int64_t *leaf_end, const uint32_t *tkey, const int32_t *leaves, int64_t n_leaves,
          double *near)
{
    __shared__ T sp[256][4];
    __shared__ double red[256][4];
    const DevLev &lv = g.lev[g.L];
    // a target leaf holding user points (past the last: the first without any)
    const bool in = block_id() < n_leaves;
    const int64_t leaf = leaves[in ? block_id() : 0];
    const int64_t ts = leaf_start[leaf], te = in ? leaf_end[leaf] : ts;
    const int64_t nt = te - ts;
    if (nt <= 0)
        return;
    const uint32_t key = tkey[lv.tbox_off + leaf];
    const int lc[3] = {(int)compact3(key), (int)compact3(key >> 1), (int)compact3(key >> 2)};
    double corner[3];
    for (int a = 0; a < 3; ++a)
        corner[a] = (double)((lc[a] - g.shift[a]) * g.b);
    const int t = threadIdx.x;
    // the runs of sources
    __shared__ int64_t rs[9], re[9];
    if (t < 9) {
        const int x0 = max(lc[0] - lv.s0[0] - 1, 0), x1 = min(lc[0] - lv.s0[0] + 1, lv.ns[0] - 1);
        const int y = lc[1] - lv.s0[1] + t % 3 - 1, z = lc[2] - lv.s0[2] + t / 3 - 1;
        const bool in = x0 <= x1 && y >= 0 && y < lv.ns[1] && z >= 0 && z < lv.ns[2];
        const int64_t row = in ? ((int64_t)z * lv.ns[1] + y) * lv.ns[0] : 0;
        rs[t] = in ? sstart[row + x0] : 0;
        re[t] = in ? sstart[row + x1 + 1] : 0;
    }
    __syncthreads();
    if (nt <= 16) {
        const SourceRuns run{rs, re};
        for (int bm = 0; bm < g.B; ++bm) {
            const double *m = mass + (int64_t)bm * nsrc;
            double *rd = &red[0][0];
            if (nt == 1)
                p2p_few<T, 1>(run, spos, m, tpos, corner, ts, te, rd, bm, g.B, near);
            else if (nt == 2)
                p2p_few<T, 2>(run, spos, m, tpos, corner, ts, te, rd, bm, g.B, near);
            else
                for (int64_t j0 = ts; j0 < te; j0 += 4)
                    p2p_few<T, 4>(run, spos, m, tpos, corner, j0, te, rd, bm, g.B, near);
        }
        return;
    }
    int TC = 1;
    while (TC < nt && TC < 256)
        TC <<= 1;
    const int S = 256 / TC;
    const int ti = t % TC, si = t / TC;
    for (int bm = 0; bm < g.B; ++bm) {
        for (int64_t c0 = 0; c0 < nt; c0 += TC) {
            const int64_t j = ts + c0 + ti;
            const bool valid = (c0 + ti) < nt;
            T tl[3] = {0, 0, 0};
            if (valid)
                for (int a = 0; a < 3; ++a)
                    tl[a] = (T)(tpos[3 * j + a] - corner[a]);
            T acc[4] = {0, 0, 0, 0};
            for (int k = 0; k < 9; ++k)
                for (int64_t s0 = rs[k]; s0 < re[k]; s0 += 256) {
                    const int nv = (int)min((int64_t)256, re[k] - s0);
                    __syncthreads();
                    if (t < nv) {
                        for (int a = 0; a < 3; ++a)
                            sp[t][a] = (T)(spos[3 * (s0 + t) + a] - corner[a]);
                        sp[t][3] = (T)mass[(int64_t)bm * nsrc + s0 + t];
                    }
                    __syncthreads();
                    if (!valid)
                        continue;
                    for (int v = si; v < nv; v += S)
                        add_pair(tl[0] - sp[v][0], tl[1] - sp[v][1], tl[2] - sp[v][2], sp[v][3], acc);
                }
            __syncthreads();
            for (int c = 0; c < 4; ++c)
                red[t][c] = (double)acc[c];
            __syncthreads();
            if (si == 0 && valid) {
                double s4[4] = {0, 0, 0, 0};
                for (int k = 0; k < S; ++k)
                    for (int c = 0; c < 4; ++c)
                        s4[c] += red[k * TC + ti][c];
                double *o = near + (j * g.B + bm) * 4;
                for (int c = 0; c < 4; ++c)
                    o[c] = s4[c];
            }
        }
    }
}

// --------------------------------------------------------------------------
// Densities in leaf blocks for the lattice near field, in the element type
// of the near-field contraction.  Cell v of a leaf (x fastest, v < b^3) is
// contraction index v = kr * 4Q + 4 q + u (Q chunks of four k steps per
// instruction sub-row kr); the blocks are stored chunk-major,
//   blk[q][kr][pl * B + model][u],
// pl = leaf index in the source block padded by one leaf on every side, so
// that the 16 columns of a wave (consecutive leaves) read four contiguous
// runs per chunk.  The padding and cells outside the mesh stay zero.  One
// thread per cell.
// --------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
k_rho_blocks(DevGeom g, const double *rho, int Qn, int64_t nplB, T *blk)
{
    const DevLev &lv = g.lev[g.L];
    const int b = g.b, b2 = b * b, b3 = b2 * b;
    const int64_t nleaf = (int64_t)lv.ns[0] * lv.ns[1] * lv.ns[2];
    const int64_t i = block_id() * blockDim.x + threadIdx.x;
    if (i >= nleaf * g.B * b3)
        return;
    const int v = (int)(i % b3);
    const int bm = (int)((i / b3) % g.B);
    const int64_t leaf = i / ((int64_t)b3 * g.B);
    const int lx = (int)(leaf % lv.ns[0]), ly = (int)((leaf / lv.ns[0]) % lv.ns[1]),
              lz = (int)(leaf / ((int64_t)lv.ns[0] * lv.ns[1]));
    const int ix = lx * b + v % b, iy = ly * b + (v / b) % b, iz = lz * b + v / b2;
    double r = 0.0;
    if (ix < g.n[0] && iy < g.n[1] && iz < g.n[2])
        r = rho[(int64_t)bm * g.n[0] * g.n[1] * g.n[2] + ((int64_t)iz * g.n[1] + iy) * g.n[0] + ix];
    const int64_t pl = ((int64_t)(lz + 1) * (lv.ns[1] + 2) + (ly + 1)) * (lv.ns[0] + 2) + (lx + 1);
    const int kr = v / (4 * Qn), q = (v % (4 * Qn)) / 4, u = v % 4;
    blk[((int64_t)(q * 4 + kr) * nplB + pl * g.B + bm) * 4 + u] = (T)r;
}

// Lattice near-field tile: GRAV_NEAR_RW32 (FP32) or GRAV_NEAR_RW64 (FP64)
// row blocks x GRAV_NEAR_CW column blocks of 16, a tile per wave on plans
// with at least GRAV_NEAR_WAVE_TILES tiles, else a tile per workgroup of
// four waves; chunks per software-pipeline step.
#ifndef GRAV_NEAR_WAVE_TILES
#define GRAV_NEAR_WAVE_TILES 8192
#endif
#ifndef GRAV_NEAR_RW32
#define GRAV_NEAR_RW32 4
#endif
#ifndef GRAV_NEAR_RW64
#define GRAV_NEAR_RW64 2
#endif
#ifndef GRAV_NEAR_CW
#define GRAV_NEAR_CW 2
#endif
#ifndef GRAV_NEAR_DEPTH32
#define GRAV_NEAR_DEPTH32 2
#endif
#ifndef GRAV_NEAR_DEPTH64
#define GRAV_NEAR_DEPTH64 2
#endif

// --------------------------------------------------------------------------
// The voxel-centre targets, fused: near field + far field + combine, for
// leaves of 1 to 3 cells a side, and of 4 on plans whose blocks of leaves would
// stay mostly empty in near.hip.
// Targets and Gauss points both sit on the lattice, so the near field of a
// leaf's b^3 cell centres is
//   near[leaf] = sum over the 27 neighbour offsets d of  A_d rho[leaf + d],
// with A_d a fixed (C b^3) x b^3 matrix (the direct sum over the same point
// pairs, precomputed in FP64, rows for the C requested output components
// only), and the far field is a fixed (C b^3) x PS matrix applied to the
// leaf's local expansion (L2P at fixed points, FP64).
// Over all leaves these are GEMMs with columns = (leaf, model).
//
// A tile is 16 CW columns x 16 RW rows (CW x RW MFMA blocks, so every
// fragment loaded feeds CW or RW instructions).  NW = 1 (large plans): each
// wave owns a tile, runs its 27 Q near chunks (chunk = neighbour d, four k
// steps) and the far-field chunks, and writes the tile straight to the
// output in descriptor order, G applied.  NW = 4: the four waves of a
// workgroup share one tile and split the contraction (wave w a quarter of
// the near chunks and every fourth far-field chunk); the four partial tiles
// meet in LDS and are added in wave order (fixed, so the result is
// deterministic).  Operand fragments are group-major sets per (d, q, rb), the
// densities chunk-major (both read with contiguous-kilobyte vector loads).
// --------------------------------------------------------------------------
template <int RW, int CW, typename T, int NW>
__global__ void __launch_bounds__(256)
k_near_lat(DevGeom g, const T *blk, int64_t nplB, const T *A, const int64_t *ctab, int RBn, int Qn,
           const double *Lm, const int32_t *tmap, const double *le, int64_t npts, int nrg, int64_t ntile,
           double *out)
{
    using vec4 = __attribute__((__vector_size__(4 * sizeof(T)))) T;
    using dvec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    const int lane = threadIdx.x & 63;
    // wave-uniform (scalar registers): everything that depends only on the
    // chunk index below is scalar arithmetic
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // NW = 4: the workgroup's four waves share one tile; NW = 1: each wave
    // owns a tile of its own
    const int64_t tile = NW == 4 ? block_id() : block_id() * 4 + wave;
    if (tile >= ntile)
        return;  // past the grid's last: whole workgroups, or waves where there is no barrier (NW = 1)
    const int64_t cg = tile / nrg;
    const int rb0 = (int)(tile % nrg) * RW;
    const DevLev &lv = g.lev[g.L];
    const int64_t nleaf = (int64_t)lv.ns[0] * lv.ns[1] * lv.ns[2];
    const int b = g.b, b2 = b * b, b3 = b2 * b;
    const int px = lv.ns[0] + 2, py = lv.ns[1] + 2;
    const int kr = lane >> 4;
    // this lane's column in each column block
    bool cvalid[CW];
    int bm[CW], lx[CW], ly[CW], lz[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) {
        const int64_t col = (cg * CW + c) * 16 + (lane & 15);
        cvalid[c] = col < nleaf * g.B;
        const int64_t leaf = cvalid[c] ? col / g.B : 0;
        bm[c] = cvalid[c] ? (int)(col % g.B) : 0;
        lx[c] = (int)(leaf % lv.ns[0]);
        ly[c] = (int)((leaf / lv.ns[0]) % lv.ns[1]);
        lz[c] = (int)(leaf / ((int64_t)lv.ns[0] * lv.ns[1]));
    }
    bool rvalid[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r)
        rvalid[r] = rb0 + r < RBn;
    vec4 acc[CW][RW];
    dvec4 far[CW][RW];
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            acc[c][r] = vec4{0, 0, 0, 0};
            far[c][r] = dvec4{0, 0, 0, 0};
        }
    // near chunks [i0, i1) of this wave; the operands of the next chunk are
    // in flight while this chunk's instructions run
    const int NI = 27 * Qn;
    const int i0 = NW == 4 ? wave * NI / 4 : 0, i1 = NW == 4 ? (wave + 1) * NI / 4 : NI;
    // per lane: its column's density block at neighbour offset (0, 0, 0)
    // (padded coordinates) and sub-row kr; a chunk adds a uniform offset
    const T *bbase[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c)
        bbase[c] = blk + ((int64_t)kr * nplB + (((int64_t)lz[c] * py + ly[c]) * px + lx[c]) * g.B + bm[c]) * 4;
    // Chunk i's offsets come from the plan's table (scalar loads).  Rows past
    // the last row block read the last one and columns past the last column
    // read leaf 0 (both in bounds): an output element depends only on its
    // own row and column, and those are never written, so nothing needs
    // zeroing.
    auto loadc = [&](int i, T (&bb)[CW][4], T (&aa)[RW][4]) {
        const int64_t boff = ctab[2 * i], aoff = ctab[2 * i + 1];
#pragma unroll
        for (int c = 0; c < CW; ++c)
            load4(bbase[c] + boff, bb[c]);
        const T *ap = A + aoff;
#pragma unroll
        for (int r = 0; r < RW; ++r)
            load_frags<T, 4>(ap + (int64_t)min(rb0 + r, RBn - 1) * 256, lane, aa[r]);
    };
    auto compute = [&](const T (&bb)[CW][4], const T (&aa)[RW][4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    if constexpr (sizeof(T) == 8)
                        acc[c][r] = __builtin_amdgcn_mfma_f64_16x16x4f64(aa[r][u], bb[c][u], acc[c][r], 0, 0, 0);
                    else
                        acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(aa[r][u], bb[c][u], acc[c][r], 0, 0, 0);
                }
    };
    // Software pipeline over steps of D chunks: each step issues the loads of
    // the next step one by one between its own matrix instructions, so a
    // load has D chunks of instructions (and the other waves' work) to
    // arrive.  The chunks past the last whole step run unpipelined.
    constexpr int D = sizeof(T) == 8 ? GRAV_NEAR_DEPTH64 : GRAV_NEAR_DEPTH32;
    constexpr int NLD = D * (CW + RW * 4 * (int)sizeof(T) / 16), NMF = D * 4 * RW * CW;
    auto load_step = [&](int st, T (&bb)[D][CW][4], T (&aa)[D][RW][4]) {
#pragma unroll
        for (int j = 0; j < D; ++j)
            loadc(i0 + st * D + j, bb[j], aa[j]);
    };
    auto compute_step = [&](const T (&bb)[D][CW][4], const T (&aa)[D][RW][4]) {
#pragma unroll
        for (int j = 0; j < D; ++j)
            compute(bb[j], aa[j]);
    };
    const int nst = (i1 - i0) / D;
    if (nst > 0) {
        T bA[D][CW][4], bB[D][CW][4];
        T aA[D][RW][4], aB[D][RW][4];
        load_step(0, bA, aA);
        __builtin_amdgcn_sched_barrier(0);
        for (int st = 0; st < nst; st += 2) {
            load_step(min(st + 1, nst - 1), bB, aB);
            compute_step(bA, aA);
            interleave_loads<NLD, NMF>();
            __builtin_amdgcn_sched_barrier(0);
            if (st + 1 < nst) {
                load_step(min(st + 2, nst - 1), bA, aA);
                compute_step(bB, aB);
                interleave_loads<NLD, NMF>();
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    for (int i = i0 + nst * D; i < i1; ++i) {
        T bb[CW][4], aa[RW][4];
        loadc(i, bb, aa);
        compute(bb, aa);
    }
    // far field from the leaf's local expansion (FP64 in both precisions):
    // chunks q = wave, wave + 4, ...
    if (g.L >= 2) {
        bool hl[CW];
        const double2 *bp[CW];
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const int64_t tl = cvalid[c] ? tmap_lookup(lv, tmap, 3, lv.s0[0] + lx[c], lv.s0[1] + ly[c],
                                                       lv.s0[2] + lz[c])
                                         : -1;
            hl[c] = tl >= 0;
            bp[c] = (const double2 *)(le + (hl[c] ? ((lv.tgt_off + tl) * g.B + bm[c]) * g.PS : 0) + kr * (g.PS / 4));
        }
        const int QL = g.PS / 16;
        for (int q = NW == 4 ? wave : 0; q < QL; q += NW) {
            double bv[CW][4];
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const double2 b01 = bp[c][2 * q], b23 = bp[c][2 * q + 1];
                bv[c][0] = hl[c] ? b01.x : 0.0;
                bv[c][1] = hl[c] ? b01.y : 0.0;
                bv[c][2] = hl[c] ? b23.x : 0.0;
                bv[c][3] = hl[c] ? b23.y : 0.0;
            }
            double av[RW][4];
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                if (rvalid[r]) {
                    load_frags<double, 4>(Lm + ((int64_t)q * RBn + rb0 + r) * 256, lane, av[r]);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        av[r][u] = 0.0;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int r = 0; r < RW; ++r)
#pragma unroll
                    for (int c = 0; c < CW; ++c)
                        far[c][r] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[r][u], bv[c][u], far[c][r], 0, 0, 0);
        }
    }
    // row block R holds targets 16 (R % RBc) + row of output component
    // R / RBc (the row order of both operators, in lattice units); the
    // lane's element k is row 4 kr + k (FP32) or kr + 4 k (FP64)
    const double sg = g.G * g.h, sp = g.G * g.h * g.h;
    const int RBc = (b3 + 15) / 16;
    auto store = [&](int c, int r, auto &&value) {
        if (!cvalid[c] || !rvalid[r])
            return;
        const int comp = (rb0 + r) / RBc, tb = 16 * ((rb0 + r) % RBc);
        const double sc = g.C == 4 && comp == 0 ? sp : sg;
        double *o = out + ((int64_t)bm[c] * g.M + npts) * g.C + comp;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int t = tb + (sizeof(T) == 8 ? kr + 4 * k : 4 * kr + k);
            const int ix = lx[c] * b + t % b, iy = ly[c] * b + (t / b) % b, iz = lz[c] * b + t / b2;
            if (t >= b3 || ix >= g.n[0] || iy >= g.n[1] || iz >= g.n[2])
                continue;
            o[(((int64_t)iz * g.n[1] + iy) * g.n[0] + ix) * g.C] = sc * value(k);
        }
    };
    if constexpr (NW == 4) {
        // partial tiles to LDS (FP64), then each wave adds the four partials
        // of its blocks in wave order (fixed, so the result is deterministic)
        __shared__ double red[4][CW * RW * 4][64];
#pragma unroll
        for (int c = 0; c < CW; ++c)
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    red[wave][(c * RW + r) * 4 + k][lane] = (double)acc[c][r][k] + far[c][r][k];
        __syncthreads();
        for (int j = wave; j < CW * RW; j += 4)
            store(j / RW, j % RW, [&](int k) {
                return ((red[0][j * 4 + k][lane] + red[1][j * 4 + k][lane]) + red[2][j * 4 + k][lane]) +
                       red[3][j * 4 + k][lane];
            });
    } else {
#pragma unroll
        for (int c = 0; c < CW; ++c)
#pragma unroll
            for (int r = 0; r < RW; ++r)
                store(c, r, [&](int k) { return (double)acc[c][r][k] + far[c][r][k]; });
    }
}

// --------------------------------------------------------------------------
// host side
// --------------------------------------------------------------------------
DevGeom make_geom(const Plan *p)
{
    DevGeom g{};
    for (int l = 0; l <= p->L && l <= kMaxLevels; ++l) {
        const LevelInfo &s = p->lev[l];
        DevLev &d = g.lev[l];
        for (int a = 0; a < 3; ++a) {
            d.s0[a] = s.s0[a];
            d.ns[a] = s.ns[a];
        }
        d.me_off = s.me_off;
        d.tgt_off = s.tgt_off;
        d.tbox_off = p->tbox_off[l];
        d.tmap_off = s.tmap_off;
        d.n_tgt = s.n_tgt;
        for (int a = 0; a < 3; ++a) {
            d.need_lo[a] = s.need_lo[a];
            d.need_hi[a] = s.need_hi[a];
        }
    }
    g.L = p->L;
    g.b = p->b;
    g.q = p->q;
    g.P = p->P;
    g.P2 = p->P2;
    g.PS = p->PS;
    g.B = p->B;
    g.C = p->C;
    g.n[0] = p->d.nx;
    g.n[1] = p->d.ny;
    g.n[2] = p->d.nz;
    for (int a = 0; a < 3; ++a)
        g.shift[a] = p->shift[a];
    g.M = p->M;
    g.G = p->d.G;
    g.h = p->d.h;
    return g;
}

void stage_begin(Plan *p, const char *name, hipStream_t s)
{
    if (!p->profiling)
        return;
    if ((int)p->stages.size() <= p->n_stage_used) {
        Stage st;
        (void)hipEventCreate(&st.a);
        (void)hipEventCreate(&st.b);
        p->stages.push_back(st);
    }
    Stage &st = p->stages[p->n_stage_used];
    st.name = name;
    (void)hipEventRecord(st.a, s);
}

void stage_end(Plan *p, hipStream_t s)
{
    if (!p->profiling)
        return;
    (void)hipEventRecord(p->stages[p->n_stage_used].b, s);
    ++p->n_stage_used;
}

static grav_status launch_near_lat(Plan *p, const DevGeom &g, const double *rho, double *out, hipStream_t s)
{
    const LevelInfo &lv = p->lev[p->L];
    const int b3 = p->b * p->b * p->b;
    const int64_t nfill = lv.n_src * p->B * b3;
    const int64_t nplB = (int64_t)(lv.ns[0] + 2) * (lv.ns[1] + 2) * (lv.ns[2] + 2) * p->B;
    const bool f64 = p->d.precision == GRAV_FP64;
    const dim3 fgrid = block_grid((nfill + 255) / 256);
    if (f64)
        hipLaunchKernelGGL((k_rho_blocks<double>), fgrid, dim3(256), 0, s, g, rho, p->lat_Q, nplB,
                           p->d_rho_blk);
    else
        hipLaunchKernelGGL((k_rho_blocks<float>), fgrid, dim3(256), 0, s, g, rho, p->lat_Q, nplB,
                           reinterpret_cast<float *>(p->d_rho_blk));
    GRAV_HIP(hipGetLastError());
    const int64_t ncol = lv.n_src * p->B;
    const int RBn = p->lat_RB, Qn = p->lat_Q;
    constexpr int CW = GRAV_NEAR_CW;
    const int RW = f64 ? GRAV_NEAR_RW64 : GRAV_NEAR_RW32;
    const int nrg = (RBn + RW - 1) / RW;
    const int64_t ncg = (ncol + 16 * CW - 1) / (16 * CW);
    if (ncg * nrg > 0x7fffffffll)
        return GRAV_EUNSUPPORTED;
    const int64_t ntile = ncg * nrg;
    // a tile per wave once there are tiles for every wave slot of the chip,
    // else four waves per tile
    const bool per_wave = ntile >= GRAV_NEAR_WAVE_TILES;
    const dim3 grid = block_grid(per_wave ? (ntile + 3) / 4 : ntile), blk(256);
    const int64_t npts = p->d.n_points;
#define NEAR_LAUNCH(NW)                                                                                            \
    if (f64)                                                                                                       \
        hipLaunchKernelGGL((k_near_lat<GRAV_NEAR_RW64, CW, double, NW>), grid, blk, 0, s, g,                       \
                           (const double *)p->d_rho_blk, nplB, (const double *)p->d_tn64,                          \
                           (const int64_t *)p->d_lat_tab, RBn, Qn, (const double *)p->d_tl2p,                      \
                           (const int32_t *)p->d_tmap, (const double *)p->d_le, npts, nrg, ntile, out);            \
    else                                                                                                           \
        hipLaunchKernelGGL((k_near_lat<GRAV_NEAR_RW32, CW, float, NW>), grid, blk, 0, s, g,                        \
                           (const float *)p->d_rho_blk, nplB, (const float *)p->d_tn32,                            \
                           (const int64_t *)p->d_lat_tab, RBn, Qn, (const double *)p->d_tl2p,                      \
                           (const int32_t *)p->d_tmap, (const double *)p->d_le, npts, nrg, ntile, out);
    if (per_wave) {
        NEAR_LAUNCH(1)
    } else {
        NEAR_LAUNCH(4)
    }
#undef NEAR_LAUNCH
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

grav_status enqueue_forward(Plan *p, const double *rho, double *out, hipStream_t s)
{
    const DevGeom g = make_geom(p);
    const int L = p->L;
    if (p->M == 0)
        return GRAV_OK;
    if (p->n_spts > 0) {
        const int64_t n = p->n_spts * p->B;
        hipLaunchKernelGGL(k_src_mass, block_grid((n + 255) / 256), dim3(256), 0, s, rho, (const double *)p->d_sw,
                           (const uint32_t *)p->d_sperm, p->n_spts, n, p->d_smass);
        GRAV_HIP(hipGetLastError());
    }
    if (L >= 2) {
        stage_begin(p, "p2m", s);
        if (p->n_spts > 0) {
            GRAV_CHECK(launch_p2m_src(p, g, s));
        } else {
            GRAV_CHECK(launch_p2m(p, g, rho, s));
        }
        stage_end(p, s);
        // expansions in FP32 for the M2L of mixed plans
        float *rows = p->d.precision == GRAV_FP64 ? nullptr : reinterpret_cast<float *>(p->d_rows);
        stage_begin(p, "m2m", s);
        // (from lattice sources, the leaves' parents are set by the P2M)
        for (int l = p->n_spts > 0 ? L : L - 1; l >= 3; --l)
            GRAV_CHECK(launch_octet_up(p, p->m2lt, l, s, p->d_m2m, p->d_me, rows));
        stage_end(p, s);
        stage_begin(p, "m2l", s);
        {
            const OctGeom og = octet_geom(p, false);
            if (!rows) {
                GRAV_CHECK(launch_m2l<double>(p, p->m2l, s, og, p->d_me));
            } else {
                if (p->n_spts > 0) {
                    const int64_t at = p->lev[L].me_off * p->B * p->PS, n4 = p->lev[L].n_src * p->B * (p->PS / 4);
                    hipLaunchKernelGGL(k_leaf_f32, block_grid((n4 + 255) / 256), dim3(256), 0, s, g,
                                       (const double *)(p->d_me + at), n4, rows + at);
                    GRAV_HIP(hipGetLastError());
                }
                GRAV_CHECK(launch_m2l<float>(p, p->m2l, s, og, rows));
            }
        }
        stage_end(p, s);
        stage_begin(p, "l2l", s);
        for (int l = 2; l <= L; ++l)
            GRAV_CHECK(launch_octet_down(p, p->m2l, l, s, p->d_l2l, p->d_le));
        stage_end(p, s);
    }
    if (p->lat_near) {
        stage_begin(p, "near_lat", s);
        GRAV_CHECK(p->near_par ? launch_near_par(p, g, rho, out, s) : launch_near_lat(p, g, rho, out, s));
        stage_end(p, s);
    }
    if (!p->lat_near || p->d.n_points > 0) {
        stage_begin(p, "p2p", s);
        // one workgroup per target leaf holding user points
        const dim3 pgrid = block_grid(std::max<int64_t>(p->n_user_leaves, 1));
        const int32_t *ul = (const int32_t *)p->d_user_leaves;
        if (p->n_user_leaves == 0) {
        } else if (p->n_spts > 0 && p->d.precision == GRAV_FP64)
            hipLaunchKernelGGL(k_p2p_src<double>, pgrid, dim3(256), 0, s, g, (const double *)p->d_smass,
                               (const double *)p->d_spos, (const int64_t *)p->d_sstart, p->n_spts, (const double *)p->d_tpos,
                               (const int64_t *)p->d_leaf_start, (const int64_t *)p->d_leaf_pend,
                               (const uint32_t *)p->d_tkey, ul, p->n_user_leaves, p->d_near);
        else if (p->n_spts > 0)
            hipLaunchKernelGGL(k_p2p_src<float>, pgrid, dim3(256), 0, s, g, (const double *)p->d_smass,
                               (const double *)p->d_spos, (const int64_t *)p->d_sstart, p->n_spts, (const double *)p->d_tpos,
                               (const int64_t *)p->d_leaf_start, (const int64_t *)p->d_leaf_pend,
                               (const uint32_t *)p->d_tkey, ul, p->n_user_leaves, p->d_near);
        else if (p->d.precision == GRAV_FP64)
            hipLaunchKernelGGL(k_p2p<double>, pgrid, dim3(256), 0, s, g, rho,
                               (const double *)p->d_tpos, (const int64_t *)p->d_leaf_start,
                               (const int64_t *)p->d_leaf_pend, (const uint32_t *)p->d_tkey, ul, p->n_user_leaves, p->d_near);
        else
            hipLaunchKernelGGL(k_p2p<float>, pgrid, dim3(256), 0, s, g, rho,
                               (const double *)p->d_tpos, (const int64_t *)p->d_leaf_start,
                               (const int64_t *)p->d_leaf_pend, (const uint32_t *)p->d_tkey, ul, p->n_user_leaves, p->d_near);
        GRAV_HIP(hipGetLastError());
        stage_end(p, s);
        stage_begin(p, "l2p", s);
        GRAV_CHECK(launch_l2p_points(p, g, out, s));
        stage_end(p, s);
    }
    return GRAV_OK;
}

// Workspace lock of a plan: a call on another stream while the previous
// call's work is still in flight returns GRAV_EBUSY.  Under stream capture
// (a HIP graph being recorded) nothing is enqueued yet, so the lock is not
// consulted or updated and no event is recorded; the replays of a captured
// call are the caller's to serialise.
static bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone;
}

grav_status begin_call(Plan *p, hipStream_t s)
{
    p->n_stage_used = 0;
    if (capturing(s))
        return p->profiling ? GRAV_EUNSUPPORTED : GRAV_OK;
    if (p->has_pending && p->last_stream != s) {
        const hipError_t q = hipEventQuery(p->done);
        if (q == hipErrorNotReady)
            return GRAV_EBUSY;
        if (q != hipSuccess)
            return GRAV_EDEVICE;
    }
    return GRAV_OK;
}

grav_status end_call(Plan *p, hipStream_t s)
{
    if (capturing(s))
        return GRAV_OK;
    GRAV_HIP(hipEventRecord(p->done, s));
    p->has_pending = true;
    p->last_stream = s;
    return GRAV_OK;
}

}  // namespace grav

using namespace grav;

extern "C" grav_status grav_eval(grav_plan_t plan, const double *rho, double *g_out, void *stream)
{
    if (!plan)
        return GRAV_EINVAL;
    Plan *p = reinterpret_cast<Plan *>(plan);
    if (p->M == 0)
        return GRAV_OK;
    if (!rho || !g_out)
        return GRAV_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    int cur = 0;
    GRAV_HIP(hipGetDevice(&cur));
    if (cur != p->device)
        GRAV_HIP(hipSetDevice(p->device));
    grav_status st = begin_call(p, s);
    if (st == GRAV_OK)
        st = enqueue_forward(p, rho, g_out, s);
    if (st == GRAV_OK)
        st = end_call(p, s);
    if (cur != p->device)
        (void)hipSetDevice(cur);
    return st;
}

extern "C" grav_status grav_set_profiling(grav_plan_t plan, int32_t enable)
{
    if (!plan)
        return GRAV_EINVAL;
    (reinterpret_cast<Plan *>(plan))->profiling = enable != 0;
    return GRAV_OK;
}

extern "C" grav_status grav_stage_times(grav_plan_t plan, const char **names, double *ms,
                                        int32_t n, int32_t *count)
{
    if (!plan)
        return GRAV_EINVAL;
    Plan *p = reinterpret_cast<Plan *>(plan);
    int k = 0;
    for (int i = 0; i < p->n_stage_used && k < n; ++i, ++k) {
        Stage &st = p->stages[i];
        GRAV_HIP(hipEventSynchronize(st.b));
        float t = 0.f;
        GRAV_HIP(hipEventElapsedTime(&t, st.a, st.b));
        if (names)
            names[k] = st.name.c_str();
        if (ms)
            ms[k] = t;
    }
    if (count)
        *count = k;
    return GRAV_OK;
}
