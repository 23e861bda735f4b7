// L2P at user points (and at every target of plans without lattice matrices)
// with the combine, and the transpose: one workgroup per run of points of a
// target leaf (transposed: per leaf) and group of models.
//
// What bounds them: the chain of the harmonics' recurrences and the arithmetic
// in FP64.  The order is a template parameter, so the recurrences' reciprocals
// are constants (a division each before), and the orders m are split over the
// four waves.  The leaf's expansions pass through LDS; a thread per point read
// its own row from memory, one dependent load after the other.  p = 10: 32
// models at 65536 stations forward 0.25 -> 0.12 ms, transpose 0.43 -> 0.09 ms
// (sums on MFMA); one model at 262144 stations among 16.8 M cell centres 0.085 ->
// 0.023 ms (the centres are no longer visited) and 0.106 -> 0.052 ms; FP64 p =
// 14, 1024 stations 0.044 -> 0.006 ms.
#include <algorithm>

#include "harmonics.hpp"
#include "octet.hpp"

namespace grav {

namespace {

constexpr int kPointModels = 8;  // models per workgroup (1 on single-model plans)
constexpr int kRunsPerWorkgroup = 16;

// Wave w of four takes the orders m = w, 7 - w, 8 + w, 15 - w: columns of
// about equal length together.
__host__ __device__ constexpr int wave_of_order(int m) { return (m & 4) ? 3 - (m & 3) : (m & 3); }

// Visits R_n^m(u) of wave w's orders, f(n, m, Re, Im); n and m are constants
// of the unrolled code.
template <int P, int W, class F>
__device__ __forceinline__ void harmonics_of_wave(double x, double y, double z, F &&f)
{
    const double r2 = x * x + y * y + z * z;
    double mmr = 1.0, mmi = 0.0;
#pragma unroll
    for (int m = 0; m < P; ++m) {
        if (m > 0) {
            const double s = 1.0 / (2.0 * m);
            const double nr = (x * mmr - y * mmi) * s;
            const double ni = (x * mmi + y * mmr) * s;
            mmr = nr;
            mmi = ni;
        }
        if (wave_of_order(m) != W)
            continue;
        double p1r = 0.0, p1i = 0.0, p2r = 0.0, p2i = 0.0;
#pragma unroll
        for (int n = m; n < P; ++n) {
            double Rr, Ri;
            if (n == m) {
                Rr = mmr;
                Ri = mmi;
            } else if (n == m + 1) {
                Rr = z * p1r;
                Ri = z * p1i;
            } else {
                const double c = 1.0 / (double)((n - m) * (n + m));
                Rr = ((2.0 * n - 1.0) * z * p1r - r2 * p2r) * c;
                Ri = ((2.0 * n - 1.0) * z * p1i - r2 * p2i) * c;
            }
            p2r = p1r;
            p2i = p1i;
            p1r = Rr;
            p1i = Ri;
            f(n, m, Rr, Ri);
        }
    }
}
template <int P, class F>
__device__ __forceinline__ void harmonics_by_wave(int w, double x, double y, double z, F &&f)
{
    if (w == 0)
        harmonics_of_wave<P, 0>(x, y, z, f);
    else if (w == 1)
        harmonics_of_wave<P, 1>(x, y, z, f);
    else if (w == 2)
        harmonics_of_wave<P, 2>(x, y, z, f);
    else
        harmonics_of_wave<P, 3>(x, y, z, f);
}

struct PointArgs {
    const double *tpos;
    const int64_t *start, *end;  // of a leaf's points in sorted order
    const uint32_t *tkey;
    const int32_t *leaves;  // the target leaves holding points
    int64_t nleaf;          // their number
    int64_t limit;          // points of the caller's order from here on are set elsewhere
};

// The forward's workgroups: nblk blocks of runs per group of models.
struct RunArgs {
    const PointRun *runs;
    int64_t n, nblk, groups;
    int lw, mg;  // runs and models per workgroup
};

// Expansions of a workgroup of several runs: within 16 KB up to p = 11, 16 above
// (all that the registers let a CU hold fit its LDS).
__host__ __device__ constexpr int l2p_slots(int P) { return P > 11 ? 16 : 2048 / (P * P) < 64 ? 2048 / (P * P) : 64; }

__device__ __forceinline__ void leaf_centre(const DevGeom &g, uint32_t key, double (&c)[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a)
        c[a] = ((double)((int)compact3(key >> a) - g.shift[a]) + 0.5) * g.b;
}

// Forward: lanes are (point, model) pairs, points fastest; the four waves' sums
// meet in LDS.  A workgroup takes a run of a leaf's points (a workgroup per leaf
// walked all of them: 1024^2 stations above 16^3 cells are 16 leaves of 65536
// points, 2.20 ms a leaf at a time, 0.07 ms in runs; a thread per point took
// 0.14).  With LW > 1 it takes rn.lw runs, at most LW, so that its lanes are not
// mostly idle (runs_per_workgroup); their (run, model) pairs share the MG LW
// expansions in LDS.  far: whether there is a far field (L >= 2).
template <int P, int MG, int LW>
__global__ void __launch_bounds__(256)
k_l2p_points(DevGeom g, PointArgs ar, RunArgs rn, const uint32_t *perm, const double *le, const double *near, int far,
             double *out)
{
    static_assert(MG == 1 || LW == 1, "the expansions in LDS are counted for one of the two");
    constexpr int P2 = P * P, LS = P2 | 1, NS = LW == 1 ? MG : l2p_slots(P);
    __shared__ double sL[NS * LS];
    __shared__ double sum[4][4][64];
    __shared__ double sc[LW][3];
    __shared__ int64_t st[LW];
    __shared__ int sn[LW + 1];  // first pair of each leaf
    const DevLev &lv = g.lev[g.L];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t blk = (uint32_t)block_id(), nblk = (uint32_t)rn.nblk;
    if (blk >= nblk * (uint32_t)rn.groups)
        return;
    const uint32_t lb = blk % nblk;
    const int mgrp = LW == 1 ? MG : rn.mg;
    const int bm0 = (int)(blk / nblk) * mgrp, nm = min(mgrp, g.B - bm0);
    const int lw = LW == 1 ? 1 : rn.lw;
    const int nl = (int)min((int64_t)lw, rn.n - (int64_t)lb * lw);
    const PointRun *runs = rn.runs + (int64_t)lb * lw;
    const double inv_w = 1.0 / (double)g.b;
    if (tid < nl) {
        const PointRun r = runs[tid];
        double c[3];
        leaf_centre(g, ar.tkey[lv.tbox_off + r.leaf], c);
#pragma unroll
        for (int a = 0; a < 3; ++a)
            sc[tid][a] = c[a];
        st[tid] = r.start;
        sn[tid + 1] = r.n;
    }
    auto fetch = [&](int sl, int l, int m, int k) {
        sL[sl * LS + k] = le[((lv.tgt_off + runs[l].leaf) * g.B + bm0 + m) * g.PS + k];
    };
    // a run's models lie side by side
    if (far && (LW == 1 || nm == 1 || P2 < 64)) {
        for (int i = tid; i < nl * nm * P2; i += 256) {
            const int sl = i / P2, l = LW == 1 ? 0 : nm == 1 ? sl : sl / nm;
            fetch(sl, l, LW == 1 ? sl : sl - l * nm, i - sl * P2);
        }
    } else if (far) {
        // (a division for each of many coefficients takes longer)
        for (int l = 0; l < nl; ++l)
            for (int i = tid; i < nm * P2; i += 256)
                fetch(l * nm + i / P2, l, i / P2, i % P2);
    }
    __syncthreads();
    if (tid == 0) {
        sn[0] = 0;
        for (int l = 0; l < nl; ++l)
            sn[l + 1] += sn[l];
    }
    __syncthreads();
    const int np = sn[nl];
    for (int64_t u0 = 0; u0 < (int64_t)np * nm; u0 += 64) {
        const int64_t u = min(u0 + lane, (int64_t)np * nm - 1);
        int mg = 0, l = 0;
        if (LW == 1 || nm > 1)
            mg = (int)(u / np);
        int64_t at = u - (int64_t)mg * np;  // among the model's points
        if constexpr (LW > 1) {
            for (int k = 1; k < nl; ++k)
                l = at >= sn[k] ? k : l;
            at -= sn[l];
        }
        const int64_t i = st[l] + at;
        if (far) {
            const double x = (ar.tpos[3 * i + 0] - sc[l][0]) * inv_w, y = (ar.tpos[3 * i + 1] - sc[l][1]) * inv_w,
                         z = (ar.tpos[3 * i + 2] - sc[l][2]) * inv_w;
            const CoefArray L{sL + (l * nm + mg) * LS};
            double phi = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
            // pairs R_n^m with the coefficients of l2p_eval_t
            harmonics_by_wave<P>(w, x, y, z, [&](int n, int m, double Rr, double Ri) {
                if (m == 0)
                    phi += L.re(n, 0) * Rr;
                else
                    phi += 2.0 * (L.re(n, m) * Rr - L.im(n, m) * Ri);
                if (n + 1 < P) {
                    const int n1 = n + 1;
                    if (m == 0) {
                        gz += Rr * L.re(n1, 0);
                        gx += Rr * L.re(n1, 1);
                        gy -= Rr * L.im(n1, 1);
                    } else {
                        gz += 2.0 * (Rr * L.re(n1, m) - Ri * L.im(n1, m));
                        gx += Rr * (L.re(n1, m + 1) - L.re(n1, m - 1)) - Ri * (L.im(n1, m + 1) - L.im(n1, m - 1));
                        gy -= Rr * (L.im(n1, m + 1) + L.im(n1, m - 1)) + Ri * (L.re(n1, m + 1) + L.re(n1, m - 1));
                    }
                }
            });
            const double s = inv_w * inv_w;
            sum[w][0][lane] = phi * inv_w;
            sum[w][1][lane] = -gx * s;  // g = -grad phi
            sum[w][2][lane] = -gy * s;
            sum[w][3][lane] = -gz * s;
        }
        __syncthreads();
        if (w == 0 && u0 + lane < (int64_t)np * nm) {
            const int64_t dst = perm[i];
            if (dst < ar.limit) {
                const double *nr = near + (i * g.B + bm0 + mg) * 4;
                double v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    v[k] = nr[k] + (far ? (sum[0][k][lane] + sum[1][k][lane]) + (sum[2][k][lane] + sum[3][k][lane]) : 0.0);
                double *o = out + ((int64_t)(bm0 + mg) * g.M + dst) * g.C;
                const double sg = g.G * g.h, sp = g.G * g.h * g.h;
                if (g.C == 1) {
                    o[0] = sg * v[3];
                } else if (g.C == 3) {
                    o[0] = sg * v[1];
                    o[1] = sg * v[2];
                    o[2] = sg * v[3];
                } else {
                    o[0] = sp * v[0];
                    o[1] = sg * v[1];
                    o[2] = sg * v[2];
                    o[3] = sg * v[3];
                }
            }
        }
        __syncthreads();  // the sums have been read
    }
}

// Transpose.  The adjoint LE of a leaf is the derivative, with respect to its
// coefficients, of the sum over the leaf's points of a phi - (b1 gx + b2 gy +
// b3 gz), with (a, b) the point's weights scaled as the combine scales the far
// field (a = w0 / w, b = w_1..3 / w^2).  With the sums
//   S_c[h] = sum over points of (a, b1, b2, b3)_c R_h(point)
// coefficient (n, m) collects a R_n^m (x2 for m > 0) and the gradient terms of
// degree n-1 and orders m-1, m, m+1, as the evaluation pairs them (d/dz R_n^m =
// R_{n-1}^m, d/dx and d/dy from R_{n-1}^{m-1} and R_{n-1}^{m+1}).  S is a
// product of the (component, model) weights and the points' harmonics, 16
// points at a time on FP64 MFMA; points past the last weigh zero.
template <int LS>
__device__ __forceinline__ double l2pt_gather(const double *S, int CS, int n, int m, int part)
{
    auto h = [&](int c, int nn, int mm, int pp) -> double {
        if (nn < 0 || mm > nn || (mm == 0 && pp == 1))
            return 0.0;
        return S[c * CS + harm_index(nn, mm, pp)];
    };
    const int q = n - 1;  // degree of the gradient terms
    double v;
    if (part == 0) {
        v = (m == 0 ? 1.0 : 2.0) * h(0, n, m, 0);
        if (q >= 0) {
            if (m == 0) {
                v += -h(3, q, 0, 0) + h(1, q, 1, 0) + h(2, q, 1, 1);
            } else {
                v += -2.0 * h(3, q, m, 0);
                if (m == 1)
                    v -= h(1, q, 0, 0);
                else
                    v += h(2, q, m - 1, 1) - h(1, q, m - 1, 0);
                v += h(1, q, m + 1, 0) + h(2, q, m + 1, 1);
            }
        }
    } else {
        v = -2.0 * h(0, n, m, 1);
        if (q >= 0) {
            v += 2.0 * h(3, q, m, 1);
            if (m == 1)
                v += h(2, q, 0, 0);
            else
                v += h(1, q, m - 1, 1) + h(2, q, m - 1, 0);
            v += h(2, q, m + 1, 0) - h(1, q, m + 1, 1);
        }
    }
    return v;
}

template <int P, int MG>
__global__ void __launch_bounds__(256)
k_t_l2p_points(DevGeom g, PointArgs ar, const double *w, double *le)
{
    using vec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int P2 = P * P, RB = (P2 + 15) / 16, PS = 16 * RB, HS = PS + 1;
    constexpr int NR = (4 * MG + 15) / 16, NH = (RB + 3) / 4;  // row blocks; column blocks per wave
    constexpr int kS = 16 * NR * HS, kH = 16 * HS;
    __shared__ double sh[kS > kH ? kS : kH];  // harmonics [16][HS], then the sums [4][MG][HS]
    __shared__ double sw[16 * NR][17];        // weights [component][model][point]
    const DevLev &lv = g.lev[g.L];
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (block_id() >= ar.nleaf)
        return;
    const int64_t leaf = ar.leaves[block_id()];
    const int bm0 = blockIdx.z * MG;
    const int64_t ts = ar.start[leaf], te = ar.end[leaf];
    double c[3];
    leaf_centre(g, ar.tkey[lv.tbox_off + leaf], c);
    const double inv_w = 1.0 / (double)g.b, inv_w2 = inv_w * inv_w;
    vec4 acc[NR][NH];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int j = 0; j < NH; ++j)
            acc[r][j] = vec4{0, 0, 0, 0};
    // (the columns past the coefficients are never read)
    for (int64_t j0 = ts; j0 < te; j0 += 16) {
        for (int i = tid; i < 16 * NR * 16; i += 256) {
            const int t = i / (16 * NR), row = i % (16 * NR), mg = row / 4, k = row % 4;
            const bool ok = j0 + t < te && mg < MG && bm0 + mg < g.B;
            const double v = ok ? w[((j0 + t) * g.B + bm0 + mg) * 4 + k] : 0.0;
            if (row < 4 * MG)
                sw[k * MG + mg][t] = v * (k == 0 ? inv_w : inv_w2);
            else
                sw[row][t] = 0.0;
        }
        if (lane < 16) {
            const int64_t j = min(j0 + lane, te - 1);
            harmonics_by_wave<P>(wv, (ar.tpos[3 * j + 0] - c[0]) * inv_w, (ar.tpos[3 * j + 1] - c[1]) * inv_w,
                                 (ar.tpos[3 * j + 2] - c[2]) * inv_w, [&](int n, int m, double Rr, double Ri) {
                                     sh[lane * HS + (m == 0 ? n * n : n * n + 2 * m - 1)] = Rr;
                                     if (m > 0)
                                         sh[lane * HS + n * n + 2 * m] = Ri;
                                 });
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            double a[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r)
                a[r] = sw[16 * r + (lane & 15)][4 * ks + kr];
#pragma unroll
            for (int j = 0; j < NH; ++j) {
                const int hb = min(wv + 4 * j, RB - 1);
                const double b = sh[(4 * ks + kr) * HS + 16 * hb + (lane & 15)];
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    acc[r][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], b, acc[r][j], 0, 0, 0);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < NH; ++j)
        if (wv + 4 * j < RB)
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    sh[(16 * r + kr + 4 * i) * HS + 16 * (wv + 4 * j) + (lane & 15)] = acc[r][j][i];
    __syncthreads();
    for (int i = tid; i < MG * PS; i += 256) {
        const int mg = i / PS, k = i % PS, bm = bm0 + mg;
        if (bm >= g.B)
            break;
        double v = 0.0;  // padding coefficients stay zero
        if (k < P2) {
            const int n = (int)sqrtf((float)k + 0.5f), r = k - n * n;
            v = l2pt_gather<HS>(sh + mg * HS, MG * HS, n, (r + 1) / 2, (r > 0 && (r & 1) == 0) ? 1 : 0);
        }
        le[((lv.tgt_off + leaf) * g.B + bm) * PS + k] = v;
    }
}

// --------------------------------------------------------------------------
// P2M of explicit sources: the expansion of a leaf is the sum over its sources
// of the mass times the multipole basis at the source (the lattice P2M's basis:
// R_n^0, Re R_n^m, -Im R_n^m at u = (x - centre) / b).  One workgroup per (leaf
// of the source block, MG models); a lane per source of a chunk forms the
// harmonics of its wave's orders, [coefficient][source] in LDS, and every
// thread adds the products of the (model, coefficient) sums it owns in source
// order (deterministic).  2.1 M sources, 64 a leaf, p = 10: 0.55 -> 0.20 ms.
// --------------------------------------------------------------------------
template <int P, int MG>
__global__ void __launch_bounds__(256)
k_p2m_src(DevGeom g, const double *spos, const double *mass, const int64_t *sstart, int64_t nsrc, double *me)
{
    constexpr int P2 = P * P, PS = (P2 + 15) / 16 * 16;
    constexpr int TC = P <= 11 ? 64 : 32, TS = TC + 1;  // sources per chunk
    constexpr int NJ = (MG * P2 + 255) / 256;           // sums per thread, o = model P2 + coefficient
    __shared__ double H[P2 * TS], W[MG * TC];
    const DevLev &lv = g.lev[g.L];
    const uint32_t leaf = (uint32_t)block_id();
    if (leaf >= (uint32_t)lv.ns[0] * lv.ns[1] * lv.ns[2])
        return;
    const int bm0 = blockIdx.z * MG;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lx = (int)(leaf % lv.ns[0]), ly = (int)((leaf / lv.ns[0]) % lv.ns[1]),
              lz = (int)(leaf / ((int64_t)lv.ns[0] * lv.ns[1]));
    const double inv_b = 1.0 / (double)g.b;
    const double centre[3] = {(lx + 0.5) * g.b, (ly + 0.5) * g.b, (lz + 0.5) * g.b};
    const int64_t ts = sstart[leaf], te = sstart[leaf + 1];
    double acc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        acc[j] = 0.0;
    for (int64_t j0 = ts; j0 < te; j0 += TC) {
        const int nt = (int)min((int64_t)TC, te - j0);
        for (int i = tid; i < nt * MG; i += 256) {
            const int t = i % nt, bm = bm0 + i / nt;
            W[i / nt * TC + t] = bm < g.B ? mass[(int64_t)bm * nsrc + j0 + t] : 0.0;
        }
        if (lane < nt) {
            const int64_t i = j0 + lane;
            harmonics_by_wave<P>(w, (spos[3 * i + 0] - centre[0]) * inv_b, (spos[3 * i + 1] - centre[1]) * inv_b,
                                 (spos[3 * i + 2] - centre[2]) * inv_b, [&](int n, int m, double Rr, double Ri) {
                                     H[(m == 0 ? n * n : n * n + 2 * m - 1) * TS + lane] = Rr;
                                     if (m > 0)
                                         H[(n * n + 2 * m) * TS + lane] = -Ri;  // the conjugate harmonic
                                 });
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int o = min(tid + 256 * j, MG * P2 - 1);
            const double *h = H + o % P2 * TS, *m = W + o / P2 * TC;
            double v = acc[j];
            for (int t = 0; t < nt; ++t)
                v += h[t] * m[t];
            acc[j] = v;
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int o = tid + 256 * j, bm = bm0 + o / P2;
        if (o < MG * P2 && bm < g.B)
            me[((lv.me_off + leaf) * g.B + bm) * PS + o % P2] = acc[j];
    }
    if constexpr (PS > P2)
        for (int i = tid; i < MG * (PS - P2); i += 256) {
            const int bm = bm0 + i / (PS - P2);
            if (bm < g.B)
                me[((lv.me_off + leaf) * g.B + bm) * PS + P2 + i % (PS - P2)] = 0.0;
        }
}

int64_t point_count(const Plan *p) { return p->lat_near ? p->d.n_points : p->M; }

PointArgs point_args(const Plan *p)
{
    return PointArgs{p->d_tpos, p->d_leaf_start, p->d_leaf_pend, p->d_tkey, p->d_user_leaves, p->n_user_leaves,
                     point_count(p)};
}

}  // namespace

#define GRAV_ORDERS(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

// Workgroups of the L2P that the GPU holds at once.
grav_status l2p_resident_workgroups(const Plan *p, int *workers)
{
    const void *fn = nullptr;
#define FN_CASE(X)                                                                                               \
    case X:                                                                                                      \
        fn = p->B == 1 ? reinterpret_cast<const void *>(&k_l2p_points<X, 1, 1>)                                  \
                       : reinterpret_cast<const void *>(&k_l2p_points<X, kPointModels, 1>);                      \
        break;
    switch (p->P) {
        GRAV_ORDERS(FN_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef FN_CASE
    int per_cu = 0, cus = 0;
    GRAV_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 256, 0));
    GRAV_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, p->device));
    *workers = std::max(per_cu * cus, 1);
    return GRAV_OK;
}

// Runs per workgroup: so many that those resident at once take all, up to 16;
// where runs are longer than a step, and so fill the lanes by themselves, so many
// that twice as many workgroups take all, up to 4; one of two steps or more with
// several models (p = 16, 4096 leaves of 20, 8 models: 161 us, with two 172).  One
// model, points per leaf, 9 unless given, us, with 1 / 2 / 4 / 8 / 16 runs:
//   p = 10 (1024 resident)  512 leaves  8.0 / 7.8 / 8.5 / 11.8 / 16.5
//     4096   24.5 / 15.7 / 10.9 / 13.0 / 16.7;  8192   43.8 / 26.2 / 16.9 / 15.6 / 18.5
//     16384 of 20   81.0 / 46.3 / 41.8 / 35.6 / 34.8;  32768   152 / 83 / 51 / 46 / 40
//     8192 of 80   69.6 / 53.8 / 51.6 / 52.2 / 75.1
//   p = 4 (2048)   4096   12.0 / 8.7 / 7.6 / 8.9 / 11.2;  of 160   23.0 / 21.3 / 27.0 / 46 / 85
//     8192 of 40   21.2 / 18.0 / 15.0 / 18.8 / 29.6
//   p = 16 (512)   2048   30.9 / 19.3 / 12.6 / 16.5 / 24.0;  8192   104 / 59 / 37 / 35 / 29
static int runs_per_workgroup(const Plan *p, int mg)
{
    const int64_t n = p->n_runs * ((p->B + mg - 1) / mg), pairs = point_count(p) * p->B;
    if (mg > 1 && pairs >= 128 * n)
        return 1;
    const bool full = pairs > 64 * n;
    const int64_t wgs = (int64_t)p->l2p_wgs * (full ? 2 : 1);
    return (int)std::clamp<int64_t>((n + wgs - 1) / wgs, 1, std::min(full ? 4 : kRunsPerWorkgroup, l2p_slots(p->P) / mg));
}

grav_status launch_l2p_points(const Plan *p, const DevGeom &g, double *out, hipStream_t s)
{
    if (p->n_runs == 0)
        return GRAV_OK;
    const int mg = std::min(p->B, kPointModels), lw = runs_per_workgroup(p, mg);
    const RunArgs rn{p->d_runs, p->n_runs, (p->n_runs + lw - 1) / lw, (p->B + mg - 1) / mg, lw, mg};
    if (rn.nblk * rn.groups > 0xffff0000ll)
        return GRAV_EUNSUPPORTED;  // (outputs of a quarter of a terabyte)
    const dim3 grid = block_grid(rn.nblk * rn.groups);
#define L2P_LAUNCH(P, MG, LW)                                                                                    \
    hipLaunchKernelGGL((k_l2p_points<P, MG, LW>), grid, dim3(256), 0, s, g, point_args(p), rn,                   \
                       (const uint32_t *)p->d_perm, (const double *)p->d_le, (const double *)p->d_near,          \
                       p->L >= 2 ? 1 : 0, out)
#define L2P_CASE(P)                                                                                              \
    case P:                                                                                                      \
        if (lw > 1)                                                                                              \
            L2P_LAUNCH(P, 1, kRunsPerWorkgroup);                                                                 \
        else if (p->B == 1)                                                                                      \
            L2P_LAUNCH(P, 1, 1);                                                                                 \
        else                                                                                                     \
            L2P_LAUNCH(P, kPointModels, 1);                                                                      \
        break;
    switch (p->P) {
        GRAV_ORDERS(L2P_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef L2P_CASE
#undef L2P_LAUNCH
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

grav_status launch_p2m_src(const Plan *p, const DevGeom &g, hipStream_t s)
{
    constexpr int kModels = 4;
    const int MG = p->B == 1 ? 1 : kModels;
    dim3 grid = block_grid(p->lev[p->L].n_src);
    grid.z = (unsigned)((p->B + MG - 1) / MG);
#define P2M_CASE(P)                                                                                              \
    case P:                                                                                                      \
        if (MG == 1)                                                                                             \
            hipLaunchKernelGGL((k_p2m_src<P, 1>), grid, dim3(256), 0, s, g, (const double *)p->d_spos,           \
                               (const double *)p->d_smass, (const int64_t *)p->d_sstart, p->n_spts, p->d_me);    \
        else                                                                                                     \
            hipLaunchKernelGGL((k_p2m_src<P, kModels>), grid, dim3(256), 0, s, g, (const double *)p->d_spos,     \
                               (const double *)p->d_smass, (const int64_t *)p->d_sstart, p->n_spts, p->d_me);    \
        break;
    switch (p->P) {
        GRAV_ORDERS(P2M_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef P2M_CASE
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

grav_status launch_t_l2p_points(const Plan *p, const DevGeom &g, hipStream_t s)
{
    const int MG = p->B == 1 ? 1 : kPointModels;
    if (p->n_user_leaves == 0)
        return GRAV_OK;
    dim3 grid = block_grid(p->n_user_leaves);
    grid.z = (unsigned)((p->B + MG - 1) / MG);
#define T_L2P_CASE(P)                                                                                            \
    case P:                                                                                                      \
        if (MG == 1)                                                                                             \
            hipLaunchKernelGGL((k_t_l2p_points<P, 1>), grid, dim3(256), 0, s, g, point_args(p),                  \
                               (const double *)p->d_near, p->d_le);                                              \
        else                                                                                                     \
            hipLaunchKernelGGL((k_t_l2p_points<P, kPointModels>), grid, dim3(256), 0, s, g, point_args(p),       \
                               (const double *)p->d_near, p->d_le);                                              \
        break;
    switch (p->P) {
        GRAV_ORDERS(T_L2P_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef T_L2P_CASE
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

}  // namespace grav
