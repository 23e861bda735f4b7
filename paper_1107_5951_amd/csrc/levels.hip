// Translations between a level's sibling octets and their parents by
// reflection parity (octet.hpp): M2M and the transposed L2L upward, L2L and the
// transposed M2M downward, the latter two together with the sums of the M2L's
// segment slots.
//
// The operator of child r is S_r T S_r with T the (+,+,+) child's, so with
// H_chi[k] = sum_r (-1)^(chi.r) (-1)^(class(k).r) X_r[k] over the children,
//   up:    Y[i] = sum_k T[i][k] H_{class(i)}[k],
//   down:  X_r[i] = (-1)^(class(i).r) sum_chi (-1)^(chi.r) G_chi[i],
//          G_chi[i] = sum_{k of class chi} T[i][k] Y[k] (+ the M2L's G_chi[i]):
// one operator's products per parent instead of eight.
//
// What bounds them: on wide levels memory (the children's expansions and the
// M2L's slots), on narrow ones the latency of a workgroup's chain of loads.
// 256^3 cells at leaf 4^3, p = 10 (0.24 GB of leaf expansions): upward 0.25 ->
// 0.12 ms (leaf level 0.078, 3.6 TB/s), downward with the slot sums 0.37 ->
// 0.23 ms (leaf level 0.16, 2.4 TB/s); p = 16 FP64: 1.13 -> 0.29 ms and 1.36 ->
// 0.52 ms.
#include <algorithm>

#include "octet.hpp"

// Up: one workgroup of 32 columns per CU.  All levels, wide against short, us:
// p = 10, 2048 columns 18.3 / 11.6, 4096 19.7 / 13.7, 8192 24.4 / 24.2, 16384 43.1 /
// 46.3, 32768 81.8 / 91.1; p = 16, 4096 51.6 / 37.5, 8192 62.9 / 78.6, 16384 108 / 150;
// p = 4, where both are short, 4096 6.7 / 7.7, 16384 9.4 / 15.9.
#ifndef GRAV_UP_WIDE_COLS
#define GRAV_UP_WIDE_COLS 8192
#endif
// Down: 64 workgroups.  4096 columns: p = 10 26.9 us wide, 49 us narrow, p = 16
// 61 and 179 us; 512 columns: 27.4 and 9.4 us, 80 and 13 us.
#ifndef GRAV_DOWN_WIDE_COLS
#define GRAV_DOWN_WIDE_COLS 2048
#endif

namespace grav {

namespace {

struct LevelArgs {
    const int32_t *child, *parent;  // of the level's first octet
    int64_t ncols;                  // octets x models
    int B;
};

// Up.  A workgroup takes 32 columns (octet, model), wave chi the rows of class
// chi; the children's expansions pass through LDS chunk by chunk as parity sums
// (the staging of the M2L), the parents leave through LDS as whole rows.
template <int P>
__global__ void __launch_bounds__(512)
k_octet_up(LevelArgs lv, const double *A, const int32_t *coef, const double *x, double *out, float *out32)
{
    using S = OctShape<P, double>;
    using C = ClassShape<P>;
    using vec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int CK = S::CK, CC = S::CC, NQ = S::NQ, PS = S::PS, US = S::US, NC = 2, NCOL = 16 * NC;
    constexpr int V = NCOL * CC <= 512 ? 1 : 2, TPC = CC / V, OP = PS + 1;
    constexpr int kTile = 8 * NC * CK * US, kOut = NCOL * OP;
    __shared__ __align__(16) double sm[kTile > kOut ? kTile : kOut];
    __shared__ double ssign[NQ * CC][3];
    __shared__ int32_t srow[NCOL];
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int chi = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < NQ * CC) {
        const int c = sign_class(tid);
        for (int a = 0; a < 3; ++a)
            ssign[tid][a] = (c >> a & 1) ? -1.0 : 1.0;
    }
    const int64_t col0 = block_id() * NCOL;
    if (col0 >= lv.ncols)
        return;
    if (tid < NCOL) {
        const int64_t col = col0 + tid;
        srow[tid] = col < lv.ncols ? lv.parent[col / lv.B] : -1;
    }
    // staging column and coefficients (threads past the last column repeat)
    const int stid = tid % (NCOL * TPC);
    const int scol = stid / TPC, sk = (stid % TPC) * V;
    const double *src[8];
    uint32_t hm = 0;
    {
        const int64_t col = min(col0 + scol, lv.ncols - 1);
        const int32_t *ch = lv.child + col / lv.B * 8;
        const int64_t bm = col % lv.B;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int32_t row = ch[7 ^ r];
            hm |= row >= 0 ? 1u << r : 0u;
            src[r] = x + ((row >= 0 ? row : 0) * (int64_t)lv.B + bm) * PS + sk;
        }
    }
    double m[8][V];
    auto load = [&](int q) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if constexpr (V == 2) {
                const double2 v = *reinterpret_cast<const double2 *>(src[r] + CC * q);
                m[r][0] = v.x;
                m[r][1] = v.y;
            } else {
                m[r][0] = src[r][CC * q];
            }
        }
    };
    vec4 acc[NC][C::RBC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int rb = 0; rb < C::RBC; ++rb)
            acc[c][rb] = vec4{0, 0, 0, 0};
    load(0);
    __syncthreads();
    const double *Ax = A + (int64_t)chi * S::KS * C::RBC * 64 + lane;
    for (int q = 0; q < NQ; ++q) {
        double a[CK][C::RBC];
#pragma unroll
        for (int u = 0; u < CK; ++u)
#pragma unroll
            for (int rb = 0; rb < C::RBC; ++rb)
                a[u][rb] = Ax[((q * CK + u) * C::RBC + rb) * 64];
        double h[V][8];
#pragma unroll
        for (int e = 0; e < V; ++e) {
#pragma unroll
            for (int r = 0; r < 8; ++r)
                h[e][r] = (hm >> r) & 1u ? m[r][e] : 0.0;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const double w = ssign[CC * q + sk + e][ax];
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    if ((r >> ax & 1) == 0) {
                        const double xx = h[e][r], y = h[e][r | 1 << ax];
                        h[e][r] = xx + w * y;
                        h[e][r | 1 << ax] = xx - w * y;
                    }
            }
        }
        if (q > 0)
            __syncthreads();  // the previous chunk's products are done
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                sm[(j * NC + (scol >> 4)) * (CK * US) + S::at((sk + e) / 4, (sk + e) % 4, scol & 15)] = h[e][j];
        load(q + 1 < NQ ? q + 1 : q);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < CK; ++u) {
            double b[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c)
                b[c] = sm[(chi * NC + c) * (CK * US) + S::at(u, kr, lane & 15)];
#pragma unroll
            for (int rb = 0; rb < C::RBC; ++rb)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    acc[c][rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][rb], b[c], acc[c][rb], 0, 0, 0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < C::RBC; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = coef[chi * 16 * C::RBC + 16 * rb + kr + 4 * r];
#pragma unroll
            for (int c = 0; c < NC; ++c)
                sm[(c * 16 + (lane & 15)) * OP + (k >= 0 ? k : PS)] = acc[c][rb][r];  // (PS: a spare place)
        }
    if constexpr (PS > P * P)
        for (int i = tid; i < NCOL * (PS - P * P); i += 512)
            sm[i / (PS - P * P) * OP + P * P + i % (PS - P * P)] = 0.0;
    __syncthreads();
    for (int i = tid; i < NCOL * PS; i += 512) {
        const int c = i / PS, k = i % PS;
        if (srow[c] < 0)
            continue;
        const int64_t o = ((int64_t)srow[c] * lv.B + (col0 + c) % lv.B) * PS + k;
        const double v = sm[c * OP + k];
        out[o] = v;
        if (out32)
            out32[o] = (float)v;
    }
}

// Up, on the levels with few columns: 16 columns per workgroup and K in chunks
// of 128 coefficients, so that up to p = 11 one pass of loads stands for the
// dozen dependent ones of k_octet_up's chunks.
template <int P>
__global__ void __launch_bounds__(512)
k_octet_up_short(LevelArgs lv, const double *A, const int32_t *coef, const double *x, double *out, float *out32)
{
    using S = OctShape<P, double>;
    using C = ClassShape<P>;
    using vec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int PS = S::PS, KS = S::KS, CS = 32, NCH = (KS + CS - 1) / CS, OP = PS + 1;
    constexpr int US = 65;  // doubles per k step and class: the staging stores of 32 lanes, one step each, spread
    constexpr int kTile = 8 * (KS < CS ? KS : CS) * US, kOut = 16 * OP;
    __shared__ double sm[kTile > kOut ? kTile : kOut];
    __shared__ int32_t srow[16];
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int chi = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t col0 = (int64_t)blockIdx.x * 16;
    if (tid < 16)
        srow[tid] = lv.parent[min(col0 + tid, lv.ncols - 1) / lv.B];
    const int scol = tid >> 5, su = tid & 31;  // staging column and k step of the chunk
    const int64_t col = min(col0 + scol, lv.ncols - 1);
    const int32_t *ch = lv.child + col / lv.B * 8;
    int32_t row[8];
#pragma unroll
    for (int r = 0; r < 8; ++r)
        row[r] = ch[7 ^ r];
    const double *Ax = A + (int64_t)chi * KS * C::RBC * 64 + lane;
    vec4 acc[C::RBC];
#pragma unroll
    for (int rb = 0; rb < C::RBC; ++rb)
        acc[rb] = vec4{0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
        constexpr int last = KS - 1;
        const int k0 = 4 * min(CS * q + su, last);
        double2 m[8][2];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const double2 *s = reinterpret_cast<const double2 *>(x + ((row[r] >= 0 ? row[r] : 0) * (int64_t)lv.B + col % lv.B) * PS + k0);
            m[r][0] = s[0];
            m[r][1] = s[1];
        }
        if (q > 0)
            __syncthreads();  // the previous chunk's products are done
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = sign_class(k0 + e);
            double h[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const double v = e & 1 ? m[r][e >> 1].y : m[r][e >> 1].x;
                h[r] = row[r] >= 0 ? v : 0.0;
            }
#pragma unroll
            for (int ax = 0; ax < 3; ++ax)
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    if ((r >> ax & 1) == 0) {
                        const double xx = h[r], y = (c >> ax & 1) ? -h[r | 1 << ax] : h[r | 1 << ax];
                        h[r] = xx + y;
                        h[r | 1 << ax] = xx - y;
                    }
            if (CS * q + su < KS)
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    sm[j * (kTile / 8) + su * US + 16 * e + scol] = h[j];
        }
        __syncthreads();
#pragma unroll 7
        for (int u = 0; u < (KS - CS * q < CS ? KS - CS * q : CS); ++u) {
            const double b = sm[chi * (kTile / 8) + u * US + 16 * kr + (lane & 15)];
#pragma unroll
            for (int rb = 0; rb < C::RBC; ++rb)
                acc[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(Ax[((CS * q + u) * C::RBC + rb) * 64], b, acc[rb], 0, 0, 0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < C::RBC; ++rb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = coef[chi * 16 * C::RBC + 16 * rb + kr + 4 * r];
            sm[(lane & 15) * OP + (k >= 0 ? k : PS)] = acc[rb][r];  // (PS: a spare place)
        }
    if constexpr (PS > P * P)
        for (int i = tid; i < 16 * (PS - P * P); i += 512)
            sm[i / (PS - P * P) * OP + P * P + i % (PS - P * P)] = 0.0;
    __syncthreads();
    for (int i = tid; i < 16 * PS; i += 512) {
        const int c = i / PS, k = i % PS;
        if (col0 + c >= lv.ncols)
            continue;
        const int64_t o = ((int64_t)srow[c] * lv.B + (col0 + c) % lv.B) * PS + k;
        const double v = sm[c * OP + k];
        out[o] = v;
        if (out32)
            out32[o] = (float)v;
    }
}

// Down.  A workgroup takes 16 NC columns, wave chi the products of class chi;
// row block by row block the eight parities meet in LDS, the slots are added,
// and the children's rows are stored.  NC = 2: all row blocks, on levels that
// fill the chip.  NC = 1, on the others: one row block (blockIdx.y), the slots
// shared by two halves of the workgroup and loaded several at a time, since
// small plans cut a unit into up to 26.
template <int P, typename T, int NC>
__global__ void __launch_bounds__(512)
k_octet_down(LevelArgs lv, SlotArgs<T> sl, const double *A, const int32_t *coef, const double *x, double *out)
{
    using S = OctShape<P, double>;
    using C = ClassShape<P>;
    using vec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int PS = S::PS, RB = S::RB, NCOL = 16 * NC, XP = PS + 1, GP = 17, KC = C::KC;
    constexpr int RS = OctShape<P, T>::RS, NX = 8 / RS, H = 2 / NC;
    constexpr int U = NC == 2 ? 1 : 32 / (int)sizeof(T);  // slots in flight per thread
    constexpr int kG = 8 * NCOL * GP, kX = NCOL * XP;
    // products of even row blocks (or of the one); parents' rows, then products
    // of odd row blocks
    __shared__ double g0[kG], g1[kX > kG ? kX : kG];
    __shared__ double hs[H == 2 ? 2 * 8 * 256 : 1];
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int chi = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (blockIdx.y: NC = 2 the grid's rows, NC = 1 the row block)
    const int64_t col0 = (NC == 2 ? block_id() : (int64_t)blockIdx.x) * NCOL;
    if (NC == 2 && col0 >= lv.ncols)
        return;
    // this thread's output: column, row of each block (and half of the slots)
    const int half = tid / (NCOL * 16), oc = tid / 16 % NCOL, orow = tid & 15;
    const int64_t col = col0 + oc;
    const bool ok = col < lv.ncols;
    const int64_t cs = ok ? col : lv.ncols - 1;
    const int64_t gi = sl.g0 + cs / sl.ncol, xs = (int64_t)sl.ncol * PS;
    int jb[RS], je[RS];
#pragma unroll
    for (int u = 0; u < RS; ++u) {
        jb[u] = sl.uslot[gi * RS + u];
        je[u] = sl.uslot[gi * RS + u + 1];
    }
    const T *pc = sl.part + cs % sl.ncol * PS + orow;
    // the parents' rows
    if (x != nullptr) {
        constexpr int NI = (NCOL * PS + 511) / 512;
        double y[NI];
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int i = min(tid + 512 * n, NCOL * PS - 1);
            const int64_t c = min(col0 + i / PS, lv.ncols - 1);
            y[n] = x[((int64_t)lv.parent[c / lv.B] * lv.B + c % lv.B) * PS + i % PS];
        }
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int i = min(tid + 512 * n, NCOL * PS - 1);
            g1[i / PS * XP + i % PS] = y[n];
        }
        __syncthreads();
    }
    double b[KC][NC];
    if (x != nullptr) {
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            const int k = coef[chi * 16 * C::RBC + 4 * q + kr];
#pragma unroll
            for (int c = 0; c < NC; ++c)
                b[q][c] = k >= 0 ? g1[(c * 16 + (lane & 15)) * XP + k] : 0.0;
        }
    }
    const int bm = (int)(cs % lv.B);
    int32_t ch[8];
#pragma unroll
    for (int r = 0; r < 8; ++r)
        ch[r] = ok ? lv.child[cs / lv.B * 8 + (7 ^ r)] : -1;
    const double *Ax = A + (int64_t)chi * KC * RB * 64 + lane;
    const int rb0 = NC == 2 ? 0 : (int)blockIdx.y, rb1 = NC == 2 ? RB : rb0 + 1;
    T w[8];  // NC == 2: the first slot's values of the next row block
    auto first = [&](int rb) {
#pragma unroll
        for (int y = 0; y < 8; ++y)
            w[y] = pc[((int64_t)jb[y / NX] * NX + y % NX) * xs + 16 * rb];
    };
    bool any[RS];
#pragma unroll
    for (int u = 0; u < RS; ++u) {
        any[u] = je[u] > jb[u];
        if (!any[u])
            jb[u] = je[u] = 0;
    }
    double a[KC];
    auto fragments = [&](int rb) {
#pragma unroll
        for (int q = 0; q < KC; ++q)
            a[q] = Ax[(q * RB + rb) * 64];
    };
    fragments(rb0);
    if constexpr (NC == 2)
        first(0);
    for (int rb = rb0; rb < rb1; ++rb) {
        const int i = 16 * rb + orow;
        // the slots' sums of this thread's element, parity by parity
        double v[8];
#pragma unroll
        for (int y = 0; y < 8; ++y)
            v[y] = NC == 2 && any[y / NX] ? (double)w[y] : 0.0;
        if constexpr (NC == 2) {
            first(min(rb + 1, RB - 1));
#pragma unroll
            for (int u = 0; u < RS; ++u)
                for (int j = jb[u] + 1; j < je[u]; ++j)
#pragma unroll
                    for (int y = 0; y < NX; ++y)
                        v[u * NX + y] += (double)pc[((int64_t)j * NX + y) * xs + 16 * rb];
        } else {
#pragma unroll
            for (int u = 0; u < RS; ++u)
                for (int j = jb[u] + half; j < je[u]; j += H * U) {
                    T p[U][NX];
#pragma unroll
                    for (int n = 0; n < U; ++n)
#pragma unroll
                        for (int y = 0; y < NX; ++y)
                            p[n][y] = pc[((int64_t)min(j + H * n, je[u] - 1) * NX + y) * xs + 16 * rb];
#pragma unroll
                    for (int n = 0; n < U; ++n)
#pragma unroll
                        for (int y = 0; y < NX; ++y)
                            v[u * NX + y] += j + H * n < je[u] ? (double)p[n][y] : 0.0;
                }
        }
        double *gs = (rb - rb0) & 1 ? g1 : g0;
        if (x != nullptr) {
            vec4 acc[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c)
                acc[c] = vec4{0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < KC; ++q)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q][c], acc[c], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    gs[(chi * NCOL + c * 16 + (lane & 15)) * GP + kr + 4 * r] = acc[c][r];
            // ahead of this block's stores: a wait for the next fragments is
            // then none for the stores
            if constexpr (NC == 2)
                fragments(min(rb + 1, RB - 1));
        }
        if constexpr (H == 2)
#pragma unroll
            for (int y = 0; y < 8; ++y)
                hs[(half * 8 + y) * 256 + oc * 16 + orow] = v[y];
        __syncthreads();
        if constexpr (H == 2)
#pragma unroll
            for (int y = 0; y < 8; ++y)
                v[y] = hs[y * 256 + oc * 16 + orow] + hs[(8 + y) * 256 + oc * 16 + orow];
        if (x != nullptr)
#pragma unroll
            for (int y = 0; y < 8; ++y)
                v[y] += gs[(y * NCOL + oc) * GP + orow];
#pragma unroll
        for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
            for (int r = 0; r < 8; ++r)
                if ((r & bit) == 0) {
                    const double xx = v[r], y = v[r | bit];
                    v[r] = xx + y;
                    v[r | bit] = xx - y;
                }
        const int s = sign_class(i);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (ch[r] >= 0 && (H == 1 || r / 4 == half))
                out[((int64_t)ch[r] * lv.B + bm) * PS + i] = odd_parity(s & r) ? -v[r] : v[r];
    }
}

// Levels with more columns than these run the kernels of 32 columns.
constexpr int64_t kUpWideCols = GRAV_UP_WIDE_COLS, kDownWideCols = GRAV_DOWN_WIDE_COLS;

LevelArgs level_args(const Plan *p, const OctPlan &o, int l)
{
    return LevelArgs{o.d_child + 8 * o.first[l], o.d_parent + o.first[l], (o.first[l + 1] - o.first[l]) * p->B, p->B};
}

}  // namespace

#define GRAV_ORDERS(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

// The expansions of the parents of level l's octets from their children's.
grav_status launch_octet_up(const Plan *p, const OctPlan &o, int l, hipStream_t s, const double *A, double *x,
                            float *out32)
{
    const LevelArgs lv = level_args(p, o, l);
    if (lv.ncols == 0)
        return GRAV_OK;
    const bool wide = lv.ncols > kUpWideCols;
    const dim3 grid = block_grid(wide ? (lv.ncols + 31) / 32 : (lv.ncols + 15) / 16);
#define UP_CASE(P)                                                                                            \
    case P:                                                                                                   \
        if (wide)                                                                                             \
            hipLaunchKernelGGL((k_octet_up<P>), grid, dim3(512), 0, s, lv, A,                                 \
                               (const int32_t *)p->d_class_coef, (const double *)x, x, out32);                \
        else                                                                                                  \
            hipLaunchKernelGGL((k_octet_up_short<P>), grid, dim3(512), 0, s, lv, A,                           \
                               (const int32_t *)p->d_class_coef, (const double *)x, x, out32);                \
        break;
    switch (p->P) {
        GRAV_ORDERS(UP_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef UP_CASE
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

// The expansions of level l's octets: the M2L's slot sums plus, from level 3
// on, the parents' translated.
template <typename T>
static grav_status octet_down(const Plan *p, const OctPlan &o, int l, hipStream_t s, const double *A, double *x)
{
    const LevelArgs lv = level_args(p, o, l);
    if (lv.ncols == 0)
        return GRAV_OK;
    const SlotArgs<T> sl{reinterpret_cast<const T *>(p->d_part), o.d_uslot, o.gfirst[l], 16 * o.nc};
    const double *in = l > 2 ? x : nullptr;
    const bool wide = lv.ncols > kDownWideCols;
    const dim3 grid = wide ? block_grid((lv.ncols + 31) / 32)
                           : dim3((unsigned)((lv.ncols + 15) / 16), (unsigned)(p->PS / 16));
#define DOWN_CASE(P)                                                                                          \
    case P:                                                                                                   \
        if (wide)                                                                                             \
            hipLaunchKernelGGL((k_octet_down<P, T, 2>), grid, dim3(512), 0, s, lv, sl, A,                     \
                               (const int32_t *)p->d_class_coef, in, x);                                      \
        else                                                                                                  \
            hipLaunchKernelGGL((k_octet_down<P, T, 1>), grid, dim3(512), 0, s, lv, sl, A,                     \
                               (const int32_t *)p->d_class_coef, in, x);                                      \
        break;
    switch (p->P) {
        GRAV_ORDERS(DOWN_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef DOWN_CASE
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

grav_status launch_octet_down(const Plan *p, const OctPlan &o, int l, hipStream_t s, const double *A, double *x)
{
    return p->d.precision == GRAV_FP64 ? octet_down<double>(p, o, l, s, A, x) : octet_down<float>(p, o, l, s, A, x);
}

}  // namespace grav
