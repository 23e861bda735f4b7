// M2L over sibling octets on MFMA (kept in its own file: its measured HBM
// traffic is tied to this source), for the forward pass and, on the
// transposed operators, for the adjoint.
#include <algorithm>
#include <type_traits>

#include "octet.hpp"

namespace grav {

// --------------------------------------------------------------------------
// A GEMM per parity chi with rows = coefficients of G_chi, columns = (octet,
// model) and contraction over (orbit, coefficient) (see octet.hpp).  A unit
// is 16 NC columns of one level and 8 / RS parities; a work item is a (unit,
// orbit) pair at which some column has a source box.  A workgroup runs its
// segments (a unit and some of its orbits, see the schedule in plan.hip) one
// after the other and writes each segment's sums to a slot of its own.
//
// Per chunk of coefficients the staging threads load the eight images of
// their (column, coefficients) from the natural-order expansions, form the
// eight H_chi with three butterfly stages and put them into LDS in B-operand
// order.  Loads run two chunks ahead (expansions) and D k steps
// ahead (operators), the LDS tile is double-buffered, and there is one
// barrier per chunk.  Each wave reads its own parity's B values and streams
// its own operator fragments, so no operator value is read twice in a
// workgroup, and all workgroups walk the orbits in the same order, so that
// the operators come from the L2.
//
// What bounds it: matrix issue.  Per octet it runs 26 x 8 operators instead
// of 8 x 189 (or 8 x 56 class-blocked ones of the reflection orbits of single
// targets, the form before this one).  Measured: 256^3 cells at leaf 4^3,
// p = 10 in FP32 6.82 -> 1.52 ms (its matrix cycles 1.0 ms), p = 16 in FP64
// 128.5 -> 17.0 ms (13.0 ms); 64^3 with two Gauss points 0.17 -> 0.05 ms and
// p = 12 in FP64 0.61 -> 0.14 ms.  A unit costs the same however few of its octets'
// children are targets or sources.  Sparse targets gain all the same, as the form
// before was bound by its loads there: 128^3 cells, p = 10, 4000 random points, about
// one target leaf per octet, 0.27 -> 0.16 ms, 200 points 0.17 -> 0.04.  Leaf grids of three boxes an axis or a
// row of boxes lose at 128 models or more: 12^3 cells have 936 products of a parity
// per model in octets and 386 of pairs, and 1024 of them, FP64 p = 14, take 1.85 ms in
// all where that form took 0.81.  The rest is building the tiles: without it
// the FP32 kernel takes 1.2 ms, without the loads behind it 1.1 ms.
// --------------------------------------------------------------------------
template <int P, typename T, int NC>
__global__ void __launch_bounds__(512)
k_m2l_octet(OctGeom g, OctTables t, const T *K, const T *in, T *part)
{
    using S = OctShape<P, T>;
    using vec4 = __attribute__((__vector_size__(4 * sizeof(T)))) T;
    constexpr int NX = S::NX, RS = S::RS, RBW = S::RBW, EA = S::EA, CK = S::CK, CC = S::CC, NQ = S::NQ, PS = S::PS,
                  D = S::D;
    constexpr int NCOL = 16 * NC;
    // V coefficients of one column per staging thread
    constexpr int V = NCOL * CC <= 512 ? 1 : NCOL * CC <= 1024 ? 2 : 4;
    constexpr int TPC = CC / V;  // staging threads per column
    static_assert(NCOL * TPC <= 512 && CC % V == 0 && CK % D == 0, "staging does not fit the workgroup");
    using vecv = __attribute__((__vector_size__(V * sizeof(T)))) T;
    __shared__ __align__(16) T hs[2][NX][NC][CK * S::US];
    // the class signs of a coefficient under the x, y and z reflections
    __shared__ __align__(16) T ssign[NQ * CC][4];
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xi = wave / RS, rpart = wave % RS;
    // staging: column scol, coefficients sk .. sk + V - 1 of each chunk; the
    // threads past the last column repeat the work of the first ones, so that
    // no load stands under a branch (the counts of loads in flight would be
    // waited for at its end)
    const int stid = tid % (NCOL * TPC);
    const int scol = stid / TPC, sk = (stid % TPC) * V;
    if (tid < NQ * CC) {
        const int c = sign_class(tid);
        for (int a = 0; a < 4; ++a)
            ssign[tid][a] = (c >> a & 1) ? (T)-1 : (T)1;
    }
    __syncthreads();
    for (int sg = t.wgseg[blockIdx.x]; sg < t.wgseg[blockIdx.x + 1]; ++sg) {
        const int unit = __builtin_amdgcn_readfirstlane(t.segs[4 * sg]);
        const uint32_t orbits = (uint32_t)__builtin_amdgcn_readfirstlane(t.segs[4 * sg + 1]);  // bit o - 1
        const OctGroup grp = t.groups[unit / RS];
        const int xh = unit % RS;  // RS = 2: which half of the parities
        const OctLev lv = g.lev[grp.level];
        // the staging thread's column
        const bool cval = scol < grp.ncol;
        int px = 0, py = 0, pz = 0, bm = 0;
        if (cval) {
            const int64_t col = grp.col0 + scol;
            const uint32_t key = t.key[grp.oct0 + col / g.B];
            bm = (int)(col % g.B);
            px = (int)compact3(key);
            py = (int)compact3(key >> 1);
            pz = (int)compact3(key >> 2);
        }
        vec4 acc[NC][RBW];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int rb = 0; rb < RBW; ++rb)
                acc[c][rb] = vec4{0, 0, 0, 0};
        // the orbit being loaded: input columns of its images (a missing box
        // reads the level's first row and counts as zero), which exist
        uint32_t row[8], hm = 0;
        auto look = [&](int o) {
            const int ox = orbit_axis(o, 0), oy = orbit_axis(o, 1), oz = orbit_axis(o, 2);
            hm = 0;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int32_t j = octet_place(lv, orbit_coord(px, ox, r & 1), orbit_coord(py, oy, r & 2),
                                              orbit_coord(pz, oz, r & 4));
                const bool have = cval && j >= 0;
                hm |= have ? 1u << r : 0u;
                row[r] = (uint32_t)((lv.row0 + (have ? j : 0)) * g.B + bm);
            }
        };
        T m[8][V];
        auto load = [&](int q) {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const T *src = in + (int64_t)row[r] * PS + CC * q + sk;
                if constexpr (V == 1) {
                    m[r][0] = *src;
                } else {
                    const vecv v = *reinterpret_cast<const vecv *>(src);
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        m[r][e] = v[e];
                }
            }
        };
        // butterflies over the images, the signs of the coefficient's class
        // folded into each stage, and one store of V coefficients per parity
        T w[V][3];
        auto signs = [&](int q) {
#pragma unroll
            for (int e = 0; e < V; ++e)
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    w[e][a] = ssign[CC * q + sk + e][a];
        };
        auto put = [&](int buf) {
            if (__ballot(hm != 0xffu) != 0) {
#pragma unroll
                for (int r = 0; r < 8; ++r)
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        m[r][e] = (hm >> r) & 1u ? m[r][e] : (T)0;
            }
#pragma unroll
            for (int e = 0; e < V; ++e) {
                if constexpr (RS == 2) {
                    const T wz = xh ? -w[e][2] : w[e][2];
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        m[r][e] += wz * m[r + 4][e];
                }
#pragma unroll
                for (int a = 0; 1 << a < NX; ++a)
#pragma unroll
                    for (int r = 0; r < NX; ++r)
                        if ((r >> a & 1) == 0) {
                            const T x = m[r][e], y = m[r | 1 << a][e];
                            m[r][e] = x + w[e][a] * y;
                            m[r | 1 << a][e] = x - w[e][a] * y;
                        }
            }
            T *dst = &hs[buf][0][scol >> 4][S::at(sk / 4, sk % 4, scol & 15)];
#pragma unroll
            for (int j = 0; j < NX; ++j)
#pragma unroll
                for (int e = 0; e < V; e += 2) {
                    T *d = dst + j * NC * CK * S::US + (S::at(0, e, 0) - S::at(0, 0, 0));
                    if constexpr (V > 1 && sizeof(T) == 4)
                        *reinterpret_cast<float2 *>(d) = make_float2(m[j][e], m[j][e + 1]);
                    else
                        *d = m[j][e];
                    if constexpr (V > 1 && sizeof(T) == 8)
                        dst[j * NC * CK * S::US + S::at(0, e + 1, 0)] = m[j][e + 1];
                }
        };
        auto ops = [&](int o) { return K + (((int64_t)(o - 1) * 8 + xh * NX + xi) * RS + rpart) * S::KOP; };
        // steps: (orbit, chunk) pairs in order; each call issues the next
        // step's loads (past the last step, the last orbit's again)
        const int NS = __builtin_popcount(orbits) * NQ;
        uint32_t lm = orbits;  // orbits not yet loaded, and the next chunk
        int lq = 0;
        look(__builtin_ctz(lm) + 1);
        auto advance = [&]() {
            load(lq);
            if (++lq == NQ) {
                lq = 0;
                lm &= lm - 1;
            }
        };
        // the masks of the step in `m`, and the next step's orbit: after put
        auto next = [&]() {
            if (lq == 0 && lm)
                look(__builtin_ctz(lm) + 1);
        };
        advance();
        uint32_t cm = orbits;  // orbits from the current one on
        const T *kp = ops(__builtin_ctz(cm) + 1);
        T an[D][EA];
#pragma unroll
        for (int d = 0; d < D; ++d)
            load_set<T, EA>(kp + d * EA * 64, lane, an[d]);
        signs(0);
        put(0);
        next();
        advance();
        __syncthreads();
        constexpr int PP = CK / 2;  // the k step that also builds the next tile
        int q = 0;
        for (int s = 0; s < NS; ++s) {
            const int buf = s & 1;
            const bool more = s + 1 < NS;
            const int qn = q + 1 < NQ ? q + 1 : 0;
            // operators of the next step (the last step reads its own again)
            if (qn == 0 && more)
                cm &= cm - 1;
            const T *kpn = qn > 0 ? kp + CK * EA * 64 : more ? ops(__builtin_ctz(cm) + 1) : kp;
            const T *bs = &hs[buf][xi][0][S::at(0, kr, lane & 15)];
            T b[2][NC];
#pragma unroll
            for (int c = 0; c < NC; ++c)
                b[0][c] = bs[c * CK * S::US];
#pragma unroll
            for (int u = 0; u < CK; ++u) {
                if (u == PP)
                    signs(qn);
                if (u + 1 < CK) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        b[(u + 1) & 1][c] = bs[c * CK * S::US + (u + 1) * S::US];
                }
#pragma unroll
                for (int rb = 0; rb < RBW; ++rb) {
                    if (RS * RBW > OctShape<P, T>::RB && rb == RBW - 1 && rpart == RS - 1)
                        continue;  // the last part is one row block short
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const T av = an[u % D][rb], bv = b[u & 1][c];
                        if constexpr (sizeof(T) == 8)
                            acc[c][rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[c][rb], 0, 0, 0);
                        else if (OctShape<P, T>::TAIL4 && rb == RBW - 1)
                            acc[c][rb] = __builtin_amdgcn_mfma_f32_4x4x1f32(av, bv, acc[c][rb], 0, 0, 0);
                        else
                            acc[c][rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[c][rb], 0, 0, 0);
                    }
                }
                // the set just used takes the k step D ahead
                load_set<T, EA>(u + D < CK ? kp + (u + D) * EA * 64 : kpn + (u + D - CK) * EA * 64, lane, an[u % D]);
                // the next step's tile, then the loads of the one after it,
                // which have a whole step to arrive
                if (u == PP) {
                    put(buf ^ 1);
                    next();
                    advance();
                }
            }
            __syncthreads();
            kp = kpn;
            q = qn;
        }
        if constexpr (S::TAIL4) {
            // the 4x4 tail: lane l holds rows 16 (RB - 1) + r of column l % 16
            // summed over its sub-row's coefficients; add the four sub-rows in
            // a fixed order into lanes 0..15, where the 16x16x4 layout puts
            // those rows (the other lanes' rows are padding: zero)
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    T v = acc[c][RBW - 1][r];
                    v += __shfl_xor(v, 16);
                    v += __shfl_xor(v, 32);
                    acc[c][RBW - 1][r] = lane < 16 ? v : (T)0;
                }
        }
        // slot [parity][column][PS]; a lane holds column lane % 16 and rows
        // 4 (lane / 16) + r (FP32) or lane / 16 + 4 r (FP64) of each block
        T *dst = part + (((int64_t)t.segs[4 * sg + 2] * NX + xi) * NCOL + (lane & 15)) * PS + 16 * rpart * RBW;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int rb = 0; rb < RBW; ++rb) {
                if (RS * RBW > S::RB && rb == RBW - 1 && rpart == RS - 1)
                    continue;
                T *d = dst + (int64_t)c * 16 * PS + 16 * rb;
                if constexpr (sizeof(T) == 4) {
                    *reinterpret_cast<vec4 *>(d + 4 * kr) = acc[c][rb];
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        d[kr + 4 * r] = acc[c][rb][r];
                }
            }
    }
}

#define GRAV_ORDERS(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

template <typename T>
grav_status launch_m2l(const Plan *p, const OctPlan &o, hipStream_t s, const OctGeom &g, const T *in)
{
    if (o.wgs == 0)
        return GRAV_OK;
    const T *K = reinterpret_cast<const T *>(o.d_ops);
    T *part = reinterpret_cast<T *>(p->d_part);
    const OctTables t = o.tables();
    const dim3 grid((unsigned)o.wgs), blk(512);
#define M2L_CASE(P)                                                                                              \
    case P:                                                                                                      \
        if (o.nc == 1)                                                                                           \
            hipLaunchKernelGGL((k_m2l_octet<P, T, 1>), grid, blk, 0, s, g, t, K, in, part);                 \
        else if (o.nc == OctShape<P, T>::NCW)                                                                    \
            hipLaunchKernelGGL((k_m2l_octet<P, T, OctShape<P, T>::NCW>), grid, blk, 0, s, g, t, K, in, part); \
        else                                                                                                     \
            return GRAV_EUNSUPPORTED;                                                                            \
        break;
    switch (p->P) {
        GRAV_ORDERS(M2L_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef M2L_CASE
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

template grav_status launch_m2l<double>(const Plan *, const OctPlan &, hipStream_t, const OctGeom &, const double *);
template grav_status launch_m2l<float>(const Plan *, const OctPlan &, hipStream_t, const OctGeom &, const float *);

OctGeom octet_geom(const Plan *p, bool transposed)
{
    OctGeom g{};
    g.B = p->B;
    for (int l = 2; l <= p->L; ++l) {
        const LevelInfo &lv = p->lev[l];
        for (int a = 0; a < 3; ++a) {
            g.lev[l].s0[a] = transposed ? lv.gs0[a] : lv.s0[a];
            g.lev[l].ns[a] = transposed ? lv.gns[a] : lv.ns[a];
        }
        g.lev[l].row0 = transposed ? lv.g_off : lv.me_off;
    }
    return g;
}

// Compile-time shape of the plan's M2L kernel for the host code that lays
// out its operators and schedule.
OctInfo octet_info(int P, bool f64)
{
    OctInfo o{};
#define INFO(T, X)                                                                                                  \
    o = OctInfo{OctShape<X, T>::RS, OctShape<X, T>::RBW, OctShape<X, T>::EA,  OctShape<X, T>::CK, \
                OctShape<X, T>::KS, OctShape<X, T>::NCW, OctShape<X, T>::TAIL4}
#define INFO_CASE(X)         \
    case X:                  \
        if (f64)             \
            INFO(double, X); \
        else                 \
            INFO(float, X);  \
        break;
    switch (P) {
        GRAV_ORDERS(INFO_CASE)
    }
#undef INFO_CASE
#undef INFO
    return o;
}

// Workgroups of the plan's M2L kernel (nc column blocks per wave) that the
// device holds at once: the size of the schedule, so that every workgroup
// is resident from the start.
grav_status m2l_resident_workgroups(const Plan *p, int nc, int *workers)
{
    const bool f64 = p->d.precision == GRAV_FP64;
    const void *fn = nullptr;
#define FN(T, X)                                                                  \
    nc == 1 ? reinterpret_cast<const void *>(&k_m2l_octet<X, T, 1>)               \
            : reinterpret_cast<const void *>(&k_m2l_octet<X, T, OctShape<X, T>::NCW>)
#define FN_CASE(X)                              \
    case X:                                     \
        fn = f64 ? (FN(double, X)) : (FN(float, X)); \
        break;
    switch (p->P) {
        GRAV_ORDERS(FN_CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef FN_CASE
#undef FN
    int per_cu = 0, n_cu = 0;
    GRAV_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 512, 0));
    GRAV_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, p->device));
    *workers = std::max(1, per_cu) * std::max(1, n_cu);
    return GRAV_OK;
}

}  // namespace grav
