// Sibling octets: the eight children of one parent box, the unit of work of
// the M2L and of the translations between levels.
//
// Reflecting the axes about the parent's centre permutes its children, and
// the source boxes of their interaction lists (the children of the parent's
// 27 neighbours, a 6 x 6 x 6 block of child boxes) among themselves.  A
// reflection r acts on an expansion by a sign per coefficient, (-1)^(s(k).r)
// with s(k) the sign class of coefficient k, and every translation operator
// commutes with it: K_r(d) = S_r K_d S_r.  So the operator from the block to
// the octet is block-diagonal in the eight parities chi of the group: with
// the Walsh-Hadamard sums over the images r of a box o of the positive octant
//   H_chi[o][k] = sum_r (-1)^(chi.r) (-1)^(s(k).r) M_{r o}[k],
// the octet's expansions are
//   L_r[i] = (-1)^(s(i).r) sum_chi (-1)^(chi.r) G_chi[i],
//   G_chi  = sum_o F_{chi,o} H_chi[o],
//   F_{chi,o}[i][k] = 1/8 sum_r (-1)^(chi.r) (-1)^(s(k).r) K_{r o - t}[i][k],
// t the (+,+,+) child and the sum over the r whose box is in t's list.  The
// positive octant holds 27 boxes, of which (1,1,1) is the octet itself: 26
// operators per parity serve eight targets, where the lists hold 189 offsets
// per target.  Reflection index r: bit a set = the negative side of axis a.
#pragma once

#include "eval_common.hpp"

namespace grav {

constexpr int kOrbits = 26;  // boxes (x, y, z) in {1, 2, 3}^3 without (1, 1, 1)

// Sign class of real coefficient c under the z, y and x reflections (bits 2,
// 1, 0): degree n block of 2n+1 values, the real part of order 0, then real
// and imaginary parts of orders 1..n; z -> -z gives (-1)^(n+m), y -> -y -1 on
// imaginary parts, x -> -x (-1)^m on real and -(-1)^m on imaginary parts.
__host__ __device__ inline int sign_class(int c)
{
    const int n = (int)sqrtf((float)c + 0.5f);  // exact: c < 2^16
    const int i = c - n * n;
    const int m = (i + 1) / 2;
    const int im = (i > 0 && (i & 1) == 0) ? 1 : 0;
    return (((n + m) & 1) << 2) | (im << 1) | ((m + im) & 1);
}

__host__ __device__ inline bool odd_parity(int v) { return ((v ^ (v >> 1) ^ (v >> 2)) & 1) != 0; }

// Orbit o in 1..26: half-widths from the parent's centre along axis a.
__host__ __device__ inline int orbit_axis(int o, int a) { return 1 + (a == 0 ? o : a == 1 ? o / 3 : o / 9) % 3; }
// Child-level coordinate at distance x on the positive or negative side of
// the centre of parent coordinate p (x = 1: p's own children 2 p + 1, 2 p).
__host__ __device__ inline int orbit_coord(int p, int x, bool neg) { return neg ? 2 * p + 1 - x : 2 * p + x; }

// One level of an M2L input: its boxes are the rows of a [row][model][PS]
// array, dense over a block of the level, x fastest.
struct OctLev {
    int s0[3], ns[3];
    int64_t row0;  // first row of the level
};
struct OctGeom {
    OctLev lev[kMaxLevels + 1];
    int B;
};
// Place of a box in its level's block, -1 outside.
__host__ __device__ inline int32_t octet_place(const OctLev &lv, int x, int y, int z)
{
    const int sx = x - lv.s0[0], sy = y - lv.s0[1], sz = z - lv.s0[2];
    // no branches: the M2L looks eight images up between matrix instructions
    const bool in = ((uint32_t)sx < (uint32_t)lv.ns[0]) & ((uint32_t)sy < (uint32_t)lv.ns[1]) &
                    ((uint32_t)sz < (uint32_t)lv.ns[2]);
    const int32_t j = (sz * lv.ns[1] + sy) * lv.ns[0] + sx;
    return in ? j : -1;
}
// The forward's input: the ME over each level's source block; the transposed
// M2L's: the adjoint LE over each level's gather region (the target boxes'
// bounding box within reach of the source block), zero where no target box is.
OctGeom octet_geom(const Plan *p, bool transposed);

// Element (lane, e) of a set of E operand values per lane: 16-byte groups
// [E / G][64 lanes][G], then the E % G values left over as [64 lanes][E % G].
// (A padded last group would load a register that holds no operand: the
// compiler puts temporaries there and waits for the load in flight first.)
template <typename T>
__host__ __device__ constexpr int frag_at(int E, int lane, int e)
{
    constexpr int G = 16 / (int)sizeof(T);
    return e < E / G * G ? ((e / G) * 64 + lane) * G + e % G : (E / G * 64) * G + lane * (E % G) + e % G;
}
template <typename T, int E>
__device__ __forceinline__ void load_set(const T *set, int lane, T (&v)[E])
{
    constexpr int G = 16 / (int)sizeof(T), R = E % G;
    using g16 = __attribute__((__vector_size__(16))) T;
#pragma unroll
    for (int j = 0; j < E / G; ++j) {
        const g16 x = reinterpret_cast<const g16 *>(set)[j * 64 + lane];
#pragma unroll
        for (int t = 0; t < G; ++t)
            v[j * G + t] = x[t];
    }
    if constexpr (R > 0) {
        const T *p = set + (E / G * 64) * G + lane * R;
#pragma unroll
        for (int t = 0; t < R; ++t)
            v[E / G * G + t] = p[t];
    }
}

// Shape of the M2L kernel at order P in type T.  A workgroup has eight
// waves: wave w takes parity w / RS and one of RS parts of the row blocks
// (RS = 2 covers the eight parities with two units), so that no wave holds
// more than 8 row blocks x 2 column blocks of FP64 sums.  The contraction over
// the coefficients is cut into NQ chunks of CK k steps: chunk q, k step u
// and sub-row kr take coefficient 4 CK q + 4 u + kr.  CK divides the k steps
// that hold coefficients wherever a small divisor exists (25 = 5 x 5 at p =
// 10), so that few instructions run on padding.  A lane's operator values of
// one k step are its RBW row blocks, in 16-byte groups and one shorter load for
// the rest (frag_at); D sets of them are in flight.
template <int P, typename T>
struct OctShape {
    static constexpr int P2 = P * P, RB = (P2 + 15) / 16, PS = 16 * RB;
    static constexpr int CK = P <= 2 ? 1 : P == 3 || P == 6 ? 3 : P == 5 || P == 7 || P == 9 ? 7 : P == 10 ? 5 : 4;
    static constexpr int CC = 4 * CK, NQ = (P2 + CC - 1) / CC, KS = NQ * CK;
    static_assert(NQ * CC <= PS, "a chunk reads past an expansion");
    static constexpr int RS = sizeof(T) == 8 && RB > 4 ? 2 : 1;
    static constexpr int RBW = (RB + RS - 1) / RS, NX = 8 / RS;
    static constexpr int EA = RBW;
    static constexpr int D = CK * EA * (int)sizeof(T) <= (sizeof(T) == 4 && RB <= 12 ? 256 : 224) ? CK : 2;  // 64 or 56 registers
    static_assert(CK % D == 0, "operator sets do not tile a chunk");
    static constexpr int64_t KOP = (int64_t)KS * EA * 64;  // elements per (orbit, parity, part)
    // LDS tile of one k step: sub-row kr and column c sit where both the
    // staging stores (a few columns, all k steps of a chunk) and the reads of
    // 32 (FP32) or 16 lanes spread over the banks
    static constexpr int US = 80;
    __host__ __device__ static constexpr int at(int u, int kr, int c)
    {
        return sizeof(T) == 4 ? US * u + 32 * (kr >> 1) + 2 * c + (kr & 1) : US * u + 20 * kr + c;
    }
    // column blocks of 16 per wave on wide plans: as many as leave two waves
    // per SIMD without spills
    static constexpr int NCW = sizeof(T) == 4 ? (RB <= 5 ? 4 : RB <= 8 ? 3 : 2) : 2;
    // FP32 with at most four coefficient rows in the last row block: that
    // block runs as 4x4x1 instructions, a quarter of the cycles
    static constexpr bool TAIL4 = sizeof(T) == 4 && P2 % 16 >= 1 && P2 % 16 <= 4;
};

// Parities' rows: class sizes are at most h (h + 1) / 2, h = ceil(P / 2).
template <int P>
struct ClassShape {
    static constexpr int h = (P + 1) / 2, MAXC = h * (h + 1) / 2;
    static constexpr int RBC = (MAXC + 15) / 16;  // row blocks of a class
    static constexpr int KC = (MAXC + 3) / 4;     // k steps of a class
};

// The M2L slots of a level's columns (T: the M2L's element type): group g0 +
// column / ncol holds column % ncol; RS units per group, 8 / RS parities each.
template <typename T>
struct SlotArgs {
    const T *part;
    const int32_t *uslot;
    int g0, ncol;
};

}  // namespace grav
