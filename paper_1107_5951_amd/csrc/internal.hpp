// Internal plan layout and shared device helpers of libgrav.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "grav.h"

namespace grav {

constexpr int kMaxP = 16;
constexpr int kMaxLevels = 10;

constexpr int kCanonOffsets = 56;  // M2L offsets d, 2 <= max |d_a| <= 3, with non-negative components
constexpr int kClassOffsets = 189; // offsets valid for one child-parity class
constexpr int kMaxLeafCells = 8;     // leaf edge cap: a leaf's densities fit one 512-entry LDS stage
constexpr int kNearChunk = 3;        // k steps per chunk of the near field by parity (54 in all)
constexpr int kMaxLatticeLeaf = 4;   // largest leaf edge with lattice near-field matrices

struct LevelInfo {
    int l = 0;
    double w = 0.0;                   // box edge
    int s0[3] = {0, 0, 0};            // source block start (root-relative box coords, x,y,z)
    int ns[3] = {0, 0, 0};            // source block size
    int64_t n_src = 0;                // ns[0]*ns[1]*ns[2]
    int64_t me_off = 0;               // offset (in expansions) of this level in the ME array
    int64_t n_tgt = 0;                // boxes holding evaluation points
    int64_t tgt_off = 0;              // offset of this level in the per-target-box arrays
    int64_t tmap_off = 0;             // offset of this level's target map (source block + halo 3)
    int need_lo[3] = {0, 0, 0};       // box range whose expansions the M2L reads (the
    int need_hi[3] = {-1, -1, -1};    // target boxes' range widened by 3, inclusive)
    // transposed M2L's input: the block of boxes that holds the target boxes
    // within reach of the source block
    int gs0[3] = {0, 0, 0}, gns[3] = {0, 0, 0};
    int64_t g_off = 0;                // first row of the level in that input
};

// One direction of the M2L over sibling octets (octet.hpp): columns are
// (octet, model) pairs, octet = a parent box, level by level.
struct OctGroup {      // 16 nc columns of one level
    int32_t level, ncol;
    int64_t col0;      // first column within the level
    int64_t oct0;      // first octet of the level
};
struct OctTables {
    const uint32_t *key;       // [noct] Morton key of the parent
    const OctGroup *groups;
    const int32_t *segs;       // [nseg][4] unit, its orbits (bit o - 1), slot, 0
    const int32_t *wgseg;      // [wgs + 1] segments of a workgroup
    const int32_t *uslot;      // [nunit + 1] slots of a unit, in orbit order
};
struct OctPlan {
    int32_t wgs = 0, nc = 1, ngroup = 0, nunit = 0;
    int64_t noct = 0, nseg = 0;
    uint32_t *d_key = nullptr;
    int64_t first[kMaxLevels + 2] = {0};  // octets of level l: [first[l], first[l + 1])
    int64_t reach[kMaxLevels + 1] = {0};  // those from reach[l] on have no M2L input
    int32_t gfirst[kMaxLevels + 1] = {0}; // first group of level l
    int32_t *d_parent = nullptr;          // [noct] row of the parent, -1 at level 2
    int32_t *d_child = nullptr;           // [noct][8] row of each child octant, -1: none
    int32_t *d_segs = nullptr, *d_wgseg = nullptr;
    int32_t *d_uslot = nullptr;
    OctGroup *d_groups = nullptr;
    void *d_ops = nullptr;  // operators as MFMA A fragments, in the M2L's element type
    OctTables tables() const
    {
        return OctTables{d_key, d_groups, d_segs, d_wgseg, d_uslot};
    }
};
// Compile-time shape of the M2L kernel (OctShape in octet.hpp).
struct OctInfo {
    int RS, RBW, EA, CK, KS, NCW;
    bool tail4;
};

// Points start .. start + n - 1 (sorted order) of a target leaf.
struct PointRun {
    int64_t start;
    int32_t leaf, n;
};

struct Stage {
    std::string name;
    hipEvent_t a = nullptr, b = nullptr;
};

struct Plan {
    grav_plan_desc d{};
    int device = 0;
    int P = 0, P2 = 0, PS = 0;     // order, p^2, padded stride (multiple of 16)
    int q = 1, nq3 = 1, b = 1;     // quadrature points per axis, per cell, leaf edge in cells
    int L = 0;                     // leaf level
    int B = 1, C = 3;
    double wl = 0.0;               // leaf edge
    double root0[3] = {0, 0, 0};   // root lower corner
    int shift[3] = {0, 0, 0};      // leaves between root corner and the mesh origin
    int64_t M = 0;                 // evaluation points
    int64_t n_spts = 0;            // explicit sources (0: the cells' quadrature points)
    int64_t n_leaf = 0;            // leaves holding evaluation points
    LevelInfo lev[kMaxLevels + 1];
    int64_t n_me = 0, n_le = 0;    // expansions (per model) in the ME / LE arrays
    int64_t n_tbox = 0;            // target boxes over all levels >= 2
    int64_t n_tmap = 0;

    // device buffers
    double *d_points = nullptr;    // [n_points][3] user points (unsorted)
    // explicit sources, sorted by their leaf (dense index in the leaf
    // level's source block): lattice-frame positions, mass per unit input
    // value (volume / h^3, or 1 / h^3), sorted -> user index, and the CSR
    // of each leaf's sources
    double *d_spos = nullptr;      // [n_spts][3]
    double *d_sw = nullptr;        // [n_spts]
    uint32_t *d_sperm = nullptr;   // [n_spts]
    double *d_smass = nullptr;     // [B][n_spts] masses of the call's input, sorted
    int64_t *d_sstart = nullptr;   // [leaves of the leaf-level source block + 1]
    uint32_t *d_perm = nullptr;    // [M] sorted position -> user index
    double *d_tpos = nullptr;      // [M][3] sorted target positions
    int64_t *d_leaf_start = nullptr; // [n_leaf + 1]
    uint32_t *d_tkey = nullptr;    // [n_tbox_all] Morton key of every target box, per level
    int64_t tbox_off[kMaxLevels + 1] = {0}; // start of each level in the array above
    OctPlan m2l, m2lt;                  // octets of the target boxes (M2L, L2L, L2L^T) and of the
                                        // source boxes (M2L^T, M2M, M2M^T)
    // the translations between levels by parity (levels.hip), operators of the
    // (+,+,+) child as MFMA A fragments, and the coefficients of each class
    double *d_m2m = nullptr, *d_l2lt = nullptr;    // up: [8][k steps][row blocks of a class][64]
    double *d_l2l = nullptr, *d_m2mt = nullptr;    // down: [8][k steps of a class][PS/16][64]
    int32_t *d_class_coef = nullptr;               // [8][16 x row blocks of a class], -1 past its end
    double *d_part = nullptr;           // segment slots, shared by both directions
    // the M2L's input where it is not the ME itself: FP32 copies of the ME
    // (mixed plans), the gathered adjoint LE
    double *d_rows = nullptr;
    int64_t n_grow = 0;                 // rows of the gathered adjoint LE
    // near field of voxel-centre targets by lattice matrices (b <= 4)
    bool lat_near = false;
    int lat_RB = 0, lat_Q = 0;                     // row blocks (C b^3 / 16); chunks of four k steps
    // near field by reflection parity (4^3-cell leaves, near.hip): operators
    // of both directions in the near field's element type, the far field at
    // the base centres and its coefficients by class
    bool near_par = false;
    void *d_near_op = nullptr, *d_near_opt = nullptr;
    double *d_near_far = nullptr, *d_near_fart = nullptr;  // and its transpose
    int32_t *d_near_coef = nullptr;
    int near_KC = 0;                               // k steps of a class
    double *d_tl2p = nullptr;                      // [PS/16][RB][64][4] far field (L2P) at the cell centres, FP64
    int64_t *d_lat_tab = nullptr;                  // [27 Q][2] per near chunk: density and operator offsets
    double *d_tn64 = nullptr;                      // [27][KS][RB][64] swizzled, FP64 plans
    float *d_tn32 = nullptr;                       // same, mixed plans
    int lat_TQ = 0;                                // adjoint: chunks of the (target, component) contraction
    double *d_tnt64 = nullptr;                     // [27][TQ][ceil(b^3/16)][64][4] transposed near field, FP64
    float *d_tnt32 = nullptr;                      // same, mixed plans
    double *d_tl2pt = nullptr;                     // [TQ][PS/16][64][4] transposed lattice L2P (FP64)
    double *d_w_blk = nullptr;                     // [TQ][4][padded leaves x B][4] adjoint weights per leaf (FP32 in mixed plans)
    int32_t *d_cell_slot = nullptr;                // [ncell] sorted slot of each voxel centre
    hipStream_t bs = nullptr;                      // plan-build stream (non-blocking), only inside grav_plan
    int direct_chunks = 1;                         // source chunks of grav_direct
    double *d_dpart = nullptr;                     // [chunks][M][B][4] its partial sums
    double *d_rho_blk = nullptr;                   // [Q][4][padded leaves x B][4] densities per leaf (FP32 in mixed plans)
    int64_t *d_leaf_pend = nullptr;                // [n_leaf] end of the user points of a leaf
    int32_t *d_pt_leaves = nullptr;                // source leaves with user points in their 27 neighbours
    int64_t n_pt_leaves = 0;                       // (any order), for the adjoint's point near field
    int32_t *d_user_leaves = nullptr;              // target leaves holding user points (any order), for
    int64_t n_user_leaves = 0;                     // the point near field
    PointRun *d_runs = nullptr;                    // their points in runs (any order), for the L2P
    int64_t n_runs = 0;
    int l2p_wgs = 0;                               // workgroups of the L2P that are resident at once
    int32_t *d_class_off = nullptr;  // [8][189][4] (dx, dy, dz, offset id)
    int32_t *d_tmap = nullptr;       // per level: target-box index over source block + halo 3
    struct DevGeom *d_geom = nullptr;

    // lattice P2M by octets (p2m.hip) as MFMA A fragments: leaf, parent by
    // class, and their transposes (rows: cells, to whole sets of row blocks)
    double *d_pm = nullptr, *d_pm_up = nullptr, *d_pmt = nullptr, *d_pmt_down = nullptr;
    double *d_me = nullptr;        // [n_me][B][PS], without the leaves' in mixed plans with lattice sources
    double *d_le = nullptr;        // [n_tbox][B][PS]
    double *d_near = nullptr;      // [M][B][4] near field (phi, gx, gy, gz), sorted order

    int64_t m2l_pairs = 0;         // box pairs translated by M2L (per model)
    int64_t p2p_pairs = 0;         // point pairs of the near-field sum (per model)
    size_t bytes_resident = 0, bytes_call = 0;
    hipStream_t last_stream = nullptr;
    hipEvent_t done = nullptr;
    bool has_pending = false;

    bool profiling = false;
    std::vector<Stage> stages;
    int n_stage_used = 0;
};

#define GRAV_HIP(call)                                                                 \
    do {                                                                               \
        hipError_t e_ = (call);                                                        \
        if (e_ != hipSuccess)                                                          \
            return GRAV_EDEVICE;                                                       \
    } while (0)

#define GRAV_CHECK(call)                                                               \
    do {                                                                               \
        grav_status s_ = (call);                                                       \
        if (s_ != GRAV_OK)                                                             \
            return s_;                                                                 \
    } while (0)

// Morton interleave of 10-bit coordinates (x in bit 0).
__host__ __device__ inline uint32_t spread3(uint32_t v)
{
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000ffu;
    v = (v | (v << 8)) & 0x0300f00fu;
    v = (v | (v << 4)) & 0x030c30c3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}
__host__ __device__ inline uint32_t compact3(uint32_t v)
{
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030c30c3u;
    v = (v | (v >> 4)) & 0x0300f00fu;
    v = (v | (v >> 8)) & 0x030000ffu;
    v = (v | (v >> 16)) & 0x000003ffu;
    return v;
}
__host__ __device__ inline uint32_t morton3(uint32_t x, uint32_t y, uint32_t z)
{
    return spread3(x) | (spread3(y) << 1) | (spread3(z) << 2);
}

// Device scans / sorts (sort.hip).
grav_status scan_exclusive_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp,
                               hipStream_t s);
size_t scan_tmp_words(int64_t n);
grav_status radix_sort_pairs(uint32_t *keys, uint32_t *vals, uint32_t *keys_tmp,
                             uint32_t *vals_tmp, int64_t n, int bits, uint32_t *scratch,
                             hipStream_t s);
size_t radix_scratch_words(int64_t n);

// Stage helpers (eval.hip)
void stage_begin(Plan *p, const char *name, hipStream_t s);
void stage_end(Plan *p, hipStream_t s);

}  // namespace grav
