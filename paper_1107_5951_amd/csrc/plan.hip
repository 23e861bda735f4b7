// grav_plan: geometry, device octree build and operator set-up.
//
// Internally every length is in cell units with the mesh origin at 0 (the
// "lattice frame"): cell (i, j, k) spans [i, i+1) x [j, j+1) x [k, k+1), a
// quadrature point has mass rho * w_a with w_a the rule's weight fraction,
// and the physical field follows as g = G h g_lat, phi = G h^2 phi_lat.
// Cell-centre evaluation points are placed at exact half-integers, so a
// point that coincides with a 1-point source has an exactly zero offset.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <new>

#include "octet.hpp"
#include "resolve.hpp"
#include "internal.hpp"
#include "operators.hpp"

// Wide M2L units (see build_octet_schedule) from this many work items per
// resident workgroup on: with two column blocks per wave and 64^3 cells, FP64 p =
// 12, 142 us wide against 166 single (three items per workgroup); with three,
// FP32 p = 10, 57 wide against 48 (one item); no difference on larger plans.
#ifndef GRAV_M2L_WIDE_ROUNDS
#define GRAV_M2L_WIDE_ROUNDS 2
#endif

// Leaves of 4^3 cells take the dense near field where the parity kernels' blocks
// (16 leaves of one model) hold at most a quarter of their leaves and there are
// more of them (over all models) than this many per leaf held and twice as many in
// all.  Dense against parity, whole calls of cell centres in us, forward and
// adjoint, p = 10 (gz; g): 4^3 cells (1 leaf) x 512 models 28 / 16, 37 / 21; 28 / 20,
// 79 / 37; x 1024 28 / 22, 37 / 31; 29 / 31, 92 / 62; x 2048 28 / 37, 37 / 53; 32 / 54,
// 94 / 113; FP64 x 512 26 / 22, 57 / 24; 28 / 28, 143 / 49; x 1024 26 / 37, 57 / 38;
// 29 / 49, 145 / 86; x 2048 28 / 67, 59 / 66; 45 / 92, 146 / 161; 8 x 8 x 4 cells (4 leaves) x 1024 29 / 24, 39 / 33; 47 / 33, 96 / 63; x 4096 53 /
// 65, 62 / 94; 127 / 101, 137 / 214.
#ifndef GRAV_NEAR_DENSE_BLOCKS
#define GRAV_NEAR_DENSE_BLOCKS 512
#endif

// Workgroups that the runs of points of single-model plans are cut for.  L2P with
// 1024 / 2048 / 4096 / 8192: one model at 1024^2 stations above 16^3 cells, p = 10,
// 68 / 65 / 68 / 71 us, FP64 p = 14 133 / 119 / 119 / 123.  Several models load their
// expansions again with every run (64 at 64^2 stations 22 / 25 / 35 / 32 us; 18 over
// 76^3 cells, 16 points a leaf, 14.7 whole and 19.0 in two runs of one step): runs of
// two steps or more, cut for the workgroups that are resident.
#ifndef GRAV_RUN_BLOCKS
#define GRAV_RUN_BLOCKS 2048
#endif

namespace grav {

namespace {

constexpr int64_t kRunBlocks = GRAV_RUN_BLOCKS;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Position (lattice frame) of evaluation point i in descriptor order.
__device__ inline void target_lattice(int64_t i, const double *pts, int64_t npts, int nx, int ny,
                                      const double org[3], double inv_h, double out[3])
{
    if (i < npts) {
        out[0] = (pts[3 * i + 0] - org[0]) * inv_h;
        out[1] = (pts[3 * i + 1] - org[1]) * inv_h;
        out[2] = (pts[3 * i + 2] - org[2]) * inv_h;
    } else {
        const int64_t c = i - npts;
        const int64_t ix = c % nx;
        const int64_t iy = (c / nx) % ny;
        const int64_t iz = c / ((int64_t)nx * ny);
        out[0] = (double)ix + 0.5;
        out[1] = (double)iy + 0.5;
        out[2] = (double)iz + 0.5;
    }
}

struct KeyArgs {
    const double *pts;
    int64_t npts, M;
    int nx, ny;
    double org[3];
    double inv_h;
    double shift_lat[3];  // shift * b: lattice distance from root corner to origin
    double inv_b;
    int kmax;             // leaves per axis - 1
    int L;
};

__global__ void k_target_keys(KeyArgs a, uint32_t *keys, uint32_t *vals)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.M)
        return;
    double u[3];
    target_lattice(i, a.pts, a.npts, a.nx, a.ny, a.org, a.inv_h, u);
    uint32_t c[3];
    for (int d = 0; d < 3; ++d) {
        double f = floor((u[d] + a.shift_lat[d]) * a.inv_b);
        f = fmin(fmax(f, 0.0), (double)a.kmax);
        c[d] = (uint32_t)f;
    }
    keys[i] = morton3(c[0], c[1], c[2]);
    vals[i] = (uint32_t)i;
}

__global__ void k_gather_targets(KeyArgs a, const uint32_t *perm, double *tpos)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.M)
        return;
    double u[3];
    target_lattice((int64_t)perm[i], a.pts, a.npts, a.nx, a.ny, a.org, a.inv_h, u);
    tpos[3 * i + 0] = u[0];
    tpos[3 * i + 1] = u[1];
    tpos[3 * i + 2] = u[2];
}

// flags[i] = 1 where (key[i] >> sh) differs from its predecessor.
__global__ void k_head_flags(const uint32_t *keys, int64_t n, int sh, uint32_t *flags)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    flags[i] = (i == 0 || (keys[i] >> sh) != (keys[i - 1] >> sh)) ? 1u : 0u;
}

// Leaf level: leaf start offsets, leaf keys.
__global__ void k_leaf_build(const uint32_t *keys, const uint32_t *flags, const uint32_t *scan,
                             int64_t n, int64_t *leaf_start, uint32_t *leaf_key)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t id = scan[i] + flags[i] - 1u;
    if (flags[i]) {
        leaf_start[id] = i;
        leaf_key[id] = keys[i];
    }
}

// Parent level from the sorted child box keys.
__global__ void k_parent_build(const uint32_t *ckeys, const uint32_t *flags, const uint32_t *scan,
                               int64_t n, uint32_t *pkeys)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t id = scan[i] + flags[i] - 1u;
    if (flags[i])
        pkeys[id] = ckeys[i] >> 3;
}

struct CountArgs {
    int s0[3], ns[3];   // source block of the level
    int n[3], shift[3];
    int b, nq3;
};

// M2L box pairs of one level: in-block offsets of each target box's class list.
__global__ void k_count_m2l(const uint32_t *bkeys, int64_t n, CountArgs a, const int32_t *cls_off,
                            unsigned long long *acc)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t k = bkeys[i];
    const int x = (int)compact3(k), y = (int)compact3(k >> 1), z = (int)compact3(k >> 2);
    const int32_t *o = cls_off + (k & 7u) * kClassOffsets * 4;
    unsigned long long c = 0;
    for (int j = 0; j < kClassOffsets; ++j) {
        const int sx = x + o[4 * j] - a.s0[0], sy = y + o[4 * j + 1] - a.s0[1],
                  sz = z + o[4 * j + 2] - a.s0[2];
        if (sx >= 0 && sy >= 0 && sz >= 0 && sx < a.ns[0] && sy < a.ns[1] && sz < a.ns[2])
            ++c;
    }
    atomicAdd(acc, c);
}

// P2P point pairs: targets of a leaf times source points in its 27 neighbours.
__global__ void k_count_p2p(const uint32_t *lkeys, const int64_t *leaf_start, int64_t n,
                            CountArgs a, unsigned long long *acc)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t k = lkeys[i];
    const int c[3] = {(int)compact3(k), (int)compact3(k >> 1), (int)compact3(k >> 2)};
    unsigned long long cells = 0;
    for (int nb = 0; nb < 27; ++nb) {
        const int d[3] = {nb % 3 - 1, (nb / 3) % 3 - 1, nb / 9 - 1};
        unsigned long long leaf_cells = 1;
        for (int ax = 0; ax < 3; ++ax) {
            const int lc = c[ax] + d[ax];
            if (lc - a.s0[ax] < 0 || lc - a.s0[ax] >= a.ns[ax]) {
                leaf_cells = 0;
                break;
            }
            const int lo = (lc - a.shift[ax]) * a.b;
            const int hi = min(lo + a.b, a.n[ax]);
            leaf_cells *= (unsigned long long)max(0, hi - max(lo, 0));
        }
        cells += leaf_cells;
    }
    atomicAdd(acc, cells * (unsigned long long)a.nq3 * (unsigned long long)(leaf_start[i + 1] - leaf_start[i]));
}

// Point pairs of the near field with explicit sources: per target leaf, its
// targets times the sources of its 27 neighbour leaves.
__global__ void k_count_p2p_src(const uint32_t *lkeys, const int64_t *leaf_start, int64_t n, CountArgs a,
                                const int64_t *sstart, unsigned long long *acc)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t k = lkeys[i];
    const int c[3] = {(int)compact3(k), (int)compact3(k >> 1), (int)compact3(k >> 2)};
    unsigned long long srcs = 0;
    for (int nb = 0; nb < 27; ++nb) {
        const int d[3] = {nb % 3 - 1, (nb / 3) % 3 - 1, nb / 9 - 1};
        int r[3];
        bool in = true;
        for (int ax = 0; ax < 3; ++ax) {
            r[ax] = c[ax] + d[ax] - a.s0[ax];
            in = in && r[ax] >= 0 && r[ax] < a.ns[ax];
        }
        if (!in)
            continue;
        const int64_t j = ((int64_t)r[2] * a.ns[1] + r[1]) * a.ns[0] + r[0];
        srcs += (unsigned long long)(sstart[j + 1] - sstart[j]);
    }
    atomicAdd(acc, srcs * (unsigned long long)(leaf_start[i + 1] - leaf_start[i]));
}

__global__ void k_fill_last(int64_t *leaf_start, int64_t n_leaf, int64_t M)
{
    if (blockIdx.x == 0 && threadIdx.x == 0)
        leaf_start[n_leaf] = M;
}

// Sorted slot of every voxel-centre target: slot[c] = j with perm[j] = npts + c.
__global__ void k_cell_slot(const uint32_t *perm, int64_t M, int64_t npts, int32_t *slot)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= M)
        return;
    const int64_t i = perm[j];
    if (i >= npts)
        slot[i - npts] = (int32_t)j;
}

// End of the user points of each leaf.  The sort is stable and the keys are
// assigned in descriptor order (points first, then voxel centres), so within a
// leaf the user points form a prefix; find its end by bisection.
__global__ void k_leaf_point_end(const uint32_t *perm, const int64_t *leaf_start, int64_t n_leaf,
                                 int64_t npts, int64_t *pend)
{
    const int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= n_leaf)
        return;
    int64_t lo = leaf_start[l], hi = leaf_start[l + 1];
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if ((int64_t)perm[mid] < npts)
            lo = mid + 1;
        else
            hi = mid;
    }
    pend[l] = lo;
}

template <class T>
grav_status dalloc(Plan *p, T **ptr, size_t count, bool resident)
{
    *ptr = nullptr;
    if (count == 0)
        return GRAV_OK;
    if (hipMalloc((void **)ptr, sizeof(T) * count) != hipSuccess) {
        *ptr = nullptr;
        return GRAV_ENOMEM;
    }
    if (resident)
        p->bytes_resident += sizeof(T) * count;
    else
        p->bytes_call += sizeof(T) * count;
    return GRAV_OK;
}

void free_plan(Plan *p)
{
    if (!p)
        return;
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(p->device);
    void *bufs[] = {p->d_points, p->d_perm, p->d_tpos, p->d_leaf_start, p->d_tkey,
                    p->d_class_off, p->d_tmap, p->d_geom, p->d_pm, p->d_pm_up, p->d_pmt, p->d_pmt_down, p->d_m2m, p->d_l2l, p->d_m2mt,
                    p->d_l2lt, p->d_class_coef, p->d_me, p->d_le, p->d_near, p->d_part, p->d_rows,
                    p->d_tn64, p->d_tn32, p->d_rho_blk, p->d_tl2p, p->d_dpart,
                    p->d_lat_tab, p->d_cell_slot, p->d_leaf_pend,
                    p->d_tnt64, p->d_tnt32, p->d_tl2pt, p->d_w_blk,
                    p->d_spos, p->d_sw, p->d_smass, p->d_sperm, p->d_sstart, p->d_pt_leaves, p->d_user_leaves, p->d_runs,
                    p->d_near_op, p->d_near_opt, p->d_near_far, p->d_near_fart, p->d_near_coef};
    for (OctPlan *o : {&p->m2l, &p->m2lt}) {
        void *ob[] = {o->d_key, o->d_child, o->d_parent, o->d_segs, o->d_wgseg, o->d_uslot, o->d_groups,
                      o->d_ops};
        for (void *b : ob)
            if (b)
                (void)hipFree(b);
    }
    for (void *b : bufs)
        if (b)
            (void)hipFree(b);
    if (p->done)
        (void)hipEventDestroy(p->done);
    for (auto &st : p->stages) {
        if (st.a)
            (void)hipEventDestroy(st.a);
        if (st.b)
            (void)hipEventDestroy(st.b);
    }
    (void)hipSetDevice(cur);
    delete p;
}

grav_status validate(const grav_plan_desc *d)
{
    if (!d)
        return GRAV_EINVAL;
    if (d->nx < 1 || d->ny < 1 || d->nz < 1)
        return GRAV_EINVAL;
    if (!(d->h > 0.0) || !std::isfinite(d->h))
        return GRAV_EINVAL;
    for (int a = 0; a < 3; ++a)
        if (!std::isfinite(d->origin[a]))
            return GRAV_EINVAL;
    if (d->quad_order != 1 && d->quad_order != 2)
        return GRAV_EINVAL;
    if (d->n_points < 0 || (d->n_points > 0 && !d->points))
        return GRAV_EINVAL;
    if (d->components != 1 && d->components != 3 && d->components != 4)
        return GRAV_EINVAL;
    if (d->p < 1)
        return GRAV_EINVAL;
    if (d->p > kMaxP)
        return GRAV_EUNSUPPORTED;
    if (d->leaf_size < 1)
        return GRAV_EINVAL;
    if (d->precision != GRAV_FP64 && d->precision != GRAV_MIXED)
        return GRAV_EINVAL;
    if (d->batch < 1)
        return GRAV_EINVAL;
    if (!std::isfinite(d->G))
        return GRAV_EINVAL;
    if (d->n_sources < 0 || (d->n_sources > 0 && (!d->sources || d->quad_order != 1)))
        return GRAV_EINVAL;
    if (d->n_sources > 0xffffffffll)
        return GRAV_EUNSUPPORTED;
    for (int64_t i = 0; i < d->n_sources; ++i) {
        for (int a = 0; a < 3; ++a) {
            const int n = a == 0 ? d->nx : a == 1 ? d->ny : d->nz;
            const double u = (d->sources[3 * i + a] - d->origin[a]) / d->h;
            if (!(u >= 0.0 && u < (double)n))
                return GRAV_EINVAL;  // outside the mesh box (or not finite)
        }
        if (d->source_volumes && !(d->source_volumes[i] > 0.0 && std::isfinite(d->source_volumes[i])))
            return GRAV_EINVAL;
    }
    const int64_t ncell = (int64_t)d->nx * d->ny * d->nz;
    const int64_t M = d->n_points + (d->voxel_centres ? ncell : 0);
    if (M > 0xffffffffll || (int64_t)d->nx > 0x3fffffff)
        return GRAV_EUNSUPPORTED;
    return GRAV_OK;
}

// Index of offset |d| (components 0..3, largest >= 2) among the 56 canonical
// ones, z slowest, x fastest.
int canon_index(int ax, int ay, int az)
{
    int k = 0;
    for (int z = 0; z <= 3; ++z)
        for (int y = 0; y <= 3; ++y)
            for (int x = 0; x <= 3; ++x) {
                if (std::max(x, std::max(y, z)) < 2)
                    continue;
                if (x == ax && y == ay && z == az)
                    return k;
                ++k;
            }
    return -1;
}

// Per child-parity class the 189 M2L offsets (2 <= |d|_inf <= 3), entries
// (dx, dy, dz, canonical index of |d|): a target box of class c sees sources
// at T + d for d_a in [-2 - c_a, 3 - c_a].
std::vector<int32_t> offsets_table()
{
    std::vector<int32_t> fwd(8 * kClassOffsets * 4, 0);
    for (int c = 0; c < 8; ++c) {
        int nf = 0;
        for (int dz = -2 - (c >> 2 & 1); dz <= 3 - (c >> 2 & 1); ++dz)
            for (int dy = -2 - (c >> 1 & 1); dy <= 3 - (c >> 1 & 1); ++dy)
                for (int dx = -2 - (c & 1); dx <= 3 - (c & 1); ++dx) {
                    const int ci = canon_index(std::abs(dx), std::abs(dy), std::abs(dz));
                    if (ci < 0)
                        continue;
                    int32_t *e = &fwd[(c * kClassOffsets + nf++) * 4];
                    e[0] = dx, e[1] = dy, e[2] = dz, e[3] = ci;
                }
    }
    return fwd;
}

// Position of value e (of E per lane) of a lane in a set of MFMA operand
// fragments stored group-major, [E / G][64 lanes][G] with G = 16 bytes /
// element size: the layout the kernels read with one 16-byte vector load per
// group (a contiguous kilobyte per wave).
static inline size_t frag_pos(int lane, int e, int G)
{
    return ((size_t)(e / G) * 64 + lane) * G + e % G;
}

template <class T>
grav_status upload(Plan *p, T **dst, const std::vector<T> &src)
{
    GRAV_CHECK(dalloc(p, dst, src.size(), true));
    if (!src.empty())
        GRAV_HIP(hipMemcpyAsync(*dst, src.data(), sizeof(T) * src.size(), hipMemcpyHostToDevice, p->bs));
    GRAV_HIP(hipStreamSynchronize(p->bs));
    return GRAV_OK;
}

// The octet M2L's operators as MFMA A fragments, [orbit - 1][parity][part of
// the row blocks][k step][EA values per lane, see frag_at].  The
// image r of orbit o lies at offset e(r) from the (+,+,+) child; the forward
// takes K_e, the transposed M2L (a source box fed by the target box at e) the
// transpose of K_{-e}, both from the canonical operators by reflection.
template <class T>
grav_status upload_octet_operators(Plan *p, const std::vector<std::vector<double>> &kc, bool transposed, OctPlan &o)
{
    const int P2 = p->P2, PS = p->PS, RB = PS / 16;
    const OctInfo in = octet_info(p->P, sizeof(T) == 8);
    const size_t blk = (size_t)in.EA * 64, per = blk * in.KS;
    std::vector<T> ops(per * kOrbits * 8 * in.RS, (T)0);
    std::vector<int> cls(P2);
    for (int k = 0; k < P2; ++k)
        cls[k] = sign_class(k);
    // sign tables: (-1)^popcount(a & b)
    double sg[8][8];
    for (int a = 0; a < 8; ++a)
        for (int b = 0; b < 8; ++b)
            sg[a][b] = odd_parity(a & b) ? -1.0 : 1.0;
    std::vector<double> f((size_t)8 * P2 * P2);  // [chi][i][k]
    for (int ob = 1; ob <= kOrbits; ++ob) {
        const double *src[8];
        int refl[8];
        for (int r = 0; r < 8; ++r) {
            int e[3];
            refl[r] = 0;
            for (int a = 0; a < 3; ++a) {
                const int x = orbit_axis(ob, a);
                e[a] = (r >> a & 1) ? -x : x - 1;
                if ((transposed ? -e[a] : e[a]) < 0)
                    refl[r] |= 1 << a;
            }
            const int ci = canon_index(std::abs(e[0]), std::abs(e[1]), std::abs(e[2]));
            src[r] = ci >= 0 ? kc[ci].data() : nullptr;
        }
        for (int i = 0; i < P2; ++i)
            for (int k = 0; k < P2; ++k) {
                const size_t at = transposed ? (size_t)k * PS + i : (size_t)i * PS + k;
                const int si = cls[i], sk = cls[k];
                double v[8];
                for (int r = 0; r < 8; ++r)
                    v[r] = src[r] ? 0.125 * sg[r][sk] * sg[refl[r]][si ^ sk] * src[r][at] : 0.0;
                for (int bit = 1; bit < 8; bit <<= 1)
                    for (int r = 0; r < 8; ++r)
                        if ((r & bit) == 0) {
                            const double x = v[r], y = v[r | bit];
                            v[r] = x + y;
                            v[r | bit] = x - y;
                        }
                for (int x = 0; x < 8; ++x)
                    f[((size_t)x * P2 + i) * P2 + k] = v[x];
            }
        for (int x = 0; x < 8; ++x)
            for (int part = 0; part < in.RS; ++part) {
                T *dst = ops.data() + (((size_t)(ob - 1) * 8 + x) * in.RS + part) * per;
                for (int ks = 0; ks < in.KS; ++ks) {
                    for (int rb = 0; rb < in.RBW; ++rb)
                        for (int lane = 0; lane < 64; ++lane) {
                            const int rbg = part * in.RBW + rb;
                            const int row = 16 * rbg + (in.tail4 && rbg == RB - 1 ? (lane & 3) : (lane & 15));
                            const int col = 4 * ks + (lane >> 4);
                            if (row < P2 && col < P2)
                                dst[ks * blk + frag_at<T>(in.EA, lane, rb)] = (T)f[((size_t)x * P2 + row) * P2 + col];
                        }
                }
            }
    }
    T *d = nullptr;
    GRAV_CHECK(upload(p, &d, ops));
    o.d_ops = d;
    return GRAV_OK;
}

// Operators of the translations between levels (levels.hip).  m and l: M2M and
// L2L of the (+,+,+) child.  Up: [class][k step][row block of the class][lane],
// row = coefficient 16 rb + lane % 16 of the class, column 4 ks + lane / 16.
// Down: [class][k step of the class][row block][lane], row 16 rb + lane % 16,
// column = coefficient 4 q + lane / 16 of the class.
static grav_status upload_level_operators(Plan *p, const std::vector<double> &m, const std::vector<double> &l)
{
    const int P2 = p->P2, PS = p->PS, RB = PS / 16;
    const int KS = octet_info(p->P, true).KS;
    std::vector<int> cls[8];
    size_t most = 0;
    for (int k = 0; k < P2; ++k) {
        cls[sign_class(k)].push_back(k);
        most = std::max(most, cls[sign_class(k)].size());
    }
    const int RBC = (int)ceil_div((int64_t)most, 16), KC = (int)ceil_div((int64_t)most, 4);
    std::vector<int32_t> coef((size_t)8 * 16 * RBC, -1);
    for (int x = 0; x < 8; ++x)
        std::copy(cls[x].begin(), cls[x].end(), coef.begin() + (size_t)x * 16 * RBC);
    GRAV_CHECK(upload(p, &p->d_class_coef, coef));
    for (int t = 0; t < 2; ++t) {
        // up: M2M, and L2L transposed; down: L2L, and M2M transposed
        std::vector<double> up((size_t)8 * KS * RBC * 64, 0.0), dn((size_t)8 * KC * RB * 64, 0.0);
        auto at_up = [&](int i, int k) { return t ? l[(size_t)k * PS + i] : m[(size_t)i * PS + k]; };
        auto at_dn = [&](int i, int k) { return t ? m[(size_t)k * PS + i] : l[(size_t)i * PS + k]; };
        for (int x = 0; x < 8; ++x)
            for (int lane = 0; lane < 64; ++lane) {
                for (int ks = 0; ks < KS; ++ks)
                    for (int rb = 0; rb < RBC; ++rb) {
                        const int n = 16 * rb + lane % 16, k = 4 * ks + lane / 16;
                        if (n < (int)cls[x].size() && k < P2)
                            up[(((size_t)x * KS + ks) * RBC + rb) * 64 + lane] = at_up(cls[x][n], k);
                    }
                for (int q = 0; q < KC; ++q)
                    for (int rb = 0; rb < RB; ++rb) {
                        const int n = 4 * q + lane / 16, i = 16 * rb + lane % 16;
                        if (n < (int)cls[x].size() && i < P2)
                            dn[(((size_t)x * KC + q) * RB + rb) * 64 + lane] = at_dn(i, cls[x][n]);
                    }
            }
        GRAV_CHECK(upload(p, t ? &p->d_l2lt : &p->d_m2m, up));
        GRAV_CHECK(upload(p, t ? &p->d_m2mt : &p->d_l2l, dn));
    }
    return GRAV_OK;
}

// Operators of the lattice P2M and its transpose by octets (p2m.hip).  m: the
// M2M of the (+,+,+) child.  Forward, in chunks of 16 cells, zero past the last:
// k step ks and sub-row kr take cell 4 ks + kr; leaf rows, in one part or two, 16 rb + 4 (lane % 4) + lane % 16 / 4 (a lane of the product then
// holds four consecutive coefficients), parent rows coefficient 16 rb + lane %
// 16 of the class.  Transpose: rows = cells 16 rb + lane % 16, to whole sets of
// row blocks; contraction over the leaf's coefficients in the order 16 (ks / 4)
// + 4 (lane / 16) + ks % 4 (four consecutive ones per lane and chunk of four k
// steps), over the parent's class in order.
static grav_status upload_lattice_p2m(Plan *p, const std::vector<double> &m)
{
    const int P = p->P, P2 = p->P2, PS = p->PS, RB = PS / 16;
    const int b3 = p->b * p->b * p->b, KV = (int)ceil_div(b3, 16) * 4;
    const int NP = RB > 8 ? 2 : 1, RBL = (int)ceil_div(RB, NP);
    const int R0 = (int)ceil_div(b3, 16), RBT = R0 <= 2 ? 2 : (int)ceil_div(R0, 4) * 4;
    std::vector<double> pm((size_t)b3 * PS), up((size_t)b3 * PS, 0.0);
    p2m_lattice(P, p->b, p->q, 1.0, PS, pm.data());
    for (int v = 0; v < b3; ++v)
        for (int i = 0; i < P2; ++i)
            for (int k = 0; k < P2; ++k)
                up[(size_t)v * PS + i] += m[(size_t)i * PS + k] * pm[(size_t)v * PS + k];
    std::vector<int> cls[8];
    size_t most = 0;
    for (int k = 0; k < P2; ++k) {
        cls[sign_class(k)].push_back(k);
        most = std::max(most, cls[sign_class(k)].size());
    }
    const int RBC = (int)ceil_div((int64_t)most, 16), KC = (int)ceil_div((int64_t)most, 4);
    std::vector<double> a((size_t)KV * NP * RBL * 64, 0.0), au((size_t)8 * KV * RBC * 64, 0.0);
    std::vector<double> t((size_t)PS / 4 * RBT * 64, 0.0), td((size_t)8 * KC * RBT * 64, 0.0);
    for (int lane = 0; lane < 64; ++lane) {
        for (int ks = 0; ks < KV; ++ks) {
            const int v = 4 * ks + lane / 16;
            if (v >= b3)
                continue;
            for (int rb = 0; rb < RB; ++rb)
                a[((((size_t)ks / 4 * NP + rb / RBL) * 4 + ks % 4) * RBL + rb % RBL) * 64 + lane] = pm[(size_t)v * PS + 16 * rb + 4 * (lane % 4) + lane % 16 / 4];
            for (int x = 0; x < 8; ++x)
                for (int rb = 0; rb < RBC; ++rb)
                    if (16 * rb + lane % 16 < (int)cls[x].size())
                        au[(((size_t)x * KV + ks) * RBC + rb) * 64 + lane] = up[(size_t)v * PS + cls[x][16 * rb + lane % 16]];
        }
        for (int rb = 0; rb < RBT; ++rb) {
            const int v = 16 * rb + lane % 16;
            if (v >= b3)
                continue;
            for (int ks = 0; ks < PS / 4; ++ks)
                t[((size_t)ks * RBT + rb) * 64 + lane] = pm[(size_t)v * PS + 16 * (ks / 4) + 4 * (lane / 16) + ks % 4];
            for (int x = 0; x < 8; ++x)
                for (int q = 0; q < KC; ++q)
                    if (4 * q + lane / 16 < (int)cls[x].size())
                        td[(((size_t)x * KC + q) * RBT + rb) * 64 + lane] = up[(size_t)v * PS + cls[x][4 * q + lane / 16]];
        }
    }
    GRAV_CHECK(upload(p, &p->d_pm, a));
    GRAV_CHECK(upload(p, &p->d_pm_up, au));
    GRAV_CHECK(upload(p, &p->d_pmt, t));
    GRAV_CHECK(upload(p, &p->d_pmt_down, td));
    return GRAV_OK;
}

grav_status build_operators(Plan *p)
{
    const int P = p->P, PS = p->PS;
    if (p->L < 2)
        return GRAV_OK;

    {
        // translations between levels by parity (levels.hip), from the
        // operators of the (+,+,+) child
        const double delta[3] = {0.25, 0.25, 0.25};
        std::vector<double> m((size_t)PS * PS), l((size_t)PS * PS);
        m2m_matrix(P, delta, PS, m.data());
        l2l_matrix(P, delta, PS, l.data());
        GRAV_CHECK(upload_level_operators(p, m, l));
        if (p->n_spts == 0)
            GRAV_CHECK(upload_lattice_p2m(p, m));
    }
    GRAV_CHECK(upload(p, &p->d_class_off, offsets_table()));
    if (p->M == 0)
        return GRAV_OK;
    // M2L over sibling octets: F_{chi,o} of both directions (octet.hpp)
    std::vector<std::vector<double>> kc(kCanonOffsets, std::vector<double>((size_t)PS * PS));
    for (int z = 0; z <= 3; ++z)
        for (int y = 0; y <= 3; ++y)
            for (int x = 0; x <= 3; ++x) {
                const int ci = canon_index(x, y, z);
                if (ci < 0)
                    continue;
                // source = target + d  =>  target centre - source centre = -d
                const double dd[3] = {-(double)x, -(double)y, -(double)z};
                m2l_matrix(P, dd, PS, kc[ci].data());
            }
    for (int t = 0; t < 2; ++t) {
        OctPlan &o = t ? p->m2lt : p->m2l;
        GRAV_CHECK(p->d.precision == GRAV_FP64 ? upload_octet_operators<double>(p, kc, t != 0, o)
                                               : upload_octet_operators<float>(p, kc, t != 0, o));
    }
    return GRAV_OK;
}

// Octets of the target or source boxes, level by level: the key of the parent,
// its row in the level above (-1 at level 2) and the rows of its children.
struct Octets {
    std::vector<uint32_t> key;
    std::vector<int32_t> child, parent;
    int64_t first[kMaxLevels + 2] = {0};  // octets of level l: [first[l], first[l + 1])
    int64_t reach[kMaxLevels + 1] = {0};  // those before reach[l] are within reach of M2L input
    void add(uint32_t k, int32_t row)
    {
        if ((int64_t)key.size() == open || key.back() != k >> 3) {
            key.push_back(k >> 3);
            child.insert(child.end(), 8, -1);
        }
        child[8 * (key.size() - 1) + (k & 7)] = row;
    }
    void level(int l)
    {
        first[l] = open = (int64_t)key.size();
        first[l + 1] = open;
    }
    void reached(int l) { reach[l] = (int64_t)key.size(); }
    void done(int l) { first[l + 1] = (int64_t)key.size(); }

private:
    int64_t open = 0;
};

// Groups, work items and schedule of one direction.  A unit is a group of
// 16 nc columns and one of RS parts of the parities; its items are the
// orbits at which some column has an input row (`has`: whether a box of a
// level has one).  A fixed number of workgroups, all resident at once: units
// that fill whole rounds of them run unsplit, one per workgroup and round, so
// that the workgroups of an XCD walk the operators together; the items of the
// remaining units are cut into equal contiguous shares, split into segments at
// unit boundaries.  Workgroups w, w + 8, ... share an XCD and take
// neighbouring units.
template <class Has>
static grav_status build_octet_schedule(Plan *p, const Octets &oc, OctPlan &o, Has &&has)
{
    const OctInfo in = octet_info(p->P, p->d.precision == GRAV_FP64);
    const int64_t B = p->B;
    o.noct = (int64_t)oc.key.size();
    std::copy(std::begin(oc.first), std::end(oc.first), std::begin(o.first));
    std::copy(std::begin(oc.reach), std::end(oc.reach), std::begin(o.reach));
    // two to four column blocks per wave once the work items (units times
    // orbits) are two for every resident workgroup; else single blocks, for more
    // items on small plans
    int resident = 0;
    GRAV_CHECK(m2l_resident_workgroups(p, in.NCW, &resident));
    int64_t near = 0;
    for (int l = 2; l <= p->L; ++l)
        near += oc.reach[l] - oc.first[l];
    o.nc = near * B * in.RS >= (int64_t)GRAV_M2L_WIDE_ROUNDS * resident * 16 * in.NCW / kOrbits ? in.NCW : 1;
    GRAV_CHECK(m2l_resident_workgroups(p, o.nc, &resident));
    const int ncol = 16 * o.nc;
    std::vector<OctGroup> groups;
    std::vector<uint32_t> umask;          // orbits of a unit
    std::vector<int32_t> live;            // units with orbits
    std::vector<int64_t> ustart(1, 0);    // first work item of each of those
    for (int l = 2; l <= p->L; ++l) {
        const int64_t cols = (oc.first[l + 1] - oc.first[l]) * B;
        o.gfirst[l] = (int32_t)groups.size();
        for (int64_t c0 = 0; c0 < cols; c0 += ncol) {
            OctGroup g{};
            g.level = l;
            g.ncol = (int32_t)std::min<int64_t>(ncol, cols - c0);
            g.col0 = c0;
            g.oct0 = oc.first[l];
            groups.push_back(g);
            uint32_t mask = 0;
            for (int ob = 1; ob <= kOrbits; ++ob) {
                bool hit = false;
                for (int64_t j = c0 / B; j <= std::min((c0 + g.ncol - 1) / B, oc.reach[l] - oc.first[l] - 1) && !hit; ++j) {
                    const uint32_t k = oc.key[oc.first[l] + j];
                    const int c[3] = {(int)compact3(k), (int)compact3(k >> 1), (int)compact3(k >> 2)};
                    for (int r = 0; r < 8 && !hit; ++r)
                        hit = has(l, orbit_coord(c[0], orbit_axis(ob, 0), r & 1),
                                  orbit_coord(c[1], orbit_axis(ob, 1), r & 2),
                                  orbit_coord(c[2], orbit_axis(ob, 2), r & 4));
                }
                if (hit)
                    mask |= 1u << (ob - 1);
            }
            for (int xh = 0; xh < in.RS; ++xh) {
                if (mask) {
                    live.push_back((int32_t)umask.size());
                    ustart.push_back(ustart.back() + __builtin_popcount(mask));
                }
                umask.push_back(mask);
            }
        }
    }
    const int64_t nunit = (int64_t)umask.size(), nlive = (int64_t)live.size(), T = ustart.back();
    const int64_t W = T == 0 ? 0 : std::min<int64_t>(resident, T);
    int64_t rounds = W > 0 ? nlive / W : 0;
    {
        // a round lasts as long as its longest unit: where units are so unequal
        // (small leaf grids) that the rounds would take 1.15 times their mean, all
        // items are shared out (p = 14 FP64, 12^3 cells x 1024: 2.07 -> 1.52 ms)
        int64_t longest = 0;
        for (int64_t r = 0; r < rounds; ++r) {
            int64_t m = 0;
            for (int64_t v = r * W; v < (r + 1) * W; ++v)
                m = std::max(m, ustart[v + 1] - ustart[v]);
            longest += m;
        }
        if (100 * longest * W > 115 * ustart[rounds * W])
            rounds = 0;
    }
    std::vector<int32_t> seg, wgseg(W + 1, 0);
    std::vector<std::vector<int32_t>> useg(nunit);
    const int64_t u0 = rounds * W, rest = T - ustart[u0];
    // position of workgroup w in its round: XCD w % 8 takes a contiguous range
    std::vector<int64_t> pos(W);
    {
        int64_t n = 0;
        for (int64_t x = 0; x < 8; ++x)
            for (int64_t w = x; w < W; w += 8)
                pos[w] = n++;
    }
    for (int64_t w = 0; w < W; ++w) {
        wgseg[w] = (int32_t)(seg.size() / 4);
        auto add = [&](int64_t v, int64_t i, int64_t j) {
            if (i >= j)
                return;
            const int32_t u = live[v];
            uint32_t left = umask[u], mask = 0;  // the i-th to (j - 1)-th orbits of the unit
            for (int64_t n = ustart[v]; n < j; ++n, left &= left - 1)
                mask |= n >= i ? left & -left : 0u;
            useg[u].push_back((int32_t)(seg.size() / 4));
            seg.insert(seg.end(), {u, (int32_t)mask, 0, 0});
        };
        for (int64_t r = 0; r < rounds; ++r) {
            const int64_t u = r * W + pos[w];
            add(u, ustart[u], ustart[u + 1]);
        }
        const int64_t ib = ustart[u0] + pos[w] * rest / W, ie = ustart[u0] + (pos[w] + 1) * rest / W;
        int64_t u = std::upper_bound(ustart.begin() + u0, ustart.end(), ib) - ustart.begin() - 1;
        for (int64_t i = ib; i < ie; ++u) {
            const int64_t j = std::min(ie, ustart[u + 1]);
            add(u, i, j);
            i = std::max(i, j);
        }
    }
    o.wgs = (int32_t)W;
    o.nseg = (int64_t)seg.size() / 4;
    o.ngroup = (int32_t)groups.size();
    o.nunit = (int32_t)nunit;
    if (W > 0)
        wgseg[W] = (int32_t)o.nseg;
    // slots: the segments of each unit in orbit order, unit by unit
    std::vector<int32_t> uslot(nunit + 1, 0);
    for (int64_t u = 0; u < nunit; ++u) {
        std::sort(useg[u].begin(), useg[u].end(), [&](int32_t a, int32_t b) { return (uint32_t)seg[4 * a + 1] < (uint32_t)seg[4 * b + 1]; });
        uslot[u + 1] = uslot[u] + (int32_t)useg[u].size();
        for (size_t j = 0; j < useg[u].size(); ++j)
            seg[4 * useg[u][j] + 2] = uslot[u] + (int32_t)j;
    }
    GRAV_CHECK(upload(p, &o.d_key, oc.key));
    GRAV_CHECK(upload(p, &o.d_child, oc.child));
    GRAV_CHECK(upload(p, &o.d_parent, oc.parent));
    GRAV_CHECK(upload(p, &o.d_groups, groups));
    GRAV_CHECK(upload(p, &o.d_segs, seg));
    GRAV_CHECK(upload(p, &o.d_wgseg, wgseg));
    GRAV_CHECK(upload(p, &o.d_uslot, uslot));
    return GRAV_OK;
}

// Octets and M2L schedules of both directions, from the target boxes' keys.
// Forward: the octets of the target boxes, fed by the source blocks.
// Transposed: the octets of all source boxes (the M2M and its transpose run
// over them too), fed by the target boxes; the octets within reach of a target
// box come first in their level, so that the M2L's groups hold few others.
static grav_status build_m2l(Plan *p)
{
    const int L = p->L;
    std::vector<std::vector<uint32_t>> key(L + 1);
    for (int l = 2; l <= L; ++l) {
        const int64_t n = p->lev[l].n_tgt;
        key[l].resize(n);
        if (n > 0)
            GRAV_HIP(hipMemcpyAsync(key[l].data(), p->d_tkey + p->tbox_off[l], 4 * n, hipMemcpyDeviceToHost, p->bs));
    }
    GRAV_HIP(hipStreamSynchronize(p->bs));
    Octets fo, to;
    std::vector<std::vector<char>> tb(L + 1);  // target boxes in a level's gather region
    p->n_grow = 0;
    for (int l = 2; l <= L; ++l) {
        LevelInfo &lv = p->lev[l];
        fo.level(l);
        int lo[3] = {INT32_MAX, INT32_MAX, INT32_MAX}, hi[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
        int blo[3] = {INT32_MAX, INT32_MAX, INT32_MAX}, bhi[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
        for (size_t i = 0; i < key[l].size(); ++i) {
            const uint32_t k = key[l][i];
            fo.add(k, (int32_t)(lv.tgt_off + (int64_t)i));
            const int c[3] = {(int)compact3(k), (int)compact3(k >> 1), (int)compact3(k >> 2)};
            bool in = true;
            for (int a = 0; a < 3; ++a) {
                lo[a] = std::min(lo[a], c[a]);
                hi[a] = std::max(hi[a], c[a]);
                in = in && c[a] >= lv.s0[a] - 3 && c[a] < lv.s0[a] + lv.ns[a] + 3;
            }
            if (!in)
                continue;
            for (int a = 0; a < 3; ++a) {
                blo[a] = std::min(blo[a], c[a]);
                bhi[a] = std::max(bhi[a], c[a]);
            }
        }
        fo.reached(l);
        fo.done(l);
        for (int64_t j = 0; j < fo.first[l + 1] - fo.first[l]; ++j)
            fo.parent.push_back(l > 2 ? (int32_t)(p->lev[l - 1].tgt_off + j) : -1);
        // boxes whose expansions the M2L can read, and the source boxes within
        // reach of a target box
        const bool any = blo[0] <= bhi[0];
        int c0[3], c1[3];
        for (int a = 0; a < 3; ++a) {
            lv.need_lo[a] = key[l].empty() ? 0 : lo[a] - 3;
            lv.need_hi[a] = key[l].empty() ? -1 : hi[a] + 3;
            c0[a] = any ? std::max(lv.s0[a], blo[a] - 3) : 1;
            c1[a] = any ? std::min(lv.s0[a] + lv.ns[a] - 1, bhi[a] + 3) : 0;
            lv.gs0[a] = any ? blo[a] : 0;
            lv.gns[a] = any ? bhi[a] - blo[a] + 1 : 0;
        }
        lv.g_off = p->n_grow;
        const int64_t gn = (int64_t)lv.gns[0] * lv.gns[1] * lv.gns[2];
        p->n_grow += gn;
        tb[l].assign((size_t)gn, 0);
        const OctLev gl{{lv.gs0[0], lv.gs0[1], lv.gs0[2]}, {lv.gns[0], lv.gns[1], lv.gns[2]}, 0};
        for (const uint32_t k : key[l]) {
            const int32_t j = octet_place(gl, (int)compact3(k), (int)compact3(k >> 1), (int)compact3(k >> 2));
            if (j >= 0)
                tb[l][j] = 1;
        }
        to.level(l);
        std::vector<uint64_t> oct;
        int p0[3], p1[3];
        for (int a = 0; a < 3; ++a) {
            p0[a] = lv.s0[a] >> 1;
            p1[a] = (lv.s0[a] + lv.ns[a] - 1) >> 1;
        }
        for (int z = p0[2]; z <= p1[2]; ++z)
            for (int y = p0[1]; y <= p1[1]; ++y)
                for (int x = p0[0]; x <= p1[0]; ++x) {
                    const int c[3] = {x, y, z};
                    uint64_t far = 0;
                    for (int a = 0; a < 3; ++a)
                        if (c[a] < c0[a] >> 1 || c[a] > c1[a] >> 1)
                            far = 1;
                    oct.push_back(far << 32 | morton3(x, y, z));
                }
        std::sort(oct.begin(), oct.end());
        const OctLev sl{{lv.s0[0], lv.s0[1], lv.s0[2]}, {lv.ns[0], lv.ns[1], lv.ns[2]}, 0};
        const size_t near = std::lower_bound(oct.begin(), oct.end(), (uint64_t)1 << 32) - oct.begin();
        // no M2L shares the others' neighbours: x fastest, so that the P2M's blocks
        // of 16 octets read and write long rows of the mesh
        std::sort(oct.begin() + near, oct.end(), [](uint64_t a, uint64_t b) {
            const uint32_t ka = (uint32_t)a, kb = (uint32_t)b;
            for (int s = 2; s >= 0; --s)
                if (compact3(ka >> s) != compact3(kb >> s))
                    return compact3(ka >> s) < compact3(kb >> s);
            return false;
        });
        for (size_t i = 0; i <= oct.size(); ++i) {
            if (i == near)
                to.reached(l);
            if (i == oct.size())
                break;
            const uint32_t k = (uint32_t)oct[i];
            const int c[3] = {2 * (int)compact3(k), 2 * (int)compact3(k >> 1), 2 * (int)compact3(k >> 2)};
            for (uint32_t r = 0; r < 8; ++r) {
                const int32_t j = octet_place(sl, c[0] + (int)(r & 1), c[1] + (int)(r >> 1 & 1), c[2] + (int)(r >> 2));
                if (j >= 0)
                    to.add(k << 3 | r, (int32_t)lv.me_off + j);
            }
        }
        to.done(l);
        for (int64_t j = to.first[l]; j < to.first[l + 1]; ++j) {
            const uint32_t k = to.key[j];
            int32_t row = -1;
            if (l > 2) {
                const LevelInfo &lp = p->lev[l - 1];
                const OctLev pl{{lp.s0[0], lp.s0[1], lp.s0[2]}, {lp.ns[0], lp.ns[1], lp.ns[2]}, 0};
                row = (int32_t)lp.me_off + octet_place(pl, (int)compact3(k), (int)compact3(k >> 1), (int)compact3(k >> 2));
            }
            to.parent.push_back(row);
        }
    }
    const OctGeom fg = octet_geom(p, false), tg = octet_geom(p, true);
    GRAV_CHECK(build_octet_schedule(p, fo, p->m2l, [&](int l, int x, int y, int z) {
        return octet_place(fg.lev[l], x, y, z) >= 0;
    }));
    return build_octet_schedule(p, to, p->m2lt, [&](int l, int x, int y, int z) {
        const int32_t j = octet_place(tg.lev[l], x, y, z);
        return j >= 0 && tb[l][j] != 0;
    });
}

__global__ void k_fill_tmap(const uint32_t *bkeys, int64_t n, int s0x, int s0y, int s0z, int mx,
                            int my, int mz, int32_t *tmap)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t k = bkeys[i];
    const int x = (int)compact3(k) - s0x + 3, y = (int)compact3(k >> 1) - s0y + 3,
              z = (int)compact3(k >> 2) - s0z + 3;
    if (x >= 0 && y >= 0 && z >= 0 && x < mx && y < my && z < mz)
        tmap[((int64_t)z * my + y) * mx + x] = (int32_t)i;
}

// Lookup tables of the adjoint: target-box maps over each level's source
// block plus a halo of 3 boxes (M2L transpose, near field transpose) and the
// first-child table of each level (L2L transpose).
// Source leaves of the leaf level with some user point in their 27
// neighbour leaves (target map entry with pend > start), appended in any
// order: the cells of the other leaves get no term from the transposed
// point near field.
__global__ void k_point_leaves(const int32_t *tmap, int64_t n_tmap, int64_t tmap_off, int nsx, int nsy, int nsz,
                               const int64_t *leaf_start, const int64_t *pend,
                               int64_t n_leaf, int32_t *list, unsigned long long *count)
{
    const int64_t sl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (sl >= (int64_t)nsx * nsy * nsz)
        return;
    const int lx = (int)(sl % nsx), ly = (int)((sl / nsx) % nsy), lz = (int)(sl / ((int64_t)nsx * nsy));
    const int mxl = nsx + 6, myl = nsy + 6, mzl = nsz + 6;
    bool active = false;
    for (int nb = 0; nb < 27 && !active; ++nb) {
        // neighbour position in the target map (source block + halo 3)
        const int mx = lx + nb % 3 - 1 + 3, my = ly + (nb / 3) % 3 - 1 + 3, mz = lz + nb / 9 - 1 + 3;
        if (mx < 0 || my < 0 || mz < 0 || mx >= mxl || my >= myl || mz >= mzl)
            continue;
        const int64_t mi = tmap_off + ((int64_t)mz * myl + my) * mxl + mx;
        if (mi >= n_tmap)
            continue;
        const int64_t tl = tmap[mi];
        if (tl >= 0 && tl < n_leaf && pend[tl] > max(leaf_start[tl], (int64_t)0))
            active = true;
    }
    if (active)
        list[atomicAdd(count, 1ull)] = (int32_t)sl;
}

// Target leaves holding user points (pend > start), appended in any order.
__global__ void k_user_leaves(const int64_t *leaf_start, const int64_t *pend, int64_t n_leaf, int32_t *list,
                              unsigned long long *count)
{
    const int64_t tl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tl < n_leaf && pend[tl] > max(leaf_start[tl], (int64_t)0))
        list[atomicAdd(count, 1ull)] = (int32_t)tl;
}

// The points of those leaves in runs of about len, multiples of `step`, in any
// order; a leaf of less than `whole` stays whole.
__global__ void k_point_runs(const int64_t *leaf_start, const int64_t *pend, const int32_t *leaves, int64_t n,
                             int64_t len, int64_t step, int64_t whole,
                             PointRun *runs, unsigned long long *count)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const int32_t leaf = leaves[i];
    const int64_t s = max(leaf_start[leaf], (int64_t)0), m = pend[leaf] - s;
    const int64_t parts = m < whole ? 1 : max(m / len, (int64_t)1), per = (m + parts * step - 1) / (parts * step) * step;
    unsigned long long at = atomicAdd(count, (unsigned long long)((m + per - 1) / per));
    for (int64_t k = 0; k < m; k += per)
        runs[at++] = PointRun{s + k, leaf, (int32_t)min(per, m - k)};
}

grav_status build_adjoint_maps(Plan *p)
{
    const int L = p->L;
    const int lo = L >= 2 ? 2 : L;
    p->n_tmap = 0;
    for (int l = lo; l <= L; ++l) {
        const LevelInfo &lv = p->lev[l];
        p->lev[l].tmap_off = p->n_tmap;
        p->n_tmap += (int64_t)(lv.ns[0] + 6) * (lv.ns[1] + 6) * (lv.ns[2] + 6);
    }
    GRAV_CHECK(dalloc(p, &p->d_tmap, (size_t)p->n_tmap, true));
    GRAV_HIP(hipMemsetAsync(p->d_tmap, 0xff, sizeof(int32_t) * p->n_tmap, p->bs));
    for (int l = lo; l <= L; ++l) {
        const LevelInfo &lv = p->lev[l];
        const int64_t n = lv.n_tgt;
        if (n == 0)
            continue;
        hipLaunchKernelGGL(k_fill_tmap, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, p->bs,
                           (const uint32_t *)(p->d_tkey + p->tbox_off[l]), n, lv.s0[0], lv.s0[1],
                           lv.s0[2], lv.ns[0] + 6, lv.ns[1] + 6, lv.ns[2] + 6,
                           p->d_tmap + lv.tmap_off);
        GRAV_HIP(hipGetLastError());
    }
    {
        // the leaf level's source leaves near user points, and the target
        // leaves holding user points
        const LevelInfo &lv = p->lev[L];
        GRAV_CHECK(dalloc(p, &p->d_pt_leaves, (size_t)std::max<int64_t>(lv.n_src, 1), true));
        GRAV_CHECK(dalloc(p, &p->d_user_leaves, (size_t)std::max<int64_t>(p->n_leaf, 1), true));
        unsigned long long *cnt = nullptr;
        GRAV_HIP(hipMalloc(&cnt, 2 * sizeof(unsigned long long)));
        grav_status st = GRAV_OK;
        unsigned long long n[2] = {0, 0};
        if (hipMemsetAsync(cnt, 0, 2 * sizeof(unsigned long long), p->bs) != hipSuccess)
            st = GRAV_EDEVICE;
        if (st == GRAV_OK && lv.n_src > 0) {
            hipLaunchKernelGGL(k_point_leaves, dim3((unsigned)ceil_div(lv.n_src, 256)), dim3(256), 0, p->bs,
                               (const int32_t *)p->d_tmap, p->n_tmap, lv.tmap_off, lv.ns[0], lv.ns[1], lv.ns[2],
                               (const int64_t *)p->d_leaf_start,
                               (const int64_t *)p->d_leaf_pend, p->n_leaf, p->d_pt_leaves, cnt);
            if (hipGetLastError() != hipSuccess)
                st = GRAV_EDEVICE;
        }
        if (st == GRAV_OK && p->n_leaf > 0) {
            hipLaunchKernelGGL(k_user_leaves, dim3((unsigned)ceil_div(p->n_leaf, 256)), dim3(256), 0, p->bs,
                               (const int64_t *)p->d_leaf_start, (const int64_t *)p->d_leaf_pend, p->n_leaf,
                               p->d_user_leaves, cnt + 1);
            if (hipGetLastError() != hipSuccess)
                st = GRAV_EDEVICE;
        }
        if (st == GRAV_OK && (hipMemcpyAsync(n, cnt, sizeof(n), hipMemcpyDeviceToHost, p->bs) != hipSuccess ||
                              hipStreamSynchronize(p->bs) != hipSuccess))
            st = GRAV_EDEVICE;
        p->n_pt_leaves = (int64_t)n[0];
        p->n_user_leaves = (int64_t)n[1];
        // runs for the L2P: steps of 64 (point, model) pairs, as many a run as
        // leave kRunBlocks workgroups, those resident with several models.
        // Leaves that a resident workgroup takes in two rounds stay whole: a few
        // cut ones more than fit the CUs at once cost a round (p = 16, 512 leaves
        // of about 100 points: 16.3 us, 24.2 with some cut)
        if (st == GRAV_OK)
            st = l2p_resident_workgroups(p, &p->l2p_wgs);
        const int64_t np = p->lat_near ? p->d.n_points : p->M, mg = std::min(p->B, 8), wgs = std::max(p->l2p_wgs, 1);
        const int64_t blocks = p->B == 1 ? kRunBlocks : wgs, least = p->B == 1 ? 1 : 2, step = 64 / mg;
        const int64_t len = std::max(ceil_div(np * p->B, 64 * blocks), least) * step;
        const int64_t whole = 2 * std::max(len, ceil_div(np * p->B, 64 * wgs) * step);
        if (st == GRAV_OK && p->n_user_leaves > 0) {
            p->n_runs = 0;
            st = dalloc(p, &p->d_runs, (size_t)(p->n_user_leaves + np / len), true);
            if (st == GRAV_OK && hipMemsetAsync(cnt, 0, sizeof(unsigned long long), p->bs) != hipSuccess)
                st = GRAV_EDEVICE;
            if (st == GRAV_OK) {
                hipLaunchKernelGGL(k_point_runs, dim3((unsigned)ceil_div(p->n_user_leaves, 256)), dim3(256), 0, p->bs,
                                   (const int64_t *)p->d_leaf_start, (const int64_t *)p->d_leaf_pend,
                                   (const int32_t *)p->d_user_leaves, p->n_user_leaves, len, step, whole, p->d_runs,
                                   cnt);
                if (hipGetLastError() != hipSuccess ||
                    hipMemcpyAsync(n, cnt, sizeof(n[0]), hipMemcpyDeviceToHost, p->bs) != hipSuccess ||
                    hipStreamSynchronize(p->bs) != hipSuccess)
                    st = GRAV_EDEVICE;
                p->n_runs = (int64_t)n[0];
            }
        }
        (void)hipFree(cnt);
        GRAV_CHECK(st);
    }
    GRAV_HIP(hipStreamSynchronize(p->bs));
    return GRAV_OK;
}

// Cell of a 4^3 leaf's 12^3 neighbourhood along one axis: base cell v of the
// positive side or its image, relative to the leaf's corner -> (neighbour
// offset, cell in that leaf).
static void near_axis(int v, bool neg, int &d, int &cell)
{
    const int x = neg ? 1 - v : 2 + v;
    d = x < 0 ? -1 : x < 4 ? 0 : 1;
    cell = x - 4 * d;
}

// Operators of the near field by parity, F_chi and F^T_chi of near.hip, from
// the dense pair terms of near_lattice.  A set holds the CK RBN values of a
// chunk per lane (frag_at), value u RBN + rb = row 16 rb + lane % 16, base
// cell 4 (CK chunk + u) + lane / 16; [parity][chunk], transposed
// [component][parity][chunk].
template <class T>
static grav_status build_near_parity(Plan *p, const std::vector<double> &dense)
{
    constexpr int b3 = 64, CK = kNearChunk, NJ = 54 / CK;
    const int C = p->C, RBN = (8 * C + 15) / 16, E = CK * RBN;
    // transposed: rows t in two groups of four (FP32 4x4x1 instructions, row
    // lane % 4), or in the first half of a block of 16
    constexpr int RT = sizeof(T) == 4 ? 2 : 1, ET = CK * RT;
    std::vector<T> op((size_t)8 * NJ * E * 64, (T)0), opt((size_t)C * 8 * NJ * ET * 64, (T)0);
    for (int s = 0; s < 216; ++s) {
        const int sb[3] = {s % 6, s / 6 % 6, s / 36};
        // per reflection: neighbour index and cell of the base cell's image
        int nb[8], nbt[8], cell[8];
        for (int r = 0; r < 8; ++r) {
            int d[3], c[3];
            for (int a = 0; a < 3; ++a)
                near_axis(sb[a], r >> a & 1, d[a], c[a]);
            nb[r] = (d[0] + 1) + 3 * (d[1] + 1) + 9 * (d[2] + 1);
            nbt[r] = (1 - d[0]) + 3 * (1 - d[1]) + 9 * (1 - d[2]);
            cell[r] = c[0] + 4 * c[1] + 16 * c[2];
        }
        const int ks = s / 4, lane4 = 16 * (s % 4), j = ks / CK, u = ks % CK;
        for (int c = 0; c < C; ++c) {
            const int comp = c + 4 - C;  // of (phi, gx, gy, gz)
            const int cls = comp == 0 ? 0 : 1 << (comp - 1);
            for (int t = 0; t < 8; ++t) {
                const int tc = (2 + (t & 1)) + 4 * (2 + (t >> 1 & 1)) + 16 * (2 + (t >> 2));
                for (int x = 0; x < 8; ++x) {
                    double f = 0.0, ft = 0.0;
                    for (int r = 0; r < 8; ++r) {
                        const double v = dense[((size_t)nb[r] * 4 * b3 + 4 * tc + comp) * b3 + cell[r]];
                        const double w = dense[((size_t)nbt[r] * 4 * b3 + 4 * cell[r] + comp) * b3 + tc];
                        f += odd_parity(x & r) ? -v : v;
                        ft += odd_parity((x ^ cls) & r) ? -w : w;
                    }
                    const int R = 8 * c + t;
                    op[((size_t)x * NJ + j) * E * 64 + frag_at<T>(E, lane4 + R % 16, u * RBN + R / 16)] = (T)(f / 8);
                    T *set = &opt[(((size_t)c * 8 + x) * NJ + j) * ET * 64];
                    if (RT == 1)
                        set[frag_at<T>(ET, lane4 + t, u)] = (T)(ft / 8);
                    else
                        for (int i = 0; i < 16; i += 4)
                            set[frag_at<T>(ET, lane4 + i + t % 4, u * RT + t / 4)] = (T)(ft / 8);
                }
            }
        }
    }
    T *d = nullptr;
    GRAV_CHECK(upload(p, &d, op));
    p->d_near_op = d;
    GRAV_CHECK(upload(p, &d, opt));
    p->d_near_opt = d;
    return GRAV_OK;
}

// The far field at the base centres by coefficient class: [parity][k step][row
// block][lane], coefficient 4 q + lane / 16 of the class (coef; past its end
// coefficient 0 with a zero operator).
static grav_status build_near_far(Plan *p, const std::vector<double> &full)
{
    const int C = p->C, RBN = (8 * C + 15) / 16, PS = p->PS;
    const bool f64 = p->d.precision == GRAV_FP64;
    std::vector<int> cls[8];
    for (int k = 0; k < p->P2; ++k)
        cls[sign_class(k)].push_back(k);
    int KC = 0;
    for (const auto &c : cls)
        KC = std::max(KC, (int)ceil_div((int64_t)c.size(), 4));
    p->near_KC = KC;
    std::vector<int32_t> coef((size_t)8 * KC * 4, 0);
    std::vector<double> lm((size_t)8 * KC * RBN * 64, 0.0);
    for (int x = 0; x < 8; ++x)
        for (size_t n = 0; n < cls[x].size(); ++n) {
            const int k = cls[x][n], q = (int)n / 4, kr = (int)n % 4;
            coef[((size_t)x * KC + q) * 4 + kr] = k;
            for (int a = 0; a < 16 * RBN; ++a) {
                // next to FP32 sums, row i holds row 4 (i % 4) + i / 4
                const int i = a % 16, R = 16 * (a / 16) + (f64 ? i : 4 * (i % 4) + i / 4);
                if (R >= 8 * C)
                    continue;
                const int t = R % 8, comp = R / 8 + 4 - C;
                const int tc = (2 + (t & 1)) + 4 * (2 + (t >> 1 & 1)) + 16 * (2 + (t >> 2));
                lm[((size_t)(x * KC + q) * RBN + a / 16) * 64 + 16 * kr + i] = full[(size_t)(4 * tc + comp) * PS + k];
            }
        }
    GRAV_CHECK(upload(p, &p->d_near_coef, coef));
    GRAV_CHECK(upload(p, &p->d_near_far, lm));
    // its transpose: [parity][k step][row block of the class][lane], row =
    // coefficient 16 rb + lane % 16 of the class, column R = 4 ks + lane / 16
    const int RBC = (int)ceil_div((int64_t)KC * 4, 16);
    std::vector<double> lt((size_t)8 * 2 * C * RBC * 64, 0.0);
    for (int x = 0; x < 8; ++x)
        for (size_t n = 0; n < cls[x].size(); ++n)
            for (int R = 0; R < 8 * C; ++R) {
                const int t = R % 8, comp = R / 8 + 4 - C;
                const int tc = (2 + (t & 1)) + 4 * (2 + (t >> 1 & 1)) + 16 * (2 + (t >> 2));
                lt[((size_t)(x * 2 * C + R / 4) * RBC + n / 16) * 64 + 16 * (R % 4) + n % 16] =
                    full[(size_t)(4 * tc + comp) * PS + cls[x][n]];
            }
    return upload(p, &p->d_near_fart, lt);
}

// Near field of voxel-centre targets as 27 dense lattice matrices (leaf
// edges b <= 4), the slot of every voxel centre in sorted order, and the end
// of the user points of every leaf (the direct near-field kernel visits only
// those).
grav_status build_near_lattice(Plan *p, hipStream_t s)
{
    const int64_t M = p->M, npts = p->d.n_points;
    // the lattice near field pairs lattice targets with lattice sources
    p->lat_near = p->d.voxel_centres && p->b <= kMaxLatticeLeaf && p->n_spts == 0;
    GRAV_CHECK(dalloc(p, &p->d_leaf_pend, p->n_leaf, true));
    hipLaunchKernelGGL(k_leaf_point_end, dim3((unsigned)ceil_div(p->n_leaf, 256)), dim3(256), 0, s,
                       (const uint32_t *)p->d_perm, (const int64_t *)p->d_leaf_start, p->n_leaf,
                       p->lat_near ? npts : M, p->d_leaf_pend);
    GRAV_HIP(hipGetLastError());
    if (!p->lat_near) {
        GRAV_HIP(hipStreamSynchronize(s));
        return GRAV_OK;
    }
    const int64_t ncell = (int64_t)p->d.nx * p->d.ny * p->d.nz;
    GRAV_CHECK(dalloc(p, &p->d_cell_slot, ncell, true));
    hipLaunchKernelGGL(k_cell_slot, dim3((unsigned)ceil_div(M, 256)), dim3(256), 0, s,
                       (const uint32_t *)p->d_perm, M, npts, p->d_cell_slot);
    GRAV_HIP(hipGetLastError());

    const int b = p->b, b3 = b * b * b;
    // rows: (output component, target) pairs for the requested components
    // only, component-major: each component owns RBc = b^3/16 (rounded up)
    // blocks of 16 targets, RBn = C RBc blocks in all; the contraction runs
    // over Qn chunks of four k steps, k step ks and instruction sub-row kr
    // taking cell kr * 4 Qn + ks (cells past b^3 are zero in both operands)
    const int C = p->d.components, RBc = (int)ceil_div(b3, 16);
    const int RBn = C * RBc, Qn = (int)ceil_div(ceil_div(b3, 4), 4);
    const int KP = 16 * Qn;
    p->lat_RB = RBn;
    p->lat_Q = Qn;
    const bool f64 = p->d.precision == GRAV_FP64;
    std::vector<double> dense((size_t)27 * 4 * b3 * b3);
    near_lattice(b, p->q, f64 ? 1e-20 : 1e-10, dense.data());
    const int TQ = (int)ceil_div(b3, 4), RBt = (int)ceil_div(b3, 16);
    p->lat_TQ = TQ;
    {
        // by parity unless its blocks of 4 x 2 x 2 leaves stay mostly empty
        // (GRAV_NEAR_DENSE_BLOCKS)
        const LevelInfo &lv = p->lev[p->L];
        const int64_t blocks = ceil_div(lv.ns[0], 4) * ceil_div(lv.ns[1], 2) * ceil_div(lv.ns[2], 2);
        p->near_par = b == 4 && (lv.n_src > 4 * blocks ||
                                 blocks * blocks * p->B <= (int64_t)GRAV_NEAR_DENSE_BLOCKS * std::max(lv.n_src, 2 * blocks));
    }
    if (p->near_par)
        GRAV_CHECK(f64 ? build_near_parity<double>(p, dense) : build_near_parity<float>(p, dense));
    auto row_target = [C, RBc](int row, int rb, bool swap, int &t, int &comp) {
        t = 16 * (rb % RBc) + (swap ? 4 * (row % 4) + row / 4 : row);
        comp = rb / RBc + 4 - C;
    };
    if (!p->near_par) {
        // Row r of block rb is target 16 (rb % RBc) + r of output component
        // rb / RBc; the lattice matrices hold (phi, gx, gy, gz), of which
        // components 1 and 3 take the trailing one or three.  The FP32
        // instruction returns rows 4 (lane / 16) + k of a block and the FP64 one
        // rows lane / 16 + 4 k, so a lane's accumulator holds four targets of one
        // component.  The far field (FP64) is added element by element to the
        // near field's accumulator, so next to an FP32 near field its rows take
        // the FP32 order (swap: row 4 i + j holds target 4 j + i).  Layout
        // [nb][q][rb][lane][u], ks = 4 q + u.
        std::vector<double> sw((size_t)27 * Qn * RBn * 64 * 4, 0.0);
        for (int nb = 0; nb < 27; ++nb)
            for (int q = 0; q < Qn; ++q)
                for (int rb = 0; rb < RBn; ++rb)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int u = 0; u < 4; ++u) {
                            int t, comp;
                            row_target(lane & 15, rb, false, t, comp);
                            const int cell = (lane >> 4) * 4 * Qn + 4 * q + u;
                            double v = 0.0;
                            if (t < b3 && cell < b3)
                                v = dense[((size_t)nb * 4 * b3 + 4 * t + comp) * b3 + cell];
                            sw[(((size_t)nb * Qn + q) * RBn + rb) * 256 + frag_pos(lane, u, f64 ? 2 : 4)] = v;
                        }
        {
            // leaf blocks of the densities, padded by one leaf per side; the
            // padding and the rows past b^3 stay zero
            const LevelInfo &lv = p->lev[p->L];
            const size_t n = (size_t)(lv.ns[0] + 2) * (lv.ns[1] + 2) * (lv.ns[2] + 2) * p->B * KP;
            GRAV_CHECK(dalloc(p, &p->d_rho_blk, n, false));
            GRAV_HIP(hipMemsetAsync(p->d_rho_blk, 0, sizeof(double) * n, p->bs));
            GRAV_HIP(hipStreamSynchronize(p->bs));
            // per near chunk i = (neighbour nb, four k steps q): element offsets
            // of its density fragment (from a column's block at nb = (0, 0, 0))
            // and of its operator fragments; the kernel reads them with scalar
            // loads instead of recomputing them
            const int64_t px = lv.ns[0] + 2, py = lv.ns[1] + 2, nplB = px * py * (lv.ns[2] + 2) * p->B;
            std::vector<int64_t> tab((size_t)27 * Qn * 2);
            for (int nb = 0; nb < 27; ++nb)
                for (int q = 0; q < Qn; ++q) {
                    const int64_t nboff = ((int64_t)(nb / 9) * py + (nb / 3) % 3) * px + nb % 3;
                    tab[((size_t)nb * Qn + q) * 2 + 0] = ((int64_t)q * 4 * nplB + nboff * p->B) * 4;
                    tab[((size_t)nb * Qn + q) * 2 + 1] = ((int64_t)nb * Qn + q) * RBn * 256;
                }
            GRAV_CHECK(upload(p, &p->d_lat_tab, tab));
        }
        if (f64) {
            GRAV_CHECK(upload(p, &p->d_tn64, sw));
        } else {
            std::vector<float> sw32(sw.begin(), sw.end());
            GRAV_CHECK(upload(p, &p->d_tn32, sw32));
        }
        // the adjoint's transposes: rows = the cells of the source leaf (RBt
        // blocks of 16), contraction over (target t, component) of the target
        // leaf (near^T: the C output components; L2P^T: chunk q and k step u
        // taking t = (lane/16) TQ + q, component u); [nb][q][rb][lane][u]
        // group-major sets
        {
            // the weights of the cell centres in leaf blocks (padded by one leaf
            // per side, 4 TQ x 4 values per leaf and model, in the near field's
            // element type); the padding and the slots past b^3 stay zero
            const LevelInfo &lv = p->lev[p->L];
            const size_t n = (size_t)(lv.ns[0] + 2) * (lv.ns[1] + 2) * (lv.ns[2] + 2) * p->B * 16 * TQ;
            const size_t nd = f64 ? n : (n + 1) / 2;  // in doubles
            GRAV_CHECK(dalloc(p, &p->d_w_blk, nd, false));
            GRAV_HIP(hipMemsetAsync(p->d_w_blk, 0, sizeof(double) * nd, p->bs));
            GRAV_HIP(hipStreamSynchronize(p->bs));
        }
        {
            // contraction over the C b^3 (centre, output component) pairs of the
            // target leaf: value e = C t + c in chunk q, sub-row kr, k step u
            // with e = 4 KQ kr + 4 q + u (the weight blocks' order)
            const int KQ = (int)ceil_div((int64_t)C * b3, 16);
            std::vector<double> swt((size_t)27 * KQ * RBt * 256, 0.0);
            for (int nb = 0; nb < 27; ++nb)
                for (int q = 0; q < KQ; ++q)
                    for (int rb = 0; rb < RBt; ++rb)
                        for (int lane = 0; lane < 64; ++lane)
                            for (int u = 0; u < 4; ++u) {
                                const int e = 4 * KQ * (lane >> 4) + 4 * q + u, cell = 16 * rb + (lane & 15);
                                const int t = e / C, comp = e % C + 4 - C;
                                const double v =
                                    t < b3 && cell < b3 ? dense[((size_t)nb * 4 * b3 + 4 * t + comp) * b3 + cell] : 0.0;
                                swt[(((size_t)nb * KQ + q) * RBt + rb) * 256 + frag_pos(lane, u, f64 ? 2 : 4)] = v;
                            }
            if (f64) {
                GRAV_CHECK(upload(p, &p->d_tnt64, swt));
            } else {
                std::vector<float> swt32(swt.begin(), swt.end());
                GRAV_CHECK(upload(p, &p->d_tnt32, swt32));
            }
        }
    }
    if (p->L >= 2) {
        // Far field at the cell centres from the leaf's local expansion, with
        // the scaling of the combine folded in (phi / w, -grad phi / w^2), as
        // FP64 MFMA A fragments over the expansion's PS/4 k steps (same
        // contraction order as the M2L: coefficient kr * PS/4 + ks).
        const int PS = p->PS, QL = PS / 16;
        std::vector<double> e(PS, 0.0), full((size_t)4 * b3 * PS, 0.0);
        const double inv_w = 1.0 / b;
        for (int t = 0; t < b3; ++t) {
            const double u[3] = {((t % b) + 0.5 - 0.5 * b) * inv_w, (((t / b) % b) + 0.5 - 0.5 * b) * inv_w,
                                 ((t / (b * b)) + 0.5 - 0.5 * b) * inv_w};
            for (int c = 0; c < p->P2; ++c) {
                e[c] = 1.0;
                double o[4];
                l2p_eval(p->P, e.data(), u[0], u[1], u[2], o);
                e[c] = 0.0;
                full[(size_t)(4 * t + 0) * PS + c] = o[0] * inv_w;
                for (int a = 0; a < 3; ++a)
                    full[(size_t)(4 * t + 1 + a) * PS + c] = -o[1 + a] * inv_w * inv_w;
            }
        }
        if (p->near_par)
            GRAV_CHECK(build_near_far(p, full));
        else {
            std::vector<double> lsw((size_t)QL * RBn * 64 * 4, 0.0);
            for (int q = 0; q < QL; ++q)
                for (int rb = 0; rb < RBn; ++rb)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int u = 0; u < 4; ++u) {
                            int t, comp;
                            row_target(lane & 15, rb, !f64, t, comp);
                            const int c = (lane >> 4) * (PS / 4) + 4 * q + u;
                            lsw[((size_t)q * RBn + rb) * 256 + frag_pos(lane, u, 2)] =
                                t < b3 ? full[(size_t)(4 * t + comp) * PS + c] : 0.0;
                        }
            GRAV_CHECK(upload(p, &p->d_tl2p, lsw));
            // its transpose for the adjoint: rows = coefficients (QL blocks),
            // contraction over (t, component) as the transposed near field
            std::vector<double> lst((size_t)TQ * QL * 256, 0.0);
            for (int q = 0; q < TQ; ++q)
                for (int rb = 0; rb < QL; ++rb)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int u = 0; u < 4; ++u) {
                            const int t = (lane >> 4) * TQ + q, c = 16 * rb + (lane & 15);
                            lst[((size_t)q * QL + rb) * 256 + frag_pos(lane, u, 2)] =
                                t < b3 ? full[(size_t)(4 * t + u) * PS + c] : 0.0;
                        }
            GRAV_CHECK(upload(p, &p->d_tl2pt, lst));
        }
    }
    GRAV_HIP(hipStreamSynchronize(s));
    return GRAV_OK;
}

grav_status count_work(Plan *p)
{
    unsigned long long *acc = nullptr;
    GRAV_HIP(hipMalloc(&acc, 2 * sizeof(unsigned long long)));
    grav_status st = GRAV_OK;
    do {
        if (hipMemsetAsync(acc, 0, 2 * sizeof(unsigned long long), p->bs) != hipSuccess) {
            st = GRAV_EDEVICE;
            break;
        }
        CountArgs a{};
        for (int ax = 0; ax < 3; ++ax) {
            a.shift[ax] = p->shift[ax];
        }
        a.n[0] = p->d.nx;
        a.n[1] = p->d.ny;
        a.n[2] = p->d.nz;
        a.b = p->b;
        a.nq3 = p->nq3;
        if (p->L >= 2 && p->d_class_off)
            for (int l = 2; l <= p->L; ++l) {
                const int64_t n = p->lev[l].n_tgt;
                if (n == 0)
                    continue;
                for (int ax = 0; ax < 3; ++ax) {
                    a.s0[ax] = p->lev[l].s0[ax];
                    a.ns[ax] = p->lev[l].ns[ax];
                }
                hipLaunchKernelGGL(k_count_m2l, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, p->bs,
                                   (const uint32_t *)(p->d_tkey + p->tbox_off[l]), n, a,
                                   (const int32_t *)p->d_class_off, acc);
            }
        if (p->n_leaf > 0) {
            for (int ax = 0; ax < 3; ++ax) {
                a.s0[ax] = p->lev[p->L].s0[ax];
                a.ns[ax] = p->lev[p->L].ns[ax];
            }
            if (p->n_spts > 0)
                hipLaunchKernelGGL(k_count_p2p_src, dim3((unsigned)ceil_div(p->n_leaf, 256)), dim3(256), 0, p->bs,
                                   (const uint32_t *)(p->d_tkey + p->tbox_off[p->L]),
                                   (const int64_t *)p->d_leaf_start, p->n_leaf, a, (const int64_t *)p->d_sstart,
                                   acc + 1);
            else
                hipLaunchKernelGGL(k_count_p2p, dim3((unsigned)ceil_div(p->n_leaf, 256)), dim3(256), 0, p->bs,
                                   (const uint32_t *)(p->d_tkey + p->tbox_off[p->L]),
                                   (const int64_t *)p->d_leaf_start, p->n_leaf, a, acc + 1);
        }
        unsigned long long h[2] = {0, 0};
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(h, acc, sizeof(h), hipMemcpyDeviceToHost, p->bs) != hipSuccess ||
            hipStreamSynchronize(p->bs) != hipSuccess) {
            st = GRAV_EDEVICE;
            break;
        }
        p->m2l_pairs = (int64_t)h[0];
        p->p2p_pairs = (int64_t)h[1];
    } while (0);
    (void)hipFree(acc);
    return st;
}

// Explicit sources: the dense index of each source's leaf in the leaf
// level's source block (the block starts at the mesh origin, so a source at
// lattice position u lies in leaf floor(u / b)), the sort key.
__global__ void k_source_keys(const double *src, int64_t n, double ox, double oy, double oz, double inv_h, int b,
                              int nsx, int nsy, int nsz, uint32_t *keys, uint32_t *vals)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const double o[3] = {ox, oy, oz};
    const int ns[3] = {nsx, nsy, nsz};
    int c[3];
    for (int a = 0; a < 3; ++a) {
        const double u = (src[3 * i + a] - o[a]) * inv_h;
        c[a] = min(max((int)floor(u / b), 0), ns[a] - 1);
    }
    keys[i] = (uint32_t)(((int64_t)c[2] * nsy + c[1]) * nsx + c[0]);
    vals[i] = (uint32_t)i;
}

// Sorted sources: lattice-frame positions and the mass per unit input value.
__global__ void k_gather_sources(const double *src, const double *vol, int64_t n, double ox, double oy, double oz,
                                 double inv_h, const uint32_t *perm, double *pos, double *w)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const int64_t u = perm[i];
    const double o[3] = {ox, oy, oz};
    for (int a = 0; a < 3; ++a)
        pos[3 * i + a] = (src[3 * u + a] - o[a]) * inv_h;
    const double ih3 = inv_h * inv_h * inv_h;
    w[i] = (vol ? vol[u] : 1.0) * ih3;
}

// CSR of the sorted sources over the leaves: sorted source i starts every
// leaf in (key[i-1], key[i]]; the last one also ends the leaves after it.
__global__ void k_source_leaf_start(const uint32_t *keys, int64_t n, int64_t nleaf, int64_t *start)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n)
        return;
    const int64_t lo = i == 0 ? 0 : (int64_t)keys[i - 1] + 1;
    const int64_t hi = i == n ? nleaf : (int64_t)keys[i];
    for (int64_t l = lo; l <= hi && l <= nleaf; ++l)
        start[l] = i;
}

// Explicit sources: sorted by leaf with the device radix sort, positions and
// masses gathered, the per-leaf CSR built.
grav_status build_sources(Plan *p, const grav_plan_desc *desc, hipStream_t s)
{
    const int64_t n = p->n_spts;
    const LevelInfo &lv = p->lev[p->L];
    const int64_t nleaf = lv.n_src;
    int bits = 1;
    while ((int64_t(1) << bits) < nleaf)
        ++bits;
    double *src = nullptr, *vol = nullptr;
    uint32_t *keys = nullptr, *vals = nullptr, *ktmp = nullptr, *vtmp = nullptr, *scr = nullptr;
    const size_t scr_words = radix_scratch_words(n);
    grav_status st = GRAV_OK;
    auto cleanup = [&]() {
        void *bufs[] = {src, vol, keys, vals, ktmp, vtmp, scr};
        for (void *b : bufs)
            if (b)
                (void)hipFree(b);
    };
    if (hipMalloc(&src, sizeof(double) * 3 * n) != hipSuccess ||
        (desc->source_volumes && hipMalloc(&vol, sizeof(double) * n) != hipSuccess) ||
        hipMalloc(&keys, 4 * n) != hipSuccess || hipMalloc(&vals, 4 * n) != hipSuccess ||
        hipMalloc(&ktmp, 4 * n) != hipSuccess || hipMalloc(&vtmp, 4 * n) != hipSuccess ||
        hipMalloc(&scr, 4 * std::max<size_t>(scr_words, 1)) != hipSuccess) {
        cleanup();
        return GRAV_ENOMEM;
    }
    do {
        if ((st = dalloc(p, &p->d_spos, 3 * n, true)) != GRAV_OK || (st = dalloc(p, &p->d_sw, n, true)) != GRAV_OK ||
            (st = dalloc(p, &p->d_sperm, n, true)) != GRAV_OK ||
            (st = dalloc(p, &p->d_smass, n * p->B, false)) != GRAV_OK ||
            (st = dalloc(p, &p->d_sstart, nleaf + 1, true)) != GRAV_OK)
            break;
        if (hipMemcpyAsync(src, desc->sources, sizeof(double) * 3 * n, hipMemcpyHostToDevice, s) != hipSuccess ||
            (vol && hipMemcpyAsync(vol, desc->source_volumes, sizeof(double) * n, hipMemcpyHostToDevice, s) !=
                        hipSuccess)) {
            st = GRAV_EDEVICE;
            break;
        }
        const dim3 g((unsigned)ceil_div(n, 256)), g1((unsigned)ceil_div(n + 1, 256));
        const double inv_h = 1.0 / desc->h;
        hipLaunchKernelGGL(k_source_keys, g, dim3(256), 0, s, (const double *)src, n, desc->origin[0],
                           desc->origin[1], desc->origin[2], inv_h, p->b, lv.ns[0], lv.ns[1], lv.ns[2], keys, vals);
        if (hipGetLastError() != hipSuccess || radix_sort_pairs(keys, vals, ktmp, vtmp, n, bits, scr, s) != GRAV_OK) {
            st = GRAV_EDEVICE;
            break;
        }
        hipLaunchKernelGGL(k_gather_sources, g, dim3(256), 0, s, (const double *)src, (const double *)vol, n,
                           desc->origin[0], desc->origin[1], desc->origin[2], inv_h, (const uint32_t *)vals,
                           p->d_spos, p->d_sw);
        hipLaunchKernelGGL(k_source_leaf_start, g1, dim3(256), 0, s, (const uint32_t *)keys, n, nleaf, p->d_sstart);
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(p->d_sperm, vals, 4 * n, hipMemcpyDeviceToDevice, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            st = GRAV_EDEVICE;
            break;
        }
    } while (0);
    cleanup();
    return st;
}

grav_status build_tree(Plan *p, hipStream_t s)
{
    const grav_plan_desc &d = p->d;
    const int64_t M = p->M;
    const int T = 256;
    // temporaries (freed at the end)
    uint32_t *keys = nullptr, *vals = nullptr, *ktmp = nullptr, *vtmp = nullptr;
    uint32_t *flags = nullptr, *scan = nullptr, *scr = nullptr;
    const int64_t nmax = std::max<int64_t>(M, 1);
    const size_t scr_words = std::max(radix_scratch_words(nmax), scan_tmp_words(nmax));
    grav_status st = GRAV_OK;
    auto fail = [&](grav_status e) {
        st = e;
        return e;
    };
    auto cleanup = [&]() {
        uint32_t *bufs[] = {keys, vals, ktmp, vtmp, flags, scan, scr};
        for (auto *b : bufs)
            if (b)
                (void)hipFree(b);
    };
    if (hipMalloc(&keys, 4 * nmax) != hipSuccess || hipMalloc(&vals, 4 * nmax) != hipSuccess ||
        hipMalloc(&ktmp, 4 * nmax) != hipSuccess || hipMalloc(&vtmp, 4 * nmax) != hipSuccess ||
        hipMalloc(&flags, 4 * nmax) != hipSuccess || hipMalloc(&scan, 4 * nmax) != hipSuccess ||
        hipMalloc(&scr, 4 * scr_words) != hipSuccess) {
        cleanup();
        return GRAV_ENOMEM;
    }

    KeyArgs ka{};
    ka.pts = p->d_points;
    ka.npts = d.n_points;
    ka.M = M;
    ka.nx = d.nx;
    ka.ny = d.ny;
    for (int a = 0; a < 3; ++a) {
        ka.org[a] = d.origin[a];
        ka.shift_lat[a] = (double)p->shift[a] * p->b;
    }
    ka.inv_h = 1.0 / d.h;
    ka.inv_b = 1.0 / p->b;
    ka.kmax = (1 << p->L) - 1;
    ka.L = p->L;

    do {
        if (dalloc(p, &p->d_perm, M, true) || dalloc(p, &p->d_tpos, 3 * M, true)) {
            fail(GRAV_ENOMEM);
            break;
        }
        const unsigned gM = (unsigned)ceil_div(M, T);
        hipLaunchKernelGGL(k_target_keys, dim3(gM), dim3(T), 0, s, ka, keys, vals);
        if (hipGetLastError() != hipSuccess) {
            fail(GRAV_EDEVICE);
            break;
        }
        if (radix_sort_pairs(keys, vals, ktmp, vtmp, M, 3 * p->L, scr, s) != GRAV_OK) {
            fail(GRAV_EDEVICE);
            break;
        }
        if (hipMemcpyAsync(p->d_perm, vals, 4 * M, hipMemcpyDeviceToDevice, s) != hipSuccess) {
            fail(GRAV_EDEVICE);
            break;
        }
        hipLaunchKernelGGL(k_gather_targets, dim3(gM), dim3(T), 0, s, ka,
                           (const uint32_t *)p->d_perm, p->d_tpos);
        // leaf level
        hipLaunchKernelGGL(k_head_flags, dim3(gM), dim3(T), 0, s, (const uint32_t *)keys, M, 0,
                           flags);
        if (scan_exclusive_u32(flags, scan, M, scr, s) != GRAV_OK) {
            fail(GRAV_EDEVICE);
            break;
        }
        uint32_t last[2] = {0, 0};
        if (hipMemcpyAsync(&last[0], scan + (M - 1), 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipMemcpyAsync(&last[1], flags + (M - 1), 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            fail(GRAV_EDEVICE);
            break;
        }
        p->n_leaf = (int64_t)last[0] + last[1];

        // Per-level target box counts: leaf level from the scan, parents by
        // repeated compaction.  Box keys of all levels go into one array.
        const int L = p->L;
        const int lo = L >= 2 ? 2 : L;
        // first pass: compute counts (needs the compaction of each level)
        std::vector<int64_t> cnt(L + 1, 0);
        cnt[L] = p->n_leaf;
        // allocate the per-level arrays with an upper bound n_leaf per level
        int64_t total = 0;
        for (int l = lo; l <= L; ++l)
            total += p->n_leaf;
        uint32_t *bk = nullptr;
        if (hipMalloc(&bk, 4 * std::max<int64_t>(total, 1)) != hipSuccess) {
            fail(GRAV_ENOMEM);
            break;
        }
        // level L at slot 0 of the bound layout
        std::vector<int64_t> off_bound(L + 1, 0);
        {
            int64_t o = 0;
            for (int l = L; l >= lo; --l) {
                off_bound[l] = o;
                o += p->n_leaf;
            }
        }
        if (dalloc(p, &p->d_leaf_start, p->n_leaf + 1, true)) {
            (void)hipFree(bk);
            fail(GRAV_ENOMEM);
            break;
        }
        hipLaunchKernelGGL(k_leaf_build, dim3(gM), dim3(T), 0, s, (const uint32_t *)keys,
                           (const uint32_t *)flags, (const uint32_t *)scan, M,
                           p->d_leaf_start, bk + off_bound[L]);
        hipLaunchKernelGGL(k_fill_last, dim3(1), dim3(1), 0, s, p->d_leaf_start, p->n_leaf, M);
        bool ok = true;
        for (int l = L - 1; l >= lo; --l) {
            const int64_t nc = cnt[l + 1];
            const unsigned g = (unsigned)ceil_div(nc, T);
            hipLaunchKernelGGL(k_head_flags, dim3(g), dim3(T), 0, s,
                               (const uint32_t *)(bk + off_bound[l + 1]), nc, 3, flags);
            if (scan_exclusive_u32(flags, scan, nc, scr, s) != GRAV_OK) {
                ok = false;
                break;
            }
            hipLaunchKernelGGL(k_parent_build, dim3(g), dim3(T), 0, s,
                               (const uint32_t *)(bk + off_bound[l + 1]), (const uint32_t *)flags,
                               (const uint32_t *)scan, nc, bk + off_bound[l]);
            if (hipMemcpyAsync(&last[0], scan + (nc - 1), 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipMemcpyAsync(&last[1], flags + (nc - 1), 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess) {
                ok = false;
                break;
            }
            cnt[l] = (int64_t)last[0] + last[1];
        }
        if (!ok) {
            (void)hipFree(bk);
            fail(GRAV_EDEVICE);
            break;
        }
        // compact layout: levels lo..L in increasing order
        int64_t o = 0;
        for (int l = 0; l <= kMaxLevels; ++l)
            p->tbox_off[l] = 0;
        for (int l = lo; l <= L; ++l) {
            p->tbox_off[l] = o;
            p->lev[l].n_tgt = cnt[l];
            o += cnt[l];
        }
        const int64_t nall = std::max<int64_t>(o, 1);
        if (dalloc(p, &p->d_tkey, nall, true)) {
            (void)hipFree(bk);
            fail(GRAV_ENOMEM);
            break;
        }
        for (int l = lo; l <= L; ++l) {
            if (hipMemcpyAsync(p->d_tkey + p->tbox_off[l], bk + off_bound[l], 4 * cnt[l],
                               hipMemcpyDeviceToDevice, s) != hipSuccess)
                ok = false;
        }
        if (hipStreamSynchronize(s) != hipSuccess)
            ok = false;
        (void)hipFree(bk);
        if (!ok) {
            fail(GRAV_EDEVICE);
            break;
        }
        p->n_tbox = 0;
        if (L >= 2)
            for (int l = 2; l <= L; ++l) {
                p->lev[l].tgt_off = p->n_tbox;
                p->n_tbox += cnt[l];
            }

    } while (0);
    cleanup();
    return st;
}

}  // namespace

}  // namespace grav

using namespace grav;

extern "C" void grav_desc_init(grav_plan_desc *d)
{
    if (!d)
        return;
    std::memset(d, 0, sizeof(*d));
    d->nx = d->ny = d->nz = 1;
    d->h = 1.0;
    d->quad_order = 1;
    d->components = 3;
    d->p = 8;
    d->leaf_size = 64;
    d->precision = GRAV_FP64;
    d->batch = 1;
    d->G = 1.0;
    d->device = 0;
}

extern "C" grav_status grav_plan(const grav_plan_desc *desc, grav_plan_t *out)
{
    if (!out)
        return GRAV_EINVAL;
    *out = nullptr;
    GRAV_CHECK(validate(desc));
    Plan *p = new (std::nothrow) Plan();
    if (!p)
        return GRAV_ENOMEM;
    p->d = *desc;
    p->d.points = nullptr;
    p->d.sources = nullptr;
    p->d.source_volumes = nullptr;
    p->n_spts = desc->n_sources;
    p->device = desc->device;
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess || hipSetDevice(desc->device) != hipSuccess) {
        delete p;
        return GRAV_EDEVICE;
    }
    grav_status st = GRAV_OK;
    hipStream_t s = nullptr;
    do {
        p->P = desc->p;
        p->P2 = p->P * p->P;
        p->PS = (int)ceil_div(p->P2, 16) * 16;
        p->q = desc->quad_order;
        p->nq3 = p->q * p->q * p->q;
        p->B = desc->batch;
        p->C = desc->components;
        int b = (int)std::floor(std::cbrt((double)desc->leaf_size / p->nq3) + 1e-9);
        p->b = std::min(kMaxLeafCells, std::max(1, b));
        const int n3[3] = {desc->nx, desc->ny, desc->nz};
        const int64_t ncell = (int64_t)desc->nx * desc->ny * desc->nz;
        p->M = desc->n_points + (desc->voxel_centres ? ncell : 0);
        // bounding box of evaluation points in the lattice frame (cell
        // centres span [1/2, n - 1/2]; the mesh itself is covered separately)
        double tmin[3] = {0.5, 0.5, 0.5};
        double tmax[3] = {n3[0] - 0.5, n3[1] - 0.5, n3[2] - 0.5};
        if (!desc->voxel_centres && desc->n_points > 0)
            for (int a = 0; a < 3; ++a) {
                tmin[a] = (desc->points[a] - desc->origin[a]) / desc->h;
                tmax[a] = tmin[a];
            }
        for (int64_t i = 0; i < desc->n_points; ++i)
            for (int a = 0; a < 3; ++a) {
                const double u = (desc->points[3 * i + a] - desc->origin[a]) / desc->h;
                if (!std::isfinite(u)) {
                    st = GRAV_EINVAL;
                    break;
                }
                tmin[a] = std::min(tmin[a], u);
                tmax[a] = std::max(tmax[a], u);
            }
        if (st != GRAV_OK)
            break;
        int64_t need = 1;
        for (int a = 0; a < 3; ++a) {
            const double sh = std::ceil(-tmin[a] / p->b - 1e-12);
            p->shift[a] = (int)std::max(0.0, sh);
            const int64_t src_hi = ceil_div(n3[a], p->b) + p->shift[a];
            const int64_t tgt_hi = (int64_t)std::floor((tmax[a] + (double)p->shift[a] * p->b) / p->b) + 1;
            need = std::max(need, std::max(src_hi, tgt_hi));
        }
        int L = 0;
        while ((int64_t(1) << L) < need)
            ++L;
        if (L > kMaxLevels) {
            st = GRAV_EUNSUPPORTED;
            break;
        }
        p->L = L;
        p->wl = (double)p->b;
        for (int a = 0; a < 3; ++a)
            p->root0[a] = -(double)p->shift[a] * p->b;
        // source blocks per level
        for (int l = 0; l <= L; ++l) {
            LevelInfo &lv = p->lev[l];
            lv.l = l;
            lv.w = (double)p->b * (double)(int64_t(1) << (L - l));
            lv.n_src = 1;
            for (int a = 0; a < 3; ++a) {
                const int s0 = p->shift[a];
                const int s1 = p->shift[a] + (int)ceil_div(n3[a], p->b) - 1;
                lv.s0[a] = s0 >> (L - l);
                lv.ns[a] = (s1 >> (L - l)) - lv.s0[a] + 1;
                lv.n_src *= lv.ns[a];
            }
        }
        p->n_me = 0;
        if (L >= 2)
            for (int l = 2; l <= L; ++l) {
                p->lev[l].me_off = p->n_me;
                p->n_me += p->lev[l].n_src;
            }
        if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) {
            st = GRAV_EDEVICE;
            break;
        }
        p->bs = s;
        if (desc->n_points > 0) {
            if ((st = dalloc(p, &p->d_points, 3 * desc->n_points, true)) != GRAV_OK)
                break;
            if (hipMemcpyAsync(p->d_points, desc->points, sizeof(double) * 3 * desc->n_points,
                               hipMemcpyHostToDevice, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess) {
                st = GRAV_EDEVICE;
                break;
            }
        }
        if (p->M > 0 && (st = build_tree(p, s)) != GRAV_OK)
            break;
        if (p->M > 0 && p->n_spts > 0 && (st = build_sources(p, desc, s)) != GRAV_OK)
            break;
        if (p->M > 0 && (st = build_near_lattice(p, s)) != GRAV_OK)
            break;
        if ((st = build_operators(p)) != GRAV_OK)
            break;
        if (p->M > 0 && p->L >= 2 && (st = build_m2l(p)) != GRAV_OK)
            break;
        if (p->M > 0 && (st = build_adjoint_maps(p)) != GRAV_OK)
            break;
        if (p->M > 0 && (st = count_work(p)) != GRAV_OK)
            break;
        // workspace
        // (mixed plans keep the expansions of lattice leaves in FP32 alone: d_rows)
        const bool leaves = p->d.precision == GRAV_FP64 || p->n_spts > 0 || p->L < 2;
        if ((st = dalloc(p, &p->d_me, (size_t)(leaves ? p->n_me : p->lev[p->L].me_off) * p->B * p->PS, false)) !=
            GRAV_OK)
            break;
        if ((st = dalloc(p, &p->d_le, (size_t)p->n_tbox * p->B * p->PS, false)) != GRAV_OK)
            break;
        if (p->L >= 2 && p->M > 0) {
            const bool f64 = p->d.precision == GRAV_FP64;
            const size_t n = (size_t)(f64 ? p->n_grow : std::max(p->n_me, p->n_grow)) * p->B * p->PS;
            if ((st = dalloc(p, &p->d_rows, f64 ? n : (n + 1) / 2, false)) != GRAV_OK)
                break;
        }
        if ((st = dalloc(p, &p->d_near, (size_t)p->M * p->B * 4, false)) != GRAV_OK)
            break;
        {
            // grav_direct: enough source chunks for ~2048 workgroups, partial
            // sums capped at 8 MB (the plan keeps them for its lifetime)
            const int64_t ncell = (int64_t)desc->nx * desc->ny * desc->nz;
            const int64_t tiles = std::max<int64_t>(1, ceil_div(p->M, 256));
            int64_t nch = std::min<int64_t>(std::max<int64_t>(1, ceil_div(2048, tiles)), ceil_div(ncell, 256));
            const int64_t per = std::max<int64_t>(1, p->M * p->B * 4 * 8);
            nch = std::max<int64_t>(1, std::min<int64_t>(nch, (8 << 20) / per));
            p->direct_chunks = (int)std::min<int64_t>(nch, 65535);
            if (p->direct_chunks > 1 &&
                (st = dalloc(p, &p->d_dpart, (size_t)p->direct_chunks * p->M * p->B * 4, false)) != GRAV_OK)
                break;
        }
        {
            // segment slots of the M2L, [parity][column][PS] each, in its
            // element type; both directions use them in turn
            const OctInfo in = octet_info(p->P, p->d.precision == GRAV_FP64);
            auto cols = [](const OctPlan &o) { return 16 * o.nc * std::max<int64_t>(o.nseg, 1); };
            const size_t slot = (size_t)std::max(cols(p->m2l), cols(p->m2lt)) * (8 / in.RS) * p->PS;
            if ((st = dalloc(p, &p->d_part, p->d.precision == GRAV_FP64 ? slot : (slot + 1) / 2, false)) != GRAV_OK)
                break;
        }
        {
            const DevGeom g = make_geom(p);
            if ((st = dalloc(p, &p->d_geom, 1, true)) != GRAV_OK)
                break;
            if (hipMemcpyAsync(p->d_geom, &g, sizeof(DevGeom), hipMemcpyHostToDevice, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess) {
                st = GRAV_EDEVICE;
                break;
            }
        }
        if (hipEventCreateWithFlags(&p->done, hipEventDisableTiming) != hipSuccess) {
            st = GRAV_EDEVICE;
            break;
        }
    } while (0);
    p->bs = nullptr;
    if (s)
        (void)hipStreamDestroy(s);
    (void)hipSetDevice(cur);
    if (st != GRAV_OK) {
        free_plan(p);
        return st;
    }
    *out = reinterpret_cast<grav_plan_t>(p);
    return GRAV_OK;
}

extern "C" void grav_plan_destroy(grav_plan_t plan)
{
    if (!plan)
        return;
    Plan *p = reinterpret_cast<Plan *>(plan);
    if (p->has_pending && p->done)
        (void)hipEventSynchronize(p->done);
    free_plan(p);
}

extern "C" grav_status grav_plan_bytes(grav_plan_t plan, size_t *resident, size_t *per_call)
{
    if (!plan)
        return GRAV_EINVAL;
    Plan *p = reinterpret_cast<Plan *>(plan);
    if (resident)
        *resident = p->bytes_resident;
    if (per_call)
        *per_call = p->bytes_call;
    return GRAV_OK;
}

extern "C" grav_status grav_plan_info(grav_plan_t plan, int64_t *n_targets, int32_t *levels,
                                      int32_t *leaf_cells, int64_t *n_target_leaves)
{
    if (!plan)
        return GRAV_EINVAL;
    Plan *p = reinterpret_cast<Plan *>(plan);
    if (n_targets)
        *n_targets = p->M;
    if (levels)
        *levels = p->L;
    if (leaf_cells)
        *leaf_cells = p->b;
    if (n_target_leaves)
        *n_target_leaves = p->n_leaf;
    return GRAV_OK;
}

extern "C" grav_status grav_plan_work(grav_plan_t plan, int64_t *m2l_pairs, int64_t *p2p_pairs,
                                      int64_t *n_sources)
{
    if (!plan)
        return GRAV_EINVAL;
    Plan *p = reinterpret_cast<Plan *>(plan);
    if (m2l_pairs)
        *m2l_pairs = p->m2l_pairs;
    if (p2p_pairs)
        *p2p_pairs = p->p2p_pairs;
    if (n_sources)
        *n_sources = p->n_spts > 0 ? p->n_spts : (int64_t)p->d.nx * p->d.ny * p->d.nz * p->nq3;
    return GRAV_OK;
}

extern "C" grav_status grav_operator(int32_t p, int32_t kind, int32_t which, int32_t dx,
                                     int32_t dy, int32_t dz, double *out)
{
    if (!out || p < 1)
        return GRAV_EINVAL;
    if (p > kMaxP)
        return GRAV_EUNSUPPORTED;
    const int P2 = p * p;
    if (kind == 0 || kind == 1) {
        if (which < 0 || which > 7)
            return GRAV_EINVAL;
        const double delta[3] = {((which & 1) - 0.5) * 0.5, (((which >> 1) & 1) - 0.5) * 0.5,
                                 (((which >> 2) & 1) - 0.5) * 0.5};
        if (kind == 0)
            m2m_matrix(p, delta, P2, out);
        else
            l2l_matrix(p, delta, P2, out);
        return GRAV_OK;
    }
    if (kind == 2) {
        const int mx = std::max(std::abs(dx), std::max(std::abs(dy), std::abs(dz)));
        if (mx < 2 || mx > 3)
            return GRAV_EINVAL;
        const double d[3] = {-(double)dx, -(double)dy, -(double)dz};
        m2l_matrix(p, d, P2, out);
        return GRAV_OK;
    }
    return GRAV_EINVAL;
}

extern "C" grav_status grav_harmonics(int32_t p, int32_t kind, double x, double y, double z,
                                      double *out)
{
    if (!out || p < 1 || (kind != 0 && kind != 1))
        return GRAV_EINVAL;
    if (p > kMaxP)
        return GRAV_EUNSUPPORTED;
    std::vector<cd> A;
    if (kind == 0)
        solid_regular(x, y, z, p, A);
    else {
        if (x == 0.0 && y == 0.0 && z == 0.0)
            return GRAV_EINVAL;
        solid_irregular(x, y, z, p, A);
    }
    for (int n = 0; n < p; ++n) {
        out[ridx(n, 0, 0)] = A[n * p].real();
        for (int m = 1; m <= n; ++m) {
            out[ridx(n, m, 0)] = A[n * p + m].real();
            out[ridx(n, m, 1)] = A[n * p + m].imag();
        }
    }
    return GRAV_OK;
}

extern "C" const char *grav_status_string(grav_status s)
{
    switch (s) {
    case GRAV_OK: return "ok";
    case GRAV_EINVAL: return "invalid argument";
    case GRAV_ENOMEM: return "out of memory";
    case GRAV_EDEVICE: return "device error";
    case GRAV_EUNSUPPORTED: return "unsupported request";
    case GRAV_EBUSY: return "plan busy on another stream";
    }
    return "unknown status";
}

extern "C" const char *grav_version(void) { return "grav-mi355x 0.1"; }
