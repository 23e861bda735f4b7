// Adjoint evaluation: the exact transpose of grav_eval's linear map rho -> g.
//
// Eq. (1) is linear in the density (Sec. 1.1), and so is every FMM stage of
// Sec. 2.3 (lattice P2M, M2M, M2L, L2L, L2P, the near-field sum of Eq. (13)
// and the combine), so the transpose of the forward map applies the
// transposed stages in reverse order:
//
//   w      = C^T r                      combine^T (scaling, descriptor order)
//   LE_L   = L2P^T w                    per target leaf
//   LE_l   = sum_children L2L_c^T LE_l+1    l = L-1 .. 2
//   ME_l   = sum_d K_d^T LE_l[S - d]    M2L^T, every source box S, levels 2 .. L
//   ME_l  += M2M_c^T ME_l-1[parent]     l = 3 .. L
//   drho   = P2M^T ME_L + NEAR^T w      per cell
//
// with the same operators (the FP32-rounded M2L matrices in mixed
// precision), the same interaction lists and the same point pairs and
// coincidence rule as the forward pass, so <A rho, r> = <rho, A^T r> holds to
// rounding.  The far field's stages are the octet kernels with transposed
// operators; every sum has a fixed order (no atomics), so results are
// deterministic.  Every index that comes from a plan table is checked against
// the size of the array it addresses, here or when the plan is checked.
#include <algorithm>

#include "harmonics.hpp"
#include "octet.hpp"
#include "resolve.hpp"

namespace grav {

namespace {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// combine^T: the weights that multiply (phi, gx, gy, gz) of a target in the
// lattice frame (G and the lattice-to-physical scale of the combine folded
// in), from its residual r (C values).
__device__ __forceinline__ void combine_weights(const DevGeom &g, const double *r, double (&o)[4])
{
    const double sg = g.G * g.h, sp = g.G * g.h * g.h;
    if (g.C == 1) {
        o[0] = o[1] = o[2] = 0.0;
        o[3] = sg * r[0];
    } else if (g.C == 3) {
        o[0] = 0.0;
        o[1] = sg * r[0];
        o[2] = sg * r[1];
        o[3] = sg * r[2];
    } else {
        o[0] = sp * r[0];
        o[1] = sg * r[1];
        o[2] = sg * r[2];
        o[3] = sg * r[3];
    }
}

// The weights of each sorted target (one thread per (sorted target,
// model)), for the targets with descriptor index below `limit`: all of them,
// or on lattice plans the user points only (the lattice kernels form the
// cell centres' weights from the residuals themselves).
__global__ void __launch_bounds__(256)
k_t_weights(DevGeom g, const double *resid, const uint32_t *perm, int64_t limit, double *w)
{
    const int64_t t = block_id() * blockDim.x + threadIdx.x;
    if (t >= g.M * g.B)
        return;
    const int64_t i = t / g.B;
    const int bm = (int)(t - i * g.B);
    const int64_t u = perm[i];
    if (u >= limit)
        return;
    double *o = w + t * 4;
    if (u < 0 || u >= g.M) {
        o[0] = o[1] = o[2] = o[3] = 0.0;
        return;
    }
    double v[4];
    combine_weights(g, resid + ((int64_t)bm * g.M + u) * g.C, v);
    o[0] = v[0];
    o[1] = v[1];
    o[2] = v[2];
    o[3] = v[3];
}

// The matrix stages below give each thread up to MT density models (a
// group), so that every operator entry or pair geometry it loads serves MT
// models; groups are ceil(B / MT).

// The near-field transpose, per cell: drho[cell] = (with `prior`, the terms
// already in drho, else 0) plus, over the targets j (with `pend`, the user
// points only: the lattice kernel takes the cell centres) of the 27 leaves
// around the cell's leaf (the forward near field pairs every target of a
// leaf with every quadrature point of its 27 neighbours), the weights times
// the pair terms (1/r, (t - x)/r^3) of each of the cell's quadrature
// points, with the forward's coincidence rule and arithmetic type T.  One
// thread per (cell, model group): the pair geometry is computed once for the
// group's models.  With `leaves` (and `prior`), only the cells of those
// source leaves (the leaves with user points around them; the other cells
// keep their prior terms), else every cell.
template <typename T, int MT>
__global__ void __launch_bounds__(256)
k_t_cells(DevGeom g, const double *tpos, const int64_t *leaf_start, const int64_t *pend, int64_t n_leaf,
          const int32_t *tmap, int64_t n_tmap, const double *w, int prior, const int32_t *leaves, int64_t n_leaves,
          double *drho)
{
    const int NG = (g.B + MT - 1) / MT;
    const int64_t ncell = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const int64_t t = block_id() * blockDim.x + threadIdx.x;
    const int b = g.b;
    const DevLev &lv = g.lev[g.L];
    int grp, ix, iy, iz;
    if (leaves) {
        const int b3 = b * b * b;
        const int64_t per = n_leaves * b3;
        if (t >= per * NG)
            return;
        grp = (int)(t / per);
        const int64_t r = t - (int64_t)grp * per;
        const int64_t sl = leaves[r / b3];
        const int v = (int)(r % b3);
        ix = (lv.s0[0] + (int)(sl % lv.ns[0]) - g.shift[0]) * b + v % b;
        iy = (lv.s0[1] + (int)((sl / lv.ns[0]) % lv.ns[1]) - g.shift[1]) * b + (v / b) % b;
        iz = (lv.s0[2] + (int)(sl / ((int64_t)lv.ns[0] * lv.ns[1])) - g.shift[2]) * b + v / (b * b);
        if (ix < 0 || iy < 0 || iz < 0 || ix >= g.n[0] || iy >= g.n[1] || iz >= g.n[2])
            return;
    } else {
        if (t >= ncell * NG)
            return;
        grp = (int)(t / ncell);
        const int64_t c = t - (int64_t)grp * ncell;
        ix = (int)(c % g.n[0]);
        iy = (int)((c / g.n[0]) % g.n[1]);
        iz = (int)(c / ((int64_t)g.n[0] * g.n[1]));
    }
    const int64_t cell = ((int64_t)iz * g.n[1] + iy) * g.n[0] + ix;
    // the cell's leaf (root-relative) and place in it
    const int lx = ix / b + g.shift[0], ly = iy / b + g.shift[1], lz = iz / b + g.shift[2];
    const int v = (ix % b) + b * ((iy % b) + b * (iz % b));
    double acc[MT];
#pragma unroll
    for (int u = 0; u < MT; ++u)
        acc[u] = 0.0;
    (void)v;
    if (prior) {
        // the terms already in drho (P2M^T, the lattice near field)
#pragma unroll
        for (int u = 0; u < MT; ++u)
            if (grp * MT + u < g.B)
                acc[u] = drho[(int64_t)(grp * MT + u) * ncell + cell];
    }
    // near field: quadrature points of this cell relative to its centre
    const T go = (T)(0.5 / 1.7320508075688772);
    const int mxl = lv.ns[0] + 6, myl = lv.ns[1] + 6, mzl = lv.ns[2] + 6;
    for (int nb = 0; nb < 27; ++nb) {
        const int tx = lx + nb % 3 - 1, ty = ly + (nb / 3) % 3 - 1, tz = lz + nb / 9 - 1;
        const int mx = tx - lv.s0[0] + 3, my = ty - lv.s0[1] + 3, mz = tz - lv.s0[2] + 3;
        if (mx < 0 || my < 0 || mz < 0 || mx >= mxl || my >= myl || mz >= mzl)
            continue;
        const int64_t mi = lv.tmap_off + ((int64_t)mz * myl + my) * mxl + mx;
        if (mi >= n_tmap)
            continue;
        const int64_t tl = tmap[mi];
        if (tl < 0 || tl >= n_leaf)
            continue;
        // target positions relative to the corner of the target leaf, as the
        // forward near field forms them, and the cell centre in that frame
        const int cx = (tx - g.shift[0]) * b, cy = (ty - g.shift[1]) * b, cz = (tz - g.shift[2]) * b;
        const T sx = (T)(ix - cx) + (T)0.5, sy = (T)(iy - cy) + (T)0.5, sz = (T)(iz - cz) + (T)0.5;
        const int64_t ts = max(leaf_start[tl], (int64_t)0);
        const int64_t te = min(pend ? pend[tl] : leaf_start[tl + 1], g.M);
        T part[MT];
#pragma unroll
        for (int u = 0; u < MT; ++u)
            part[u] = 0;
        for (int64_t j = ts; j < te; ++j) {
            const T ux = (T)(tpos[3 * j + 0] - (double)cx) - sx;
            const T uy = (T)(tpos[3 * j + 1] - (double)cy) - sy;
            const T uz = (T)(tpos[3 * j + 2] - (double)cz) - sz;
            // the pair geometry of the cell's quadrature points: (1/r, d/r^3)
            T f[8][4];
            const int np = g.q == 1 ? 1 : 8;
#pragma unroll
            for (int gp = 0; gp < 8; ++gp) {
                if (gp >= np) {
                    f[gp][0] = f[gp][1] = f[gp][2] = f[gp][3] = 0;
                    continue;
                }
                const T px = g.q == 1 ? ux : ux - ((gp & 1) ? go : -go);
                const T py = g.q == 1 ? uy : uy - ((gp & 2) ? go : -go);
                const T pz = g.q == 1 ? uz : uz - ((gp & 4) ? go : -go);
                const T r2 = px * px + py * py + pz * pz;
                const T wq = g.q == 1 ? (T)1 : (T)0.125;
                if (r2 > coincident2<T>()) {
                    const T ri = rsqrt_t(r2);
                    const T ri3 = ri * ri * ri;
                    f[gp][0] = wq * ri;
                    f[gp][1] = wq * px * ri3;
                    f[gp][2] = wq * py * ri3;
                    f[gp][3] = wq * pz * ri3;
                } else {
                    f[gp][0] = f[gp][1] = f[gp][2] = f[gp][3] = 0;
                }
            }
#pragma unroll
            for (int u = 0; u < MT; ++u) {
                const int bm = grp * MT + u;
                if (bm >= g.B)
                    continue;
                const double *wj = w + (j * g.B + bm) * 4;
                const T w0 = (T)wj[0], w1 = (T)wj[1], w2 = (T)wj[2], w3 = (T)wj[3];
                T sum = 0;
#pragma unroll
                for (int gp = 0; gp < 8; ++gp)
                    if (gp < np)
                        sum += w0 * f[gp][0] + (w1 * f[gp][1] + w2 * f[gp][2] + w3 * f[gp][3]);
                part[u] += sum;
            }
        }
#pragma unroll
        for (int u = 0; u < MT; ++u)
            acc[u] += (double)part[u];
    }
#pragma unroll
    for (int u = 0; u < MT; ++u) {
        const int bm = grp * MT + u;
        if (bm < g.B)
            drho[(int64_t)bm * ncell + cell] = acc[u];
    }
}

// Explicit sources, the transposes of P2M and of the near field per source:
// drho[source] = mass per unit value x (the derivative of the leaf
// expansion's contribution, multipole_basis_dot against ME_L^T, plus the
// pair terms of the targets of the 27 leaves around the source's leaf with
// their weights, formed as the forward near field forms them: relative to
// the target leaf's corner, in type T, with its coincidence rule).  One
// thread per (sorted source, model group).
template <typename T, int MT>
__global__ void __launch_bounds__(256)
k_t_src(DevGeom g, const double *spos, const double *sw, const uint32_t *sperm, int64_t nsrc, const double *tpos,
        const int64_t *leaf_start, int64_t n_leaf, const int32_t *tmap, int64_t n_tmap, const double *w,
        const double *me, double *drho)
{
    const int NG = (g.B + MT - 1) / MT;
    const int64_t t = block_id() * blockDim.x + threadIdx.x;
    if (t >= nsrc * NG)
        return;
    const int grp = (int)(t / nsrc);
    const int64_t i = t - (int64_t)grp * nsrc;
    const int nm = min(MT, g.B - grp * MT);
    const int b = g.b;
    const DevLev &lv = g.lev[g.L];
    const double x[3] = {spos[3 * i + 0], spos[3 * i + 1], spos[3 * i + 2]};
    // the source's leaf (block-relative, as the sort key)
    int lc[3];
    for (int a = 0; a < 3; ++a)
        lc[a] = min(max((int)floor(x[a] / b), 0), lv.ns[a] - 1);
    double acc[MT];
#pragma unroll
    for (int u = 0; u < MT; ++u)
        acc[u] = 0.0;
    if (g.L >= 2) {
        const int64_t leaf = ((int64_t)lc[2] * lv.ns[1] + lc[1]) * lv.ns[0] + lc[0];
        const double inv_b = 1.0 / (double)b;
        multipole_basis_dot<MT>(g.P, (x[0] - (lc[0] + 0.5) * b) * inv_b, (x[1] - (lc[1] + 0.5) * b) * inv_b,
                                (x[2] - (lc[2] + 0.5) * b) * inv_b,
                                me + ((lv.me_off + leaf) * g.B + grp * MT) * g.PS, g.PS, nm, acc);
    }
    const int mxl = lv.ns[0] + 6, myl = lv.ns[1] + 6, mzl = lv.ns[2] + 6;
    for (int nb = 0; nb < 27; ++nb) {
        // target leaf (root coordinates) and its place in the target map
        const int tx = lc[0] + lv.s0[0] + nb % 3 - 1, ty = lc[1] + lv.s0[1] + (nb / 3) % 3 - 1,
                  tz = lc[2] + lv.s0[2] + nb / 9 - 1;
        const int mx = tx - lv.s0[0] + 3, my = ty - lv.s0[1] + 3, mz = tz - lv.s0[2] + 3;
        if (mx < 0 || my < 0 || mz < 0 || mx >= mxl || my >= myl || mz >= mzl)
            continue;
        const int64_t mi = lv.tmap_off + ((int64_t)mz * myl + my) * mxl + mx;
        if (mi >= n_tmap)
            continue;
        const int64_t tl = tmap[mi];
        if (tl < 0 || tl >= n_leaf)
            continue;
        const double corner[3] = {(double)((tx - g.shift[0]) * b), (double)((ty - g.shift[1]) * b),
                                  (double)((tz - g.shift[2]) * b)};
        const T sx = (T)(x[0] - corner[0]), sy = (T)(x[1] - corner[1]), sz = (T)(x[2] - corner[2]);
        const int64_t ts = max(leaf_start[tl], (int64_t)0), te = min(leaf_start[tl + 1], g.M);
        T part[MT];
#pragma unroll
        for (int u = 0; u < MT; ++u)
            part[u] = 0;
        for (int64_t j = ts; j < te; ++j) {
            const T cx = (T)(tpos[3 * j + 0] - corner[0]) - sx;
            const T cy = (T)(tpos[3 * j + 1] - corner[1]) - sy;
            const T cz = (T)(tpos[3 * j + 2] - corner[2]) - sz;
            const T r2 = cx * cx + cy * cy + cz * cz;
            if (!(r2 > coincident2<T>()))
                continue;
            const T ri = rsqrt_t(r2);
            const T ri3 = ri * ri * ri;
#pragma unroll
            for (int u = 0; u < MT; ++u) {
                if (u >= nm)
                    break;
                const double *wj = w + (j * g.B + grp * MT + u) * 4;
                part[u] += (T)wj[0] * ri + ((T)wj[1] * (cx * ri3) + (T)wj[2] * (cy * ri3) + (T)wj[3] * (cz * ri3));
            }
        }
#pragma unroll
        for (int u = 0; u < MT; ++u)
            acc[u] += (double)part[u];
    }
    const uint32_t user = sperm[i];
#pragma unroll
    for (int u = 0; u < MT; ++u)
        if (u < nm)
            drho[(int64_t)(grp * MT + u) * nsrc + user] = sw[i] * acc[u];
}

__global__ void __launch_bounds__(256) k_t_zero(double *x, int64_t n)
{
    const int64_t i = block_id() * blockDim.x + threadIdx.x;
    if (i < n)
        x[i] = 0.0;
}

}  // namespace

// The transposed M2L's input in its element type: the adjoint LE over each
// level's gather region, zero where the region has no target box (found
// through the level's target map, the source block plus a halo of 3, which
// holds the region).  One thread per four coefficients.
template <typename T>
__global__ void __launch_bounds__(256)
k_le_rows(DevGeom g, OctGeom og, const int32_t *tmap, const double *le, int64_t n4, T *out)
{
    const int64_t i = block_id() * blockDim.x + threadIdx.x;
    if (i >= n4)
        return;
    const int P4 = g.PS / 4;
    const int k4 = (int)(i % P4);
    const int64_t col = i / P4;  // row * B + model
    const int64_t row = col / g.B;
    const int bm = (int)(col - row * g.B);
    int l = 2;
    while (l < g.L && row >= og.lev[l + 1].row0)
        ++l;
    const OctLev &lt = og.lev[l];
    const DevLev &lv = g.lev[l];
    const int64_t j = row - lt.row0;
    const int64_t tb = tmap_lookup(lv, tmap, 3, lt.s0[0] + (int)(j % lt.ns[0]), lt.s0[1] + (int)((j / lt.ns[0]) % lt.ns[1]),
                                   lt.s0[2] + (int)(j / ((int64_t)lt.ns[0] * lt.ns[1])));
    double2 a = double2{0.0, 0.0}, b = a;
    if (tb >= 0 && tb < lv.n_tgt) {
        const double2 *src = reinterpret_cast<const double2 *>(le + ((lv.tgt_off + tb) * g.B + bm) * g.PS) + 2 * k4;
        a = src[0];
        b = src[1];
    }
    if constexpr (sizeof(T) == 4) {
        reinterpret_cast<float4 *>(out)[i] = make_float4((float)a.x, (float)a.y, (float)b.x, (float)b.y);
    } else {
        reinterpret_cast<double2 *>(out)[2 * i] = a;
        reinterpret_cast<double2 *>(out)[2 * i + 1] = b;
    }
}

// M2L^T on the forward's kernel with the transposed operators: columns are
// the octets of source boxes.
template <typename T>
static grav_status enqueue_m2l_transposed(Plan *p, const DevGeom &g, hipStream_t s)
{
    const OctGeom og = octet_geom(p, true);
    T *rows = reinterpret_cast<T *>(p->d_rows);
    const int64_t n4 = p->n_grow * p->B * (p->PS / 4);
    if (n4 > 0) {
        hipLaunchKernelGGL((k_le_rows<T>), block_grid(ceil_div(n4, 256)), dim3(256), 0, s, g, og,
                           (const int32_t *)p->d_tmap, (const double *)p->d_le, n4, rows);
        GRAV_HIP(hipGetLastError());
    }
    return launch_m2l<T>(p, p->m2lt, s, og, rows);
}

// The lattice transposes for voxel-centre targets (see k_near_lat): with w_T
// the combine^T weights of target leaf T's b^3 cell centres (4 per centre),
//   drho[S] (+)= sum over the 27 neighbours d of A_d^T w_{S - d}   (near^T)
//   LE[T]   (+)= Lm^T w_T                                          (L2P^T)
// GEMMs with columns = (leaf, model) and contraction over (centre t,
// component) of the target leaf.  L2P^T: chunk q and k step u take t =
// (lane/16) TQ + q and component u, so a lane's four k steps are the four
// weights of one centre.  near^T: only the C output components, value e =
// C t + c in chunk q, sub-row kr and k step u with e = 4 KQ kr + 4 q + u,
// read from the weight blocks.  A centre's weights come straight from its
// residual (the centres follow the npts user points in descriptor order, x
// fastest); centres outside the mesh or past b^3 read zero.
__device__ __forceinline__ void lattice_weights(const DevGeom &g, const double *resid, int64_t npts, int tx, int ty,
                                                int tz, int t, int bm, bool in, double (&v)[4])
{
    const int b = g.b;
    v[0] = v[1] = v[2] = v[3] = 0.0;
    if (!in || t >= b * b * b)
        return;
    const int ix = tx * b + t % b, iy = ty * b + (t / b) % b, iz = tz * b + t / (b * b);
    if (ix >= g.n[0] || iy >= g.n[1] || iz >= g.n[2])
        return;
    const int64_t cell = ((int64_t)iz * g.n[1] + iy) * g.n[0] + ix;
    combine_weights(g, resid + ((int64_t)bm * g.M + npts + cell) * g.C, v);
}

// The weights of the cell centres in leaf blocks for near^T, as k_rho_blocks
// lays out the densities, for the C output components only: value e =
// C t + c (centre t, component c of the C) of a leaf sits at
// blk[q][kr][pl * B + model][u] with e = 4 KQ kr + 4 q + u, pl = the leaf's
// index in the source block padded by one leaf per side (padding and
// e >= C b^3 zero).  One thread per (leaf, model, centre).
template <typename T>
__global__ void __launch_bounds__(256)
k_t_wblocks(DevGeom g, const double *resid, int64_t npts, int KQ, int64_t nplB, T *blk)
{
    const DevLev &lv = g.lev[g.L];
    const int b = g.b, b3 = b * b * b;
    const int64_t nleaf = (int64_t)lv.ns[0] * lv.ns[1] * lv.ns[2];
    const int64_t i = block_id() * blockDim.x + threadIdx.x;
    if (i >= nleaf * g.B * b3)
        return;
    const int t = (int)(i % b3);
    const int bm = (int)((i / b3) % g.B);
    const int64_t leaf = i / ((int64_t)b3 * g.B);
    const int lx = (int)(leaf % lv.ns[0]), ly = (int)((leaf / lv.ns[0]) % lv.ns[1]),
              lz = (int)(leaf / ((int64_t)lv.ns[0] * lv.ns[1]));
    double v[4];
    lattice_weights(g, resid, npts, lx, ly, lz, t, bm, true, v);
    const int64_t pl = ((int64_t)(lz + 1) * (lv.ns[1] + 2) + (ly + 1)) * (lv.ns[0] + 2) + (lx + 1);
    for (int c = 0; c < g.C; ++c) {
        const int e = g.C * t + c, kr = e / (4 * KQ), q = (e / 4) % KQ;
        blk[((int64_t)(q * 4 + kr) * nplB + pl * g.B + bm) * 4 + e % 4] = (T)v[c + 4 - g.C];
    }
}

// near^T of the plans that k_near_lat serves (the others: near.hip): a workgroup
// owns CW blocks of 16 (source leaf, model) columns and the (up to four) 16-cell
// row blocks; its four waves split the 27 KQ
// chunks (neighbour d, chunk q of the target leaf's C b^3 weights) and add
// their partial tiles through LDS in wave order (deterministic), as
// k_near_lat does.  Target leaf T = S - d reads the padded weight blocks (no
// bounds test).
template <int CW, typename T>
__global__ void __launch_bounds__(256)
k_t_near_lat(DevGeom g, const T *blk, int64_t nplB, const T *A, int RBt, int KQ, int add, double *drho)
{
    using vec4 = __attribute__((__vector_size__(4 * sizeof(T)))) T;
    __shared__ double red[4][CW * 4 * 4][64];
    const int lane = threadIdx.x & 63, kr = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const DevLev &lv = g.lev[g.L];
    const int64_t nleaf = (int64_t)lv.ns[0] * lv.ns[1] * lv.ns[2];
    const int b = g.b, b3 = b * b * b;
    const int px = lv.ns[0] + 2, py = lv.ns[1] + 2;
    bool cvalid[CW];
    int bm[CW], sx[CW], sy[CW], sz[CW];
    const T *bbase[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) {
        const int64_t col = (block_id() * CW + c) * 16 + (lane & 15);
        cvalid[c] = col < nleaf * g.B;
        const int64_t leaf = cvalid[c] ? col / g.B : 0;
        bm[c] = cvalid[c] ? (int)(col % g.B) : 0;
        sx[c] = (int)(leaf % lv.ns[0]);
        sy[c] = (int)((leaf / lv.ns[0]) % lv.ns[1]);
        sz[c] = (int)(leaf / ((int64_t)lv.ns[0] * lv.ns[1]));
        bbase[c] = blk + ((int64_t)kr * nplB + (((int64_t)(sz[c] + 1) * py + (sy[c] + 1)) * px + (sx[c] + 1)) * g.B +
                          bm[c]) * 4;
    }
    vec4 acc[CW][4];
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            acc[c][r] = vec4{0, 0, 0, 0};
    const int NI = 27 * KQ;
    const int i0 = wave * NI / 4, i1 = (wave + 1) * NI / 4;
    for (int i = i0; i < i1; ++i) {
        const int nb = i / KQ, q = i - nb * KQ;
        // the forward pairs target leaf T with source leaf T + d: T = S - d
        const int dx = nb % 3 - 1, dy = (nb / 3) % 3 - 1, dz = nb / 9 - 1;
        const int64_t boff = ((int64_t)q * 4 * nplB + (((int64_t)(-dz) * py - dy) * px - dx) * g.B) * 4;
        T bb[CW][4];
#pragma unroll
        for (int c = 0; c < CW; ++c)
            load4(bbase[c] + boff, bb[c]);
        T av[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            load_frags<T, 4>(A + (((int64_t)nb * KQ + q) * RBt + min(r, RBt - 1)) * 256, lane, av[r]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    if constexpr (sizeof(T) == 8)
                        acc[c][r] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[r][u], bb[c][u], acc[c][r], 0, 0, 0);
                    else
                        acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[r][u], bb[c][u], acc[c][r], 0, 0, 0);
                }
    }
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                red[wave][(c * 4 + r) * 4 + k][lane] = (double)acc[c][r][k];
    __syncthreads();
    // output rows: FP32 instruction rows 4 (lane/16) + i, FP64 rows lane/16 + 4 i
    const int64_t ncell = (int64_t)g.n[0] * g.n[1] * g.n[2];
    for (int j = wave; j < CW * 4; j += 4) {
        const int c = j / 4, r = j % 4;
        if (!cvalid[c] || r >= RBt)
            continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = 16 * r + (sizeof(T) == 8 ? kr + 4 * i : 4 * kr + i);
            if (v >= b3)
                continue;
            const int ix = sx[c] * b + v % b, iy = sy[c] * b + (v / b) % b, iz = sz[c] * b + v / (b * b);
            if (ix >= g.n[0] || iy >= g.n[1] || iz >= g.n[2])
                continue;
            const double sum = ((red[0][j * 4 + i][lane] + red[1][j * 4 + i][lane]) + red[2][j * 4 + i][lane]) +
                               red[3][j * 4 + i][lane];
            double *o = drho + (int64_t)bm[c] * ncell + ((int64_t)iz * g.n[1] + iy) * g.n[0] + ix;
            *o = add ? *o + sum : sum;
        }
    }
}

// L2P^T at the cell centres (FP64): one wave owns 16 (leaf, model) columns
// and all RB coefficient blocks; the column's target leaf is found in the
// leaf level's target map.  With `add`, the LE of a leaf that also holds
// user points (written by k_t_l2p_points) is added to, every other one set.
template <int RB>
__global__ void __launch_bounds__(64)
k_t_l2p_lat(DevGeom g, const double *A, int TQ, const int32_t *tmap, const double *resid, int64_t npts,
            int add, const int64_t *leaf_start, const int64_t *pend, double *le)
{
    using vec4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
    constexpr int PS = 16 * RB;
    const int lane = threadIdx.x, kr = lane >> 4;
    const DevLev &lv = g.lev[g.L];
    const int64_t nleaf = (int64_t)lv.ns[0] * lv.ns[1] * lv.ns[2];
    const int64_t col = block_id() * 16 + (lane & 15);
    const bool cvalid = col < nleaf * g.B;
    const int64_t leaf = cvalid ? col / g.B : 0;
    const int bm = cvalid ? (int)(col % g.B) : 0;
    const int sx = (int)(leaf % lv.ns[0]), sy = (int)((leaf / lv.ns[0]) % lv.ns[1]),
              sz = (int)(leaf / ((int64_t)lv.ns[0] * lv.ns[1]));
    const int64_t tl =
        cvalid ? tmap_lookup(lv, tmap, 3, lv.s0[0] + sx, lv.s0[1] + sy, lv.s0[2] + sz) : -1;
    vec4 acc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
        acc[r] = vec4{0, 0, 0, 0};
    for (int q = 0; q < TQ; ++q) {
        double bv[4];
        lattice_weights(g, resid, npts, sx, sy, sz, kr * TQ + q, bm, tl >= 0, bv);
        double av[RB][4];
#pragma unroll
        for (int r = 0; r < RB; ++r)
            load_frags<double, 4>(A + ((int64_t)q * RB + r) * 256, lane, av[r]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < RB; ++r)
                acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[r][u], bv[u], acc[r], 0, 0, 0);
    }
    if (tl < 0 || tl >= lv.n_tgt)
        return;
    const bool addc = add && pend[tl] > max(leaf_start[tl], (int64_t)0);
    double *dst = le + ((lv.tgt_off + tl) * g.B + bm) * PS;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double *o = dst + 16 * r + kr + 4 * i;
            *o = addc ? *o + acc[r][i] : acc[r][i];
        }
}

#define GRAV_T_RB_CASES(X) X(1) X(2) X(3) X(4) X(6) X(7) X(8) X(9) X(11) X(13) X(15) X(16)

static grav_status launch_t_l2p_lat(Plan *p, const DevGeom &g, const double *resid, int add, hipStream_t s)
{
    const dim3 grid = block_grid(ceil_div(p->lev[p->L].n_src * p->B, 16));
#define CASE(R)                                                                                             \
    case R:                                                                                                 \
        hipLaunchKernelGGL((k_t_l2p_lat<R>), grid, dim3(64), 0, s, g, (const double *)p->d_tl2pt, p->lat_TQ, \
                           (const int32_t *)p->d_tmap, resid, p->d.n_points,                              \
                           add, (const int64_t *)p->d_leaf_start, (const int64_t *)p->d_leaf_pend, p->d_le); \
        break;
    switch (p->PS / 16) {
        GRAV_T_RB_CASES(CASE)
    default:
        return GRAV_EUNSUPPORTED;
    }
#undef CASE
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

static grav_status launch_t_near_lat(Plan *p, const DevGeom &g, const double *resid, int add, double *drho,
                                     hipStream_t s)
{
    constexpr int CW = 2;
    const LevelInfo &lv = p->lev[p->L];
    const int b3 = p->b * p->b * p->b, RBt = (int)ceil_div(b3, 16);
    // chunks of 16 weights over the C b^3 (centre, component) pairs of a leaf
    const int KQ = (int)ceil_div((int64_t)p->d.components * b3, 16);
    const int64_t nplB = (int64_t)(lv.ns[0] + 2) * (lv.ns[1] + 2) * (lv.ns[2] + 2) * p->B;
    const bool f64 = p->d.precision == GRAV_FP64;
    const dim3 fgrid = block_grid(ceil_div(lv.n_src * p->B * b3, 256));
    const dim3 grid = block_grid(ceil_div(lv.n_src * p->B, 16 * CW));
    if (f64) {
        hipLaunchKernelGGL((k_t_wblocks<double>), fgrid, dim3(256), 0, s, g, resid, p->d.n_points, KQ, nplB,
                           p->d_w_blk);
        hipLaunchKernelGGL((k_t_near_lat<CW, double>), grid, dim3(256), 0, s, g, (const double *)p->d_w_blk, nplB,
                           (const double *)p->d_tnt64, RBt, KQ, add, drho);
    } else {
        float *wb = reinterpret_cast<float *>(p->d_w_blk);
        hipLaunchKernelGGL((k_t_wblocks<float>), fgrid, dim3(256), 0, s, g, resid, p->d.n_points, KQ, nplB,
                           wb);
        hipLaunchKernelGGL((k_t_near_lat<CW, float>), grid, dim3(256), 0, s, g, (const float *)wb, nplB,
                           (const float *)p->d_tnt32, RBt, KQ, add, drho);
    }
    GRAV_HIP(hipGetLastError());
    return GRAV_OK;
}

template <int MT>
static grav_status enqueue_adjoint_mt(Plan *p, const double *resid, double *drho, hipStream_t s)
{
    const DevGeom g = make_geom(p);
    const int L = p->L;
    const int64_t ncell = (int64_t)p->d.nx * p->d.ny * p->d.nz;
    const int64_t NG = (p->B + MT - 1) / MT;
    const dim3 blk(256);
    auto grid = [](int64_t n) { return block_grid(ceil_div(n, 256)); };
    if (ncell * NG > 0x7fffffffll * 256 || p->n_me > 0x7fffffffll || p->P2 > 256)
        return GRAV_EUNSUPPORTED;
    stage_begin(p, "weights", s);
    hipLaunchKernelGGL(k_t_weights, grid(p->M * p->B), blk, 0, s, g, resid, (const uint32_t *)p->d_perm,
                       p->lat_near ? p->d.n_points : p->M, p->d_near);
    GRAV_HIP(hipGetLastError());
    stage_end(p, s);
    if (L >= 2) {
        stage_begin(p, "l2pT", s);
        // user points by the transposed recurrence; cell centres of lattice
        // plans by the transposed lattice L2P
        const bool pts = !p->lat_near || p->d.n_points > 0;
        if (p->n_leaf > 0 && pts)
            GRAV_CHECK(launch_t_l2p_points(p, g, s));
        if (p->lat_near)
            GRAV_CHECK(p->near_par ? launch_t_l2p_par(p, g, resid, pts ? 1 : 0, s)
                                   : launch_t_l2p_lat(p, g, resid, pts ? 1 : 0, s));
        stage_end(p, s);
        stage_begin(p, "l2lT", s);
        for (int l = L; l >= 3; --l)
            GRAV_CHECK(launch_octet_up(p, p->m2l, l, s, p->d_l2lt, p->d_le, nullptr));
        stage_end(p, s);
        stage_begin(p, "m2lT", s);
        if (p->d.precision == GRAV_FP64)
            GRAV_CHECK(enqueue_m2l_transposed<double>(p, g, s));
        else
            GRAV_CHECK(enqueue_m2l_transposed<float>(p, g, s));
        stage_end(p, s);
        stage_begin(p, "m2mT", s);
        // (to lattice sources, the P2M^T goes on from the level above)
        for (int l = 2; l <= (p->n_spts > 0 ? L : L - 1); ++l)
            GRAV_CHECK(launch_octet_down(p, p->m2lt, l, s, p->d_m2mt, p->d_me));
        stage_end(p, s);
        if (p->n_spts == 0) {
            stage_begin(p, "p2mT", s);
            GRAV_CHECK(launch_t_p2m(p, g, drho, s));
            stage_end(p, s);
        }
    }
    if (p->n_spts > 0) {
        // explicit sources: P2M^T and near^T per source
        stage_begin(p, "srcT", s);
        const int64_t n = p->n_spts * NG;
        if (p->d.precision == GRAV_FP64)
            hipLaunchKernelGGL((k_t_src<double, MT>), grid(n), blk, 0, s, g, (const double *)p->d_spos,
                               (const double *)p->d_sw, (const uint32_t *)p->d_sperm, p->n_spts,
                               (const double *)p->d_tpos, (const int64_t *)p->d_leaf_start, p->n_leaf,
                               (const int32_t *)p->d_tmap, p->n_tmap, (const double *)p->d_near,
                               (const double *)p->d_me, drho);
        else
            hipLaunchKernelGGL((k_t_src<float, MT>), grid(n), blk, 0, s, g, (const double *)p->d_spos,
                               (const double *)p->d_sw, (const uint32_t *)p->d_sperm, p->n_spts,
                               (const double *)p->d_tpos, (const int64_t *)p->d_leaf_start, p->n_leaf,
                               (const int32_t *)p->d_tmap, p->n_tmap, (const double *)p->d_near,
                               (const double *)p->d_me, drho);
        GRAV_HIP(hipGetLastError());
        stage_end(p, s);
        return GRAV_OK;
    }
    // the near field's transpose (with no far field it also sets drho):
    // cell centres of lattice plans on MFMA, user points (or all targets of
    // other plans) pair by pair
    if (p->lat_near) {
        stage_begin(p, "nearT", s);
        GRAV_CHECK(p->near_par ? launch_t_near_par(p, g, resid, L >= 2 ? 1 : 0, drho, s)
                               : launch_t_near_lat(p, g, resid, L >= 2 ? 1 : 0, drho, s));
        stage_end(p, s);
    }
    const bool pts = p->lat_near ? p->d.n_points > 0 : (p->p2p_pairs > 0 || L < 2);
    if (pts) {
        const int prior = (L >= 2 || p->lat_near) ? 1 : 0;
        const int64_t *pend = p->lat_near ? (const int64_t *)p->d_leaf_pend : nullptr;
        stage_begin(p, "nearT_pts", s);
        // with prior terms only the cells of the leaves near user points
        // change (none when the points lie away from the mesh)
        const int32_t *leaves = prior ? p->d_pt_leaves : nullptr;
        const int64_t nthr = leaves ? p->n_pt_leaves * p->b * p->b * p->b * NG : ncell * NG;
        if (nthr > 0) {
            if (p->d.precision == GRAV_FP64)
                hipLaunchKernelGGL((k_t_cells<double, MT>), grid(nthr), blk, 0, s, g, (const double *)p->d_tpos,
                                   (const int64_t *)p->d_leaf_start, pend, p->n_leaf, (const int32_t *)p->d_tmap,
                                   p->n_tmap, (const double *)p->d_near, prior, leaves, p->n_pt_leaves, drho);
            else
                hipLaunchKernelGGL((k_t_cells<float, MT>), grid(nthr), blk, 0, s, g, (const double *)p->d_tpos,
                                   (const int64_t *)p->d_leaf_start, pend, p->n_leaf, (const int32_t *)p->d_tmap,
                                   p->n_tmap, (const double *)p->d_near, prior, leaves, p->n_pt_leaves, drho);
            GRAV_HIP(hipGetLastError());
        }
        stage_end(p, s);
    }
    return GRAV_OK;
}

grav_status enqueue_adjoint(Plan *p, const double *resid, double *drho, hipStream_t s)
{
    // one model per thread for single-model plans, groups of eight otherwise
    return p->B == 1 ? enqueue_adjoint_mt<1>(p, resid, drho, s) : enqueue_adjoint_mt<8>(p, resid, drho, s);
}

}  // namespace grav

using namespace grav;

extern "C" grav_status grav_adjoint(grav_plan_t plan, const double *resid, double *drho_out, void *stream)
{
    if (!plan)
        return GRAV_EINVAL;
    Plan *p = reinterpret_cast<Plan *>(plan);
    if (!drho_out || (p->M > 0 && !resid))
        return GRAV_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    int cur = 0;
    GRAV_HIP(hipGetDevice(&cur));
    if (cur != p->device)
        GRAV_HIP(hipSetDevice(p->device));
    grav_status st = begin_call(p, s);
    if (st == GRAV_OK) {
        if (p->M == 0) {
            // no evaluation points: the transpose is zero (a fill kernel, not a
            // memset, so that the call can be recorded in a graph)
            const int64_t n = (p->n_spts > 0 ? p->n_spts : (int64_t)p->d.nx * p->d.ny * p->d.nz) * p->B;
            hipLaunchKernelGGL(k_t_zero, block_grid(ceil_div(n, 256)), dim3(256), 0, s, drho_out, n);
            st = hipGetLastError() == hipSuccess ? GRAV_OK : GRAV_EDEVICE;
        } else {
            st = enqueue_adjoint(p, resid, drho_out, s);
        }
    }
    if (st == GRAV_OK)
        st = end_call(p, s);
    if (cur != p->device)
        (void)hipSetDevice(cur);
    return st;
}
