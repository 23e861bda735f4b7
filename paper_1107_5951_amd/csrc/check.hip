// grav_plan_check: host-side validation of a plan's index tables.
//
// Copies the plan's device tables back and runs, on the host, the same
// column/term resolvers the M2L kernels use (they are compiled for both
// sides), plus the tree tables the other kernels index,
// checking every expansion, matrix, target-range and cell index against the
// size of the buffer it addresses, and that no two columns of one stage
// write the same expansion.  No compute kernel is launched.
#include <algorithm>
#include <functional>
#include <cstdio>
#include <string>
#include <tuple>
#include <vector>

#include "octet.hpp"
#include "resolve.hpp"

namespace grav {

namespace {

template <class T>
std::vector<T> fetch(const T *d, size_t n)
{
    std::vector<T> h(n);
    if (n && d && hipMemcpy(h.data(), d, n * sizeof(T), hipMemcpyDeviceToHost) != hipSuccess)
        h.clear();
    return h;
}

struct Checker {
    bool ok = true;
    std::string msg;
    void fail(const char *stage, const char *what, long long a, long long b)
    {
        if (ok) {
            char buf[256];
            std::snprintf(buf, sizeof buf, "%s: %s (%lld vs %lld)", stage, what, a, b);
            msg = buf;
        }
        ok = false;
    }
};

// One M2L direction: the groups cover every column of every level, the
// segments every orbit of a unit with a source once, in one slot each, every
// input row lies in [0, nin), and every output row is written by exactly one octet.
void check_octets(Checker &ck, const char *name, const Plan *p, const OctPlan &o, const OctGeom &g,
                  int64_t nin, int64_t nout, const std::function<bool(int, int32_t)> &present)
{
    const OctInfo in = octet_info(p->P, p->d.precision == GRAV_FP64);
    const auto key = fetch(o.d_key, (size_t)o.noct);
    const auto child = fetch(o.d_child, (size_t)o.noct * 8);
    const auto groups = fetch(o.d_groups, (size_t)o.ngroup);
    const auto segs = fetch(o.d_segs, (size_t)o.nseg * 4);
    const auto wgseg = fetch(o.d_wgseg, (size_t)o.wgs + (o.wgs > 0 ? 1 : 0));
    const auto uslot = fetch(o.d_uslot, (size_t)o.nunit + 1);
    // segment of each slot
    std::vector<int32_t> slot_seg((size_t)o.nseg, -1);
    for (int64_t sg = 0; sg < o.nseg && ck.ok; ++sg) {
        const int32_t sl = segs[4 * sg + 2];
        if (sl < 0 || sl >= o.nseg || slot_seg[sl] >= 0)
            ck.fail(name, "slot out of range or repeated", sg, sl);
        else
            slot_seg[sl] = (int32_t)sg;
    }
    std::vector<char> written((size_t)nout, 0);
    for (int64_t i = 0; i < o.noct * 8 && ck.ok; ++i)
        if (child[i] >= 0 && (child[i] >= nout || written[child[i]]++))
            ck.fail(name, "output row out of range or repeated", i, child[i]);
    for (int64_t i = 0; i < nout && ck.ok; ++i)
        if (!written[i])
            ck.fail(name, "expansion never written", i, nout);
    // the parent of an octet is the box of its key in the level above, whose own
    // row is a child of exactly one octet there
    const auto parent = fetch(o.d_parent, (size_t)o.noct);
    std::vector<int64_t> octet_of((size_t)nout, -1);
    for (int64_t i = 0; i < o.noct * 8 && ck.ok; ++i)
        if (child[i] >= 0)
            octet_of[child[i]] = i;
    for (int l = 2; l <= p->L && ck.ok; ++l)
        for (int64_t i = o.first[l]; i < o.first[l + 1] && ck.ok; ++i) {
            if (l == 2 ? parent[i] != -1 : parent[i] < 0 || parent[i] >= nout)
                ck.fail(name, "parent row out of range", i, parent[i]);
            else if (l > 2) {
                const int64_t at = octet_of[parent[i]];
                if (at < 8 * o.first[l - 1] || at >= 8 * o.first[l] || ((key[at / 8] << 3) | (uint32_t)(at % 8)) != key[i])
                    ck.fail(name, "parent row is another box's", i, parent[i]);
            }
        }
    int64_t covered = 0;
    for (int64_t i = 0; i < o.ngroup && ck.ok; ++i) {
        const OctGroup &gr = groups[i];
        covered += gr.ncol;
        if (gr.level < 2 || gr.level > p->L || gr.ncol < 1 || gr.ncol > 16 * o.nc || gr.col0 < 0 ||
            gr.oct0 + (gr.col0 + gr.ncol - 1) / p->B >= o.noct)
            ck.fail(name, "group out of range", i, gr.level);
    }
    if (ck.ok && covered != o.noct * p->B)
        ck.fail(name, "groups do not cover the columns", covered, o.noct * p->B);
    if (ck.ok && o.nunit != (int64_t)o.ngroup * in.RS)
        ck.fail(name, "units do not match the groups", o.nunit, o.ngroup);
    if (ck.ok && o.wgs > 0 && (wgseg[0] != 0 || wgseg[o.wgs] != o.nseg))
        ck.fail(name, "segment ranges do not cover the segments", wgseg[0], o.nseg);
    if (ck.ok && (uslot[0] != 0 || uslot[o.nunit] != o.nseg))
        ck.fail(name, "unit slots do not cover the segments", uslot[o.nunit], o.nseg);
    for (int64_t u = 0; u < o.nunit && ck.ok; ++u) {
        const OctGroup &gr = groups[u / in.RS];
        uint32_t done = 0;
        for (int32_t j = uslot[u]; j < uslot[u + 1] && ck.ok; ++j) {
            const int32_t sg = slot_seg[j];
            const uint32_t mask = (uint32_t)segs[4 * sg + 1];
            if (segs[4 * sg] != u || mask == 0 || (mask & done) || mask >> kOrbits)
                ck.fail(name, "unit's segments inconsistent", u, sg);
            done |= mask;
        }
        for (int ob = 1; ob <= kOrbits && ck.ok; ++ob)
            for (int64_t c = 0; c < gr.ncol && ck.ok; c += p->B - (gr.col0 + c) % p->B) {
                const uint32_t k = key[gr.oct0 + (gr.col0 + c) / p->B];
                const OctLev &lv = g.lev[gr.level];
                for (int r = 0; r < 8 && ck.ok; ++r) {
                    const int32_t j = octet_place(lv, orbit_coord((int)compact3(k), orbit_axis(ob, 0), r & 1),
                                                  orbit_coord((int)compact3(k >> 1), orbit_axis(ob, 1), r & 2),
                                                  orbit_coord((int)compact3(k >> 2), orbit_axis(ob, 2), r & 4));
                    if (j < 0)
                        continue;
                    if (lv.row0 + j >= nin)
                        ck.fail(name, "input row out of range", lv.row0 + j, nin);
                    if (present && !present(gr.level, j))
                        continue;
                    if (!((done >> (ob - 1)) & 1u))
                        ck.fail(name, "an orbit with a source is in no segment", u, ob);
                }
            }
    }
}

}  // namespace

}  // namespace grav

using namespace grav;

extern "C" grav_status grav_plan_check(grav_plan_t plan, char *msg, int32_t msglen)
{
    if (!plan)
        return GRAV_EINVAL;
    Plan *p = reinterpret_cast<Plan *>(plan);
    Checker ck;
    auto report = [&]() {
        if (msg && msglen > 0) {
            std::snprintf(msg, (size_t)msglen, "%s", ck.ok ? "ok" : ck.msg.c_str());
        }
        return ck.ok ? GRAV_OK : GRAV_EINVAL;
    };
    if (p->M == 0)
        return report();
    int cur = 0;
    GRAV_HIP(hipGetDevice(&cur));
    GRAV_HIP(hipSetDevice(p->device));
    GRAV_HIP(hipDeviceSynchronize());
    const DevGeom g = make_geom(p);
    const int L = p->L;
    int64_t ntb = 0;
    const int lo = L >= 2 ? 2 : L;
    for (int l = lo; l <= L; ++l)
        ntb = std::max<int64_t>(ntb, p->tbox_off[l] + p->lev[l].n_tgt);
    const auto tkey = fetch(p->d_tkey, (size_t)ntb);
    const auto tmap = fetch(p->d_tmap, (size_t)p->n_tmap);
    const auto leaf_start = fetch(p->d_leaf_start, (size_t)p->n_leaf + 1);
    const auto perm = fetch(p->d_perm, (size_t)p->M);
    const auto leaf_pend = fetch(p->d_leaf_pend, (size_t)p->n_leaf);
    const int64_t ncell = (int64_t)p->d.nx * p->d.ny * p->d.nz;
    const auto cell_slot = p->lat_near ? fetch(p->d_cell_slot, (size_t)ncell) : std::vector<int32_t>();
    (void)hipSetDevice(cur);

    // target tables
    for (int64_t i = 0; i < p->n_leaf && ck.ok; ++i)
        if (leaf_start[i] >= leaf_start[i + 1])
            ck.fail("tree", "empty or unordered leaf range", leaf_start[i], leaf_start[i + 1]);
    if (ck.ok && leaf_start[p->n_leaf] != p->M)
        ck.fail("tree", "leaf ranges do not cover the targets", leaf_start[p->n_leaf], p->M);
    std::vector<char> seen(p->M, 0);
    for (int64_t i = 0; i < p->M && ck.ok; ++i) {
        if (perm[i] >= (uint64_t)p->M || seen[perm[i]])
            ck.fail("tree", "permutation not a bijection", perm[i], p->M);
        else
            seen[perm[i]] = 1;
    }
    // user points first within each leaf; voxel-centre slots invert perm
    const int64_t npts = p->lat_near ? p->d.n_points : p->M;
    for (int64_t i = 0; i < p->n_leaf && ck.ok; ++i) {
        const int64_t e = leaf_pend[i];
        if (e < leaf_start[i] || e > leaf_start[i + 1])
            ck.fail("tree", "user-point end outside its leaf", e, i);
        for (int64_t j = leaf_start[i]; j < leaf_start[i + 1] && ck.ok; ++j)
            if (((int64_t)perm[j] < npts) != (j < e))
                ck.fail("tree", "user points not a prefix of their leaf", j, i);
    }
    if (p->lat_near) {
        if ((int64_t)cell_slot.size() != ncell)
            ck.fail("lattice", "cell slots not readable", (long long)cell_slot.size(), ncell);
        for (int64_t c = 0; c < ncell && ck.ok; ++c) {
            const int64_t j = cell_slot[c];
            if (j < 0 || j >= p->M || (int64_t)perm[j] != p->d.n_points + c)
                ck.fail("lattice", "cell slot does not invert the permutation", c, j);
        }
    }
    for (int l = lo; l <= L && ck.ok; ++l) {
        const DevLev &lv = g.lev[l];
        for (int64_t i = 0; i < p->lev[l].n_tgt && ck.ok; ++i) {
            const uint32_t k = tkey[lv.tbox_off + i];
            if (i > 0 && k <= tkey[lv.tbox_off + i - 1])
                ck.fail("tree", "box keys not strictly increasing", l, i);
        }
        // target map entries
        const int64_t msz = (int64_t)(lv.ns[0] + 6) * (lv.ns[1] + 6) * (lv.ns[2] + 6);
        for (int64_t i = 0; i < msz && ck.ok; ++i) {
            const int32_t v = tmap[lv.tmap_off + i];
            if (v < -1 || v >= p->lev[l].n_tgt)
                ck.fail("tmap", "entry out of range", v, p->lev[l].n_tgt);
        }
    }
    // near field / leaf kernels: neighbour leaves within the source block or skipped
    if (ck.ok && L >= 0) {
        const DevLev &lv = g.lev[L];
        for (int64_t i = 0; i < p->n_leaf && ck.ok; ++i) {
            const uint32_t k = tkey[lv.tbox_off + i];
            const int c[3] = {(int)compact3(k), (int)compact3(k >> 1), (int)compact3(k >> 2)};
            for (int a = 0; a < 3; ++a)
                if (c[a] >= (1 << L))
                    ck.fail("leaf", "leaf coordinate outside the root", c[a], 1 << L);
        }
    }

    if (L >= 2 && ck.ok) {
        // the octets of the target and of the source boxes
        const OctGeom fg = octet_geom(p, false), tg = octet_geom(p, true);
        check_octets(ck, "m2l", p, p->m2l, fg, p->n_me, p->n_tbox, nullptr);
        // the gather regions hold every target box within reach and lie in
        // the target maps (source block + halo 3)
        for (int l = 2; l <= L && ck.ok; ++l)
            for (int a = 0; a < 3 && ck.ok; ++a)
                if (tg.lev[l].ns[a] > 0 && (tg.lev[l].s0[a] < p->lev[l].s0[a] - 3 ||
                                            tg.lev[l].s0[a] + tg.lev[l].ns[a] > p->lev[l].s0[a] + p->lev[l].ns[a] + 3))
                    ck.fail("m2lT", "gather region outside the target map", l, a);
        check_octets(ck, "m2lT", p, p->m2lt, tg, p->n_grow, p->n_me, [&](int l, int32_t j) {
            const OctLev &t = tg.lev[l];
            return tmap_lookup(g.lev[l], tmap.data(), 3, t.s0[0] + j % t.ns[0], t.s0[1] + j / t.ns[0] % t.ns[1],
                               t.s0[2] + j / (t.ns[0] * t.ns[1])) >= 0;
        });
    }
    if (L >= 2 && ck.ok) {
        // M2M / M2M^T: every parent of a level >= 3 box lies in the block above
        for (int l = 3; l <= L && ck.ok; ++l) {
            const DevLev &lv = g.lev[l];
            for (int z = 0; z < lv.ns[2] && ck.ok; ++z)
                for (int y = 0; y < lv.ns[1] && ck.ok; ++y)
                    for (int x = 0; x < lv.ns[0] && ck.ok; ++x)
                        if (dense_index(g.lev[l - 1], (lv.s0[0] + x) >> 1, (lv.s0[1] + y) >> 1,
                                        (lv.s0[2] + z) >> 1) < 0)
                            ck.fail("m2mT", "parent outside the source block", l, x);
        }
    }
    // explicit sources: the per-leaf CSR is monotone and covers every
    // source; the permutation is a permutation
    if (ck.ok && p->n_spts > 0) {
        const int64_t nleaf = p->lev[L].n_src;
        const auto st = fetch(p->d_sstart, (size_t)nleaf + 1);
        const auto pm = fetch(p->d_sperm, (size_t)p->n_spts);
        if (st[0] != 0 || st[nleaf] != p->n_spts)
            ck.fail("sources", "leaf ranges do not cover the sources", st[0], st[nleaf]);
        for (int64_t j = 0; j < nleaf && ck.ok; ++j)
            if (st[j + 1] < st[j])
                ck.fail("sources", "leaf ranges out of order", j, st[j]);
        std::vector<char> seen((size_t)p->n_spts, 0);
        for (int64_t i = 0; i < p->n_spts && ck.ok; ++i)
            if (pm[i] >= (uint32_t)p->n_spts || seen[pm[i]]++)
                ck.fail("sources", "sorted order is not a permutation", i, pm[i]);
    }
    return report();
}
