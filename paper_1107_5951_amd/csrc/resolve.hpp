// Index helpers shared by the kernels and the host's plan checks.
#pragma once

#include "eval_common.hpp"

namespace grav {

__host__ __device__ inline int64_t dense_index(const DevLev &lv, int x, int y, int z)
{
    const int sx = x - lv.s0[0], sy = y - lv.s0[1], sz = z - lv.s0[2];
    if (sx < 0 || sy < 0 || sz < 0 || sx >= lv.ns[0] || sy >= lv.ns[1] || sz >= lv.ns[2])
        return -1;
    return ((int64_t)sz * lv.ns[1] + sy) * lv.ns[0] + sx;
}

// Target-box map around a level's source block (halo H): index or -1.
__host__ __device__ inline int64_t tmap_lookup(const DevLev &lv, const int32_t *tmap, int H, int x, int y, int z)
{
    const int mx = lv.ns[0] + 2 * H, my = lv.ns[1] + 2 * H, mz = lv.ns[2] + 2 * H;
    const int sx = x - lv.s0[0] + H, sy = y - lv.s0[1] + H, sz = z - lv.s0[2] + H;
    if (sx < 0 || sy < 0 || sz < 0 || sx >= mx || sy >= my || sz >= mz)
        return -1;
    return tmap[lv.tmap_off + ((int64_t)sz * my + sy) * mx + sx];
}

}  // namespace grav
