// Internal launch interface of the volume renderer.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace hlb {

// Block map of the rendered volume: grid[(gx * gdim[1] + gy) * gdim[2] + gz] is the
// record index of block (blo + g), or -1 where no site lies; rec[k] holds that
// block's fluid mask and first site; values holds one value per site (site order).
// far[g] is the distance, in blocks along the axis where it is largest and 16 at most, from
// block blo + g to the nearest that holds a site; near[(hx * (gdim[1] + 1) + hy) * (gdim[2]
// + 1) + hz] likewise from block blo - 1 + h to the nearest from which a trilinear sample
// reaches a site, that is, with one among it + {0, 1}^3 that holds a site.
struct RenderVolume {
    const int32_t* grid;
    const BlockRec* rec;
    const float* values;
    const uint8_t* near;
    const uint8_t* far;
    int32_t blo[3];
    int32_t gdim[3];
};

// Fixed-point view (2^20 units per lattice spacing), as in hemelb_view_t.
struct RenderView {
    int64_t origin[3];
    int64_t right[3];
    int64_t up[3];
    int64_t dir[3];
    int64_t dir_right[3], dir_up[3];  // ray (i, j) steps dir + i dir_right + j dir_up
    int32_t width, height, steps;
    float scale, offset;
    int32_t filter;  // 0: nearest voxel, 1: trilinear
};

// image [height][width][4] of the volume seen through view v; lut: device [256][4]
hipError_t launch_render(const RenderVolume& V, const RenderView& v, const float* lut, float* image,
                         hipStream_t s);

// Distance map of dim[0] x dim[1] x dim[2] cells into out: from each to the nearest with
// grid >= 0, or near != 0 where grid is null.  tmp: as many bytes, near itself if need be.
#ifdef HLB_NO_DEVICE  // host-only builds of the planner: no kernels to launch
inline hipError_t launch_render_far(const int32_t*, const uint8_t*, const int32_t (&)[3], uint8_t*,
                                    uint8_t*, hipStream_t) {
    return hipErrorNoDevice;
}
#else
hipError_t launch_render_far(const int32_t* grid, const uint8_t* near, const int32_t (&dim)[3],
                             uint8_t* tmp, uint8_t* out, hipStream_t s);
#endif

// out[m] = in[perm[m]] (perm null: identity), m < n
hipError_t launch_permute(const float* in, const int32_t* perm, int64_t n, float* out,
                          hipStream_t s);

}  // namespace hlb
