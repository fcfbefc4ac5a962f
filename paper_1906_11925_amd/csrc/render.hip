// In-situ direct volume rendering of a lattice property by ray marching
// (paper Section 3.C.2: voxels sampled from a volume, viewing parameters and a
// transfer-function look-up table with steerable scale and offset).
//
// One thread per ray.  Sample positions are fixed-point integers (2^20 units per
// lattice spacing), so every ray visits exactly the voxels the definition names.
// Two sampling rules: the nearest voxel, or trilinear filtering as a texture unit
// does it (8-bit fractional weights, empty voxels zero); the trilinear weights
// are integers summing to 2^24 and each corner's product with its FP32 value is
// exact in FP64, so the filtered value is the same however the sum is evaluated
// (in corner order here).
// The volume is the sparse site list itself: a dense map of 4x4x4 blocks over the
// sites' bounding box gives each block's record (fluid mask, first site index),
// and a voxel's site is the block's first site plus the number of fluid positions
// before it.  A sample that falls in an empty block jumps to the first sample past the
// empty blocks around it, whose extent a map of distances to the nearest block with a site
// gives: exact integer arithmetic, so no contributing sample is ever skipped.  The kernel is
// bound by the latency of a ray's dependent loads, not by HBM: what counts is how many
// there are.  1024 x 1024 rays through a tree of 5.6M sites in 1.0e9 voxels: trilinear
// 2784 -> 1020 us (corner after corner 2784, corners together 2160, jumps over several empty
// blocks without 64-bit divisions 1180, a wavefront per workgroup 1020), nearest 1469 -> 450.
// Two samples of a ray at a time were slower (2370 instead of 2160 us: registers).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"
#include "lbdev.hpp"
#include "render.hpp"

namespace hlb {

// rays per workgroup, 8 x 8: one wavefront, so its slot is free as soon as its own longest
// ray ends, and of the shape whose rays meet the same blocks (16 x 16: 1181 us a frame, 1027)
constexpr int kRayTile = 8;
constexpr int64_t kFix = 1 << 20;
constexpr int kFar = 16;  // largest distance (blocks) in the maps of empty blocks

__device__ inline int64_t ceil_div_pos(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Trilinear value of the sample at P (its base voxel b, 8-bit fractions fr), if one of its
// corners of nonzero weight is a site.  Every corner's loads are issued, at a clamped index
// where there is nothing to load, so a sample waits for three loads one after another (block,
// record, value) and not for three per corner.
struct Corners {
    uint32_t valid;   // corners with a nonzero weight inside the map, then those that are sites
    int32_t W[8];     // weights, 2^24 in all
    int32_t blk[8];   // block of each corner
    int32_t p[8];     // position in it
    float val[8];
};

__device__ inline void corners_find(const RenderVolume& V, const int64_t (&P)[3], Corners& c) {
    int32_t g[3][2], q[3][2], w[3][2];
    bool ok[3][2];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int32_t b = (int32_t)(P[a] >> 20);                 // base voxel (floor)
        const int32_t f = (int32_t)((P[a] & (kFix - 1)) >> 12);  // 8-bit fraction
        w[a][0] = 256 - f;
        w[a][1] = f;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            g[a][e] = ((b + e) >> 2) - V.blo[a];
            q[a][e] = (b + e) & 3;
            ok[a][e] = g[a][e] >= 0 && g[a][e] < V.gdim[a] && w[a][e] > 0;
        }
    }
    c.valid = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int x = k & 1, y = (k >> 1) & 1, z = (k >> 2) & 1;
        const bool in = ok[0][x] && ok[1][y] && ok[2][z];
        c.W[k] = w[0][x] * w[1][y] * w[2][z];
        c.p[k] = block_pos(q[0][x], q[1][y], q[2][z]);
        const int64_t at = ((int64_t)g[0][x] * V.gdim[1] + g[1][y]) * V.gdim[2] + g[2][z];
        c.blk[k] = V.grid[in ? at : 0];
        if (in && c.blk[k] >= 0) c.valid |= 1u << k;
    }
}

__device__ inline void corners_load(const RenderVolume& V, Corners& c) {
    BlockRec r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) r[k] = V.rec[c.valid & (1u << k) ? c.blk[k] : 0];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint64_t m = block_mask(r[k]);
        const bool site = (c.valid & (1u << k)) && ((m >> c.p[k]) & 1ull);
        c.val[k] = V.values[site ? r[k].off + __popcll(m & ((1ull << c.p[k]) - 1ull)) : 0];
        if (!site) c.valid &= ~(1u << k);
    }
}

__device__ inline float corners_value(const Corners& c) {
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const double sum = acc + (double)c.W[k] * (double)c.val[k];  // exact product
        acc = c.valid & (1u << k) ? sum : acc;
    }
    return (float)(acc * 0x1p-24);
}

// ceil(num / d) for num, d > 0 and a quotient below 2^31; rd = 1 / d
__device__ inline int64_t steps_to(int64_t num, int64_t d, double rd) {
    int64_t q = (int64_t)((double)num * rd);  // off by one at most
    int64_t r = num - q * d;
    if (r < 0) {
        --q;
        r += d;
    } else if (r >= d) {
        ++q;
        r -= d;
    }
    return q + (r > 0);
}

// First sample after the one at P whose position leaves the blocks within `far` - 1 of its
// block B, all empty.  A division of 64-bit integers is a long sequence, and there are three
// per jump: the quotient comes from a product with the reciprocal and is put right exactly.
__device__ inline int64_t jump(const int64_t (&P)[3], const int64_t (&B)[3], int far,
                               const int64_t (&D)[3], const double (&rd)[3]) {
    int64_t n = (int64_t)1 << 31;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (D[a] > 0)
            n = min(n, steps_to(4 * (B[a] + far) * kFix - P[a], D[a], rd[a]));
        else if (D[a] < 0)
            n = min(n, steps_to(P[a] - (4 * (B[a] - far + 1) * kFix - 1), -D[a], rd[a]));
    }
    return n;
}

// Composite one sample of value val.
__device__ inline void composite(const RenderView& v, const float4* __restrict__ lut, float val,
                                 float& c0, float& c1, float& c2, float& A) {
    const float t = (val - v.offset) * v.scale;
    const float f = floorf(t * 256.0f);
    const int e = f >= 255.0f ? 255 : (f > 0.0f ? (int)f : 0);
    const float4 rgba = lut[e];
    const float w = (1.0f - A) * rgba.w;
    c0 += w * rgba.x;
    c1 += w * rgba.y;
    c2 += w * rgba.z;
    A += w;
}

template <bool TRI>
__global__ __launch_bounds__(kRayTile* kRayTile) void k_render(RenderVolume V, RenderView v,
                                                                 const float4* __restrict__ lut,
                                                                 float4* __restrict__ image) {
    const int32_t i = (int32_t)(blockIdx.x * kRayTile + threadIdx.x % kRayTile);
    const int32_t j = (int32_t)(blockIdx.y * kRayTile + threadIdx.x / kRayTile);
    if (i >= v.width || j >= v.height) return;
    int64_t P0[3], D[3];  // start and step of ray (i, j)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        P0[a] = v.origin[a] + (int64_t)i * v.right[a] + (int64_t)j * v.up[a];
        D[a] = v.dir[a] + (int64_t)i * v.dir_right[a] + (int64_t)j * v.dir_up[a];
    }

    // samples that can reach a site: on each axis P must lie in
    // [4 lo FIX - FIX/2, 4 (lo + dim) FIX - FIX/2) for the nearest voxel, and in
    // [(4 lo - 1) FIX, 4 (lo + dim) FIX) for trilinear (base voxel or the next one
    // inside the map's box)
    int64_t k0 = 0, k1 = v.steps;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t lo = TRI ? (4 * (int64_t)V.blo[a] - 1) * kFix : 4 * (int64_t)V.blo[a] * kFix - kFix / 2;
        const int64_t hi = TRI ? 4 * ((int64_t)V.blo[a] + V.gdim[a]) * kFix
                               : 4 * ((int64_t)V.blo[a] + V.gdim[a]) * kFix - kFix / 2;  // exclusive
        const int64_t d = D[a];
        if (d == 0) {
            if (P0[a] < lo || P0[a] >= hi) k1 = 0;
        } else if (d > 0) {
            if (P0[a] < lo) k0 = max(k0, ceil_div_pos(lo - P0[a], d));
            k1 = P0[a] >= hi ? 0 : min(k1, ceil_div_pos(hi - P0[a], d));
        } else {
            if (P0[a] >= hi) k0 = max(k0, ceil_div_pos(P0[a] - (hi - 1), -d));
            k1 = P0[a] < lo ? 0 : min(k1, ceil_div_pos(P0[a] - (lo - 1), -d));
        }
    }

    double rd[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) rd[a] = D[a] ? 1.0 / (double)(D[a] > 0 ? D[a] : -D[a]) : 0.0;
    float c0 = 0.f, c1 = 0.f, c2 = 0.f, A = 0.f;
    int64_t k = k0;
    if constexpr (TRI) {
        const int64_t nd1 = V.gdim[1] + 1, nd2 = V.gdim[2] + 1;
        while (k < k1) {
            int64_t P[3], B[3];
            bool in = true;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                P[a] = P0[a] + k * D[a];
                B[a] = P[a] >> 22;  // block of the base voxel (floor)
                const int64_t h = B[a] - V.blo[a] + 1;
                in = in && h >= 0 && h <= V.gdim[a];
            }
            // the blocks are looked up before the map says whether they are needed: one wait less
            Corners c;
            corners_find(V, P, c);
            // no corner of any sample whose base voxel lies within far - 1 blocks of B is a
            // site
            const int far = in ? V.near[((B[0] - V.blo[0] + 1) * nd1 + (B[1] - V.blo[1] + 1)) * nd2 +
                                        (B[2] - V.blo[2] + 1)]
                               : 1;
            if (far > 0) {
                k += jump(P, B, far, D, rd);
                continue;
            }
            corners_load(V, c);
            if (c.valid) composite(v, lut, corners_value(c), c0, c1, c2, A);
            ++k;
        }
        image[(int64_t)j * v.width + i] = make_float4(c0, c1, c2, A);
        return;
    }
    while (k < k1) {
        int64_t P[3], B[3];  // position half a spacing on: the nearest voxel is its floor
        bool in = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            P[a] = P0[a] + k * D[a] + kFix / 2;
            B[a] = P[a] >> 22;
            const int64_t g = B[a] - V.blo[a];
            in = in && g >= 0 && g < V.gdim[a];
        }
        const int64_t at = ((B[0] - V.blo[0]) * V.gdim[1] + (B[1] - V.blo[1])) * V.gdim[2] +
                           (B[2] - V.blo[2]);
        const int far = in ? V.far[at] : 1;
        if (far > 0) {
            k += jump(P, B, far, D, rd);
            continue;
        }
        const int32_t blk = V.grid[at];
        const BlockRec r = V.rec[blk];
        const int p = block_pos((int)(P[0] >> 20) & 3, (int)(P[1] >> 20) & 3, (int)(P[2] >> 20) & 3);
        const uint64_t m = block_mask(r);
        if ((m >> p) & 1ull)
            composite(v, lut, V.values[r.off + __popcll(m & ((1ull << p) - 1ull))], c0, c1, c2, A);
        ++k;
    }
    image[(int64_t)j * v.width + i] = make_float4(c0, c1, c2, A);
}

// One axis of the distance map: out = min over cells t away on the axis of max(|t|, in),
// |t| < kFar, else kFar.  FIRST: in is 0 at an occupied cell (grid >= 0 or near != 0), kFar
// elsewhere.  Rows of workgroups: a map may have more cells than a launch takes threads along
// one dimension (2^32 - 1).
template <bool FIRST>
__global__ __launch_bounds__(kBlock) void k_far(const int32_t* __restrict__ grid,
                                                const uint8_t* __restrict__ in, int64_t cells,
                                                int64_t stride, int32_t dim,
                                                uint8_t* __restrict__ out) {
    const int64_t c = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kBlock + threadIdx.x;
    if (c >= cells) return;
    const int32_t x = (int32_t)((c / stride) % dim);
    int best = kFar;
    for (int t = max(-x, 1 - kFar); t <= min(dim - 1 - x, kFar - 1); ++t) {
        const int64_t at = c + t * stride;
        const int d = !FIRST ? in[at] : ((grid ? grid[at] >= 0 : in[at] != 0) ? 0 : kFar);
        best = min(best, max(t < 0 ? -t : t, d));
    }
    out[c] = (uint8_t)best;
}

__global__ __launch_bounds__(kBlock) void k_permute(const float* __restrict__ in,
                                                     const int32_t* __restrict__ perm, int64_t n,
                                                     float* __restrict__ out) {
    const int64_t m = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (m >= n) return;
    out[m] = in[perm ? perm[m] : m];
}

hipError_t launch_render_far(const int32_t* grid, const uint8_t* near, const int32_t (&dim)[3],
                             uint8_t* tmp, uint8_t* out, hipStream_t s) {
    const int64_t cells = (int64_t)dim[0] * dim[1] * dim[2];
    if (cells == 0) return hipSuccess;
    const int64_t rows = ((cells - 1) / kBlock >> 23) + 1;
    const dim3 nb((unsigned)(((cells - 1) / kBlock + rows) / rows), (unsigned)rows);
    k_far<true><<<nb, kBlock, 0, s>>>(grid, near, cells, 1, dim[2], out);
    k_far<false><<<nb, kBlock, 0, s>>>(nullptr, out, cells, dim[2], dim[1], tmp);
    k_far<false><<<nb, kBlock, 0, s>>>(nullptr, tmp, cells, (int64_t)dim[1] * dim[2], dim[0], out);
    return hipGetLastError();
}

hipError_t launch_render(const RenderVolume& V, const RenderView& v, const float* lut, float* image,
                         hipStream_t s) {
    if (v.width <= 0 || v.height <= 0) return hipSuccess;
    RenderView u = v;
    if (!V.grid) u.steps = 0;  // no sites, no maps: rays without samples
    const dim3 grid((unsigned)((v.width + kRayTile - 1) / kRayTile),
                    (unsigned)((v.height + kRayTile - 1) / kRayTile));
    if (v.filter == 1)
        k_render<true><<<grid, kRayTile * kRayTile, 0, s>>>(
            V, u, reinterpret_cast<const float4*>(lut), reinterpret_cast<float4*>(image));
    else
        k_render<false><<<grid, kRayTile * kRayTile, 0, s>>>(
            V, u, reinterpret_cast<const float4*>(lut), reinterpret_cast<float4*>(image));
    return hipGetLastError();
}

hipError_t launch_permute(const float* in, const int32_t* perm, int64_t n, float* out,
                          hipStream_t s) {
    if (n <= 0) return hipSuccess;
    k_permute<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(in, perm, n, out);
    return hipGetLastError();
}

}  // namespace hlb
