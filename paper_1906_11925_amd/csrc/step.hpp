// The fused pull-stream + LBGK-collide step of one site and one workgroup, shared
// by the step kernel and the adjoint's recompute.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"
#include "lattice.hpp"
#include "lbdev.hpp"

namespace hlb {

// ---------------------------------------------------------------------------
// fused pull stream + LBGK collide
// ---------------------------------------------------------------------------
// Build-time tuning knobs (every variant computes the same result):
//   HLB_NT_STORE  nontemporal stores of the post-collision populations
//   HLB_NT_TABLE  nontemporal loads of the neighbour table
#ifndef HLB_NT_STORE
#define HLB_NT_STORE 1
#endif
#ifndef HLB_NT_TABLE
#define HLB_NT_TABLE 1
#endif
// One workgroup covers one group of four tiles (the unit of the staged block
// records).  Groups of 8 or 16 tiles per workgroup (more neighbours sharing one
// L1) measured no faster with the explicit tables.
constexpr int kScBlock = 4 * kTile;

template <class T>
__device__ inline void st_pop(T* p, T v) {
#if HLB_NT_STORE
    __builtin_nontemporal_store(v, p);
#else
    *p = v;
#endif
}

// Incoming population of an iolet link (direction i; its iolet's kind and value v, the
// link's coefficient) of a site whose stored populations decode to vs (the definition the
// ghost-fill kernel applies).  Both the step kernel's epilogue and the ghost-fill kernel
// inline it; without contraction every product and sum rounds on its own in both, so a
// state restored from a checkpoint gets the same ghost values, bit for bit, as the step that
// produced it (the moment sums it calls multiply only by 0 and +-1, which is exact either
// way).
template <int Q>
__device__ inline float ghost_value(int kind, double v, float coef, int i, const float (&vs)[Q]) {
#pragma clang fp contract(off)
    using Lt = Lat<Q>;
    if (kind == 0) {
        float drho, mx, my, mz;
        moments<Q>(vs, drho, mx, my, mz);
        const float ir = 1.0f / (1.0f + drho);
        const float ux = mx * ir, uy = my * ir, uz = mz * ir;
        const float cu = (float)Lt::cx[i] * ux + (float)Lt::cy[i] * uy + (float)Lt::cz[i] * uz;
        const float usq = ux * ux + uy * uy + uz * uz;
        const float rk = (float)v, rk1 = (float)(v - 1.0);
        return Lt::w[i] * (rk1 + rk * (3.0f * cu + 4.5f * cu * cu - 1.5f * usq));
    }
    return vs[opp(i)] + coef * (float)v;
}
// the same for iolet link l at time t; a velocity iolet's coefficient alone is loaded
template <int Q>
__device__ inline float ghost_value(const Ghosts& G, int64_t l, int i, const float (&vs)[Q],
                                    int64_t t) {
    const int k = G.iolet[l];
    const double v = G.vals[(t - G.vals_t0) * G.n_iolets + k];
    const int kind = G.iolets[k].kind;
    return ghost_value<Q>(kind, v, kind == 0 ? 0.f : G.coef[l], i, vs);
}

// With HLB_FUSE_GHOSTS, a site that owns iolet links also writes the incoming
// populations of those links for the next step (time t_next) into dst's ghost
// slots, from its freshly stored populations; the separate ghost fill is then
// only needed for a state that did not come out of this kernel.
#ifndef HLB_FUSE_GHOSTS
#define HLB_FUSE_GHOSTS 1
#endif

// The pulled (pre-collision) deviations of one site and what the epilogue needs
// about its iolet links.
template <int Q>
struct Pulled {
    float d[Q];
    uint32_t gmask;  // directions of the site's iolet links (fused ghost epilogue)
    int64_t gl;      // the first of those links
};

// Pull the populations of site s whose links are decoded in j; load(dir, site) gives the
// stored value.
template <int Q, int ST, bool SC, bool BFL, class Load>
__device__ inline void site_pull(const typename Store<ST>::T* __restrict__ src, int32_t n,
                                 const Ghosts& G, int32_t s, const int32_t (&j)[Q], Pulled<Q>& P,
                                 Load&& load) {
    using C = Codec<Q, ST, SC>;
    P.d[0] = C::dec(0, load(0, s));
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        int dir;
        int32_t site;
        link_src(i, j[i], s, dir, site);
        P.d[i] = C::dec(i, load(dir, site));
    }
    if constexpr (BFL) apply_bfl<Q, ST, SC>(src, s, n, j, P.d);
    P.gmask = 0;
    P.gl = -1;
#if HLB_FUSE_GHOSTS
    // directions of the site's iolet links and the first of those links (they are
    // consecutive in the link list, in direction order), for the epilogue
    int32_t top = j[1];  // walls are negative, sites below n, ghost slots from n
#pragma unroll
    for (int i = 2; i < Q; ++i) top = max(top, j[i]);
    if (top >= n) {
#pragma unroll
        for (int i = 1; i < Q; ++i) P.gmask |= j[i] >= n ? 1u << i : 0u;
        const int first = __builtin_ctz(P.gmask);
        int32_t slot = 0;
#pragma unroll
        for (int i = 1; i < Q; ++i) slot = i == first ? j[i] : slot;
        P.gl = ghost_link<Q>(G, n, slot, first);
    }
#else
    (void)G;
#endif
}

// Post-collision populations e (in storage format) of site s from the pulled ones.
template <int Q, int ST, bool SC, bool BRINK>
__device__ inline void site_collide(const float (&d)[Q], float omega,
                                    const float* __restrict__ alpha, int32_t s,
                                    typename Store<ST>::T (&e)[Q]) {
    using C = Codec<Q, ST, SC>;
    float drho, mx, my, mz;
    moments<Q>(d, drho, mx, my, mz);
    const float rho = 1.0f + drho;
    const float ir = 1.0f / rho;
    float ux = mx * ir, uy = my * ir, uz = mz * ir;
    if constexpr (BRINK) {
        const float a = 1.0f - alpha[s];
        ux *= a;
        uy *= a;
        uz *= a;
    }
    float deq[Q];
    eq_dev<Q>(drho, rho, ux, uy, uz, deq);
#pragma unroll
    for (int i = 0; i < Q; ++i) e[i] = C::enc(i, d[i] - omega * (d[i] - deq[i]));
}

// Collide the pulled populations of site s and store them (and, with the fused
// ghost epilogue, the incoming populations of its iolet links for time t_next).
// FOUT: also store the pulled populations themselves into fout, in the site's own
// slots, for the reverse sweep (exact: each is a stored value decoded; halfway
// walls only).
template <int Q, int ST, bool SC, bool BRINK, bool FOUT = false>
__device__ inline void site_collide_store(typename Store<ST>::T* __restrict__ dst, int32_t n,
                                          float omega, const float* __restrict__ alpha,
                                          const Ghosts& G, int64_t t_next, int32_t s,
                                          const Pulled<Q>& P,
                                          typename Store<ST>::T* __restrict__ fout) {
    using C = Codec<Q, ST, SC>;
    const float(&d)[Q] = P.d;
    if constexpr (FOUT) {
#pragma unroll
        for (int i = 0; i < Q; ++i) st_pop(fout + tix<Q>(i, s), C::enc(i, d[i]));
    } else {
        (void)fout;
    }
    typename Store<ST>::T e[Q];
    site_collide<Q, ST, SC, BRINK>(d, omega, alpha, s, e);
    float vs[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        st_pop(dst + tix<Q>(i, s), e[i]);
        vs[i] = C::dec(i, e[i]);
    }
#if HLB_FUSE_GHOSTS
    // The iolet links of a site are consecutive in the link list, in direction
    // order.  With one slot per link (table encodings) the first one is the
    // smallest ghost slot the site pulls from; with shared ghost cells (block
    // addressing) it is found through the cell's link list.
    // The few workgroups with iolet sites set the length of a small lattice's step: what
    // kLinkBatch links name is loaded at once, and what the first link's iolet names only
    // once (a link of another iolet loads its own).  With the ghost records in LDS
    // (staged_refs) a single step of a tree of 8k sites went from 10.8 to 8.6 us, of 61k
    // from 11.9 to 9.1, of a 13k-site pipe from 8.4 to 7.5.
    if (P.gmask) {
        const int64_t at = (t_next - G.vals_t0) * G.n_iolets;
        const int k0 = G.iolet[P.gl];
        const int kind0 = G.iolets[k0].kind;
        const double val0 = G.vals[at + k0];
        int64_t l = P.gl;
#pragma unroll
        for (int i0 = 1; i0 < Q; i0 += kLinkBatch) {
            int kio[kLinkBatch];
            int32_t slot[kLinkBatch];
            float coef[kLinkBatch];
#pragma unroll
            for (int i = i0; i < i0 + kLinkBatch && i < Q; ++i)
                if (P.gmask & (1u << i)) {
                    kio[i - i0] = G.iolet[l];
                    slot[i - i0] = ghost_slot(G, n, l);
                    coef[i - i0] = G.coef[l];
                    ++l;
                }
#pragma unroll
            for (int i = i0; i < i0 + kLinkBatch && i < Q; ++i)
                if (P.gmask & (1u << i)) {
                    const int k = kio[i - i0];
                    const float v = ghost_value<Q>(k == k0 ? kind0 : G.iolets[k].kind,
                                                   k == k0 ? val0 : G.vals[at + k], coef[i - i0], i,
                                                   vs);
                    dst[tix<Q>(i, slot[i - i0])] = C::enc(i, v);
                }
        }
    }
#else
    (void)vs;
    (void)G;
    (void)t_next;
    (void)n;
#endif
}

// Pull, collide and store one site whose links are decoded in j.
template <int Q, int ST, bool SC, bool BRINK, bool BFL, bool FOUT = false>
__device__ inline void site_update(const typename Store<ST>::T* __restrict__ src,
                                   typename Store<ST>::T* __restrict__ dst, int32_t n, float omega,
                                   const float* __restrict__ alpha, const Ghosts& G,
                                   int64_t t_next, int32_t s, const int32_t (&j)[Q],
                                   typename Store<ST>::T* __restrict__ fout) {
    Pulled<Q> P;
    site_pull<Q, ST, SC, BFL>(src, n, G, s, j, P,
                              [&](int dir, int32_t site) { return src[tix<Q>(dir, site)]; });
    site_collide_store<Q, ST, SC, BRINK, FOUT>(dst, n, omega, alpha, G, t_next, s, P, fout);
}

// Block ids are dealt round-robin to the 8 XCDs (each with its own L2).  With
// groups of G > 0, every XCD takes G consecutive blocks of a window of 8G
// blocks, so neighbouring sites share an L2 while all XCDs still sweep the
// Morton order together (and share the last-level cache).  code (xcd_code): G, or
// -1 - log2 G for a power of two, which needs no division.
__device__ inline int32_t xcd_block(int32_t b, int32_t code) {
    if (code < 0) {
        const int32_t sh = -1 - code, w = 8 << sh;
        return (b & -w) + ((b & 7) << sh) + ((b >> 3) & ((1 << sh) - 1));
    }
    if (code > 0) {
        const int32_t w = 8 * code;
        b = (b / w) * w + (b & 7) * code + (b >> 3) % code;
    }
    return b;
}
inline int32_t xcd_code(int32_t group) {
    return group > 0 && (group & (group - 1)) == 0 ? -1 - __builtin_ctz((unsigned)group) : group;
}

// One workgroup (group g of four tiles) of the fused step.  Every thread of the
// workgroup calls it.  FOUT: also store the pulled populations into fout.
template <int Q, int ST, bool SC, bool BRINK, bool BFL, bool FOUT = false>
__device__ inline void stream_collide_group(const typename Store<ST>::T* __restrict__ src,
                                            typename Store<ST>::T* __restrict__ dst,
                                            const Table& tb, int32_t n, int32_t g, float omega,
                                            const float* __restrict__ alpha, const Ghosts& G,
                                            int64_t t_next, StageLds& lds, LinkLds<Q>& links,
                                            typename Store<ST>::T* __restrict__ fout = nullptr) {
    constexpr int SZ = sizeof(typename Store<ST>::T);
    if (g * kScBlock >= n) return;  // the whole workgroup lies past the end
    const int32_t s = g * kScBlock + (int32_t)threadIdx.x;
    const bool live = (s & ~(kTile - 1)) < n;  // the wavefront's tile has sites
    if constexpr (!BFL) {
        if (tb.grp)
            stage_links<Q>(__builtin_amdgcn_readfirstlane((int)threadIdx.x >> kTileShift),
                           (int)threadIdx.x & (kTile - 1), links);
        const StageHdr h = tb.grp ? stage_header(tb, g) : StageHdr{0, 0, 0, false};
        if (h.nown > 0) {
            const int64_t base = group_base(tb.wide, 4 * g, Q);
            stage(tb, h, g, (int)threadIdx.x, lds);
            lds_loads_done();
            __syncthreads();
            if (s >= n) return;
            const uint32_t own = slot_ref<Q, SZ>(s, (uint32_t)base);
            uint32_t e[Q];
            Pulled<Q> P;
            staged_refs<Q, SZ>(tb, h, (int)threadIdx.x, (uint32_t)base, own, lds, links, e,
                                P.gmask);
            refs_gather<Q, ST, SC>(src, base, own, e, P.d);
            P.gl = P.gmask ? staged_link<Q, SZ>(G, n, base, e, 0u, P.gmask) : -1;
            site_collide_store<Q, ST, SC, BRINK, FOUT>(dst, n, omega, alpha, G, t_next, s, P, fout);
            return;
        }
    }
    // all link decoding, then all population gathers, before any arithmetic
    if (!live) return;
    int32_t j[Q];
    links_wave<Q, HLB_NT_TABLE != 0>(tb, s, j);
    if (s >= n) return;
    site_update<Q, ST, SC, BRINK, BFL, FOUT>(src, dst, n, omega, alpha, G, t_next, s, j, fout);
}

// The fused step for a workgroup of W consecutive tiles (64 W threads) that first
// copies its own tiles' populations into LDS with coalesced loads: a link whose
// upstream site (or ghost slot) lies in those tiles reads LDS, any other reads
// global memory, so each wavefront's gathers touch only the lines of tiles outside
// the workgroup.  Block addressing, halfway walls.  Every thread calls it.  With DMA
// the copy uses loads that write LDS directly; pops must then be 16-byte aligned.
template <int Q, int ST, bool SC, bool BRINK, int W, bool DMA = false, bool FOUT = false>
__device__ inline void stream_collide_staged(const typename Store<ST>::T* __restrict__ src,
                                             typename Store<ST>::T* __restrict__ dst,
                                             const Table& tb, int32_t n, int32_t tiles_alloc,
                                             int32_t T0, float omega,
                                             const float* __restrict__ alpha, const Ghosts& G,
                                             int64_t t_next,
                                             typename Store<ST>::T (&pops)[W][Q][kTile],
                                             StageLds (&lds)[W / 4], LinkLds<Q>& links,
                                             typename Store<ST>::T* __restrict__ fout = nullptr) {
    using T = typename Store<ST>::T;
    using C = Codec<Q, ST, SC>;
    constexpr int SZ = sizeof(T), kRow = kRowSize<SZ>, kTileBytes = Q * kRow;
    static_assert(W * kTileBytes + kRow <= ((int64_t)1 << 32) - kRefSpan * 4,
                  "a reference below lo must not wrap into the span");
    if (((int64_t)T0 << kTileShift) >= n) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> kTileShift);
    const int lane = (int)threadIdx.x & (kTile - 1);
    const int32_t staged = min(W, tiles_alloc - T0);  // tiles of the array in this workgroup
    stage_links<Q>(wave, lane, links);
    if (wave < staged) {
        if constexpr (DMA) {
            // A tile's Q rows are one contiguous block, in memory as in LDS: copy it
            // with 16 bytes per lane per load, written straight into LDS (no
            // registers, no LDS store instructions).
            constexpr int kBytes = kTileBytes;
            const char* gp = reinterpret_cast<const char*>(src + (int64_t)(T0 + wave) * (Q * kTile));
            char* l = reinterpret_cast<char*>(&pops[wave][0][0]);
#pragma unroll
            for (int c = 0; c < (kBytes + 1023) / 1024; ++c)
                if (c * 1024 + lane * 16 < kBytes)
                    load_lds16(gp + c * 1024 + lane * 16, l + c * 1024);
        } else {
            const int32_t s = ((T0 + wave) << kTileShift) + lane;
#pragma unroll
            for (int i = 0; i < Q; ++i) pops[wave][i][lane] = src[tix<Q>(i, s)];
        }
    }
    // this thread's group of four tiles; the group's 256 threads stage its records
    const int32_t g = (T0 >> 2) + (wave >> 2);
    const int t = (int)threadIdx.x & (kScBlock - 1);
    StageLds& map = lds[wave >> 2];
    StageHdr h{0, 0, 0, false};
    if (((int64_t)g << 8) < n) h = stage_header(tb, g);
    StageHdr hs = h;
    if (h.far) hs.nown = h.far;
    if (hs.nown > 0) stage(tb, hs, g, t, map);
    const int64_t base = group_base(tb.wide, 4 * g, Q);
    lds_loads_done();
    __syncthreads();
    const int32_t s = (T0 << kTileShift) + (int32_t)threadIdx.x;
    if ((s & ~(kTile - 1)) >= n) return;
    if (__builtin_expect(h.nown == 0, 0)) {  // out of the way of the others' code: 0.1%
        int32_t j[Q];
        if (h.far) {
            if (s >= n) return;
            staged_slots<Q>(tb, hs, t, map, links, j);
            // From LDS what lies in these tiles: 395M sites, where 8% of the groups are such,
            // 9250 us a step with all of it from memory, so 9080.  Not in the forms that no
            // such lattice runs by default.
            if constexpr (DMA && !FOUT) {
                Pulled<Q> P;
                site_pull<Q, ST, SC, false>(src, n, G, s, j, P, [&](int dir, int32_t site) {
                    const uint32_t w = (uint32_t)((site >> kTileShift) - T0);
                    return w < (uint32_t)staged ? pops[w][dir][site & (kTile - 1)]
                                                : src[tix<Q>(dir, site)];
                });
                site_collide_store<Q, ST, SC, BRINK>(dst, n, omega, alpha, G, t_next, s, P, fout);
                return;
            }
        } else {
            links_blocks_wave<Q>(tb, s, j);
            if (s >= n) return;
        }
        site_update<Q, ST, SC, BRINK, false, FOUT>(src, dst, n, omega, alpha, G, t_next, s, j, fout);
        return;
    }
    if (s >= n) return;
    const char* sb = reinterpret_cast<const char*>(src + base);
    const char* pb = reinterpret_cast<const char*>(&pops[0][0][0]);
    const uint32_t lo = (uint32_t)((int64_t)T0 * (Q * kTile) - base) * SZ;
    const uint32_t span = (uint32_t)(staged * kTileBytes + kRow);
    const uint32_t own = (uint32_t)(wave * kTileBytes + kRow + lane * SZ);  // from lo
    uint32_t e[Q];  // from lo
    Pulled<Q> P;
    staged_refs<Q, SZ>(tb, h, t, (uint32_t)base + (uint32_t)(lo / SZ), own, map, links, e,
                        P.gmask);
    P.d[0] = C::dec(0, pops[wave][0][lane]);
    // LDS first, then the lanes whose source lies outside the workgroup overwrite
    T v[Q];
#pragma unroll
    for (int i = 1; i < Q; ++i)
        v[i] = *reinterpret_cast<const T*>(pb + (e[i] < span ? e[i] : own) + (i - 1) * kRow);
#pragma unroll
    for (int i = 1; i < Q; ++i)
        if (e[i] >= span) v[i] = *reinterpret_cast<const T*>(sb + (e[i] + lo) + (i - 1) * kRow);
#pragma unroll
    for (int i = 1; i < Q; ++i) P.d[i] = C::dec(i, v[i]);
    P.gl = P.gmask ? staged_link<Q, SZ>(G, n, base, e, lo, P.gmask) : -1;
    site_collide_store<Q, ST, SC, BRINK, FOUT>(dst, n, omega, alpha, G, t_next, s, P, fout);
}

}  // namespace hlb
