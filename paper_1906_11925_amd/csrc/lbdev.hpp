// Device helpers shared by the forward and adjoint kernels: template dispatch,
// tiled indexing, table decoding, moments, equilibrium and iolet time series.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"
#include "lattice.hpp"

namespace hlb {

template <int Q_, int ST_, bool SC_>
struct Tag {
    static constexpr int Q = Q_;
    static constexpr int ST = ST_;
    static constexpr bool SC = SC_;
};

template <class F>
inline hipError_t dispatch(int q, int st, bool scaled, F&& f) {
    if (q == 15) {
        if (st == ST_F32) return f(Tag<15, ST_F32, false>{});
        if (st == ST_F16) return scaled ? f(Tag<15, ST_F16, true>{}) : f(Tag<15, ST_F16, false>{});
        if (st == ST_BF16) return scaled ? f(Tag<15, ST_BF16, true>{}) : f(Tag<15, ST_BF16, false>{});
    } else if (q == 19) {
        if (st == ST_F32) return f(Tag<19, ST_F32, false>{});
        if (st == ST_F16) return scaled ? f(Tag<19, ST_F16, true>{}) : f(Tag<19, ST_F16, false>{});
        if (st == ST_BF16) return scaled ? f(Tag<19, ST_BF16, true>{}) : f(Tag<19, ST_BF16, false>{});
    }
    return hipErrorInvalidValue;
}

// element (direction i, site s) of a tiled array with R rows per tile
template <int R>
__device__ inline int64_t tix(int i, int32_t s) {
    return ((int64_t)(s >> kTileShift) * R + i) * kTile + (s & (kTile - 1));
}

// decode a table entry j for direction i of site s: (source direction, source site).
// A wall link (bit 31 set) reads the opposite population of the site itself; its
// low 15 bits hold the interpolated-wall fraction (0: halfway bounce-back).
__device__ inline void link_src(int i, int32_t j, int32_t s, int& dir, int32_t& site) {
    const bool wall = j < 0;
    dir = wall ? opp(i) : i;
    site = wall ? s : j;
}

// Interpolated (BFL, linear) walls on gathered pre-collision deviations d: for a
// wall link i with fraction q = code / 2^15 (o = opp(i), d[i] holding A[o][s]):
//   q <  1/2: d_i = 2q A[o][s] + (1 - 2q) A[o][s + c_i]   (the value pulled for o,
//             when link o is a fluid link; halfway bounce-back otherwise)
//   q >= 1/2: d_i = A[o][s] / (2q) + (2q - 1)/(2q) A[i][s]
// The weights sum to one, so the rule applies to deviations unchanged.
template <int Q, int ST, bool SC>
__device__ inline void apply_bfl(const typename Store<ST>::T* __restrict__ A, int32_t s, int32_t n,
                                 const int32_t (&j)[Q], float (&d)[Q]) {
    using C = Codec<Q, ST, SC>;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const int32_t code = j[i] & 0x7fff;
        if (j[i] < 0 && code != 0) {
            const int o = opp(i);
            const float q = (float)code * (1.0f / 32768.0f);
            const float bb = d[i];
            if (q < 0.5f) {
                if (j[o] >= 0 && j[o] < n) d[i] = 2.0f * q * bb + (1.0f - 2.0f * q) * d[o];
            } else {
                const float own = C::dec(i, A[tix<Q>(i, s)]);
                d[i] = bb / (2.0f * q) + (2.0f * q - 1.0f) / (2.0f * q) * own;
            }
        }
    }
}

template <bool NT, class T>
__device__ inline T ld_maybe_nt(const T* p) {
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

// Links j[1..Q-1] of site s (decoded form).  Wave form: all 64 lanes of the
// wavefront call it for the sites of one tile (lane = s & 63), lanes past n
// included, because the compact decoding exchanges the tile's source list
// between lanes.  Split into the loads (load_codes) and the decoding
// (decode_codes) so that a caller can issue the loads of the next tile early.
template <int Q, bool NT>
__device__ inline void load_codes(const Table& tb, int32_t s, uint32_t (&c)[Q], int32_t& e0,
                                  int32_t& e1) {
    if (tb.t16 == nullptr) {
#pragma unroll
        for (int i = 1; i < Q; ++i) c[i] = (uint32_t)ld_maybe_nt<NT>(tb.t32 + tix<Q - 1>(i - 1, s));
        e0 = e1 = 0;
        return;
    }
    const int32_t T = s >> kTileShift;
    const int32_t off = tb.toff[T];
    const int32_t cnt = tb.toff[T + 1] - off;
    const int lane = s & (kTile - 1);
    e0 = lane < cnt ? tb.tlist[off + lane] : 0;
    e1 = lane + kTile < cnt ? tb.tlist[off + kTile + lane] : 0;
#pragma unroll
    for (int i = 1; i < Q; ++i) c[i] = ld_maybe_nt<NT>(tb.t16 + tix<Q - 1>(i - 1, s));
}

template <int Q>
__device__ inline void decode_codes(const Table& tb, int32_t s, const uint32_t (&c)[Q], int32_t e0,
                                    int32_t e1, int32_t (&j)[Q]) {
    if (tb.t16 == nullptr) {
#pragma unroll
        for (int i = 1; i < Q; ++i) j[i] = (int32_t)c[i];
        return;
    }
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const int slot = (int)((c[i] >> kTileShift) & 0x1ffu);
        const int32_t a = __shfl(e0, slot & (kTile - 1), kTile);
        const int32_t b = __shfl(e1, slot & (kTile - 1), kTile);
        const int32_t tile = slot < kTile ? a : b;
        j[i] = (c[i] & 0x8000u) ? (int32_t)(0x80000000u | (c[i] & 0x7fffu))
                                : ((tile << kTileShift) | (int32_t)(c[i] & (kTile - 1)));
    }
}

// ---- two-level block addressing -------------------------------------------
__device__ inline uint64_t block_mask(const BlockRec& r) {
    return ((uint64_t)r.mask_hi << 32) | (uint64_t)r.mask_lo;
}

// position of the set bit of rank r (counted from 0) of m; the result stays in
// [0, 63] for any m and r
__device__ inline int select_bit(uint64_t m, int r) {
    uint32_t x = (uint32_t)m;
    int p = 0;
    int c = __popc(x);
    if (r >= c) {
        r -= c;
        x = (uint32_t)(m >> 32);
        p = 32;
    }
    c = __popc(x & 0xffffu);
    if (r >= c) {
        r -= c;
        x >>= 16;
        p += 16;
    }
    c = __popc(x & 0xffu);
    if (r >= c) {
        r -= c;
        x >>= 8;
        p += 8;
    }
    c = __popc(x & 0xfu);
    if (r >= c) {
        r -= c;
        x >>= 4;
        p += 4;
    }
    c = __popc(x & 0x3u);
    if (r >= c) {
        r -= c;
        x >>= 2;
        p += 2;
    }
    if (r >= (int)(x & 1u)) p += 1;
    return p;
}

// position of local coordinates (x, y, z) in [0, 4)^3: z fastest, then y, then x
__device__ inline int block_pos(int x, int y, int z) { return z | (y << 2) | (x << 4); }

// Links j[1..Q-1] of the site at local coordinates (bx, by, bz) of block bl.
template <int Q>
__device__ inline void block_links(const Table& tb, int32_t bl, int bx, int by, int bz,
                                   int32_t (&j)[Q]) {
    using Lt = Lat<Q>;
    const int32_t* nb = tb.bnbr + (int64_t)bl * 27;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const int ux = bx - Lt::cx[i], uy = by - Lt::cy[i], uz = bz - Lt::cz[i];  // in [-1, 4]
        const int d = ((ux >> 2) + 1) + 3 * ((uy >> 2) + 1) + 9 * ((uz >> 2) + 1);
        const int32_t b2 = nb[d];
        int32_t v = (int32_t)0x80000000u;  // wall
        if (b2 >= 0) {
            const BlockRec r = tb.brec[b2];
            const uint64_t m = block_mask(r);
            const int p = block_pos(ux & 3, uy & 3, uz & 3);
            const uint64_t below = (1ull << p) - 1ull;
            if ((m >> p) & 1ull) {
                v = r.off + __popcll(m & below);
            } else if (r.goff >= 0) {
                const uint64_t g = tb.gmask[b2];
                if ((g >> p) & 1ull) v = tb.n + r.goff + __popcll(g & below);
            }
        }
        j[i] = v;
    }
}

// the site's block bl (given a first guess b0 <= bl) and its local coordinates
__device__ inline void block_site(const Table& tb, int32_t s, int32_t bl, int& bx, int& by,
                                  int& bz) {
    const BlockRec r = tb.brec[bl];
    const int p = select_bit(block_mask(r), s - r.off);
    bx = p >> 4;
    by = (p >> 2) & 3;
    bz = p & 3;
}

// Wave form: the blocks that the tile's sites fall into are found with
// wave-uniform loads of their first-site offsets.
template <int Q>
__device__ inline void links_blocks_wave(const Table& tb, int32_t s, int32_t (&j)[Q]) {
    const int32_t T = __builtin_amdgcn_readfirstlane(s >> kTileShift);
    const int32_t end = (T + 1) << kTileShift;
    const int32_t b0 = tb.tblock[T];
    int32_t bl = b0;
    for (int32_t b = b0 + 1; b < tb.nfluid; ++b) {
        const int32_t o = tb.brec[b].off;
        if (o >= end) break;
        if (s >= o) bl = b;
    }
    int bx, by, bz;
    block_site(tb, s, bl, bx, by, bz);
    block_links<Q>(tb, bl, bx, by, bz, j);
}

// Per position p of a block and moving direction i: where the upstream position lies.
// Bits 16..: byte offset of its block in a group's row (2 bytes per neighbour block);
// bits 0..5: 63 - its position there.
template <int Q>
struct LinkTable {
    static constexpr int quads = (Q - 1 + 3) / 4;
    struct alignas(16) Quad {
        uint32_t x, y, z, w;
    };
    Quad q[quads][kTile];
};
template <int Q>
constexpr uint32_t link_entry(int p, int i) {
    if (i >= Q) return 0u;
    const int ux = (p >> 4) - Lat<Q>::cx[i], uy = ((p >> 2) & 3) - Lat<Q>::cy[i],
              uz = (p & 3) - Lat<Q>::cz[i];  // each in [-1, 4]
    const int d = ((ux + 4) / 4) + 3 * ((uy + 4) / 4) + 9 * ((uz + 4) / 4);
    const int pos = (uz & 3) | ((uy & 3) << 2) | ((ux & 3) << 4);
    return ((uint32_t)(2 * d) << 16) | (uint32_t)(63 - pos);
}
template <int Q>
constexpr LinkTable<Q> make_link_table() {
    LinkTable<Q> t{};
    for (int c = 0; c < LinkTable<Q>::quads; ++c)
        for (int p = 0; p < kTile; ++p) {
            t.q[c][p].x = link_entry<Q>(p, 4 * c + 1);
            t.q[c][p].y = link_entry<Q>(p, 4 * c + 2);
            t.q[c][p].z = link_entry<Q>(p, 4 * c + 3);
            t.q[c][p].w = link_entry<Q>(p, 4 * c + 4);
        }
    return t;
}
template <int Q>
__device__ const LinkTable<Q> kLinkTable = make_link_table<Q>();

// LDS of one group: its staged block records and the own block and position of each of
// its sites (at: block << 6 | position); and, one for the workgroup, the link table.
struct StageLds {
    uint4 chunk[kStageChunks];
    uint16_t at[4 * kTile];
};
template <int Q>
struct LinkLds {
    alignas(16) typename LinkTable<Q>::Quad q[LinkTable<Q>::quads][kTile];
};

// A group's staged blob: where it starts and how many own blocks and records it
// holds (nown = 0: the group's records did not fit and its links decode from the
// global records).  Uniform over the workgroup.
struct StageHdr {
    int32_t off;
    int nown, nrec;
    bool ghosts;
    // own blocks of a group with records but sources too far apart for references (nown
    // is 0 then): the step decodes its links to slots (staged_slots), other kernels take
    // the global records
    int far = 0;
};

// The group entries never change during a launch: read them through the constant
// address space, so that they come in through the scalar cache even after the
// kernel has stored populations (a vector load would have to wait for those
// stores before its value could be used).
__device__ inline StageHdr stage_header(const Table& tb, int32_t g) {
    const __attribute__((address_space(4))) int32_t* grp =
        (const __attribute__((address_space(4))) int32_t*)tb.grp;
    const int32_t cnt = grp[2 * g + 1];
    const bool far = (cnt & kGroupFar) != 0;
    return StageHdr{grp[2 * g], far ? 0 : cnt & 0xff, cnt >> 16, (cnt & kGroupGhosts) != 0,
                    far ? cnt & 0xff : 0};
}

// Iolet links whose data are loaded together: of each, a chain of dependent loads.  More at a
// time cost registers that all sites pay for (D3Q15 FP32 staged 55 VGPRs, 60 with 5, 78 with
// all 14; D3Q19 69, 75 with 5, which is a wave less per SIMD).
constexpr int kLinkBatch = 3;

// bytes of one population row of a tile
template <int SZ>
constexpr int kRowSize = kTile * SZ;

// byte reference of slot j (site or ghost), for elements of SZ bytes
template <int Q, int SZ>
__device__ inline uint32_t slot_ref(int32_t j, uint32_t base) {
    const uint32_t e = (uint32_t)j + __umul24((uint32_t)j >> kTileShift, (Q - 1) * kTile);
    return e * SZ + (kTile - base) * SZ;
}

// slot of a byte reference
template <int Q, int SZ>
__device__ inline int32_t ref_slot(uint32_t ref, int64_t base) {
    const int64_t e = (int64_t)(ref / SZ) - kTile + base;
    const int32_t T = (int32_t)(e / (Q * kTile));
    return (T << kTileShift) | (int32_t)(e - (int64_t)T * (Q * kTile));
}

// 16 bytes per lane from global memory into LDS (no registers, no LDS store): lane l of
// the wavefront writes to + 16 l; `to` is uniform.  lds_loads_done() before the barrier.
__device__ inline void load_lds16(const void* from, void* to) {
    __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
}
__device__ inline void lds_loads_done() { __builtin_amdgcn_s_waitcnt(0); }

// Start the copy of the link table by the workgroup's first four wavefronts.
template <int Q>
__device__ inline void stage_links(int wave, int lane, LinkLds<Q>& links) {
    constexpr int quads = LinkTable<Q>::quads;
    if (wave < 4) load_lds16(&kLinkTable<Q>.q[wave][lane], &links.q[wave][0]);
    if (wave < quads - 4) load_lds16(&kLinkTable<Q>.q[4 + wave][lane], &links.q[4 + wave][0]);
}

// One thread's share of staging a group with records (t: thread index within the
// group's 256 threads): the records, and where each site lies (each wavefront takes
// every fourth own block, whose record is uniform).  The loads are issued before the
// first value is used, so that the stage costs one memory latency after the header's.
// A row of 64 bytes makes block << 6 the byte offset of the block's row.
__device__ inline void stage(const Table& tb, const StageHdr& h, int32_t g, int t, StageLds& lds) {
    const int lane = t & (kTile - 1), wave = __builtin_amdgcn_readfirstlane(t >> kTileShift);
    const int rows = h.nown * (kRowBytes / 16);
    if (t < rows + h.nrec) load_lds16(tb.gblob + h.off + t, &lds.chunk[wave * kTile]);
    const __attribute__((address_space(4))) uint32_t* recs =
        (const __attribute__((address_space(4))) uint32_t*)(tb.gblob + h.off + rows);
    const int k0 = min(wave, h.nown - 1), k1 = min(wave + 4, h.nown - 1);
    const uint32_t a0 = recs[4 * k0], a1 = recs[4 * k0 + 1], a2 = recs[4 * k0 + 2];
    const uint32_t b0 = recs[4 * k1], b1 = recs[4 * k1 + 1], b2 = recs[4 * k1 + 2];
    auto place = [&](int k, uint32_t lo, uint32_t hi, uint32_t off) {
        const uint64_t m = ((uint64_t)hi << 32) | lo;
        const uint32_t at = __builtin_amdgcn_mbcnt_hi(
            hi, __builtin_amdgcn_mbcnt_lo(lo, off + 1u - (uint32_t)(g * 4 * kTile)));
        if (((m >> lane) & 1ull) && at < 4 * kTile) lds.at[at] = (uint16_t)((k << 6) | lane);
    };
    place(k0, a0, a1, a2);  // a block placed twice (few own blocks) gets the same values
    place(k1, b0, b1, b2);
    for (int k = wave + 8; k < h.nown; k += 4) place(k, recs[4 * k], recs[4 * k + 1], recs[4 * k + 2]);
}

// Source references of the links of the group's site t (its own reference: own), from
// the group's LDS (h.nown > 0).  A wall link gets the site's own row: the reference
// less (i - 1) rows is then the address of population opp(i).  gmask, if the group has
// ghost cells: the directions of the site's iolet links.
template <int Q, int SZ>
__device__ inline void staged_refs(const Table& tb, const StageHdr& h, int t, uint32_t base,
                                   uint32_t own, const StageLds& lds, const LinkLds<Q>& links,
                                   uint32_t (&e)[Q], uint32_t& gmask) {
    const char* raw = reinterpret_cast<const char*>(lds.chunk);
    const uint32_t at = lds.at[t];
    const uint32_t p = at & 63u;
    const uint32_t row = at & ~63u;
    uint32_t lk[LinkTable<Q>::quads * 4];
#pragma unroll
    for (int c = 0; c < LinkTable<Q>::quads; ++c) {
        const typename LinkTable<Q>::Quad v = links.q[c][p];
        lk[4 * c] = v.x;
        lk[4 * c + 1] = v.y;
        lk[4 * c + 2] = v.z;
        lk[4 * c + 3] = v.w;
    }
    auto rec = [&](int i) {
        const uint32_t a = *reinterpret_cast<const uint16_t*>(raw + row + (lk[i - 1] >> 16));
        return *reinterpret_cast<const uint4*>(raw + a);
    };
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        // the mask shifted so that the position is the top bit: sign = a fluid site,
        // population count = its rank + 1
        const uint4 r = rec(i);
        const uint64_t m = (((uint64_t)r.y << 32) | r.x) << (lk[i - 1] & 63u);
        const int32_t j = (int32_t)r.z + __popc((uint32_t)m) + __popc((uint32_t)(m >> 32));
        const uint32_t ref = slot_ref<Q, SZ>(j, base);
        e[i] = (int64_t)m < 0 ? ref : own + (opp(i) - i) * kRowSize<SZ>;
    }
    gmask = 0;
    if (!h.ghosts) return;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        if (e[i] != own + (opp(i) - i) * kRowSize<SZ>) continue;
        const int32_t at = (int32_t)rec(i).w;  // the block's ghost record
        if (at < 0) continue;
        const uint4 g = *reinterpret_cast<const uint4*>(raw + at);
        const uint64_t gm = (((uint64_t)g.y << 32) | g.x) << (lk[i - 1] & 63u);
        if ((int64_t)gm < 0) {
            e[i] = slot_ref<Q, SZ>((int32_t)g.z + __popcll(gm), base);
            gmask |= 1u << i;
        }
    }
}

// As staged_refs, but the links themselves (sites, walls, ghost slots), for groups whose
// sources lie too far apart for 32-bit references.  8% of the groups of a 395M-site tree
// are such: with the global records for them its step took 11.15 ms, so 9.08.
template <int Q>
__device__ inline void staged_slots(const Table& tb, const StageHdr& h, int t, const StageLds& lds,
                                    const LinkLds<Q>& links, int32_t (&j)[Q]) {
    const char* raw = reinterpret_cast<const char*>(lds.chunk);
    const uint32_t at = lds.at[t];
    const uint32_t* lk = reinterpret_cast<const uint32_t*>(&links.q[0][at & 63u]);
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const uint32_t l = lk[(i - 1) / 4 * (kTile * 4) + (i - 1) % 4];
        const uint32_t a = *reinterpret_cast<const uint16_t*>(raw + (at & ~63u) + (l >> 16));
        const uint4 r = *reinterpret_cast<const uint4*>(raw + a);
        const uint64_t m = (((uint64_t)r.y << 32) | r.x) << (l & 63u);
        j[i] = (int64_t)m < 0 ? (int32_t)r.z + __popcll(m) : (int32_t)0x80000000u;
        if (!h.ghosts || (int64_t)m < 0 || (int32_t)r.w < 0) continue;
        const uint4 g = *reinterpret_cast<const uint4*>(raw + (int32_t)r.w);
        const uint64_t gm = (((uint64_t)g.y << 32) | g.x) << (l & 63u);
        if ((int64_t)gm < 0) j[i] = (int32_t)g.z + __popcll(gm);
    }
}

// Gather the pre-collision deviations of the site with row reference own: a reference
// is the load's 32-bit offset from a uniform base, the direction's row its constant
// offset.
template <int Q, int ST, bool SC>
__device__ inline void refs_gather(const typename Store<ST>::T* __restrict__ A, int64_t base,
                                   uint32_t own, const uint32_t (&e)[Q], float (&d)[Q]) {
    using T = typename Store<ST>::T;
    using C = Codec<Q, ST, SC>;
    constexpr int kRow = kRowSize<sizeof(T)>;
    const char* ab = reinterpret_cast<const char*>(A + base);
    T v[Q];
    v[0] = *reinterpret_cast<const T*>(ab + own - kRow);
#pragma unroll
    for (int i = 1; i < Q; ++i) v[i] = *reinterpret_cast<const T*>(ab + e[i] + (i - 1) * kRow);
#pragma unroll
    for (int i = 0; i < Q; ++i) d[i] = C::dec(i, v[i]);
}

// Wave form of the link decode (all lanes of a wavefront call it); block
// addressing decodes from the global records here.
template <int Q, bool NT>
__device__ inline void links_wave(const Table& tb, int32_t s, int32_t (&j)[Q]) {
    if (tb.brec) {
        links_blocks_wave<Q>(tb, s, j);
        return;
    }
    uint32_t c[Q];
    int32_t e0, e1;
    load_codes<Q, NT>(tb, s, c, e0, e1);
    decode_codes<Q>(tb, s, c, e0, e1, j);
}

// All links of an arbitrary site (no lane exchange; any lane may call it).
template <int Q>
__device__ inline void links_site(const Table& tb, int32_t s, int32_t (&j)[Q]) {
    if (tb.brec) {
        int32_t bl = tb.tblock[s >> kTileShift];
        while (bl + 1 < tb.nfluid && tb.brec[bl + 1].off <= s) ++bl;
        int bx, by, bz;
        block_site(tb, s, bl, bx, by, bz);
        block_links<Q>(tb, bl, bx, by, bz, j);
        return;
    }
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        if (tb.t16 == nullptr) {
            j[i] = tb.t32[tix<Q - 1>(i - 1, s)];
            continue;
        }
        const uint32_t c = tb.t16[tix<Q - 1>(i - 1, s)];
        if (c & 0x8000u) {
            j[i] = (int32_t)(0x80000000u | (c & 0x7fffu));
        } else {
            const int32_t tile =
                tb.tlist[tb.toff[s >> kTileShift] + (int)((c >> kTileShift) & 0x1ffu)];
            j[i] = (tile << kTileShift) | (int32_t)(c & (kTile - 1));
        }
    }
}

// slot holding the incoming population of iolet link l
__device__ inline int32_t ghost_slot(const Ghosts& G, int32_t n, int64_t l) {
    return G.slot ? G.slot[l] : n + (int32_t)l;
}

// iolet link that pulls direction i from ghost slot `slot`
template <int Q>
__device__ inline int64_t ghost_link(const Ghosts& G, int32_t n, int32_t slot, int i) {
    return G.slot ? (int64_t)G.cell_link[(int64_t)(slot - n) * Q + i] : (int64_t)(slot - n);
}

// the first iolet link of a site with iolet directions gmask and references e + lo
template <int Q, int SZ>
__device__ inline int64_t staged_link(const Ghosts& G, int32_t n, int64_t base,
                                      const uint32_t (&e)[Q], uint32_t lo, uint32_t gmask) {
    const int first = __builtin_ctz(gmask);
    uint32_t ref = 0;
#pragma unroll
    for (int i = 1; i < Q; ++i) ref = i == first ? e[i] + lo : ref;
    return ghost_link<Q>(G, n, ref_slot<Q, SZ>(ref, base), first);
}

// moments of FP32 deviations: drho = sum d, m = sum c d (constant-folded per lattice)
template <int Q>
__device__ inline void moments(const float (&d)[Q], float& drho, float& mx, float& my, float& mz) {
    using Lt = Lat<Q>;
    drho = d[0];
    mx = my = mz = 0.f;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        drho += d[i];
        if (Lt::cx[i] > 0) mx += d[i];
        if (Lt::cx[i] < 0) mx -= d[i];
        if (Lt::cy[i] > 0) my += d[i];
        if (Lt::cy[i] < 0) my -= d[i];
        if (Lt::cz[i] > 0) mz += d[i];
        if (Lt::cz[i] < 0) mz -= d[i];
    }
}

// equilibrium deviations deq_i = f_i^eq(rho, u) - w_i for all i (pairs share the
// even part of the quadratic)
template <int Q>
__device__ inline void eq_dev(float drho, float rho, float ux, float uy, float uz,
                              float (&deq)[Q]) {
    using Lt = Lat<Q>;
    const float usq15 = 1.5f * (ux * ux + uy * uy + uz * uz);
    deq[0] = Lt::w[0] * (drho - rho * usq15);
#pragma unroll
    for (int k = 1; k < Q; k += 2) {
        const float cu = (float)Lt::cx[k] * ux + (float)Lt::cy[k] * uy + (float)Lt::cz[k] * uz;
        const float sym = Lt::w[k] * (drho + rho * (4.5f * cu * cu - usq15));
        const float asym = Lt::w[k] * rho * 3.0f * cu;
        deq[k] = sym + asym;
        deq[k + 1] = sym - asym;
    }
}

__device__ inline double iolet_value(const DevIolet& io, const double* harm, double t) {
    double v = io.mean;
    for (int h = 1; h <= io.n_harm; ++h) {
        const double ph = fmod((double)h * t, io.period) / io.period;  // in [0, 1)
        double sv, cv;
        sincospi(2.0 * ph, &sv, &cv);
        v += harm[io.harm_off + h - 1] * cv + harm[io.harm_off + io.n_harm + h - 1] * sv;
    }
    return v;
}

}  // namespace hlb
