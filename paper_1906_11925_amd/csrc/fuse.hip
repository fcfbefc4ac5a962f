// Several time steps per launch for lattices too small to fill the GPU.
//
// A step of a small lattice is bound by latency, not by bytes: one launch is a chain
// of dependent memory accesses (addressing data, gather, store) that a single round of
// workgroups cannot hide.  Here every workgroup advances its own sites by K steps
// without talking to the others: it starts from the sites that can reach its own in
// K - 1 steps, makes the first step on all of them from global memory, keeps the
// result in LDS, and makes the remaining steps there on sets that shrink by one layer
// each.  The sites around a group are computed by several groups (the same arithmetic
// on the same values, so the same bits); in return K - 1 of K launches and their
// memory latencies are gone.  What bounds it then is the vector instructions of the
// sites computed more than once, so a link costs one instruction in LDS: its code is
// the LDS address of what it pulls, walls included.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "fuse.hpp"
#include "kernels.hpp"
#include "lattice.hpp"
#include "lbdev.hpp"
#include "step.hpp"

namespace hlb {

template <int Q, bool BFL>
struct FuseRow {
    uint32_t w[fuse_row_words(Q, BFL)];
    __device__ uint32_t code(int i) const { return (w[(i - 1) >> 1] >> (16 * ((i - 1) & 1))) & 0xffffu; }
    // directions of the iolet links (bit i) and the first of them
    __device__ uint32_t mask() const { return Q == 15 ? (w[7] & 0x3fffu) << 1 : w[10]; }
    __device__ int32_t first_link() const { return (int32_t)(Q == 15 ? w[7] >> 14 : w[9]); }
    __device__ int32_t walls() const { return (int32_t)w[Q == 15 ? 8 : 11]; }
};

template <int Q, bool BFL>
__device__ inline FuseRow<Q, BFL> fuse_row(const uint4* __restrict__ rows, int32_t pitch, int32_t x) {
    FuseRow<Q, BFL> r;
#pragma unroll
    for (int c = 0; c < fuse_row_words(Q, BFL) / 4; ++c) {
        const uint4 v = rows[c * pitch + x];
        r.w[4 * c] = v.x;
        r.w[4 * c + 1] = v.y;
        r.w[4 * c + 2] = v.z;
        r.w[4 * c + 3] = v.w;
    }
    return r;
}

// Interpolated walls on pulled deviations (the rule of apply_bfl); own(i): the site's
// own stored population i.
template <int Q, class Own>
__device__ inline void fuse_bfl(const uint16_t* __restrict__ frac, uint32_t iolets, float (&d)[Q],
                                Own&& own) {
    uint16_t code[Q];
#pragma unroll
    for (int i = 1; i < Q; ++i) code[i] = frac[i - 1];
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        if (code[i] == 0) continue;
        const int o = opp(i);
        const float q = (float)code[i] * (1.0f / 32768.0f);
        const float bb = d[i];
        if (q < 0.5f) {
            if (code[o] == 0 && !(iolets & (1u << o))) d[i] = 2.0f * q * bb + (1.0f - 2.0f * q) * d[o];
        } else {
            d[i] = bb / (2.0f * q) + (2.0f * q - 1.0f) / (2.0f * q) * own(i);
        }
    }
}

template <int Q, int ST, bool SC, bool BRINK, bool BFL, int PITCH>
__global__ __launch_bounds__(kFuseMaxThreads) void k_fused_steps(
    const typename Store<ST>::T* __restrict__ src, typename Store<ST>::T* __restrict__ dst,
    typename Store<ST>::T* __restrict__ prev, Fuse F, int32_t n, float omega,
    const float* __restrict__ alpha, Ghosts G, int64_t t) {
    using T = typename Store<ST>::T;
    using C = Codec<Q, ST, SC>;
    constexpr int SZ = sizeof(T), kRow = kRowSize<SZ>, kPitch = fuse_row_bytes(Q, PITCH);
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* pops = lds;  // [Q][kPitch bytes]
    uint32_t* list = reinterpret_cast<uint32_t*>(lds + Q * kPitch);
    // consecutive groups on one XCD (workgroups go round the 8 XCDs in turn)
    const int32_t per = (F.groups + 7) >> 3;
    const int32_t g = ((int32_t)blockIdx.x & 7) * per + ((int32_t)blockIdx.x >> 3);
    if (g >= F.groups) return;
    const __attribute__((address_space(4))) int32_t* h =
        (const __attribute__((address_space(4))) int32_t*)(F.hdr + (int64_t)g * kFuseHdr);
    const int K = F.steps, tid = (int)threadIdx.x, nthr = (int)blockDim.x;
    const int32_t s0 = h[0], nrow = h[4 + K - 1], nloc = h[4 + K];
    const uint4* rows = F.rows + h[2];
    const uint32_t* glist = F.list + h[1];
    const char* sb = reinterpret_cast<const char*>(src);

    // the first row of this thread serves every step
    FuseRow<Q, BFL> r0{};
    if (tid < nrow) r0 = fuse_row<Q, BFL>(rows, nrow, tid);
    const int32_t gap = h[3];
    for (int32_t k = tid; k < nloc; k += nthr) list[k < nrow ? k : k + gap] = glist[k];
    __syncthreads();

    // step 1: from global memory, on R_{K-1}
    for (int32_t x = tid; x < nrow; x += nthr) {
        const FuseRow<Q, BFL> r = x == tid ? r0 : fuse_row<Q, BFL>(rows, nrow, x);
        const uint32_t own = list[x];
        T v[Q];
        v[0] = *reinterpret_cast<const T*>(sb + own - kRow);
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            const uint32_t c = r.code(i);
            const bool wall = c == (uint32_t)(x * SZ + (1 + opp(i) - i) * kPitch);
            const uint32_t ref = list[wall ? (uint32_t)x : (c - kPitch) / SZ] + (wall ? (opp(i) - i) * kRow : 0);
            v[i] = *reinterpret_cast<const T*>(sb + ref + (i - 1) * kRow);
        }
        float d[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) d[i] = C::dec(i, v[i]);
        const uint32_t mask = r.mask();
        if (mask) {
            int64_t l = r.first_link();
#pragma unroll
            for (int i = 1; i < Q; ++i)
                if (mask & (1u << i)) d[i] = C::dec(i, src[tix<Q>(i, ghost_slot(G, n, l++))]);
        }
        if constexpr (BFL) {
            if (r.walls() >= 0)
                fuse_bfl<Q>(F.frac + (int64_t)r.walls() * (Q - 1), mask, d, [&](int i) {
                    return C::dec(i, *reinterpret_cast<const T*>(sb + own + (i - 1) * kRow));
                });
        }
        T e[Q];
        site_collide<Q, ST, SC, BRINK>(d, omega, alpha, BRINK ? ref_slot<Q, SZ>(own, 0) : 0, e);
#pragma unroll
        for (int i = 0; i < Q; ++i) *reinterpret_cast<T*>(pops + i * kPitch + x * SZ) = e[i];
    }

    // the other steps, in LDS.  Those before the last have at most one site per thread
    // and write their results where they read: pull, barrier, store, barrier.
    for (int p = 2; p <= K; ++p) {
        __syncthreads();
        const bool last = p == K;
        const int32_t np = h[4 + K - p];
        for (int32_t x0 = 0; x0 < np; x0 += nthr) {
            const int32_t x = x0 + tid;
            const bool mine = x < np;
            Pulled<Q> P;
            P.gmask = 0;
            P.gl = -1;
            T e[Q];
            if (mine) {
                const FuseRow<Q, BFL> r = x0 == 0 ? r0 : fuse_row<Q, BFL>(rows, nrow, x);
                P.d[0] = C::dec(0, *reinterpret_cast<const T*>(pops + x * SZ));
#pragma unroll
                for (int i = 1; i < Q; ++i)
                    P.d[i] = C::dec(i, *reinterpret_cast<const T*>(pops + r.code(i) + (i - 1) * kPitch));
                auto own = [&](int i) {
                    return *reinterpret_cast<const T*>(pops + i * kPitch + x * SZ);
                };
                const bool keep = last && prev != nullptr;
                const int32_t s = s0 + x;  // of own sites
                P.gmask = r.mask();
                if (P.gmask) {
                    P.gl = r.first_link();
                    float vs[Q];
#pragma unroll
                    for (int i = 0; i < Q; ++i) vs[i] = C::dec(i, own(i));
                    int64_t l = P.gl;
#pragma unroll
                    for (int i = 1; i < Q; ++i)
                        if (P.gmask & (1u << i)) {
                            const T v = C::enc(i, ghost_value<Q>(G, l, i, vs, t + p - 1));
                            if (keep) prev[tix<Q>(i, ghost_slot(G, n, l))] = v;
                            P.d[i] = C::dec(i, v);
                            ++l;
                        }
                }
                if constexpr (BFL) {
                    if (r.walls() >= 0)
                        fuse_bfl<Q>(F.frac + (int64_t)r.walls() * (Q - 1), P.gmask, P.d,
                                    [&](int i) { return C::dec(i, own(i)); });
                }
                if (last) {
                    if (keep) {
#pragma unroll
                        for (int i = 0; i < Q; ++i) st_pop(prev + tix<Q>(i, s), own(i));
                    }
                    site_collide_store<Q, ST, SC, BRINK>(dst, n, omega, alpha, G, t + K, s, P, dst);
                } else {
                    site_collide<Q, ST, SC, BRINK>(P.d, omega, alpha,
                                                   BRINK ? ref_slot<Q, SZ>(list[x], 0) : 0, e);
                }
            }
            if (last) continue;
            __syncthreads();
            if (mine) {
#pragma unroll
                for (int i = 0; i < Q; ++i) *reinterpret_cast<T*>(pops + i * kPitch + x * SZ) = e[i];
            }
        }
    }
}

template <class F>
static hipError_t fuse_dispatch(const Layout& L, bool brink, int pitch, F&& f) {
    return dispatch(L.q, L.storage, L.scaled, [&](auto tag) {
        using Tg = decltype(tag);
        auto pick = [&](auto w) {
            constexpr int W = decltype(w)::value;
            if (brink)
                return L.bfl ? f(tag, k_fused_steps<Tg::Q, Tg::ST, Tg::SC, true, true, W>)
                             : f(tag, k_fused_steps<Tg::Q, Tg::ST, Tg::SC, true, false, W>);
            return L.bfl ? f(tag, k_fused_steps<Tg::Q, Tg::ST, Tg::SC, false, true, W>)
                         : f(tag, k_fused_steps<Tg::Q, Tg::ST, Tg::SC, false, false, W>);
        };
        return pitch == 0   ? pick(std::integral_constant<int, 0>{})
               : pitch == 1 ? pick(std::integral_constant<int, 1>{})
                            : pick(std::integral_constant<int, 2>{});
    });
}

hipError_t fuse_prepare(const Layout& L, const Fuse& F, bool brink) {
    return fuse_dispatch(L, brink, F.pitch, [&](auto, auto kernel) {
        // the limit belongs to the kernel, not to the handle: the same for all of them
        return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, kFuseMaxLds);
    });
}

hipError_t launch_fused_steps(const Layout& L, const Ghosts& G, const Fuse& F, const void* src,
                              void* dst, void* prev, float omega, const float* alpha, int64_t t,
                              hipStream_t s) {
    if (L.n == 0 || F.groups == 0) return hipSuccess;
    return fuse_dispatch(L, alpha != nullptr, F.pitch, [&](auto tag, auto kernel) {
        using T = typename Store<decltype(tag)::ST>::T;
        kernel<<<(unsigned)(((F.groups + 7) / 8) * 8), (unsigned)F.threads, (size_t)F.lds, s>>>(
            static_cast<const T*>(src), static_cast<T*>(dst), static_cast<T*>(prev), F, (int32_t)L.n,
            omega, alpha, G, t);
        return hipGetLastError();
    });
}

}  // namespace hlb
