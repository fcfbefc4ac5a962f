// Internal interface of the several-steps-per-launch kernel for small lattices.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace hlb {

constexpr int kFuseMaxSteps = 4;       // most time steps one launch makes
constexpr int kFuseMaxThreads = 1024;  // most threads of a workgroup
constexpr int kFuseMaxLds = 160 * 1024;
constexpr int kFuseHdr = 16;           // 32-bit words per group header

// Host-built description of the groups (one workgroup each).  Group g owns the
// consecutive sites [first, first + count[0]), whole tiles; R_m is the set of sites whose
// populations at the launch's start can reach them in m steps (R_0 the own sites),
// numbered so that R_m is the first count[m] of the group's local sites.
//  * hdr[g]: words 0 = first own site, 1 = first word of its list, 2 = first 16-byte
//    chunk of its rows, 3 = gap, 4 + m = count[m] for m = 0 .. steps;
//  * list: byte reference (kernels.hpp, base 0) of every local site below count[steps];
//  * rows: for the local sites below count[steps - 1], 16-byte chunk c of site x at
//    c * count[steps - 1] + x.  A row holds
//      one 16-bit code per moving direction: the byte offset, from row i - 1 of a
//      population array of row pitch P (fuse_pitch), of the value that link i pulls: P + y
//      elements for the local upstream site y, P + x + (opp(i) - i) P for a wall (the
//      site's own opposite population), P + x for an iolet link.  The outermost sites
//      (from count[steps - 1], only ever read from global memory) count from
//      count[steps - 1] + gap, gap = P where they would pass P, so that no code of a
//      site reads as another's wall (the host builds no group whose codes pass 16 bits);
//      then the first iolet link and the mask of the iolet directions (D3Q15: link << 14
//      | mask >> 1 in one word; D3Q19: two words), and with interpolated walls the entry
//      of the site in frac (-1: none);
//  * frac: (q - 1) 16-bit wall fractions per entry (units of 2^-15, 0: no wall).
struct Fuse {
    const int32_t* hdr;
    const uint32_t* list;
    const uint4* rows;
    const uint16_t* frac;
    int32_t groups;
    int32_t steps;
    int32_t threads;
    int32_t pitch;  // which row pitch (fuse_row_bytes)
    int32_t lds;   // bytes of LDS per workgroup
};

constexpr int fuse_row_words(int q, bool bfl) { return q == 15 && !bfl ? 8 : 12; }

// Row pitch in bytes of the population array in LDS.  Constants, so that a row is a
// load's or store's immediate offset (below 2^16 for every row).
constexpr int kFusePitches = 3;
constexpr int fuse_row_bytes(int q, int pitch) {
    return pitch == 0 ? 2048 : pitch == 1 ? 3072 : q == 15 ? 4096 : 3584;
}

// LDS bytes of a workgroup whose groups have at most nloc local numbers
inline int32_t fuse_lds(int q, int pitch, int32_t nloc) {
    return ((nloc * 4 + 15) & ~15) + q * fuse_row_bytes(q, pitch);
}

#ifdef HLB_NO_DEVICE  // host-only builds of the planner: no kernels to launch
inline hipError_t fuse_prepare(const Layout&, const Fuse&, bool) { return hipErrorNoDevice; }
inline hipError_t launch_fused_steps(const Layout&, const Ghosts&, const Fuse&, const void*, void*,
                                     void*, float, const float*, int64_t, hipStream_t) {
    return hipErrorNoDevice;
}
#else
// Let the handle's kernel use up to kFuseMaxLds bytes of LDS on the current device.
hipError_t fuse_prepare(const Layout& L, const Fuse& F, bool brink);

// fuse.steps time steps src -> dst in one launch; src's ghost slots hold the incoming
// values for time t, dst's receive those for time t + steps.  prev (optional): also
// receives the state at time t + steps - 1 with its ghost slots.
hipError_t launch_fused_steps(const Layout& L, const Ghosts& G, const Fuse& F, const void* src,
                              void* dst, void* prev, float omega, const float* alpha, int64_t t,
                              hipStream_t s);
#endif

}  // namespace hlb
