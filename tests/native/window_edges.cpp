// Host-only check of the staged step's choice between LDS and memory at the edges of the
// 32-bit window (group_base, kRefSpan): a source belongs to the workgroup's own W tiles
// exactly if its reference less theirs, in 32 bits, is below their span.
#include <cstdio>

#include "../../paper_1906_11925_amd/csrc/kernels.hpp"

int main() {
    using namespace hlb;
    int bad = 0;
    for (int q : {15, 19})
        for (int sz : {2, 4})
            for (int w : {4, 8, 16}) {
                const int64_t tile = (int64_t)q * kTile, last = (kRefSpan - 1) / tile;
                const uint32_t span = (uint32_t)((w * tile + kTile) * sz);
                // the lowest and the highest tile that a window can hold, and their neighbours
                for (int64_t t0 = 0; t0 <= last; t0 = t0 == 2 * w ? last - 2 * w : t0 + 1)
                    for (int64_t t = 0; t <= last; t = t == 2 * w ? last - 2 * w : t + 1)
                        for (int lane : {0, kTile - 1}) {
                            const uint32_t ref = (uint32_t)((t * tile + kTile + lane) * sz);
                            const uint32_t e = ref - (uint32_t)(t0 * tile * sz);
                            const bool own = t >= t0 && t < t0 + w;
                            if ((e < span) != own && bad++ < 5)
                                printf("q %d elem %d w %d: tile %lld seen from %lld\n", q, sz, w,
                                       (long long)t, (long long)t0);
                        }
            }
    printf("%d\n", bad);
    return bad != 0;
}
