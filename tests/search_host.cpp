// Searches of csrc/smmo_device.hpp on bitmaps as a search can meet them while
// another wavefront is between two levels, run by a wavefront of one lane on
// the host (built and run by tests/test_search_host.py; no GPU is touched).
#include <cstdio>

#include "one_lane/heap.hpp"

int main()
{
    // windows of 4,096 blocks below one level-2 container: the first `behind`
    // are claimed to the last block, their bits there still set
    int bad = 0;
    for (uint32_t behind : {0u, 1u, 2u, 5u}) {
        for (uint32_t seed = 0; seed < 200; ++seed) {
            Host m(7 * 4096, true);
            for (uint32_t w = 0; w < behind; ++w) {
                *m.h.bm_word(BM_FREE, 1, w) = 0;
                for (uint32_t c = 0; c < 64; ++c) *m.h.bm_word(BM_FREE, 0, 64 * w + c) = 0;
            }
            const uint32_t b = m.claim(hash32(seed));
            if (b == kNoBlock || b < behind * 4096 || m.ctrl[CTRL_ERR]) ++bad;
            // nothing behind: the first window, as the claims of a growing class want it
            if (behind == 0 && b >= 4096) ++bad;
        }
    }
    Host none(7 * 4096, false);
    const bool exhausted = none.claim(1) == kNoBlock && none.ctrl[CTRL_ERR] == 0;
    // every block once, then none
    Host all(2 * 4096 + 17, true);
    std::vector<int> got(all.h.M, 0);
    uint32_t n = 0;
    for (uint32_t b; (b = all.claim(hash32(n))) != kNoBlock; ++n) ++got[b];
    bool once = n == all.h.M;
    for (int g : got) once = once && g == 1;
    for (uint64_t w : all.bm) once = once && w == 0;
    std::printf("missed %d exhausted %d once %d\n", bad, exhausted, once);
    return 0;
}
