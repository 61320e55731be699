// Searches of csrc/smmo_device.hpp on bitmaps as a search can meet them while
// another wavefront is between two levels, run by a wavefront of one lane on
// the host (built and run by tests/test_search_host.py; no GPU is touched).
#include <cstdio>
#include <vector>

#include "../paper_1908_05845_amd/csrc/smmo_device.hpp"

using namespace smmo;

struct Host {
    HeapView h{};
    std::vector<uint32_t> ctrl, type;
    std::vector<uint64_t> bm, alloc_bm;

    // M blocks, one class, all free or all taken
    Host(uint32_t M, bool free)
    {
        h.M = M;
        h.nclasses = 1;
        h.rotation = 1;
        h.spin_limit = 1u << 16;
        for (uint32_t n = M;;) {
            n = (n + 63) / 64;
            h.lvl_off[h.nlev] = h.bm_words;
            h.lvl_n[h.nlev++] = n;
            h.bm_words += n;
            if (n == 1) break;
        }
        ctrl.assign(kCtrlWords, 0);
        type.assign(M, kNull);
        alloc_bm.assign(M, ~0ull);
        bm.assign(3ull * h.bm_words, 0);
        h.ctrl = ctrl.data();
        h.type = type.data();
        h.alloc_bm = alloc_bm.data();
        h.bm = bm.data();
        for (uint32_t l = 0, n = M; free && l < h.nlev; n = h.lvl_n[l++])
            for (uint32_t i = 0; i < n; ++i) *h.bm_word(BM_FREE, l, i / 64) |= 1ull << (i % 64);
    }
    uint32_t claim(uint32_t seed) { return claim_free_block(h, 0, seed); }
};

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
