// A heap's bookkeeping in host memory, for a wavefront of one lane.
#pragma once
#include <vector>

#include "../../paper_1908_05845_amd/csrc/smmo_device.hpp"

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
