// Releases of csrc/smmo_device.hpp (give_back_slots, release_beside) by a
// wavefront of one lane on the host (built and run by tests/test_release_host.py;
// no GPU is touched): random slots of random blocks until all are free, every
// bitmap, type and counter compared with a plain model after each release.
#include <cstdio>
#include <random>

#include "one_lane/heap.hpp"

struct Model {
    uint32_t M;
    std::vector<uint64_t> slots;             // live slots; a block without any is free
    bool agrees(const Host &m) const
    {
        std::vector<uint64_t> want(m.bm.size(), 0);
        HeapView v = m.h;
        v.bm = want.data();
        auto set = [&](uint32_t bmid, uint32_t pos) {
            for (uint32_t l = 0; l < v.nlev; ++l, pos >>= 6) *v.bm_word(bmid, l, pos >> 6) |= 1ull << (pos & 63);
        };
        for (uint32_t b = 0; b < M; ++b) {
            if (!slots[b]) set(BM_FREE, b);
            else set(bm_alloc(0), b);
            if (slots[b] && slots[b] != ~0ull) set(bm_active(0), b);
            if (m.type[b] != (slots[b] ? 0 : kNull) || m.alloc_bm[b] != (slots[b] ? slots[b] : ~0ull)) return false;
        }
        return want == m.bm;
    }
};

int main()
{
    int wrong = 0, errors = 0;
    for (uint32_t M : {1u, 63u, 64u, 65u, 300u, 4097u}) {
        for (int beside = 0; beside < 2; ++beside) {
            std::mt19937_64 rng(M + beside);
            Host m(M, true);
            Model w{M, std::vector<uint64_t>(M)};
            for (uint32_t b = 0; b < M; ++b) {           // full blocks, some with free slots, some free
                const uint32_t r = rng() % 8;
                const uint64_t s = r == 0 ? 0 : r == 1 ? rng() : r == 2 ? 1ull << rng() % 64 : ~0ull;
                if (!s) continue;
                w.slots[b] = m.alloc_bm[b] = s;
                m.type[b] = 0;
                switch_bit_one(m.h, 0, BM_FREE, b, -1);
                switch_bit_one(m.h, 0, bm_alloc(0), b, +1);
                if (s != ~0ull) switch_bit_one(m.h, 0, bm_active(0), b, +1);
            }
            wrong += !w.agrees(m);
            for (uint32_t n = 0, left = M; left && n < 40 * M; ++n) {
                const uint32_t b = rng() % M;
                if (!w.slots[b]) continue;
                uint64_t mask = w.slots[b] & (n % 3 ? rng() & rng() : ~0ull);
                if (!mask) mask = w.slots[b] & -w.slots[b];
                if (beside) errors += !release_beside(m.h, 0, b, mask);
                else give_back_slots(m.h, 0, 0, b, mask);
                w.slots[b] &= ~mask;
                if (M < 100 || n % 64 == 0) wrong += !w.agrees(m);
            }
            wrong += !w.agrees(m);
            errors += m.ctrl[CTRL_ERR] != 0;
            // a free slot: reported, nothing changed
            if (M < 2) continue;
            for (uint32_t b = 0; b < M; ++b)
                if (w.slots[b] && w.slots[b] != ~0ull) {
                    const uint64_t mask = ~w.slots[b] & (w.slots[b] + 1);
                    if (beside) errors += release_beside(m.h, 0, b, mask);
                    else give_back_slots(m.h, 0, 0, b, mask);
                    errors += m.ctrl[CTRL_ERR] != ERR_BADHANDLE;
                    wrong += !w.agrees(m);
                    break;
                }
        }
    }
    std::printf("wrong %d errors %d\n", wrong, errors);
    return 0;
}
