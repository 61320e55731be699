// Device side of the SMMO heap: hierarchical bitmaps, block slot reservation
// and release, block invalidation, and wavefront-aggregated allocation and
// deallocation.  Follows the DynaSOAr allocator (Springer, Ch.5 sec.5.2 and
// sec.5.3, correctness argument in sec.5.4), re-expressed for CDNA wave64:
//   - a block holds 64 objects, so its 64-bit allocation bitmap is exactly a
//     wavefront ballot; one wavefront processes one block, one lane per slot;
//   - the leader of an aggregated allocation is the lowest requesting lane,
//     results are broadcast by readlane and ranks come from the ballot;
//   - CDNA has no independent thread scheduling, so every retrying bitmap
//     update runs in a converged loop in which each lane tries each of its
//     pending updates once per iteration (the deadlock-free deallocation of
//     sec.5.4.4, applied to every multi-lane bitmap update);
//   - every retry loop is bounded; exceeding the bound raises a device error
//     instead of hanging the GPU.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "smmo_layout.hpp"

namespace smmo {

// ---------------------------------------------------------------- atomics --
// Bitmap words and block headers are shared mutable state; all accesses go
// through agent-scope atomics, which are performed at the device's point of
// coherence (past the per-CU L1 and the per-XCD L2).  They are relaxed: an
// acquire or release at agent scope makes the compiler write back and
// invalidate the whole L2 of the XCD around the atomic, which on this chip
// costs far more than the atomic.  The orderings the allocator needs are
// among these atomics themselves: a thread's atomic whose result it uses has
// been performed before its next access is issued, and a block-type store is
// made complete (complete_prior) before the bitmap update that publishes
// it.  Object data written by methods is published at kernel boundaries.
__device__ __forceinline__ uint64_t ald(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ald32(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t aor(uint64_t *p, uint64_t v)
{
    return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t aand(uint64_t *p, uint64_t v)
{
    return __hip_atomic_fetch_and(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// waits until every earlier memory access of this thread (stores included)
// has been performed
__device__ __forceinline__ void complete_prior() { __builtin_amdgcn_s_waitcnt(0); }

__device__ __forceinline__ void raise_error(const HeapView &h, uint32_t bits)
{
    __hip_atomic_fetch_or(h.ctrl + CTRL_ERR, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// adds n to event counter `ev` in this wavefront's stripe
__device__ __forceinline__ void count_events(const HeapView &h, uint32_t ev, uint64_t n)
{
    const uint32_t wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    uint32_t *w = h.ctrl + CTRL_EVENTS + (wave % kEventStripes) * kStripeWords + ev;
    __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(w), (unsigned long long)n,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void count_event(const HeapView &h, uint32_t ev) { count_events(h, ev, 1); }

// the block list of class cls (wave-uniform)
__device__ __forceinline__ BlockList block_list(const HeapView &h, uint32_t cls)
{
    BlockList L;
    L.R = h.R + (uint64_t)cls * h.M;
    L.M = h.M;
    L.direct = (h.direct >> cls) & 1;
    if (L.direct) {
        L.r = L.nd = h.M;
        return L;
    }
    L.r = __builtin_amdgcn_readfirstlane(__hip_atomic_load(h.ctrl + CTRL_RFINAL + cls, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT));
    const uint32_t ns = __builtin_amdgcn_readfirstlane(__hip_atomic_load(h.ctrl + CTRL_RSFINAL + cls,
                                                                         __ATOMIC_RELAXED,
                                                                         __HIP_MEMORY_SCOPE_AGENT));
    L.nd = L.r - ns;
    return L;
}

__device__ __forceinline__ bool heap_failed(const HeapView &h)
{
    return ald32(h.ctrl + CTRL_ERR) != 0;
}

// ------------------------------------------------------------ bit helpers --
__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// lane `from`'s value (from wave-uniform), in scalar registers
__device__ __forceinline__ uint64_t lane64(uint64_t v, uint32_t from)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)from);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), (int)from);
    return ((uint64_t)hi << 32) | lo;
}

// a value every lane holds alike, moved to scalar registers
__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// index of the n-th (0-based) set bit of b, or 64 if b has fewer bits
// (Alg. nth_set_bit: clear the lowest set bit n times, then find first set)
__device__ __forceinline__ uint32_t nth_set_bit(uint64_t b, uint32_t n)
{
    for (uint32_t i = 0; i < n && b; ++i) b &= b - 1;
    return b ? (uint32_t)(__ffsll((unsigned long long)b) - 1) : 64u;
}

// the lowest n set bits of b
__device__ __forceinline__ uint64_t lowest_bits(uint64_t b, uint32_t n)
{
    if ((uint32_t)__popcll(b) <= n) return b;
    uint32_t p = nth_set_bit(b, n);   // first bit not taken
    return b & ((1ull << p) - 1);
}

// the lowest n set bits of a wave-uniform b, n <= 64 (a lane per bit instead of
// a loop over the bits; converged)
__device__ __forceinline__ uint64_t wave_lowest_bits(uint64_t b, uint32_t n)
{
    const uint32_t lane = lane_id();
    return __ballot(((b >> lane) & 1) && (uint32_t)__popcll(b & ((1ull << lane) - 1)) < n);
}

// Lane r of the result is the position of the r-th set bit of a wave-uniform
// b, for r < popcount(b) (a permutation of the lanes; converged).
__device__ __forceinline__ uint32_t wave_set_bits(uint64_t b)
{
    const uint32_t lane = lane_id();
    const uint32_t below = (uint32_t)__popcll(b & ((1ull << lane) - 1));
    const uint32_t to = (b >> lane) & 1 ? below : (uint32_t)__popcll(b) + lane - below;
    return (uint32_t)__builtin_amdgcn_ds_permute((int)(to << 2), (int)lane);
}

__device__ __forceinline__ uint32_t hash32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352dU;
    x ^= x >> 15;
    x *= 0x846ca68bU;
    x ^= x >> 16;
    return x;
}

__device__ __forceinline__ uint32_t global_wave_id()
{
    return blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
}

// ---------------------------------------------------- hierarchical bitmap --
// A bitmap of M bits is a stack of levels; level l+1 has one bit per 64-bit
// container of level l, set iff that container is non-zero ("container
// consistency", sec.5.3.1).  Levels are only eventually consistent while
// kernels run; they are consistent whenever no kernel runs on the heap.

// One pending switch of a bit: dir +1 = set (0 -> 1), -1 = clear (1 -> 0).
// A successful switch that sets the first bit of a container, or clears its
// last bit, continues as the same switch one level up (Alg. try_clear).
struct BitOp {
    uint32_t pos;
    uint16_t bmid;
    int8_t lvl;
    int8_t dir;
};

// Invalidation attempts of one block (Alg. invalidate with rollback) before
// the release that emptied it gives up.  A further attempt follows only where
// slots were reserved and released again between two atomics of this one.
constexpr int kInvalidateAttempts = 3;

// The most switches that one release calls for: a re-activation, a rollback
// per failed attempt but the last, and the three of a successful invalidation.
// Releases make each as it falls due; a queue has room for as many, and its
// users (a destroy's settling launch and defragmentation) fill at most three.
constexpr int kMaxReleaseOps = 1 + (kInvalidateAttempts - 1) + 3;
constexpr int kMaxOps = kMaxReleaseOps;

// A lane's queue of pending switches.  A push into a full queue is not
// dropped silently: it marks the queue, and completing the queue raises
// ERR_INTERNAL (run_ops_wave, run_ops_lane).
struct OpQueue {
    BitOp op[kMaxOps];
    bool overflow;
    __host__ __device__ __forceinline__ void reset()
    {
#pragma unroll
        for (int i = 0; i < kMaxOps; ++i) op[i].dir = 0;
        overflow = false;
    }
    __host__ __device__ __forceinline__ bool push(uint32_t bmid, uint32_t pos, int dir)
    {
#pragma unroll
        for (int i = 0; i < kMaxOps; ++i)
            if (op[i].dir == 0) {
                op[i].pos = pos;
                op[i].bmid = (uint16_t)bmid;
                op[i].lvl = 0;
                op[i].dir = (int8_t)dir;
                return true;
            }
        overflow = true;
        return false;
    }
    __host__ __device__ __forceinline__ bool pending() const
    {
        bool p = false;
#pragma unroll
        for (int i = 0; i < kMaxOps; ++i) p |= op[i].dir != 0;
        return p;
    }
};

// One attempt of a pending switch.  A failed attempt (the bit already has the
// target value: another thread's opposite switch is still on its way) leaves
// the op pending; the caller retries it later.
__device__ __forceinline__ void bitop_try(const HeapView &h, BitOp &o)
{
    uint64_t *w = h.bm_word(o.bmid, (uint32_t)o.lvl, o.pos >> 6);
    const uint64_t bit = 1ull << (o.pos & 63);
    if (o.dir > 0) {
        const uint64_t prev = aor(w, bit);
        if (prev & bit) return;
        if (prev == 0 && (uint32_t)o.lvl + 1 < h.nlev) {
            o.lvl++;
            o.pos >>= 6;
            return;
        }
        o.dir = 0;
    } else {
        const uint64_t prev = aand(w, ~bit);
        if (!(prev & bit)) return;
        if (prev == bit && (uint32_t)o.lvl + 1 < h.nlev) {
            o.lvl++;
            o.pos >>= 6;
            return;
        }
        o.dir = 0;
    }
}

// Converged completion of every lane's pending switches.  All lanes of the
// wavefront that may hold pending switches must call this together; each
// iteration every lane tries each of its pending switches once, so a switch
// that waits for another lane's switch cannot block it.
__device__ __forceinline__ void run_ops_wave(const HeapView &h, OpQueue &q)
{
    if (q.overflow) raise_error(h, ERR_INTERNAL);
    for (uint32_t it = 0;; ++it) {
        bool pend = false;
#pragma unroll
        for (int i = 0; i < kMaxOps; ++i)
            if (q.op[i].dir) {
                bitop_try(h, q.op[i]);
                pend |= q.op[i].dir != 0;
            }
        const uint64_t pending = __ballot(pend);
        if (pending == 0) break;
        if (lane_id() == (uint32_t)(__ffsll((unsigned long long)pending) - 1)) count_event(h, EV_SPIN);
        if (it >= h.spin_limit) {
            if (pend) raise_error(h, ERR_SPIN);
            break;
        }
    }
}

// The same for a single lane running alone (no other lane of its wavefront
// holds pending switches while it runs).
__device__ __forceinline__ void run_ops_lane(const HeapView &h, OpQueue &q)
{
    if (q.overflow) raise_error(h, ERR_INTERNAL);
    for (uint32_t it = 0; q.pending(); ++it) {
        if (it >= h.spin_limit) {
            raise_error(h, ERR_SPIN);
            return;
        }
        if (it) count_event(h, EV_SPIN);
#pragma unroll
        for (int i = 0; i < kMaxOps; ++i)
            if (q.op[i].dir) bitop_try(h, q.op[i]);
    }
}

// Atomics of an allocating wavefront: made by lane `who`, their results known
// to every lane (converged).
__device__ __forceinline__ uint64_t aor_one(uint32_t who, uint64_t *p, uint64_t v)
{
    uint64_t prev = 0;
    if (lane_id() == who) prev = aor(p, v);
    return lane64(prev, who);
}

__device__ __forceinline__ uint64_t aand_one(uint32_t who, uint64_t *p, uint64_t v)
{
    uint64_t prev = 0;
    if (lane_id() == who) prev = aand(p, v);
    return lane64(prev, who);
}

__device__ __forceinline__ void count_event_one(const HeapView &h, uint32_t who, uint32_t ev, uint32_t n = 1)
{
    if (lane_id() == who) count_events(h, ev, n);
}

// Completes one switch, beginning at level lvl, for a wavefront whose lanes
// hold no other pending switch (converged; all arguments wave-uniform).
__device__ __forceinline__ void switch_bit_one(const HeapView &h, uint32_t who, uint32_t bmid, uint32_t pos, int dir,
                                               uint32_t lvl = 0)
{
    for (uint32_t it = 0;; ++it) {
        if (it >= h.spin_limit) {
            if (lane_id() == who) raise_error(h, ERR_SPIN);
            return;
        }
        uint64_t *const w = h.bm_word(bmid, lvl, pos >> 6);
        const uint64_t bit = 1ull << (pos & 63);
        const uint64_t prev = dir > 0 ? aor_one(who, w, bit) : aand_one(who, w, ~bit);
        const bool was = (prev & bit) != 0;
        if (was != (dir > 0)) {                      // switched here
            if ((dir > 0 ? prev != 0 : prev != bit) || lvl + 1 >= h.nlev) return;
            ++lvl;
            pos >>= 6;
        }
        count_event_one(h, who, EV_SPIN);
    }
}

// The set bit of container c != 0 that a search at level lvl takes: the first
// one at or after a seed-dependent position ("Bitmap Rotation", sec.5.3.2), or
// the lowest one with rotation off.  The position is drawn between the lowest
// and the highest set bit, not over all 64: a class's blocks are clusters of
// neighbouring bits, and from a position outside the cluster every search
// would land on the cluster's first bit.  Seven containers of the top level
// in use, as for 256 x 256 cells, gave the first of them 90 % of the
// searches, and 29 % of the reservations lost their block to another one.
__device__ __forceinline__ uint32_t pick_bit(const HeapView &h, uint64_t c, uint32_t seed, uint32_t lvl)
{
    const uint32_t lo = (uint32_t)(__ffsll((unsigned long long)c) - 1);
    if (!h.rotation) return lo;
    const uint32_t span = 64u - (uint32_t)__clzll((long long)c) - lo;
    const uint32_t at = lo + __umulhi(hash32(seed + 0x9E3779B9u * (lvl + 1)), span);
    return at + (uint32_t)(__ffsll((unsigned long long)(c >> at)) - 1);
}

// Alg. try_find_set: top-down descent, at each level the container's set bit
// that pick_bit takes.  May fail spuriously while levels are inconsistent.
// Searches for a free block take the lowest bit above level 1, so that blocks
// are claimed from one window of 4,096 after the other: the blocks of the
// classes that grow then lie together, and the drawn positions of the later
// searches for their active blocks find them evenly.  Claimed anywhere in the
// heap, a few of them in every container, they drew as many requests as the
// full containers did: 4096 x 4096 cells took 2.5 ms a generation (3.3 M of
// 10.2 M searches wasted over twelve), 0.74 ms now (0.3 M of 4.2 M); 256 x 256
// cells 29 us before both changes, 21.5 us now.  `anywhere` draws there too.
// Converged call, every argument and the result wave-uniform.
__device__ __forceinline__ uint32_t find_set(const HeapView &h, uint32_t who, uint32_t bmid, uint32_t seed,
                                             bool anywhere = false)
{
    count_event_one(h, who, EV_FIND);
    uint32_t idx = 0;
    for (int lvl = (int)h.nlev - 1; lvl >= 0; --lvl) {
        const uint64_t c = uniform64(ald(h.bm_word(bmid, (uint32_t)lvl, idx)));
        if (!c) return kNoBlock;
        const uint32_t b = bmid == BM_FREE && lvl >= 2 && !anywhere ? (uint32_t)(__ffsll((unsigned long long)c) - 1)
                                                                    : pick_bit(h, c, seed, (uint32_t)lvl);
        idx = idx * 64u + b;
    }
    return idx;
}

// Bitmap::clear() on the free-block bitmap: find a set bit and switch it off;
// retry the search if another thread switched it first.  Returns kNoBlock when
// no free block is found (the thesis spins forever here; we report exhaustion).
// Converged call, wave-uniform as find_set.
__device__ __forceinline__ uint32_t claim_free_block(const HeapView &h, uint32_t who, uint32_t seed)
{
    // Misses at the lowest window before the search draws at every level, and
    // misses in a row after that which mean that the heap is exhausted: the
    // window's summary bits may be behind, cleared by a claimer that has yet to
    // pass it on, while the other windows have blocks.  Drawn from the first
    // miss on, the claims scatter (4096 x 4096 cells, a frame of two
    // generations 1180 us, 987 so; ten wa-tor iterations on 1024 x 1024 cells
    // 4289 and 3432).
    constexpr uint32_t kWindowMisses = 64, kDrawnMisses = 128;
    uint32_t misses = 0;
    for (uint32_t t = 0; t < h.spin_limit; ++t) {
        const uint32_t b = find_set(h, who, BM_FREE, seed + t * 0x632BE5ABu, misses >= kWindowMisses);
        if (b == kNoBlock) {
            // A search can miss while another thread is between two levels
            // of the hierarchy; only a run of consecutive misses means the
            // heap is exhausted.  Races lost to other claimers (below) are
            // progress of others and do not count.
            if (++misses > kWindowMisses + kDrawnMisses) return kNoBlock;
            __builtin_amdgcn_s_sleep(4);
            continue;
        }
        misses = 0;
        const uint64_t bit = 1ull << (b & 63);
        const uint64_t prev = aand_one(who, h.bm_word(BM_FREE, 0, b >> 6), ~bit);
        if (!(prev & bit)) continue;           // someone else took it
        if (prev == bit && h.nlev > 1)         // cleared the container's last bit
            switch_bit_one(h, who, BM_FREE, b >> 6, -1, 1);
        return b;
    }
    if (lane_id() == who) raise_error(h, ERR_SPIN);
    return kNoBlock;
}

// Alg. initialize_block: publish the type, then reset the allocation bitmap
// (every class has capacity 64, so no tail bits are pre-set); both complete
// before the caller sets the block's allocated and active bits.
__device__ __forceinline__ void initialize_block(const HeapView &h, uint32_t bid, uint32_t cls)
{
    __hip_atomic_store(h.type + bid, cls, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    complete_prior();
    __hip_atomic_store(h.alloc_bm + bid, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    complete_prior();
}

// Block::reserve, extended to up to n slots at once (reserve_multiple):
// returns the mask of slots this call switched 0 -> 1 (0 = block full or
// invalidated) and whether this call made the block full.  Converged call,
// wave-uniform as find_set.
__device__ __forceinline__ uint64_t reserve_slots(const HeapView &h, uint32_t who, uint32_t bid, uint32_t n,
                                                  bool &filled)
{
    uint64_t *p = h.alloc_bm + bid;
    uint64_t cur = uniform64(ald(p));
    filled = false;
    for (int it = 0; it < 64; ++it) {
        const uint64_t want = wave_lowest_bits(~cur, n);
        if (!want) return 0;
        const uint64_t prev = aor_one(who, p, want);
        const uint64_t got = want & ~prev;
        if (got) {
            filled = (prev | want) == ~0ull;
            return got;
        }
        cur = prev | want;   // all wanted slots were taken meanwhile; look again
    }
    return 0;
}

// ------------------------------------------------------------- allocation --
// Block::deallocate for a set of slots of one block, with the block-state
// consequences of Alg. deallocate: the release that frees the first slot of a
// full block re-activates it; the release that empties it invalidates it (Alg.
// invalidate: try to switch all 64 slots to 1 so that no reservation can
// succeed; on success the block is empty and can be freed; if some slot was
// reserved meanwhile, roll back, and owe the deferred active-bit clear when a
// concurrent release saw the block as full).  Releasing a free slot raises the
// bad-handle error.  Each switch is completed before the next is begun: one
// only ever waits for a switch that an earlier change of its block's bitmap
// calls for, and every wavefront makes its own in the order of its changes, so
// no two can wait for each other.

// ... for one block, by lane `who` (converged, arguments wave-uniform).
__device__ __forceinline__ void give_back_slots(const HeapView &h, uint32_t who, uint32_t cls, uint32_t bid,
                                                uint64_t mask)
{
    uint64_t *const p = h.alloc_bm + bid;
    const uint64_t prev = aand_one(who, p, ~mask);
    if ((prev & mask) != mask) {
        if (lane_id() == who) raise_error(h, ERR_BADHANDLE);
        return;
    }
    count_event_one(h, who, EV_DELS, (uint32_t)__popcll(mask));
    if (prev == ~0ull) switch_bit_one(h, who, bm_active(cls), bid, +1);
    if ((prev & ~mask) != 0) return;
    for (int attempt = 0; attempt < kInvalidateAttempts; ++attempt) {
        const uint64_t before = aor_one(who, p, ~0ull);
        if (before == ~0ull) return;
        const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)ald32(h.type + bid));
        if (before == 0) {
            // The block is ours and empty.  Retire its type before it is
            // marked free, so a stale block list sees it as not of class t
            // and a later initialize_block's store of a new type comes after.
            if (lane_id() == who)
                __hip_atomic_store(h.type + bid, kNull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            complete_prior();
            switch_bit_one(h, who, bm_active(t), bid, -1);
            switch_bit_one(h, who, bm_alloc(t), bid, -1);
            switch_bit_one(h, who, BM_FREE, bid, +1);
            return;
        }
        const uint64_t before_rb = aand_one(who, p, before);
        if (before_rb != ~0ull) switch_bit_one(h, who, bm_active(t), bid, -1);
        if ((before_rb & before) != 0) return;
        // empty again: retry the invalidation
    }
}

// One switch a lane, where todo, beginning at level lvl, completed by all of
// them together (converged; the lanes' switches go the same way in bitmaps of
// one kind, so none of them waits for another one of these).
__device__ __forceinline__ void switch_bits(const HeapView &h, bool todo, uint32_t bmid, uint32_t pos, int dir,
                                            uint32_t lvl = 0)
{
    for (uint32_t it = 0;; ++it) {
        if (todo) {
            uint64_t *const w = h.bm_word(bmid, lvl, pos >> 6);
            const uint64_t bit = 1ull << (pos & 63);
            const uint64_t prev = dir > 0 ? aor(w, bit) : aand(w, ~bit);
            const bool was = (prev & bit) != 0;
            if (was != (dir > 0)) {
                todo = !(dir > 0 ? prev != 0 : prev != bit) && lvl + 1 < h.nlev;
                ++lvl;
                pos >>= 6;
            }
        }
        const uint64_t pending = __ballot(todo);
        if (pending == 0) return;
        if (lane_id() == (uint32_t)(__ffsll((unsigned long long)pending) - 1)) count_event(h, EV_SPIN);
        if (it >= h.spin_limit) {
            if (todo) raise_error(h, ERR_SPIN);
            return;
        }
    }
}

// ... for a block a lane, the lanes' blocks distinct (mask 0 = none), side by
// side.  Returns whether the lane's slots were live; the caller counts the
// deletions.  Converged call.  A step for all lanes after the other, not a
// queue of switches a lane: 28 vector registers less.
__device__ __forceinline__ bool release_beside(const HeapView &h, uint32_t cls, uint32_t bid, uint64_t mask)
{
    uint64_t *const p = h.alloc_bm + bid;
    const uint64_t prev = mask ? aand(p, ~mask) : 0;
    const bool ok = mask && (prev & mask) == mask;
    if (mask && !ok) raise_error(h, ERR_BADHANDLE);
    switch_bits(h, ok && prev == ~0ull, bm_active(cls), bid, +1);
    bool empty = ok && (prev & ~mask) == 0;
    for (int attempt = 0; attempt < kInvalidateAttempts && __ballot(empty); ++attempt) {
        bool freed = false, owed = false;
        uint32_t t = 0;
        if (empty) {
            const uint64_t before = aor(p, ~0ull);
            empty = before != ~0ull;
            if (empty) {
                t = ald32(h.type + bid);
                if (before == 0) {
                    __hip_atomic_store(h.type + bid, kNull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    freed = true;
                } else {
                    const uint64_t before_rb = aand(p, before);
                    owed = before_rb != ~0ull;
                    empty = (before_rb & before) == 0;
                }
            }
        }
        complete_prior();
        switch_bits(h, freed || owed, bm_active(t), bid, -1);
        switch_bits(h, freed, bm_alloc(t), bid, -1);
        switch_bits(h, freed, BM_FREE, bid, +1);
        empty = empty && !freed;
    }
    return ok;
}

// The leader's part of Alg. allocate with request coalescing: find an active
// block of the class (lookup retry with rotation), else initialize a free
// block (slow path); reserve up to n slots; deactivate the block if this
// filled it; roll back if the block's type changed meanwhile.
// The whole wavefront runs it, with wave-uniform values in scalar registers;
// lane `who` makes the atomics.  Run by that lane alone, its values were in
// vector registers, 104 of them in a kernel that allocates: four wavefronts a
// SIMD, where an allocation, a chain of dependent accesses, wants as many in
// flight as there can be.  69 and seven now: death and birth of a generation of
// 4096 x 4096 cells 600 us before, 457 so, 401 with the deaths' releases made
// the same way; births of 256 x 256 cells 14.3 us and 12.5.
__device__ __forceinline__ uint32_t leader_allocate(const HeapView &h, uint32_t who, uint32_t cls, uint32_t n,
                                                    uint64_t &got, uint32_t seed, uint32_t first = kNoBlock)
{
    got = 0;
    for (uint32_t attempt = 0; attempt < h.spin_limit; ++attempt) {
        // the first attempt may start from a block found in a prefetched
        // view of the active bitmap (wave_allocate with an ActiveView)
        uint32_t bid = attempt == 0 ? first : kNoBlock;
        for (uint32_t t = 0; t < h.retries && bid == kNoBlock; ++t)
            bid = find_set(h, who, bm_active(cls), hash32(seed + attempt * 977u + t * 131u));
        if (bid == kNoBlock) {
            bid = claim_free_block(h, who, hash32(seed ^ (attempt * 0x27d4eb2fu)));
            if (bid == kNoBlock) {
                if (lane_id() == who) raise_error(h, ERR_NOMEM);
                return kNoBlock;
            }
            if (lane_id() == who) initialize_block(h, bid, cls);
            switch_bit_one(h, who, bm_alloc(cls), bid, +1);
            switch_bit_one(h, who, bm_active(cls), bid, +1);
            count_event_one(h, who, EV_SLOW);
        }
        bool filled;
        const uint64_t g = reserve_slots(h, who, bid, n, filled);
        if (g) {
            // issued after the reservation has been performed (its result
            // is used), so it sees the type published before the reset
            const uint32_t t = __builtin_amdgcn_readfirstlane(ald32(h.type + bid));
            if (filled) switch_bit_one(h, who, bm_active(t), bid, -1);
            if (t == cls) {
                got = g;
                count_event_one(h, who, EV_NEWS, (uint32_t)__popcll(g));
                return bid;
            }
            give_back_slots(h, who, t, bid, g);   // block re-typed meanwhile: roll back
        }
        count_event_one(h, who, EV_RETRY);
    }
    if (lane_id() == who) raise_error(h, ERR_SPIN);
    return kNoBlock;
}

// A prefetched view of the upper part of class cls's active-block bitmap:
// lane i holds container i of level L = max(nlev - 2, 0), which has at most
// 64 containers (the level above it is one container).  Taken with plain
// loads before a method's allocation, in the same batch as the method's own
// loads, it lets the allocating wavefront skip the two top levels of the
// active-block search.  It is a hint: the reservation checks the block it
// picks, and a block that filled since the view was taken costs one retry
// through the ordinary search.
struct ActiveView {
    uint64_t w;
};

__device__ __forceinline__ ActiveView active_view(const HeapView &h, uint32_t cls)
{
    const uint32_t lvl = h.nlev >= 2 ? h.nlev - 2 : 0;
    const uint32_t lane = lane_id();
    ActiveView v;
    v.w = lane < h.lvl_n[lvl] ? *h.bm_word(bm_active(cls), lvl, lane) : 0ull;
    return v;
}

// The rest of Alg. try_find_set from a view: the container at level L and the
// bit in it picked as find_set picks them, then the levels below L by loads.  Converged call; the result is
// wave-uniform (kNoBlock if the view shows no active block).
__device__ __forceinline__ uint32_t find_set_from_view(const HeapView &h, uint32_t bmid, const ActiveView &v,
                                                      uint32_t seed)
{
    const int lvl = h.nlev >= 2 ? (int)h.nlev - 2 : 0;
    const uint64_t nz = __ballot(v.w != 0);
    if (!nz) return kNoBlock;
    uint32_t idx = 0;
    if (h.nlev >= 2) idx = pick_bit(h, nz, seed, (uint32_t)lvl + 1);   // the single container above L, as the ballot
    uint64_t c = lane64(v.w, idx);
    for (int l = lvl;; --l) {
        idx = idx * 64u + pick_bit(h, c, seed, (uint32_t)l);
        if (l == 0) break;
        c = uniform64(ald(h.bm_word(bmid, (uint32_t)l - 1, idx)));
        if (!c) return kNoBlock;
    }
    return idx;
}

// Allocation of one object of class `cls` for every lane with want = true.
// Must be called by all lanes of the wavefront together (converged).  With
// coalescing the lowest requesting lane allocates for all requesting lanes;
// each lane takes the slot whose rank among the reserved slots equals its
// rank among the requesting lanes.  Returns the handle, or SMMO_NULL when
// want is false or the heap is exhausted.
__device__ __forceinline__ uint32_t wave_allocate(const HeapView &h, uint32_t cls, bool want,
                                                  const ActiveView *view = nullptr)
{
    uint32_t result = kNull;
    uint64_t pending = __ballot(want);
    const uint32_t lane = lane_id();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)global_wave_id());
    const uint32_t seed = hash32(wave * 0x9E3779B1u + 0x51ED27u);
    for (uint32_t round = 0; pending; ++round) {
        const uint32_t leader = (uint32_t)(__ffsll((unsigned long long)pending) - 1);
        const uint32_t n = h.coalescing ? (uint32_t)__popcll(pending) : 1u;
        uint64_t got;
        const uint32_t rseed = seed + round * 0x85ebca6bu;
        // the first round's first lookup from the view (seeded as the
        // ordinary search's first lookup would be)
        uint32_t first = kNoBlock;
        if (view && round == 0) {
            count_event_one(h, leader, EV_FIND);
            first = find_set_from_view(h, bm_active(cls), *view, hash32(rseed));
        }
        const uint32_t bid = leader_allocate(h, leader, cls, n, got, rseed, first);
        if (bid == kNoBlock) break;
        const uint32_t k = (uint32_t)__popcll(got);
        // the lane of rank r takes the r-th reserved slot
        const uint32_t rank = (uint32_t)__popcll(pending & ((1ull << lane) - 1));
        const uint32_t slot = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((rank & 63) << 2), (int)wave_set_bits(got));
        const bool served = ((pending >> lane) & 1) && rank < k;
        if (served) result = (bid << 6) | slot;
        pending &= ~__ballot(served);
    }
    return result;
}

// OR of v over the lanes of the wavefront (butterfly over both halves)
__device__ __forceinline__ uint64_t wave_or64(uint64_t v)
{
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        lo |= (uint32_t)__shfl_xor((int)lo, d);
        hi |= (uint32_t)__shfl_xor((int)hi, d);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Deallocation of the objects named by `handle` (one per lane with want), the
// class of each block given by cls_of(block), which may raise an error and
// return kNull to leave the block alone.  Converged call.  Lanes whose objects
// share a block are released together, one atomic per distinct block (the
// multi-slot release of sec.5.3.2), and all the wavefront's blocks side by
// side: the first lane of each group holds the group's slots and makes its
// release.
// A release is a chain of dependent atomics (the block's bitmap, then a
// switch per level it passes on to), 1-2 us however many lanes make it: one
// block after the other, as handles in no order name them, took 7 times as
// long (64 distinct blocks a wavefront: 924 us for a million deletions in
// shuffled order, side by side 144).
// The grouping itself is scalar work on ballots; finding the lanes without a
// partner first, by a ballot per bit of the block index, gave nothing.
template <class ClassOf>
__device__ __forceinline__ void wave_release_handles(const HeapView &h, uint32_t handle, bool want, ClassOf &&cls_of)
{
    const uint32_t lane = lane_id();
    uint64_t pending = __ballot(want);
    if (!pending) return;
    const uint32_t first = (uint32_t)(__ffsll((unsigned long long)pending) - 1);
    uint64_t mine = 0;
    uint32_t count = 0;
    while (pending) {
        const uint32_t leader = (uint32_t)(__ffsll((unsigned long long)pending) - 1);
        const uint32_t b = (uint32_t)__builtin_amdgcn_readlane(handle, leader) >> 6;
        const uint64_t group = __ballot((handle >> 6) == b) & pending;
        pending &= ~group;
        uint64_t slots = 0;
        for (uint64_t g = group; g; g &= g - 1)
            slots |= 1ull << (__builtin_amdgcn_readlane(handle, (uint32_t)(__ffsll((unsigned long long)g) - 1)) & 63);
        const uint32_t n = (uint32_t)__popcll(slots);
        count += n;
        if (lane == leader) {
            mine = slots;
            // two lanes naming one object: released once, reported as a bad handle
            if (n != (uint32_t)__popcll(group)) raise_error(h, ERR_BADHANDLE);
        }
    }
    const uint32_t cls = mine ? cls_of(handle >> 6) : kNull;
    const bool failed = !release_beside(h, cls, handle >> 6, cls == kNull ? 0 : mine) && mine;
    for (uint64_t f = __ballot(failed); f; f &= f - 1)
        count -= (uint32_t)__builtin_amdgcn_readlane(__popcll(mine), (uint32_t)(__ffsll((unsigned long long)f) - 1));
    if (lane == first && count) count_events(h, EV_DELS, count);
}

// Deallocation of arbitrary handles of class `cls` (one per lane with want).
// Converged call.  Handles must name live objects of the class.
__device__ __forceinline__ void wave_deallocate(const HeapView &h, uint32_t cls, uint32_t handle,
                                                bool want)
{
    wave_release_handles(h, handle, want, [&](uint32_t) { return cls; });
}

// Deallocation of objects that delete themselves inside a method: the
// wavefront processes one block, so all its releases go to that block and
// are combined into one atomic (the multi-slot release of sec.5.3.2).
// Converged call; `mask` is the ballot of the lanes deleting their object.
// One release at a time, as an allocating wavefront gives slots back: 24 vector
// registers for Alive::death where the queue took 59.
__device__ __forceinline__ void wave_release_own_block(const HeapView &h, uint32_t cls, uint32_t bid,
                                                       uint64_t mask)
{
    if (!mask) return;
    give_back_slots(h, (uint32_t)(__ffsll((unsigned long long)mask) - 1), cls,
                    (uint32_t)__builtin_amdgcn_readfirstlane((int)bid), mask);
}

} // namespace smmo
