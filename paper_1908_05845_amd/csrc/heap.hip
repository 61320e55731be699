// libsmmo: schema, heap and SMMO operations (C ABI in include/smmo.h).
//
// Heap operations follow the DynaSOAr design (Springer, Ch.5): equal-size
// blocks of one class each, hierarchical block-state bitmaps, the lock-free
// object allocator, and do-all enumeration over a compacted list of
// allocated blocks (sec.5.2.7, with the bitmap `indices` operation of
// sec.5.3.1).  Device code is in smmo_device.hpp; methods in methods.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>

#include "smmo_device.hpp"
#include "smmo_host.hpp"

using namespace smmo;

namespace {

thread_local std::string g_last_error;

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct Layout {
    uint32_t nlev = 0;
    uint32_t lvl_n[kMaxLevels] = {};
    uint32_t lvl_off[kMaxLevels] = {};
    uint32_t bm_words = 0;
    size_t ctrl = 0, bm = 0, type = 0, alloc = 0, iter = 0, R = 0, claim = 0, blocks = 0, total = 0;
};

void layout_for(uint32_t nclasses, uint64_t M, uint32_t block_bytes, Layout &L)
{
    L = Layout{};
    uint64_t n = (M + 63) / 64;
    uint32_t off = 0;
    for (;;) {
        L.lvl_n[L.nlev] = (uint32_t)n;
        L.lvl_off[L.nlev] = off;
        off += (uint32_t)n;
        L.nlev++;
        if (n == 1) break;
        n = (n + 63) / 64;
    }
    L.bm_words = off;
    const uint64_t nbm = 1 + 2ull * nclasses;
    size_t p = 0;
    L.ctrl = p;   p += align256(kCtrlWords * 4);
    L.bm = p;     p += align256(nbm * L.bm_words * 8);
    L.type = p;   p += align256(M * 4);
    L.alloc = p;  p += align256(M * 8);
    L.iter = p;   p += align256(M * 8);
    L.R = p;      p += align256((size_t)nclasses * M * 4);
    L.claim = p;  p += align256(M * 4);
    L.blocks = p; p += (size_t)M * block_bytes;
    L.total = p;
}

uint32_t schema_block_bytes(const smmo_schema *s)
{
    uint32_t b = 256;
    for (uint32_t c = 0; c < s->nclasses; ++c) b = std::max(b, s->c[c].data_bytes);
    return b;
}

bool heap_ok(const smmo_heap *h) { return h && h->schema && h->base; }

smmo_status check_class(const smmo_heap *h, uint32_t cls)
{
    if (!heap_ok(h)) return fail(SMMO_EINVAL, "heap is NULL or freed");
    if (cls >= h->schema->nclasses) return fail(SMMO_EINVAL, "class id out of range");
    return SMMO_OK;
}

// ----------------------------------------------------------------- kernels --

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    const uint32_t lane = lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(v, (unsigned)d);
        if (lane >= (uint32_t)d) v += y;
    }
    return v;
}

// exclusive scan over a work-group of up to 1024 threads; *total = sum
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *s_w, uint32_t &total)
{
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint32_t incl = wave_incl_scan(v);
    if (lane == 63) s_w[w] = incl;
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (uint32_t i = 0; i < nw; ++i) {
        const uint32_t x = s_w[i];
        if (i < w) before += x;
        tot += x;
    }
    __syncthreads();
    total = tot;
    return before + incl - v;
}

// All blocks free (free bitmap full, allocation bitmaps all-ones as if
// invalidated, type unset), other bitmaps empty, control words zero.
__global__ void k_heap_init(HeapView h)
{
    const uint64_t nbw = (1ull + 2ull * h.nclasses) * h.bm_words;
    const uint64_t total = std::max<uint64_t>(std::max<uint64_t>(h.M, nbw), kCtrlWords);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        if (i < h.M) {
            h.type[i] = kNull;
            h.alloc_bm[i] = ~0ull;
            h.iter_bm[i] = 0;
        }
        if (i < nbw) {
            const uint32_t bmid = (uint32_t)(i / h.bm_words);
            const uint32_t w = (uint32_t)(i % h.bm_words);
            uint64_t val = 0;
            if (bmid == BM_FREE) {
                uint32_t l = 0;
                while (l + 1 < h.nlev && w >= h.lvl_off[l + 1]) ++l;
                const uint32_t c = w - h.lvl_off[l];
                const uint64_t nchild = l == 0 ? h.M : h.lvl_n[l - 1];
                const uint64_t lo = (uint64_t)c * 64;
                const uint64_t cnt = nchild > lo ? std::min<uint64_t>(64, nchild - lo) : 0;
                val = cnt == 64 ? ~0ull : ((1ull << cnt) - 1);
            }
            h.bm[i] = val;
        }
        if (i < kCtrlWords) h.ctrl[i] = 0;
    }
}

// Enumeration pre-pass (sec.5.2.7 with Alg. indices of sec.5.3.1): compact
// the set bits of allocated[cls] into R.  A wavefront takes kPer containers
// of level 0 (a lane reads one), a work-group the 16 kPer of its wavefronts (every container is
// read: the level-1 summary would only add a dependent load for 8 bytes per
// 64 blocks).  A lane takes one block of a container, so bitmaps are read and
// R is written in runs.  The packing plan (split): blocks with more than 32
// live objects are dense.  Without it every block counts as dense.
// The work-group's place in R:
//   in order    (at most 1,024 containers) it counts the blocks of the
//               work-groups before it itself, from all the containers, one a
//               thread; for a plan also from their blocks' bitmaps.  R is in
//               block order, and nothing is shared between work-groups.
//   as it comes it reserves its ranges (dense blocks at the front, sparse
//               ones at the back) and counts itself finished with one 64-bit
//               atomic add on the class's packed counter, so R is ordered
//               within a work-group's ranges only.  The work-group whose add
//               finds every other one finished knows the totals: it publishes
//               the lengths and zeroes the counter, so the pass needs no
//               reset launch and can be captured in a graph.
// (The lengths are read by later launches only.)
// Bound by its chain of dependent accesses and the launch, as long as there
// are work-groups for the CUs: with 1,024 containers a work-group, a thread
// writing the entries of each, one CU wrote what 65,536 blocks list.  A full
// list of 294,000 blocks 50 us, 7.6 now; wa-tor on 1024 x 1024 cells 9 and
// 5.3.  With snapshot and plan, launch included, 65,536 full blocks 53 us and
// 11, 1M 59 and 14, 4M 59 and 20, 16M 60 and 42; 4,096 15 and 10.5.  Empty
// containers are passed over by a ballot: 1,024 full blocks in a heap of 2^24
// 12.0 us and 9.5.
constexpr uint64_t kPackMask = (1ull << 25) - 1;
constexpr uint32_t kFewContainers = 1024;     // in order: one container a thread
// beyond: 16 and 64 containers a wavefront, for the atomics' sake
constexpr uint32_t kManyContainers = 16384, kMostContainers = 65536;
static_assert(kMaxBlocks <= kPackMask, "block counts must fit the packed enumeration counter");
static_assert((kMaxBlocks / 64 + 1024) / 1024 < (1u << 14) && kMostContainers / 256 < (1u << 14) &&
                  kManyContainers / 64 < (1u << 14),
              "work-group counts must fit the packed enumeration counter");

template <int kPer>
__global__ __launch_bounds__(1024) void k_enumerate(HeapView h, uint32_t cls, uint32_t snapshot, uint32_t split,
                                                    uint32_t ordered)
{
    constexpr int kBatch = kPer < 8 ? kPer : 8;
    constexpr uint32_t kGroup = 16 * kPer;
    __shared__ uint64_t s_all[kFewContainers];
    __shared__ uint32_t s_nd[16], s_ns[16], s_bd[16], s_bs[16];
    __shared__ uint32_t s_kd, s_ks;
    const uint32_t lane = lane_id(), wig = threadIdx.x >> 6;
    const uint32_t n0 = h.lvl_n[0];
    const uint32_t base = blockIdx.x * kGroup;
    const uint32_t first = base + wig * kPer;            // the wavefront's first container
    const uint64_t *const C = h.bm_word(bm_alloc(cls), 0, 0);
    const bool ok = ald32(h.ctrl + CTRL_ERR) == 0;       // a failed heap lists nothing
    // No wavefront changes a bitmap while this kernel runs, so plain loads
    // are enough.
    const uint64_t mine = ok && ordered && threadIdx.x < n0 ? C[threadIdx.x] : 0ull;
    // lane j: container first + j and its dense blocks
    const uint64_t cl = ok && lane < kPer && first + lane < n0 ? C[first + lane] : 0ull;
    const uint64_t some = __ballot(cl != 0);
    uint64_t dl = cl;
    if (snapshot | split) {
        for (uint64_t g = some; g;) {
            uint32_t j[kBatch];
            uint64_t c[kBatch], bm[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                j[u] = g ? (uint32_t)(__ffsll((unsigned long long)g) - 1) : 0u;
                c[u] = g ? lane64(cl, j[u]) : 0ull;
                g &= g - 1;
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                bm[u] = (c[u] >> lane) & 1 ? h.alloc_bm[(uint64_t)(first + j[u]) * 64 + lane] : 0ull;
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const bool in = (c[u] >> lane) & 1;
                if (snapshot && in) h.iter_bm[(uint64_t)(first + j[u]) * 64 + lane] = bm[u];
                const uint64_t d = __ballot(in && __popcll(bm[u]) > 32);
                if (split && c[u] && lane == j[u]) dl = d;
            }
        }
    }
    uint32_t nd = (uint32_t)__popcll(dl), ns = (uint32_t)__popcll(cl & ~dl);
#pragma unroll
    for (int d = 1; d < kPer; d <<= 1) {
        nd += (uint32_t)__shfl_xor((int)nd, d);
        ns += (uint32_t)__shfl_xor((int)ns, d);
    }
    uint32_t bd = 0, bs = 0;                             // of the work-groups before this one
    if (ordered) {
        if (split) {
            s_all[threadIdx.x] = mine;
            __syncthreads();
            for (uint32_t j0 = wig; j0 < base; j0 += 256) {
                uint64_t c[16], bm[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) c[u] = j0 + 16 * u < base ? s_all[j0 + 16 * u] : 0ull;
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    bm[u] = (c[u] >> lane) & 1 ? h.alloc_bm[(uint64_t)(j0 + 16 * u) * 64 + lane] : 0ull;
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const uint32_t d = (uint32_t)__popcll(__ballot(__popcll(bm[u]) > 32));
                    bd += d;
                    bs += (uint32_t)__popcll(c[u]) - d;
                }
            }
        } else {
            uint32_t k = threadIdx.x < base ? (uint32_t)__popcll(mine) : 0u;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) k += (uint32_t)__shfl_xor((int)k, d);
            bd = k;
        }
    }
    if (lane == 0) {
        s_nd[wig] = nd;
        s_ns[wig] = ns;
        s_bd[wig] = bd;
        s_bs[wig] = bs;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t td = 0, ts = 0, kd = 0, ks = 0;
        for (int k = 0; k < 16; ++k) {
            td += s_nd[k];
            ts += s_ns[k];
            kd += s_bd[k];
            ks += s_bs[k];
        }
        bool last;
        uint64_t *pack = reinterpret_cast<uint64_t *>(h.ctrl + CTRL_RPACK + 2 * cls);
        if (ordered) {
            last = blockIdx.x == gridDim.x - 1;
        } else {
            const uint64_t add = (uint64_t)td | ((uint64_t)ts << 25) | (1ull << 50);
            const uint64_t old = __hip_atomic_fetch_add(pack, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            kd = (uint32_t)(old & kPackMask);
            ks = (uint32_t)((old >> 25) & kPackMask);
            last = (old >> 50) == gridDim.x - 1;
            if (last) __hip_atomic_store(pack, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (last) {
            __hip_atomic_store(h.ctrl + CTRL_RFINAL + cls, kd + td + ks + ts, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(h.ctrl + CTRL_RSFINAL + cls, ks + ts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        s_kd = kd;
        s_ks = ks;
    }
    __syncthreads();
    uint32_t kd = s_kd, ks = s_ks;
    for (uint32_t k = 0; k < wig; ++k) {      // the ranges of the group's earlier wavefronts
        kd += s_nd[k];
        ks += s_ns[k];
    }
    uint32_t *R = h.R + (uint64_t)cls * h.M;
    const uint64_t below = (1ull << lane) - 1;
    for (uint64_t g = some; g; g &= g - 1) {
        const uint32_t j = (uint32_t)(__ffsll((unsigned long long)g) - 1), b = (first + j) * 64 + lane;
        const uint64_t c = lane64(cl, j), d = lane64(dl, j), sp = c & ~d;
        if ((d >> lane) & 1) R[kd + (uint32_t)__popcll(d & below)] = b;
        else if ((sp >> lane) & 1) R[h.M - 1 - (ks + (uint32_t)__popcll(sp & below))] = b;
        kd += (uint32_t)__popcll(d);
        ks += (uint32_t)__popcll(sp);
    }
}

struct FieldCopy {
    uint32_t offset;     // byte offset of element 0's array in a block
    uint32_t stride;     // bytes between inner elements' arrays
    uint32_t size;       // bytes per element (1 or 4)
    uint32_t count;      // inner elements
    const void *src;     // dense source (NULL = zero fill), or destination for gather
};

struct FieldSet {
    uint32_t nf;
    FieldCopy f[SMMO_MAX_FIELDS];
};

__device__ __forceinline__ void init_object(const HeapView &h, const FieldSet &fs, uint32_t handle,
                                            uint64_t i)
{
    char *base = h.block(handle >> 6);
    const uint32_t slot = handle & 63;
    for (uint32_t f = 0; f < fs.nf; ++f) {
        const FieldCopy &fc = fs.f[f];
        for (uint32_t q = 0; q < fc.count; ++q) {
            char *dst = base + fc.offset + q * fc.stride + slot * fc.size;
            const uint64_t e = i * fc.count + q;
            if (fc.size == 4) {
                *reinterpret_cast<uint32_t *>(dst) =
                    fc.src ? reinterpret_cast<const uint32_t *>(fc.src)[e] : 0u;
            } else {
                *reinterpret_cast<uint8_t *>(dst) =
                    fc.src ? reinterpret_cast<const uint8_t *>(fc.src)[e] : (uint8_t)0;
            }
        }
    }
}

// Ordered bulk claim for parallel_new: one work-group takes the `need` lowest
// free blocks in ascending order, clears their free bits, recomputes the free
// bitmap's summary levels over the touched range, and marks the blocks as
// allocated (and the last one active when it is only partly filled).  Runs
// while no other kernel uses the heap (calls on a heap are stream-ordered),
// so plain read-modify-write suffices.
// Bound by its chain of scans and by what its one CU can store.  A wavefront
// looks at 64 consecutive containers, which are one container of the next
// level, so it makes one OR per summary level, not 64; and it writes the
// claimed ids container by container, a lane per bit.
__global__ __launch_bounds__(1024) void k_bulk_claim(HeapView h, uint32_t cls, uint32_t need,
                                                     uint32_t partial)
{
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_lo, s_hi;
    if (heap_failed(h)) return;
    const uint32_t t = threadIdx.x, lane = t & 63;
    const uint32_t n0 = h.lvl_n[0];
    uint64_t *F0 = h.bm_word(BM_FREE, 0, 0);

    uint32_t cnt = 0;
    for (uint32_t c = t; c < n0; c += blockDim.x) cnt += (uint32_t)__popcll(F0[c]);
    uint32_t total;
    block_excl_scan(cnt, s_w, total);
    if (total < need) {
        if (t == 0) raise_error(h, ERR_NOMEM);
        return;
    }
    if (t == 0) {
        s_lo = 0xFFFFFFFFu;
        s_hi = 0;
    }
    __syncthreads();
    uint32_t found = 0;
    for (uint32_t base = 0; base < n0 && found < need; base += blockDim.x) {
        const uint32_t c = base + t;
        const uint64_t v = c < n0 ? F0[c] : 0ull;
        const uint32_t k = (uint32_t)__popcll(v);
        uint32_t T;
        const uint32_t p = block_excl_scan(k, s_w, T);
        uint64_t taken = 0;
        if (k && found + p < need) {
            taken = lowest_bits(v, std::min(k, need - found - p));
            F0[c] = v & ~taken;
            // the container's blocks join allocated[cls]
            aor(h.bm_word(bm_alloc(cls), 0, c), taken);
        }
        const uint64_t some = __ballot(taken != 0);
        if (some) {
            const uint32_t c0 = c - lane;              // the wavefront's first container
            if (lane == 0) {
                for (uint32_t l = 1; l < h.nlev; ++l)
                    aor(h.bm_word(bm_alloc(cls), l, c0 >> (6 * l)),
                        l == 1 ? some : 1ull << ((c0 >> (6 * (l - 1))) & 63));
                atomicMin(&s_lo, c0 + (uint32_t)(__ffsll((unsigned long long)some) - 1));
                atomicMax(&s_hi, c0 + 63u - (uint32_t)__clzll((long long)some));
            }
            for (uint64_t g = some; g; g &= g - 1) {
                const uint32_t from = (uint32_t)(__ffsll((unsigned long long)g) - 1);
                const uint64_t bits = __shfl((unsigned long long)taken, (int)from);
                const uint32_t o = found + (uint32_t)__shfl((int)p, (int)from);
                if ((bits >> lane) & 1)
                    h.claim[o + (uint32_t)__popcll(bits & ((1ull << lane) - 1))] = (c0 + from) * 64 + lane;
            }
        }
        found += T;
    }
    __syncthreads();
    uint32_t lo = s_lo, hi = s_hi;
    for (uint32_t l = 1; l < h.nlev; ++l) {
        lo >>= 6;
        hi >>= 6;
        for (uint32_t j = lo + (t >> 6); j <= hi; j += blockDim.x >> 6) {
            const uint32_t child = j * 64 + lane;
            const uint64_t v = __ballot(child < h.lvl_n[l - 1] && *h.bm_word(BM_FREE, l - 1, child) != 0);
            if (lane == 0) *h.bm_word(BM_FREE, l, j) = v;
        }
        __syncthreads();
    }
    // the partly filled last block is active (it has free slots)
    if (partial && t == 0) {
        uint32_t pos = h.claim[need - 1];
        for (uint32_t l = 0; l < h.nlev; ++l, pos >>= 6)
            aor(h.bm_word(bm_active(cls), l, pos >> 6), 1ull << (pos & 63));
    }
}

// Fills the objects of an ordered bulk claim: object i -> block claim[i/64],
// slot i%64 (64 consecutive objects share a block, so every field write of a
// wavefront is one contiguous run), and the block's header (type, allocation
// bitmap) with its first object.  The heap is quiescent during a bulk
// parallel_new, so the launch boundaries order these stores against the
// bitmaps written by k_bulk_claim.
__global__ __launch_bounds__(256) void k_bulk_init(HeapView h, uint32_t cls, FieldSet fs, uint32_t n,
                                                   uint32_t *out_handles)
{
    if (heap_failed(h)) return;
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t bid = h.claim[i >> 6];
    const uint32_t handle = (bid << 6) | (uint32_t)(i & 63);
    if ((i & 63) == 0) {
        h.type[bid] = cls;
        h.alloc_bm[bid] = n - i >= 64 ? ~0ull : (1ull << (n - i)) - 1;
    }
    init_object(h, fs, handle, i);
    if (out_handles) out_handles[i] = handle;
}

// parallel_new through the device allocator: every object is allocated by
// wavefront-aggregated device new (Alg. allocate with request coalescing)
// and then initialized, as in the thesis's parallel_new kernel.
__global__ __launch_bounds__(256) void k_new_device(HeapView h, uint32_t cls, FieldSet fs, uint32_t n,
                                                    uint32_t *out_handles)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (heap_failed(h)) return;                // uniform: one word for everyone
    const bool want = i < n;
    const uint32_t handle = wave_allocate(h, cls, want);
    if (!want) return;
    if (handle != kNull) init_object(h, fs, handle, i);
    if (out_handles) out_handles[i] = handle;
}

// Host-initiated destroy of a few objects: one wavefront that releases them as
// a method would, each handle checked first (a live object of the class; one
// named twice is released once).  By one wavefront only: between the check and
// the release of another one the block could be freed.
__global__ __launch_bounds__(64) void k_destroy_few(HeapView h, uint32_t cls, const uint32_t *handles, uint32_t n)
{
    if (heap_failed(h)) return;
    const uint32_t i = threadIdx.x, hd = i < n ? handles[i] : kNull, bid = hd >> 6;
    const bool live = hd != kNull && bid < h.M && ald32(h.type + bid) == cls &&
                      ((ald(h.alloc_bm + bid) >> (hd & 63)) & 1);
    if (i < n && !live) raise_error(h, ERR_BADHANDLE);
    wave_deallocate(h, cls, hd, live);
}

// Host-initiated destroy, first launch: frees the slots of the live objects
// that the handles name.  No block is freed and no type changes here, so the
// type check is a plain load and the slot's old bit tells whether the handle
// named a live object, once for an object named twice.
// Bound by the rate of the atomics on the blocks' bitmaps: lanes that follow
// one another in a block, as handles in the order of creation do, make one of
// them (a million 120 us with one a lane, 23 us so); in no order each lane
// makes its own (a million 62 us; 165 us with a load of the bitmap before
// each, and with the blocks' states settled by the releases).
__global__ __launch_bounds__(256) void k_destroy(HeapView h, uint32_t cls, const uint32_t *handles,
                                                 uint32_t n)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (heap_failed(h)) return;
    const uint32_t lane = lane_id(), hd = i < n ? handles[i] : kNull, bid = hd >> 6;
    const uint64_t bit = 1ull << (hd & 63);
    const bool named = hd != kNull && bid < h.M && h.type[bid] == cls;
    uint64_t pending = __ballot(named);
    uint32_t count = 0;
    bool gone = false, bad = i < n && !named;
    while (pending) {
        const uint32_t leader = (uint32_t)(__ffsll((unsigned long long)pending) - 1);
        const bool in = ((pending >> lane) & 1) && bid == (uint32_t)__builtin_amdgcn_readlane(bid, leader);
        const uint64_t group = __ballot(in);
        if (__popcll(group) < 8) break;
        const uint64_t slots = wave_or64(in ? bit : 0);
        if (lane == leader) {
            const uint32_t k = (uint32_t)__popcll(aand(h.alloc_bm + bid, ~slots) & slots);
            count += k;
            bad |= k != (uint32_t)__popcll(group);
        }
        pending &= ~group;
    }
    if ((pending >> lane) & 1) {
        gone = aand(h.alloc_bm + bid, ~bit) & bit;
        bad |= !gone;
    }
    if (bad) {
        raise_error(h, ERR_BADHANDLE);
        __hip_atomic_store(h.ctrl + CTRL_DESTROY, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    count += (uint32_t)__popcll(__ballot(gone)) * (lane == 0);
    for (int d = 1; d < 64; d <<= 1) count += (uint32_t)__shfl_xor((int)count, d);
    if (lane == 0 && count) count_events(h, EV_DELS, count);
}

// The second launch of a destroy on a heap that had failed before the call does
// nothing, as the first one did.  An error that the first launch has raised
// itself does not keep it from settling what was deleted until then; its last
// work-group then takes the mark of that back (every one has read it by then).
__device__ __forceinline__ bool destroy_begins_settling(const HeapView &h, uint32_t &err)
{
    const uint32_t own = ald32(h.ctrl + CTRL_DESTROY);
    err = ald32(h.ctrl + CTRL_ERR);
    return !err || own;
}

__device__ __forceinline__ void destroy_ends_settling(const HeapView &h, uint32_t err)
{
    if (!err) return;
    __syncthreads();
    if (threadIdx.x != 0) return;
    uint32_t *const done = h.ctrl + CTRL_DESTROY + 1;
    if (__hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != gridDim.x - 1) return;
    __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(h.ctrl + CTRL_DESTROY, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Second launch: brings the states of the class's blocks in line with their
// slots, a container's 64 blocks at a time, `per` containers a wavefront (a
// lane reads one, those without blocks of the class are passed over).  A block without objects
// becomes free (its type unset, its slots all taken, as a release
// leaves it), one with free slots active.  Nothing else runs on the heap, so
// a container is its wavefront's own; what passes on to the next levels goes
// through the switches that other wavefronts' containers meet there.
__global__ __launch_bounds__(256) void k_destroy_settle(HeapView h, uint32_t cls, uint32_t per)
{
    uint32_t err;
    if (!destroy_begins_settling(h, err)) return;
    const uint32_t lane = lane_id(), waves = gridDim.x * (blockDim.x >> 6);
    const uint32_t c0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)global_wave_id());
    // (every waves-th container: a class's blocks lie together)
    const uint64_t at = (uint64_t)lane * waves + c0;
    const uint64_t owned = lane < per && at < h.lvl_n[0] ? *h.bm_word(bm_alloc(cls), 0, (uint32_t)at) : 0ull;
    for (uint64_t g = __ballot(owned != 0); g; g &= g - 1) {
        const uint32_t j = (uint32_t)(__ffsll((unsigned long long)g) - 1), c = j * waves + c0;
        uint64_t *const alloc = h.bm_word(bm_alloc(cls), 0, c), *const active = h.bm_word(bm_active(cls), 0, c);
        const uint64_t mine = lane64(owned, j);
        const uint64_t was = uniform64(*active);
        const uint32_t bid = c * 64 + lane;
        const uint64_t slots = (mine >> lane) & 1 ? h.alloc_bm[bid] : ~0ull;
        const uint64_t empty = __ballot(slots == 0), some = __ballot(slots != 0 && slots != ~0ull);
        if (!empty && some == was) continue;
        if (slots == 0) {
            h.type[bid] = kNull;
            h.alloc_bm[bid] = ~0ull;
        }
        if (lane == 0) {
            OpQueue q;
            q.reset();
            *active = some;
            if (!was != !some && h.nlev > 1) q.op[0] = BitOp{c, (uint16_t)bm_active(cls), 1, (int8_t)(some ? 1 : -1)};
            if (empty) {
                *alloc = mine & ~empty;
                if (mine == empty && h.nlev > 1) q.op[1] = BitOp{c, (uint16_t)bm_alloc(cls), 1, -1};
                uint64_t *const free_ = h.bm_word(BM_FREE, 0, c);
                const uint64_t f = *free_;
                *free_ = f | empty;
                if (!f && h.nlev > 1) q.op[2] = BitOp{c, (uint16_t)BM_FREE, 1, 1};
            }
            run_ops_lane(h, q);
        }
    }
    destroy_ends_settling(h, err);
}

// The second launch for handles that are few beside the class's blocks: of the
// blocks that they name alone, a lane a handle (the first of those that follow
// one another in a block).  Several lanes may still name one block: the one whose exchange unsets an empty block's type
// frees it, and the one whose OR sets a block's active bit passes that on.
// Activations come before the frees of any lane, so that a wavefront's
// switches wait for none of its own that is still to come.
// Bound by its chain of atomics, 5 to 8 of them, whatever the class's size.
__global__ __launch_bounds__(256) void k_destroy_settle_named(HeapView h, uint32_t cls, const uint32_t *handles,
                                                              uint32_t n)
{
    uint32_t err;
    if (!destroy_begins_settling(h, err)) return;
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t hd = i < n ? handles[i] : kNull, bid = hd >> 6, c = bid >> 6;
    const uint64_t bit = 1ull << (bid & 63);
    const uint32_t before = (uint32_t)__shfl_up((int)bid, 1);
    const bool up = h.nlev > 1, again = lane_id() != 0 && bid == before;
    const bool named = hd != kNull && !again && bid < h.M && ald32(h.type + bid) == cls;
    const uint64_t slots = named ? ald(h.alloc_bm + bid) : ~0ull;
    bool freed = false;
    if (slots == 0) {
        uint32_t t = cls;
        freed = __hip_atomic_compare_exchange_strong(h.type + bid, &t, kNull, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
    }
    const bool some = slots != 0 && slots != ~0ull;
    uint64_t prev = some ? aor(h.bm_word(bm_active(cls), 0, c), bit) : ~0ull;
    switch_bits(h, up && prev == 0, bm_active(cls), c, +1, 1);
    if (freed) {
        __hip_atomic_store(h.alloc_bm + bid, ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        prev = aand(h.bm_word(bm_active(cls), 0, c), ~bit);
    }
    switch_bits(h, up && freed && prev == bit, bm_active(cls), c, -1, 1);
    if (freed) prev = aand(h.bm_word(bm_alloc(cls), 0, c), ~bit);
    switch_bits(h, up && freed && prev == bit, bm_alloc(cls), c, -1, 1);
    if (freed) prev = aor(h.bm_word(BM_FREE, 0, c), bit);
    switch_bits(h, up && freed && prev == 0, BM_FREE, c, +1, 1);
    destroy_ends_settling(h, err);
}

// One run of a block's 64 slots that a gather copies: a field array of 1- or
// 4-byte elements, or four consecutive inner elements of a 4-byte field whose
// dense rows take 16-byte stores.
struct GatherPlane {
    uint32_t offset;     // of the (first) array inside a block
    uint32_t stride;     // bytes to the next inner element's array (16-byte planes)
    uint32_t count;      // inner elements per object
    uint32_t q;          // the (first) inner element
    void *dst;
};

// a 16-byte plane stands for four arrays, so a class's arrays bound the planes
struct GatherSet {
    uint32_t n16, n4, n1;    // planes of 16-, 4- and 1-byte stores, in this order
    GatherPlane p[SMMO_MAX_FIELDS];
};

constexpr uint32_t kGatherThreads = 1024;
constexpr uint32_t kGatherGroups = 512;
constexpr uint32_t kGatherBlocks = 4;        // blocks whose loads a wavefront has in flight

// Copies fields of the live objects (block by block, in R order) into dense
// arrays; the last work-group publishes the count.
// Bound by the copy (each byte read and written once); what held it up before
// was its bookkeeping: one atomic per block and one per wavefront, all on one
// word, where each takes 12 ns whatever the grid: 2.29 ms for the 164,000
// blocks of 10.4M springs, 0.91 ms for 3M.  So a work-group takes one
// contiguous stretch of R, counts its live objects first (a type and a bitmap
// per block, one block per thread) and reserves its whole range, and reports
// itself done, with one 64-bit atomic; 512 work-groups of 16 wavefronts fill
// the chip with two per CU.  A wavefront then copies whole blocks, lane =
// slot, four of them at once, so that four blocks' loads are in flight
// (handle, id, count and state of 16.8M cells, 437 MB read and written:
// 125 us one block after the other, 100 us so).
__global__ __launch_bounds__(kGatherThreads) void k_gather(HeapView h, uint32_t cls, GatherSet gs,
                                                           uint32_t *out_handles, uint32_t capacity,
                                                           uint32_t *out_count)
{
    __shared__ uint64_t s_bm[kGatherThreads];
    __shared__ uint32_t s_bid[kGatherThreads], s_pos[kGatherThreads], s_w[16], s_base;
    const uint32_t t = threadIdx.x, lane = lane_id(), w = t >> 6;
    const uint32_t err = ald32(h.ctrl + CTRL_ERR);
    const BlockList L = block_list(h, cls);
    const uint32_t r = err ? 0u : L.r;          // a failed heap lists nothing
    const uint32_t lo = (uint32_t)((uint64_t)r * blockIdx.x / gridDim.x);
    const uint32_t hi = (uint32_t)((uint64_t)r * (blockIdx.x + 1) / gridDim.x);
    unsigned long long *pack = reinterpret_cast<unsigned long long *>(h.ctrl + CTRL_GATHER);
    for (uint32_t first = lo;; first += kGatherThreads) {
        const bool last = hi - first <= kGatherThreads;
        const uint32_t n = last ? hi - first : kGatherThreads;
        uint64_t bm = 0;
        if (t < n) {
            const uint32_t bid = L.at(first + t);
            const uint32_t ty = h.type[bid];
            const uint64_t b = h.alloc_bm[bid];
            bm = ty == cls ? b : 0ull;          // a listed block may have changed class
            s_bid[t] = bid;
            s_bm[t] = bm;
        }
        uint32_t total;
        const uint32_t before = block_excl_scan((uint32_t)__popcll(bm), s_w, total);
        if (t < n) s_pos[t] = before;
        if (t == 0) {
            const unsigned long long add = total | (last ? 1ull << 32 : 0ull);
            const unsigned long long old = __hip_atomic_fetch_add(pack, add, __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_AGENT);
            s_base = (uint32_t)old;
            if (last && (uint32_t)(old >> 32) == gridDim.x - 1) {   // every other group has counted
                *out_count = (uint32_t)old + total;
                __hip_atomic_store(pack, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
        const uint32_t base = s_base;
        for (uint32_t i0 = w; i0 < n; i0 += kGatherBlocks * (kGatherThreads / 64)) {
            uint64_t idx[kGatherBlocks];
            uint32_t bid[kGatherBlocks];
            bool copy[kGatherBlocks];
#pragma unroll
            for (uint32_t u = 0; u < kGatherBlocks; ++u) {
                const uint32_t i = i0 + u * (kGatherThreads / 64);
                const uint64_t live = i < n ? uniform64(s_bm[i]) : 0ull;
                bid[u] = __builtin_amdgcn_readfirstlane(s_bid[i < n ? i : i0]);
                idx[u] = (uint64_t)base + (i < n ? s_pos[i] : 0u) + (uint32_t)__popcll(live & ((1ull << lane) - 1));
                copy[u] = ((live >> lane) & 1) && idx[u] < capacity;
            }
            uint32_t j = 0;
            for (; j < gs.n16; ++j) {
                const GatherPlane &p = gs.p[j];
                const uint32_t st = p.stride / 4;
                uint4 v[kGatherBlocks];
#pragma unroll
                for (uint32_t u = 0; u < kGatherBlocks; ++u)
                    if (copy[u]) {
                        const uint32_t *a = reinterpret_cast<const uint32_t *>(h.block(bid[u]) + p.offset) + lane;
                        v[u] = make_uint4(a[0], a[st], a[2 * st], a[3 * st]);
                    }
#pragma unroll
                for (uint32_t u = 0; u < kGatherBlocks; ++u)
                    if (copy[u]) reinterpret_cast<uint4 *>(p.dst)[(idx[u] * p.count + p.q) / 4] = v[u];
            }
            for (; j < gs.n16 + gs.n4; ++j) {
                const GatherPlane &p = gs.p[j];
                uint32_t v[kGatherBlocks];
#pragma unroll
                for (uint32_t u = 0; u < kGatherBlocks; ++u)
                    if (copy[u]) v[u] = reinterpret_cast<const uint32_t *>(h.block(bid[u]) + p.offset)[lane];
#pragma unroll
                for (uint32_t u = 0; u < kGatherBlocks; ++u)
                    if (copy[u]) reinterpret_cast<uint32_t *>(p.dst)[idx[u] * p.count + p.q] = v[u];
            }
            for (; j < gs.n16 + gs.n4 + gs.n1; ++j) {
                const GatherPlane &p = gs.p[j];
                uint8_t v[kGatherBlocks];
#pragma unroll
                for (uint32_t u = 0; u < kGatherBlocks; ++u)
                    if (copy[u]) v[u] = reinterpret_cast<const uint8_t *>(h.block(bid[u]) + p.offset)[lane];
#pragma unroll
                for (uint32_t u = 0; u < kGatherBlocks; ++u)
                    if (copy[u]) reinterpret_cast<uint8_t *>(p.dst)[idx[u] * p.count + p.q] = v[u];
            }
            if (out_handles) {
#pragma unroll
                for (uint32_t u = 0; u < kGatherBlocks; ++u)
                    if (copy[u]) out_handles[idx[u]] = (bid[u] << 6) | lane;
            }
        }
        if (last) break;
        __syncthreads();                        // the lists above are rewritten
    }
}

__global__ void k_zero_words(uint32_t *p, uint32_t n)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

__device__ __forceinline__ bool bm_bit(const HeapView &h, uint32_t bmid, uint32_t pos)
{
    return (ald(h.bm_word(bmid, 0, pos >> 6)) >> (pos & 63)) & 1;
}

// Statistics and invariant check of a quiescent heap.
__global__ __launch_bounds__(256) void k_stats(HeapView h)
{
    unsigned long long *st = reinterpret_cast<unsigned long long *>(h.ctrl + CTRL_STATS);
    const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t gsz = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t b = gid; b < h.M; b += gsz) {
        const uint32_t bid = (uint32_t)b;
        const bool fr = bm_bit(h, BM_FREE, bid);
        const uint32_t t = h.type[bid];
        const uint64_t bm = h.alloc_bm[bid];
        uint32_t nalloc = 0;
        for (uint32_t c = 0; c < h.nclasses; ++c) {
            const bool a = bm_bit(h, bm_alloc(c), bid);
            const bool act = bm_bit(h, bm_active(c), bid);
            if (a) {
                nalloc++;
                if (t != c) {
                    atomicAdd(st + ST_TYPE, 1ull);
                } else {
                    atomicAdd(st + ST_LIVE + c, (unsigned long long)__popcll(bm));
                    atomicAdd(st + ST_BLOCKS + c, 1ull);
                    if (bm == 0) atomicAdd(st + ST_EMPTY, 1ull);
                    if (act != (bm != ~0ull)) atomicAdd(st + ST_ACTIVE, 1ull);
                }
            } else if (act) {
                atomicAdd(st + ST_ACTIVE, 1ull);
            }
        }
        if (fr) {
            atomicAdd(st + ST_FREE, 1ull);
            if (nalloc || t != kNull) atomicAdd(st + ST_STATE, 1ull);
        } else if (nalloc != 1) {
            atomicAdd(st + ST_STATE, 1ull);
        }
    }
    // container consistency of every summary level, and no bits past the end
    const uint64_t nbm = 1ull + 2ull * h.nclasses;
    const uint64_t words = nbm * h.bm_words;
    for (uint64_t i = gid; i < words; i += gsz) {
        const uint32_t bmid = (uint32_t)(i / h.bm_words);
        const uint32_t w = (uint32_t)(i % h.bm_words);
        uint32_t l = 0;
        while (l + 1 < h.nlev && w >= h.lvl_off[l + 1]) ++l;
        const uint32_t c = w - h.lvl_off[l];
        const uint64_t actual = h.bm[i];
        const uint64_t nchild = l == 0 ? h.M : h.lvl_n[l - 1];
        uint64_t expect_mask = ~0ull;
        const uint64_t lo = (uint64_t)c * 64;
        const uint64_t cnt = nchild > lo ? std::min<uint64_t>(64, nchild - lo) : 0;
        if (cnt < 64) expect_mask = (1ull << cnt) - 1;
        bool bad = (actual & ~expect_mask) != 0;
        if (l > 0) {
            uint64_t expect = 0;
            for (uint32_t b = 0; b < cnt; ++b)
                if (*h.bm_word(bmid, l - 1, c * 64 + b) != 0) expect |= 1ull << b;
            bad |= expect != actual;
        }
        if (bad) atomicAdd(st + ST_HIER, 1ull);
    }
}

smmo_status launch_check(const char *what)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, what);
    return SMMO_OK;
}

// The planes of a gather of fields `ids` into `ptrs`.
smmo_status build_gatherset(const smmo_heap *h, uint32_t cls, const uint32_t *ids, uint32_t n, void *const *ptrs,
                            GatherSet &gs)
{
    const smmo_class_info &ci = h->schema->c[cls];
    for (uint32_t j = 0; j < n; ++j) {
        if (ids[j] >= ci.nfields) return fail(SMMO_EINVAL, "field id out of range");
        for (uint32_t k = 0; k < j; ++k)
            if (ids[k] == ids[j]) return fail(SMMO_EINVAL, "field listed twice");
    }
    uint32_t np = 0;
    // 16-byte rows where a 4-byte field's objects start at multiples of 16
    // bytes: an inner length that is a multiple of four in an aligned array
    auto rows16 = [&](uint32_t j) {
        const smmo_field_info &fi = ci.f[ids[j]];
        return fi.size == 4 && fi.count % 4 == 0 && (reinterpret_cast<uintptr_t>(ptrs[j]) & 15) == 0;
    };
    for (uint32_t pass = 0; pass < 3; ++pass) {
        const uint32_t before = np;
        for (uint32_t j = 0; j < n; ++j) {
            const smmo_field_info &fi = ci.f[ids[j]];
            const uint32_t kind = rows16(j) ? 0 : fi.size == 4 ? 1 : 2;
            if (kind != pass) continue;
            for (uint32_t q = 0; q < fi.count; q += kind == 0 ? 4 : 1)
                gs.p[np++] = GatherPlane{fi.offset + q * fi.stride, fi.stride, fi.count, q, ptrs[j]};
        }
        (pass == 0 ? gs.n16 : pass == 1 ? gs.n4 : gs.n1) = np - before;
    }
    return SMMO_OK;
}

smmo_status read_ctrl(smmo_heap *h, uint32_t first_word, uint32_t nwords)
{
    hipError_t e = hipStreamSynchronize(h->last);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    e = hipMemcpy(reinterpret_cast<char *>(h->host_ctrl) + first_word * 4,
                  h->v.ctrl + first_word, (size_t)nwords * 4, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpy(control words)");
    return SMMO_OK;
}

smmo_status map_device_error(uint32_t err)
{
    if (!err) return SMMO_OK;
    if (err == ERR_NOMEM) return fail(SMMO_ENOMEM, "device: heap exhausted during allocation");
    std::string m = "device error:";
    if (err & ERR_NOMEM) m += " heap exhausted;";
    if (err & ERR_SPIN) m += " retry bound exceeded;";
    if (err & ERR_BADHANDLE) m += " handle not a live object of the class;";
    if (err & ERR_INTERNAL) m += " internal limit;";
    return fail(SMMO_EDEVICE, m);
}

smmo_status run_stats(smmo_heap *h, hipStream_t st)
{
    const uint32_t nw = ST_WORDS * 2;
    hipLaunchKernelGGL(k_zero_words, dim3((nw + 255) / 256), dim3(256), 0, st,
                       h->v.ctrl + CTRL_STATS, nw);
    const uint64_t work = std::max<uint64_t>(h->v.M, (1ull + 2ull * h->v.nclasses) * h->v.bm_words);
    const uint32_t grid = (uint32_t)std::min<uint64_t>((work + 255) / 256, 4096);
    hipLaunchKernelGGL(k_stats, dim3(grid), dim3(256), 0, st, h->v);
    smmo_status s = launch_check("k_stats");
    if (s) return s;
    h->last = st;
    return read_ctrl(h, 0, kCtrlWords);
}

} // namespace

// ------------------------------------------------------- internal helpers --
namespace smmo {

smmo_status heap_check_class(const smmo_heap *h, uint32_t cls) { return check_class(h, cls); }
smmo_status heap_read_ctrl(smmo_heap *h, uint32_t first_word, uint32_t nwords)
{
    return read_ctrl(h, first_word, nwords);
}
smmo_status heap_launch_check(const char *what) { return launch_check(what); }

smmo_status fail(smmo_status st, const std::string &msg)
{
    g_last_error = msg;
    return st;
}

smmo_status hip_fail(hipError_t e, const char *what)
{
    return fail(SMMO_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

uint32_t dtype_size(int32_t dtype)
{
    switch (dtype) {
    case SMMO_U8: return 1;
    case SMMO_I32:
    case SMMO_U32:
    case SMMO_F32:
    case SMMO_HANDLE: return 4;
    default: return 0;
    }
}

smmo_status bind_field(const smmo_schema *s, uint32_t cls, const char *name, int32_t dtype,
                       uint32_t count, uint32_t *offset, uint32_t *stride)
{
    if (cls >= s->nclasses) return fail(SMMO_EINVAL, "class id out of range");
    const smmo_class_info &ci = s->c[cls];
    for (uint32_t j = 0; j < ci.nfields; ++j) {
        const smmo_field_info &f = ci.f[j];
        if (strcmp(f.name, name) != 0) continue;
        if (f.dtype != dtype || (count && f.count != count))
            return fail(SMMO_EINVAL, std::string("class '") + ci.name + "': field '" + name +
                                         "' has the wrong type or length for this method");
        *offset = f.offset;
        if (stride) *stride = f.stride;
        return SMMO_OK;
    }
    return fail(SMMO_EINVAL, std::string("class '") + ci.name + "' has no field '" + name +
                                 "' required by this method");
}

namespace {
// The state of class cls's list as launches on stream st will find it.  A
// launch that is being captured does not run now, and runs again with every
// replay: an enumeration inside the capture says nothing about the list that
// launches outside find, and a list that is valid when the capture begins may
// be stale at a replay (objects created since by eager calls, by other graphs
// or by a later launch of this one), so the first walk of a class in a capture
// records an enumeration: about 5 us a class and replay.
int &list_state(smmo_heap *h, uint32_t cls, hipStream_t st)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (hipStreamGetCaptureInfo(st, &cap, &id) != hipSuccess) {
        (void)hipGetLastError();
        cap = hipStreamCaptureStatusNone;
    }
    if (cap == hipStreamCaptureStatusNone) {
        if (h->replayed[cls]) h->rstate[cls] = R_DIRTY;
        return h->rstate[cls];
    }
    if (h->capture != id) {
        h->capture = id;
        for (int &state : h->capture_rstate) state = R_DIRTY;
    }
    return h->capture_rstate[cls];
}
} // namespace

smmo_status ensure_enumerated(smmo_heap *h, uint32_t cls, bool snapshot, hipStream_t st, bool split,
                              bool allow_direct, bool in_order)
{
    // a do-all that uses a snapshot from smmo_snapshot walks that list as it is
    if ((h->v.snap >> cls) & 1) return SMMO_OK;
    int &state = list_state(h, cls, st);
    if (!snapshot && (state == R_SPLIT || (state == R_VALID && !split))) {
        h->v.direct &= ~(1u << cls);
        return SMMO_OK;
    }
    // A walk that needs neither the iteration snapshot nor the packing plan
    // reads nothing of R but its entries; on a small heap the walk over all
    // blocks costs less than the enumeration launch it replaces, for a class
    // whose list goes stale at every launch that creates its objects.  The
    // list stays stale (rstate unchanged); every such launch walks directly.
    if (allow_direct && !snapshot && !split && h->churn[cls] && h->v.M <= kDirectMaxBlocks) {
        h->v.direct |= 1u << cls;
        return SMMO_OK;
    }
    h->v.direct &= ~(1u << cls);
    h->snap_pending &= ~(1u << cls);     // the list is rebuilt: a snapshot taken before is gone
    // In block order where a work-group can count what lies before it.  For a
    // plan that costs a read of those blocks' bitmaps, and only the walks of a
    // snapshot that smmo_snapshot takes may depend on the order: any method
    // can use it, a packed one of its own visits objects in no order.
    const uint32_t n0 = h->v.lvl_n[0];
    const uint32_t ordered = n0 <= kFewContainers && (!split || in_order) ? 1u : 0u;
    const uint32_t per = n0 <= kManyContainers ? 4 : n0 <= kMostContainers ? 16 : 64;
    hipLaunchKernelGGL(per == 4 ? k_enumerate<4> : per == 16 ? k_enumerate<16> : k_enumerate<64>,
                       dim3((n0 + 16 * per - 1) / (16 * per)), dim3(1024), 0, st, h->v, cls, snapshot ? 1u : 0u,
                       split ? 1u : 0u, ordered);
    smmo_status s = launch_check("k_enumerate");
    if (s) return s;
    state = split ? R_SPLIT : R_VALID;
    return SMMO_OK;
}

bool packing_wanted(const smmo_heap *h, uint32_t cls, const LaunchShape &ls)
{
    const uint64_t waves = (uint64_t)ls.grid.x * (ls.block.x / 64);
    return h->cfg.sparse_packing == 2 || (h->cfg.sparse_packing == 1 && h->ub_blocks[cls] > waves);
}

LaunchShape method_shape(const smmo_heap *h, uint32_t cls, uint32_t def_group, uint32_t def_wg, uint32_t def_waves_per_cu)
{
    uint32_t wg = def_wg;
    uint64_t waves = h->cfg.grid_waves ? h->cfg.grid_waves : (uint64_t)def_waves_per_cu * h->cu_count;
    uint32_t group = def_group == 0 ? 1 : h->cfg.block_group ? h->cfg.block_group : def_group;
    if (h->cur_method < 64) {
        if (h->launch_wg[h->cur_method][cls]) wg = h->launch_wg[h->cur_method][cls];
        if (h->launch_waves[h->cur_method][cls]) waves = h->launch_waves[h->cur_method][cls];
        if (def_group && h->launch_group[h->cur_method][cls]) group = h->launch_group[h->cur_method][cls];
    }
    const uint64_t groups = (std::max<uint64_t>(1, h->ub_blocks[cls]) + group - 1) / group;
    waves = std::min<uint64_t>(waves, groups);
    const uint32_t wpg = wg / 64;
    LaunchShape ls;
    ls.grid = dim3((uint32_t)((waves + wpg - 1) / wpg));
    ls.block = dim3(wg);
    ls.group = group;
    return ls;
}

bool stream_captured(hipStream_t st)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) {
        (void)hipGetLastError();
        return true;           // (the null stream while another one is captured)
    }
    return cap != hipStreamCaptureStatusNone;
}

namespace {
void release_workspace(smmo_heap *h, smmo_heap::Workspace *w)
{
    if (h->owner.release) h->owner.release(w->p, w->bytes, h->owner.ctx);
    else (void)hipFree(w->p);
    delete w;
}
} // namespace

void *class_workspace(smmo_heap *h, uint32_t cls, size_t bytes, size_t most, hipStream_t st)
{
    smmo_heap::Workspace *&cur = h->work[cls];
    const bool captured = stream_captured(st);
    if (cur && cur->bytes >= bytes) {
        cur->last = st;
        cur->captured |= captured;
        return cur->p;
    }
    if (captured) return nullptr;
    // (another stream may be captured just now, which a wait, an allocation or
    // a release in the thread's default mode would break)
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    // room to grow by half, so that a growing class does not take one each time
    const size_t want = cur ? std::min(bytes + bytes / 2, std::max(bytes, most)) : bytes;
    if (cur && !cur->captured) {
        if (!stream_captured(cur->last) && hipStreamSynchronize(cur->last) == hipSuccess) {
            smmo_heap::Workspace *const older = cur->older;
            release_workspace(h, cur);
            cur = older;
        } else {
            (void)hipGetLastError();
        }
    }
    smmo_heap::Workspace *w = new (std::nothrow) smmo_heap::Workspace();
    if (w) {
        w->bytes = want;
        if (h->owner.alloc) {
            w->p = h->owner.alloc(w->bytes, h->owner.ctx);
        } else if (hipMalloc(&w->p, w->bytes) != hipSuccess) {
            (void)hipGetLastError();
            w->p = nullptr;
        }
        if (!w->p) {
            delete w;
            w = nullptr;
        }
    }
    if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (!w) return nullptr;
    w->last = st;
    w->older = cur;
    cur = w;
    return w->p;
}

uint32_t class_family(const smmo_schema *s, uint32_t cls)
{
    uint32_t fam = 0;
    for (uint32_t c = 0; c < s->nclasses; ++c)
        for (uint32_t a = c; a != SMMO_NO_PARENT; a = s->c[a].parent)
            if (a == cls) {
                fam |= 1u << c;
                break;
            }
    return fam;
}

void note_allocation(smmo_heap *h, uint32_t cls, uint64_t max_new_objects, hipStream_t st, bool in_method)
{
    if (in_method) h->churn[cls] = true;
    const uint64_t add = (max_new_objects + 63) / 64 + 1;
    h->ub_blocks[cls] = std::min<uint64_t>(h->v.M, h->ub_blocks[cls] + add);
    int &state = list_state(h, cls, st);
    state = R_DIRTY;
    // every replay of a captured launch creates the objects again, unseen by
    // the host: neither the class's list nor its block bound may be trusted
    if (&state != &h->rstate[cls]) h->replayed[cls] = true;
}

} // namespace smmo

// ===================================================================== ABI ==
extern "C" {

void smmo_config_default(smmo_config *cfg)
{
    if (!cfg) return;
    memset(cfg, 0, sizeof *cfg);
    cfg->lookup_retries = 5;
    cfg->rotation = 1;
    cfg->coalescing = 1;
    cfg->bulk_ordered = 1;
    cfg->spin_limit = 1u << 20;
    cfg->grid_waves = 0;
}

smmo_status smmo_schema_create(smmo_schema **out)
{
    if (!out) return fail(SMMO_EINVAL, "out is NULL");
    *out = new (std::nothrow) smmo_schema();
    return *out ? SMMO_OK : fail(SMMO_ENOMEM, "host allocation failed");
}

smmo_status smmo_schema_free(smmo_schema *s)
{
    delete s;
    return SMMO_OK;
}

smmo_status smmo_define_class(smmo_schema *s, const char *name, const smmo_field_desc *fields,
                              uint32_t nfields, uint32_t *class_id)
{
    if (!fields) return fail(SMMO_EINVAL, "NULL argument");
    return smmo_define_subclass(s, name, SMMO_NO_PARENT, 0, fields, nfields, class_id);
}

smmo_status smmo_define_subclass(smmo_schema *s, const char *name, uint32_t parent, uint32_t flags,
                                 const smmo_field_desc *fields, uint32_t nfields, uint32_t *class_id)
{
    if (!s || !name || !class_id || (nfields && !fields)) return fail(SMMO_EINVAL, "NULL argument");
    if (s->frozen) return fail(SMMO_ESTATE, "schema is frozen: a heap was created from it");
    if (s->nclasses >= SMMO_MAX_CLASSES) return fail(SMMO_ENOMEM, "too many classes");
    if (flags & ~SMMO_CLASS_ABSTRACT) return fail(SMMO_EINVAL, "unknown class flags");
    if (parent != SMMO_NO_PARENT && parent >= s->nclasses) return fail(SMMO_EINVAL, "parent class id out of range");
    const size_t nl = strlen(name);
    if (nl == 0 || nl > 31) return fail(SMMO_EINVAL, "class name must have 1..31 characters");
    for (uint32_t c = 0; c < s->nclasses; ++c)
        if (strcmp(s->c[c].name, name) == 0) return fail(SMMO_EINVAL, "duplicate class name");
    // the inherited fields first (same order, hence the same offsets), then the new ones
    smmo_field_desc all[SMMO_MAX_FIELDS];
    uint32_t ninh = 0;
    if (parent != SMMO_NO_PARENT) {
        const smmo_class_info &pc = s->c[parent];
        for (uint32_t j = 0; j < pc.nfields; ++j)
            all[ninh++] = smmo_field_desc{pc.f[j].name, pc.f[j].dtype, pc.f[j].count};
    }
    if (nfields > SMMO_MAX_FIELDS - ninh) return fail(SMMO_EINVAL, "bad field count");
    for (uint32_t j = 0; j < nfields; ++j) all[ninh + j] = fields[j];
    nfields += ninh;
    if (nfields == 0) return fail(SMMO_EINVAL, "bad field count");
    smmo_class_info ci{};
    memcpy(ci.name, name, nl + 1);
    ci.nfields = nfields;
    ci.parent = parent;
    ci.flags = flags;
    uint32_t cur = 0, arrays = 0;
    for (uint32_t j = 0; j < nfields; ++j) {
        const smmo_field_desc &fd = all[j];
        if (!fd.name) return fail(SMMO_EINVAL, "field name is NULL");
        const size_t fl = strlen(fd.name);
        if (fl == 0 || fl > 31) return fail(SMMO_EINVAL, "field name must have 1..31 characters");
        for (uint32_t k = 0; k < j; ++k)
            if (strcmp(ci.f[k].name, fd.name) == 0) return fail(SMMO_EINVAL, "duplicate field name");
        const uint32_t sz = dtype_size(fd.dtype);
        if (!sz) return fail(SMMO_EINVAL, std::string("field '") + fd.name + "': bad dtype");
        if (fd.count == 0) return fail(SMMO_EINVAL, std::string("field '") + fd.name + "': count 0");
        arrays += fd.count;
        if (arrays > SMMO_MAX_FIELDS) return fail(SMMO_EINVAL, "too many field arrays in class");
        smmo_field_info &fi = ci.f[j];
        memcpy(fi.name, fd.name, fl + 1);
        fi.dtype = fd.dtype;
        fi.count = fd.count;
        fi.size = sz;
        // one 64-entry array per element, aligned to its own size (<= 256 B)
        const uint32_t arr = SMMO_BLOCK_CAPACITY * sz;
        const uint32_t al = std::min<uint32_t>(256, arr);
        cur = (cur + al - 1) / al * al;
        fi.offset = cur;
        fi.stride = (arr + al - 1) / al * al;
        cur += fi.stride * fd.count;
    }
    ci.narrays = arrays;
    ci.data_bytes = (uint32_t)align256(cur);
    s->c[s->nclasses] = ci;
    *class_id = s->nclasses++;
    return SMMO_OK;
}

smmo_status smmo_class_is_a(const smmo_schema *s, uint32_t cls, uint32_t ancestor, uint32_t *out)
{
    if (!s || !out) return fail(SMMO_EINVAL, "NULL argument");
    if (cls >= s->nclasses || ancestor >= s->nclasses) return fail(SMMO_EINVAL, "class id out of range");
    *out = (smmo::class_family(s, ancestor) >> cls) & 1u;
    return SMMO_OK;
}

smmo_status smmo_field_id(const smmo_schema *s, uint32_t class_id, const char *name, uint32_t *field_id)
{
    if (!s || !name || !field_id) return fail(SMMO_EINVAL, "NULL argument");
    if (class_id >= s->nclasses) return fail(SMMO_EINVAL, "class id out of range");
    const smmo_class_info &ci = s->c[class_id];
    for (uint32_t j = 0; j < ci.nfields; ++j)
        if (strcmp(ci.f[j].name, name) == 0) {
            *field_id = j;
            return SMMO_OK;
        }
    return fail(SMMO_EINVAL, std::string("no field '") + name + "'");
}

smmo_status smmo_block_bytes(const smmo_schema *s, uint32_t *block_bytes)
{
    if (!s || !block_bytes) return fail(SMMO_EINVAL, "NULL argument");
    if (!s->nclasses) return fail(SMMO_ESTATE, "schema has no classes");
    *block_bytes = schema_block_bytes(s);
    return SMMO_OK;
}

smmo_status smmo_heap_bytes(const smmo_schema *s, uint64_t blocks, uint64_t *bytes)
{
    if (!s || !bytes) return fail(SMMO_EINVAL, "NULL argument");
    if (!s->nclasses) return fail(SMMO_ESTATE, "schema has no classes");
    if (blocks == 0 || blocks > kMaxBlocks) return fail(SMMO_EINVAL, "block count out of range");
    Layout L;
    layout_for(s->nclasses, blocks, schema_block_bytes(s), L);
    *bytes = L.total;
    return SMMO_OK;
}

namespace {
std::mutex allocator_mu;
smmo_allocator allocator_set{};   // alloc == nullptr: none

smmo_status create_heap(smmo_schema *s, void *dev_buf, size_t bytes, const smmo_config *cfg, smmo_stream stream,
                        smmo_heap **out);
} // namespace

smmo_status smmo_set_allocator(const smmo_allocator *a)
{
    if (a && (!a->alloc || !a->release)) return fail(SMMO_EINVAL, "allocator: alloc and release must be set");
    std::lock_guard<std::mutex> lock(allocator_mu);
    allocator_set = a ? *a : smmo_allocator{};
    return SMMO_OK;
}

smmo_status smmo_alloc_heap(smmo_schema *s, void *dev_buf, size_t bytes, const smmo_config *cfg,
                            smmo_stream stream, smmo_heap **out)
{
    if (!s || !out) return fail(SMMO_EINVAL, "NULL argument");
    if (dev_buf) return create_heap(s, dev_buf, bytes, cfg, stream, out);
    smmo_allocator a;
    {
        std::lock_guard<std::mutex> lock(allocator_mu);
        a = allocator_set;
    }
    if (!a.alloc) return fail(SMMO_EINVAL, "dev_buf is NULL and no allocator is set (smmo_set_allocator)");
    void *p = a.alloc(bytes, a.ctx);
    if (!p) return fail(SMMO_ENOMEM, "the allocator returned NULL");
    const smmo_status st = create_heap(s, p, bytes, cfg, stream, out);
    if (st) {
        a.release(p, bytes, a.ctx);
        return st;
    }
    (*out)->owner = a;
    return SMMO_OK;
}

namespace {
smmo_status create_heap(smmo_schema *s, void *dev_buf, size_t bytes, const smmo_config *cfg, smmo_stream stream,
                        smmo_heap **out)
{
    if (!s->nclasses) return fail(SMMO_ESTATE, "schema has no classes");
    if (reinterpret_cast<uintptr_t>(dev_buf) & 255) return fail(SMMO_EINVAL, "dev_buf must be 256-byte aligned");
    smmo_config c;
    if (cfg) c = *cfg;
    else smmo_config_default(&c);
    if (c.lookup_retries == 0) c.lookup_retries = 1;
    if (c.spin_limit < 1024) c.spin_limit = 1024;
    if (c.block_group != 0 && c.block_group != 1 && c.block_group != 2 && c.block_group != 4)
        return fail(SMMO_EINVAL, "block_group must be 0, 1, 2 or 4");
    if (c.sparse_packing > 2) return fail(SMMO_EINVAL, "sparse_packing must be 0, 1 or 2");
    if (c.streaming_loads > 2) return fail(SMMO_EINVAL, "streaming_loads must be 0, 1 or 2");
    const uint32_t bb = schema_block_bytes(s);
    // largest M whose layout fits
    uint64_t lo = 0, hi = std::min<uint64_t>(bytes / bb, kMaxBlocks);
    Layout L;
    while (lo < hi) {
        const uint64_t mid = (lo + hi + 1) / 2;
        layout_for(s->nclasses, mid, bb, L);
        if (L.total <= bytes) lo = mid;
        else hi = mid - 1;
    }
    if (lo == 0) return fail(SMMO_ENOMEM, "buffer too small for one block");
    const uint64_t M = lo;
    layout_for(s->nclasses, M, bb, L);

    smmo_heap *h = new (std::nothrow) smmo_heap();
    if (!h) return fail(SMMO_ENOMEM, "host allocation failed");
    hipError_t e = hipGetDevice(&h->device);
    if (e != hipSuccess) {
        delete h;
        return hip_fail(e, "hipGetDevice");
    }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, h->device) == hipSuccess && cus > 0)
        h->cu_count = (uint32_t)cus;
    e = hipHostMalloc(reinterpret_cast<void **>(&h->host_ctrl), kCtrlWords * 4, hipHostMallocDefault);
    if (e != hipSuccess) {
        delete h;
        return hip_fail(e, "hipHostMalloc");
    }
    char *b = static_cast<char *>(dev_buf);
    HeapView &v = h->v;
    v.ctrl = reinterpret_cast<uint32_t *>(b + L.ctrl);
    v.bm = reinterpret_cast<uint64_t *>(b + L.bm);
    v.type = reinterpret_cast<uint32_t *>(b + L.type);
    v.alloc_bm = reinterpret_cast<uint64_t *>(b + L.alloc);
    v.iter_bm = reinterpret_cast<uint64_t *>(b + L.iter);
    v.R = reinterpret_cast<uint32_t *>(b + L.R);
    v.claim = reinterpret_cast<uint32_t *>(b + L.claim);
    v.blocks = b + L.blocks;
    v.block_bytes = bb;
    v.M = (uint32_t)M;
    v.nclasses = s->nclasses;
    v.nlev = L.nlev;
    v.bm_words = L.bm_words;
    for (uint32_t l = 0; l < kMaxLevels; ++l) {
        v.lvl_off[l] = L.lvl_off[l];
        v.lvl_n[l] = L.lvl_n[l];
    }
    v.retries = c.lookup_retries;
    v.rotation = c.rotation ? 1u : 0u;
    v.coalescing = c.coalescing ? 1u : 0u;
    v.spin_limit = c.spin_limit;
    v.sparse_packing = c.sparse_packing;
    h->schema = s;
    h->base = dev_buf;
    h->bytes = bytes;
    h->cfg = c;
    h->last = static_cast<hipStream_t>(stream);
    const uint64_t work = std::max<uint64_t>(std::max<uint64_t>(M, (1ull + 2ull * s->nclasses) * L.bm_words),
                                             kCtrlWords);
    const uint32_t grid = (uint32_t)std::min<uint64_t>((work + 255) / 256, 16384);
    hipLaunchKernelGGL(k_heap_init, dim3(grid), dim3(256), 0, h->last, v);
    smmo_status st = launch_check("k_heap_init");
    if (st) {
        (void)hipHostFree(h->host_ctrl);
        delete h;
        return st;
    }
    s->frozen = true;
    *out = h;
    return SMMO_OK;
}
} // namespace

smmo_status smmo_heap_free(smmo_heap *h)
{
    if (!h) return SMMO_OK;
    if (h->base) (void)hipStreamSynchronize(h->last);
    for (smmo_heap::Workspace *&w : h->work)
        while (w) {
            smmo_heap::Workspace *const older = w->older;
            release_workspace(h, w);
            w = older;
        }
    if (h->host_ctrl) (void)hipHostFree(h->host_ctrl);
    if (h->base && h->owner.release) h->owner.release(h->base, h->bytes, h->owner.ctx);
    h->base = nullptr;
    delete h;
    return SMMO_OK;
}

smmo_status smmo_parallel_new(smmo_heap *h, uint32_t class_id, uint32_t n, const smmo_field_init *init,
                              uint32_t ninit, uint32_t *out_handles, smmo_stream stream)
{
    smmo_status s = check_class(h, class_id);
    if (s) return s;
    if (class_abstract(h->schema, class_id)) return fail(SMMO_EINVAL, "class is abstract");
    if (ninit && !init) return fail(SMMO_EINVAL, "init is NULL");
    if (n == 0) return SMMO_OK;
    if ((uint64_t)n > 64ull * h->v.M) return fail(SMMO_ENOMEM, "more objects than the heap has slots");
    const smmo_class_info &ci = h->schema->c[class_id];
    if (ninit > ci.nfields) return fail(SMMO_EINVAL, "more initializers than fields");
    FieldSet fs{};
    fs.nf = ci.nfields;
    for (uint32_t j = 0; j < ci.nfields; ++j) {
        const smmo_field_info &fi = ci.f[j];
        fs.f[j] = FieldCopy{fi.offset, fi.stride, fi.size, fi.count, nullptr};
    }
    for (uint32_t k = 0; k < ninit; ++k) {
        if (init[k].field_id >= ci.nfields) return fail(SMMO_EINVAL, "initializer field id out of range");
        if (!init[k].values) return fail(SMMO_EINVAL, "initializer values is NULL");
        if (fs.f[init[k].field_id].src) return fail(SMMO_EINVAL, "field initialized twice");
        fs.f[init[k].field_id].src = init[k].values;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t grid = (uint32_t)(((uint64_t)n + 255) / 256);
    if (h->cfg.bulk_ordered) {
        const uint32_t need = (uint32_t)(((uint64_t)n + 63) / 64);
        hipLaunchKernelGGL(k_bulk_claim, dim3(1), dim3(1024), 0, st, h->v, class_id, need, n % 64);
        if ((s = launch_check("k_bulk_claim"))) return s;
        hipLaunchKernelGGL(k_bulk_init, dim3(grid), dim3(256), 0, st, h->v, class_id, fs, n, out_handles);
        if ((s = launch_check("k_bulk_init"))) return s;
    } else {
        hipLaunchKernelGGL(k_new_device, dim3(grid), dim3(256), 0, st, h->v, class_id, fs, n, out_handles);
        if ((s = launch_check("k_new_device"))) return s;
    }
    note_allocation(h, class_id, n, st, false);
    h->last = st;
    return SMMO_OK;
}

smmo_status smmo_parallel_do(smmo_heap *h, uint32_t class_id, uint32_t method_id, const void *args,
                             size_t args_bytes, smmo_stream stream)
{
    smmo_status s = check_class(h, class_id);
    if (s) return s;
    uint32_t nm = 0;
    const MethodEntry *tab = method_table(&nm);
    if (method_id >= nm) return fail(SMMO_EINVAL, "unknown method id");
    const MethodEntry &m = tab[method_id];
    if (args_bytes != m.args_bytes || (m.args_bytes && !args))
        return fail(SMMO_EINVAL, std::string("method '") + m.name + "': wrong argument size");
    hipStream_t st = static_cast<hipStream_t>(stream);
    // the class and its descendants: one launch per concrete class, or one
    // for the whole family where the method covers it
    const uint32_t fam = (m.flags & kFamilyLaunch) ? 1u << class_id : class_family(h->schema, class_id);
    // snapshots that smmo_snapshot took of the walked classes are used here,
    // once
    const uint32_t snap = h->snap_pending & class_family(h->schema, class_id);
    h->v.snap = snap;
    for (uint32_t c = 0; c < h->schema->nclasses && !s; ++c) {
        if ((m.flags & kFamilyLaunch) && c == class_id) {
            h->cur_method = method_id;
            s = m.launch(h, c, args, st);
            h->cur_method = 0xFFFFFFFFu;
            continue;
        }
        if (!((fam >> c) & 1) || class_abstract(h->schema, c)) continue;
        h->cur_method = method_id;
        s = m.launch(h, c, args, st);
        h->cur_method = 0xFFFFFFFFu;
    }
    h->v.snap = 0;
    h->snap_pending &= ~snap;
    if (s) return s;
    h->last = st;
    return SMMO_OK;
}

smmo_status smmo_snapshot(smmo_heap *h, uint32_t class_id, smmo_stream stream)
{
    smmo_status s = check_class(h, class_id);
    if (s) return s;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t fam = class_family(h->schema, class_id);
    for (uint32_t c = 0; c < h->schema->nclasses; ++c) {
        if (!((fam >> c) & 1) || class_abstract(h->schema, c)) continue;
        // with the packing plan whenever a packed do-all may ask for it
        if ((s = ensure_enumerated(h, c, true, st, h->cfg.sparse_packing != 0, false, true))) return s;
    }
    h->snap_pending |= fam;
    h->last = st;
    return SMMO_OK;
}

smmo_status smmo_set_launch(smmo_heap *h, uint32_t method_id, uint32_t class_id, uint32_t wg_threads,
                            uint32_t grid_waves, uint32_t group)
{
    smmo_status s = check_class(h, class_id);
    if (s) return s;
    uint32_t nm = 0;
    method_table(&nm);
    if (method_id >= nm || method_id >= 64) return fail(SMMO_EINVAL, "unknown method id");
    if (wg_threads != 0 && wg_threads != 64 && wg_threads != 128 && wg_threads != 256 && wg_threads != 512 &&
        wg_threads != 1024)
        return fail(SMMO_EINVAL, "work-group size must be 0 or one of 64, 128, 256, 512, 1024");
    if (group != 0 && group != 1 && group != 2 && group != 4)
        return fail(SMMO_EINVAL, "group must be 0, 1, 2 or 4");
    h->launch_wg[method_id][class_id] = (uint16_t)wg_threads;
    h->launch_group[method_id][class_id] = (uint8_t)group;
    h->launch_waves[method_id][class_id] = grid_waves;
    return SMMO_OK;
}

namespace {
// The routes of a destroy (us; handles of consecutive objects, of random ones).
// Up to 16 handles one launch is the faster: 7.6, 9.1 in a class of 1,600
// blocks against 9.4, 9.8 with the settling launch; 24 handles 7.9, 10.1
// against 9.5, 9.9.  The settling launch of the whole class reads 8 bytes a
// block, which begins to show at half a million of them; that of the named
// blocks costs by the handle.  160,000 blocks, 256 handles: 10.5, 12.1 and 11.2,
// 12.3; 800,000 blocks, 16,384: 13.5, 23.6 and 13.6, 16.5, and 65,536: 13.5,
// 31.1 and 17.1, 21.6; 16M blocks, 1,024: 51.4, 48.8 and 12.4, 13.6, and 262,144:
// 54.5, 101 and 24.1, 51.3.
constexpr uint32_t kDestroyFew = 16;
constexpr uint64_t kDestroyManyBlocks = 1u << 19, kDestroyBlocksPerHandle = 32;
static_assert(kDestroyFew <= 64, "k_destroy_few is one wavefront");
} // namespace

smmo_status smmo_destroy(smmo_heap *h, uint32_t class_id, const uint32_t *handles, uint32_t n,
                         smmo_stream stream)
{
    smmo_status s = check_class(h, class_id);
    if (s) return s;
    if (n == 0) return SMMO_OK;
    if (!handles) return fail(SMMO_EINVAL, "handles is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    h->snap_pending &= ~(1u << class_id);   // a snapshot would still list the deleted objects
    if (n <= kDestroyFew) {
        hipLaunchKernelGGL(k_destroy_few, dim3(1), dim3(64), 0, st, h->v, class_id, handles, n);
        if ((s = launch_check("k_destroy_few"))) return s;
        h->last = st;
        return SMMO_OK;
    }
    const uint32_t grid = (uint32_t)(((uint64_t)n + 255) / 256);
    hipLaunchKernelGGL(k_destroy, dim3(grid), dim3(256), 0, st, h->v, class_id, handles, n);
    if ((s = launch_check("k_destroy"))) return s;
    if (h->ub_blocks[class_id] >= kDestroyManyBlocks && n <= h->ub_blocks[class_id] / kDestroyBlocksPerHandle) {
        hipLaunchKernelGGL(k_destroy_settle_named, dim3(grid), dim3(256), 0, st, h->v, class_id, handles, n);
    } else {
        // a container a wavefront as long as 8,192 wavefronts do
        const uint32_t per = (h->v.lvl_n[0] + 8191) / 8192;
        static_assert((kMaxBlocks / 64 + 1 + 8191) / 8192 <= 64, "a wavefront's containers must fit its lanes");
        hipLaunchKernelGGL(k_destroy_settle, dim3((h->v.lvl_n[0] + 4 * per - 1) / (4 * per)), dim3(256), 0, st, h->v,
                           class_id, per);
    }
    if ((s = launch_check("k_destroy_settle"))) return s;
    h->last = st;
    return SMMO_OK;
}

smmo_status smmo_gather_soa(smmo_heap *h, uint32_t class_id, const uint32_t *field_ids, uint32_t nfields,
                            void *const *out_ptrs, uint32_t *out_handles, uint32_t capacity,
                            uint32_t *out_count, smmo_stream stream)
{
    smmo_status s = check_class(h, class_id);
    if (s) return s;
    if (!out_count) return fail(SMMO_EINVAL, "out_count is NULL");
    if (nfields && (!field_ids || !out_ptrs)) return fail(SMMO_EINVAL, "NULL field list");
    if (nfields > SMMO_MAX_FIELDS) return fail(SMMO_EINVAL, "too many fields");
    for (uint32_t j = 0; j < nfields; ++j)
        if (!out_ptrs[j] && capacity) return fail(SMMO_EINVAL, "output pointer is NULL");
    GatherSet gs{};
    if ((s = build_gatherset(h, class_id, field_ids, nfields, out_ptrs, gs))) return s;
    hipStream_t st = static_cast<hipStream_t>(stream);
    h->snap_pending &= ~(1u << class_id);
    if ((s = ensure_enumerated(h, class_id, false, st))) return s;
    // a wavefront per block until the work-groups fill the chip; fewer where
    // the heap's configuration bounds the wavefronts of a launch
    constexpr uint32_t wpg = kGatherThreads / 64;
    uint64_t groups = std::min<uint64_t>((std::max<uint64_t>(1, h->ub_blocks[class_id]) + wpg - 1) / wpg,
                                         kGatherGroups);
    if (h->cfg.grid_waves) groups = std::min<uint64_t>(groups, (h->cfg.grid_waves + wpg - 1) / wpg);
    hipLaunchKernelGGL(k_gather, dim3((uint32_t)groups), dim3(kGatherThreads), 0, st, h->v, class_id, gs,
                       out_handles, capacity, out_count);
    if ((s = launch_check("k_gather"))) return s;
    h->last = st;
    return SMMO_OK;
}

smmo_status smmo_sync(smmo_heap *h)
{
    if (!heap_ok(h)) return fail(SMMO_EINVAL, "heap is NULL or freed");
    smmo_status s = read_ctrl(h, CTRL_ERR, 1);
    if (s) return s;
    return map_device_error(reinterpret_cast<uint32_t *>(h->host_ctrl)[CTRL_ERR]);
}

smmo_status smmo_heap_stats(smmo_heap *h, smmo_stats *out)
{
    if (!heap_ok(h) || !out) return fail(SMMO_EINVAL, "NULL argument");
    smmo_status s = run_stats(h, h->last);
    if (s) return s;
    const uint32_t *w = reinterpret_cast<const uint32_t *>(h->host_ctrl);
    const uint64_t *st = reinterpret_cast<const uint64_t *>(w + CTRL_STATS);
    memset(out, 0, sizeof *out);
    uint64_t slots = 0, used = 0;
    for (uint32_t c = 0; c < h->v.nclasses; ++c) {
        out->live_objects[c] = st[ST_LIVE + c];
        out->blocks[c] = st[ST_BLOCKS + c];
        slots += 64 * st[ST_BLOCKS + c];
        used += st[ST_LIVE + c];
    }
    out->free_blocks = st[ST_FREE];
    out->total_blocks = h->v.M;
    out->fragmentation = slots ? (double)(slots - used) / (double)slots : 0.0;
    out->block_bytes = (uint32_t)h->v.block_bytes;
    for (uint32_t k = 0; k < kEventStripes; ++k) {
        const uint32_t *e = w + CTRL_EVENTS + k * kStripeWords;
        out->slow_paths += *reinterpret_cast<const uint64_t *>(e + EV_SLOW);
        out->alloc_retries += *reinterpret_cast<const uint64_t *>(e + EV_RETRY);
        out->device_news += *reinterpret_cast<const uint64_t *>(e + EV_NEWS);
        out->device_deletes += *reinterpret_cast<const uint64_t *>(e + EV_DELS);
        out->bitmap_spins += *reinterpret_cast<const uint64_t *>(e + EV_SPIN);
        out->lookups += *reinterpret_cast<const uint64_t *>(e + EV_FIND);
    }
    const uint32_t err = w[CTRL_ERR];
    out->device_error = err == 0 ? SMMO_OK : (err == ERR_NOMEM ? SMMO_ENOMEM : SMMO_EDEVICE);
    return SMMO_OK;
}

smmo_status smmo_check_invariants(smmo_heap *h, smmo_invariants *inv)
{
    if (!heap_ok(h) || !inv) return fail(SMMO_EINVAL, "NULL argument");
    smmo_status s = run_stats(h, h->last);
    if (s) return s;
    const uint64_t *st = reinterpret_cast<const uint64_t *>(
        reinterpret_cast<const uint32_t *>(h->host_ctrl) + CTRL_STATS);
    inv->hierarchy_violations = st[ST_HIER];
    inv->state_violations = st[ST_STATE];
    inv->active_violations = st[ST_ACTIVE];
    inv->type_violations = st[ST_TYPE];
    inv->empty_allocated = st[ST_EMPTY];
    return SMMO_OK;
}

smmo_status smmo_clear_error(smmo_heap *h, smmo_stream stream)
{
    if (!heap_ok(h)) return fail(SMMO_EINVAL, "heap is NULL or freed");
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, st, h->v.ctrl + CTRL_ERR, 1u);
    smmo_status s = launch_check("k_zero_words");
    if (s) return s;
    h->last = st;
    return SMMO_OK;
}

smmo_status smmo_heap_info(const smmo_heap *h, uint64_t *blocks, uint32_t *block_bytes)
{
    if (!heap_ok(h)) return fail(SMMO_EINVAL, "heap is NULL or freed");
    if (blocks) *blocks = h->v.M;
    if (block_bytes) *block_bytes = (uint32_t)h->v.block_bytes;
    return SMMO_OK;
}

smmo_status smmo_method_id(const char *name, uint32_t *method_id)
{
    if (!name || !method_id) return fail(SMMO_EINVAL, "NULL argument");
    uint32_t n = 0;
    const MethodEntry *t = method_table(&n);
    for (uint32_t i = 0; i < n; ++i)
        if (strcmp(t[i].name, name) == 0) {
            *method_id = i;
            return SMMO_OK;
        }
    return fail(SMMO_EINVAL, std::string("unknown method '") + name + "'");
}

smmo_status smmo_last_error(char *buf, size_t n)
{
    if (!buf || n == 0) return SMMO_EINVAL;
    const size_t k = std::min(n - 1, g_last_error.size());
    memcpy(buf, g_last_error.data(), k);
    buf[k] = 0;
    return SMMO_OK;
}

#ifndef SMMO_SOURCE_HASH
#error "SMMO_SOURCE_HASH is set by the build (paper_1908_05845_amd/build.py)"
#endif
const char *smmo_source_hash(void) { return SMMO_SOURCE_HASH; }

} // extern "C"
