// n-body (Ch.7 "nbody"): the all-pairs force (a device_do over the class) and
// the update; field contracts in include/smmo_methods.h.
//
// Two force kernels.  A small class (or one too large for the pair form's
// partial sums) takes k_nbody_force, one work-group per block of bodies.  The
// others take k_nbody_pairs, which evaluates every unordered pair once and
// gives it to both bodies, and k_nbody_sum, which adds up each body's partial
// sums in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "../../include/smmo_methods.h"
#include "method_common.hpp"

using namespace smmo;

namespace {

struct NbodyK {
    uint32_t cls;
    uint32_t o_x, o_y, o_vx, o_vy, o_fx, o_fy, o_m;
    float G, eps2, dt;
};

// Body::compute_force with device_do over all bodies (Ch.7 "nbody").  A
// work-group owns one block of 64 bodies i (one per lane in every wave);
// its four wavefronts split the other bodies j block-wise (wave w takes
// every fourth block of R), stage each j-block in LDS and read it back as
// broadcasts.  Each wave sums one j-block (64 terms) into a fresh float32
// partial and adds the partial to its running sum with Kahan compensation;
// the four running sums are combined in wave order.  The thesis leaves this
// shared-memory tiling as future work (its "Further Optimizations").
template <bool kGuard>
__device__ __forceinline__ void nbody_force_walk(const HeapView &h, const NbodyK &p, const BlockList &L,
                                                 float4 (*tile)[64], float2 (*red)[64])
{
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (uint32_t ib = xcd_logical_wg(); ib < L.r; ib += gridDim.x) {
        const uint32_t bid = L.at(ib);
        if (ald32(h.type + bid) != p.cls) continue;     // same for the whole work-group
        const uint64_t bmi = ald(h.alloc_bm + bid);
        const float xi = farr<float>(h, bid, p.o_x)[lane];
        const float yi = farr<float>(h, bid, p.o_y)[lane];
        float ax = 0.f, ay = 0.f, cx = 0.f, cy = 0.f;
        for (uint32_t j0 = 0; j0 < L.r; j0 += 4) {
            const uint32_t jt = j0 + w;
            if (jt >= L.r) break;                        // wave-uniform
            const uint32_t jb = __builtin_amdgcn_readfirstlane(L.at(jt));
            if (__builtin_amdgcn_readfirstlane(ald32(h.type + jb)) != p.cls) continue;
            const uint64_t bmj = uniform64(ald(h.alloc_bm + jb));
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if ((bmj >> lane) & 1)
                v = make_float4(farr<float>(h, jb, p.o_x)[lane], farr<float>(h, jb, p.o_y)[lane],
                                farr<float>(h, jb, p.o_m)[lane], 0.f);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            tile[w][lane] = v;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            float tx = 0.f, ty = 0.f;
#pragma unroll 8
            for (int j = 0; j < 64; ++j) {
                const float4 q = tile[w][j];
                const float dx = q.x - xi, dy = q.y - yi;
                const float r2 = fmaf(dx, dx, fmaf(dy, dy, p.eps2));
                float inv = __frsqrt_rn(r2);
                if (kGuard) inv = r2 > 0.f ? inv : 0.f;
                const float sc = q.z * inv * (inv * inv);
                tx = fmaf(dx, sc, tx);
                ty = fmaf(dy, sc, ty);
            }
            float yx = tx - cx, t = ax + yx;
            cx = (t - ax) - yx;
            ax = t;
            float yy = ty - cy;
            t = ay + yy;
            cy = (t - ay) - yy;
            ay = t;
        }
        red[w][lane] = make_float2(ax, ay);
        __syncthreads();
        if (w == 0 && ((bmi >> lane) & 1)) {
            float sx = 0.f, sy = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                sx += red[k][lane].x;
                sy += red[k][lane].y;
            }
            const float gm = p.G * farr<float>(h, bid, p.o_m)[lane];
            farr<float>(h, bid, p.o_fx)[lane] = gm * sx;
            farr<float>(h, bid, p.o_fy)[lane] = gm * sy;
        }
        __syncthreads();
    }
}

template <bool kGuard>
__global__ __launch_bounds__(256) void k_nbody_force(HeapView h, NbodyK p)
{
    __shared__ float4 tile[4][64];
    __shared__ float2 red[4][64];
    if (heap_failed(h)) return;
    nbody_force_walk<kGuard>(h, p, block_list(h, p.cls), tile, red);
}

// ---- each pair once --------------------------------------------------------
// The bodies are the class's slots in list order (64 per listed block, empty
// slots as bodies without mass).  A work-group owns I = 32 W consecutive
// slots, 32 per wavefront, and one segment of J slots not before them: its
// wavefronts meet the segment's bodies 32 at a time, j = lane mod 32, their
// own 32 bodies in the 16 rows that a lane's registers hold of a 32 x 32
// matrix-core tile.  The tile of the coordinate differences is a product of
// rank two, (-x_i, 1) (1, x_j)^T, which the matrix cores form exactly as a
// float32 subtraction does and beside the vector units; per pair these are
// left with 11 full-rate instructions and a reciprocal root for two bodies,
// against 9 and one for each body in k_nbody_force.  Bound by their issue
// (91 % of the cycles).  65,536 bodies: 1437 us a pass with k_nbody_force, 874 with this
// kernel and k_nbody_sum; 3,000 bodies: 29.8 and 10.5 us (the class's 47
// blocks are 47 work-groups there, 300 here).  Handing the sums over i to the
// matrix cores too (4 x 4 x 1 products with the masses) was slower, 1196 us:
// those issue for as long as they run.
//
// The sums over j of a wavefront's own bodies stay in registers, one addend
// per 32 bodies and lane, and are combined over the lanes at the end of the
// segment (at most 64 addends each); the sums over i of the segment's bodies
// (16 addends a lane) meet in LDS, where a chunk of 128 bodies at a time is
// added up over the wavefronts and stored.  The two kinds of partial sums of
// a body take one slot each of `part` (rows of `stride` bodies): for the
// bodies of group g, slot a < g holds what group a sent them, and slot
// g + k what they took from their k-th segment.  Pairs inside a group are
// evaluated in both orders.  Nothing is summed by atomics: the result does
// not depend on the schedule.
//
// A captured launch finds, at a replay, the list of a class that may have grown
// since.  As long as the list fits the rows of `part` (whole groups, so up to
// W / 2 - 1 blocks more than the host's bound), the launch's segments and the
// work-groups of k_nbody_sum cover it; beyond, the captured k_nbody_sum walks
// all pairs as k_nbody_force does (kCaptured; the kernels of launches that are
// not captured do without the walk and its registers).
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr uint32_t kPairChunk = 128;

struct PairPlan {
    float2 *part;
    uint32_t stride;     // bodies per slot row: the class's slots, rounded up to whole groups
    uint32_t J;          // slots per segment, a multiple of kPairChunk
};

// the body in list slot s (empty past the list's end and in free slots)
__device__ __forceinline__ float3 pair_body(const HeapView &h, const NbodyK &p, const BlockList &L, uint32_t s)
{
    float3 b = make_float3(0.f, 0.f, 0.f);
    if ((s >> 6) >= L.r) return b;
    const uint32_t bid = L.at(s >> 6), l = s & 63;
    const uint32_t t = h.type[bid];
    const uint64_t bm = h.alloc_bm[bid];
    const float3 v = make_float3(farr<float>(h, bid, p.o_x)[l], farr<float>(h, bid, p.o_y)[l],
                                 farr<float>(h, bid, p.o_m)[l]);
    return t == p.cls && ((bm >> l) & 1) ? v : b;
}

template <int W, bool kGuard, bool kCaptured>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_nbody_pairs(HeapView h,
                                                                                                  NbodyK p,
                                                                                                  PairPlan pl)
{
    constexpr uint32_t I = 32 * W;
    __shared__ float s_x[2][kPairChunk], s_y[2][kPairChunk], s_m[2][kPairChunk];
    __shared__ float2 s_a[2][W][kPairChunk];
    const uint32_t err = ald32(h.ctrl + CTRL_ERR);
    const BlockList L = block_list(h, p.cls);
    const uint32_t n = 64 * L.r;
    // segment s meets the groups 0 .. (s + 1) J / I - 1: the launch numbers
    // the pairs segment by segment, so that the XCDs (work-group number mod 8)
    // share them evenly
    const uint32_t per = pl.J / I, q = blockIdx.x / per;
    uint32_t seg = (uint32_t)((sqrtf(8.f * (float)q + 1.f) - 1.f) * 0.5f);
    while (seg * (seg + 1) / 2 > q) --seg;
    while ((seg + 1) * (seg + 2) / 2 <= q) ++seg;
    const uint32_t a = blockIdx.x - per * (seg * (seg + 1) / 2), i0 = a * I;
    if (n > pl.stride) {                                // only a replay finds more than the host's bound
        if (!kCaptured && threadIdx.x == 0) raise_error(h, ERR_INTERNAL);
        return;
    }
    if (err || i0 >= n || seg * pl.J >= n) return;
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6, col = lane & 31, hi = lane >> 5;
    const uint32_t ib = i0 + 32 * w;
    // this wavefront's bodies: the matrix operands, and the masses by row
    const float3 own = pair_body(h, p, L, ib + col);
    const float ax = hi ? 1.f : -own.x, ay = hi ? 1.f : -own.y;
    float mi[16], sx[16], sy[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        mi[r] = __shfl(own.z, 8 * (r / 4) + 4 * (int)hi + r % 4);
        sx[r] = sy[r] = 0.f;
    }
    uint32_t c = std::max(seg * pl.J, i0);              // a multiple of the chunk
    const uint32_t end = std::min((seg + 1) * pl.J, n);
    if (threadIdx.x < kPairChunk) {
        const float3 b = pair_body(h, p, L, c + threadIdx.x);
        s_x[0][threadIdx.x] = b.x;
        s_y[0][threadIdx.x] = b.y;
        s_m[0][threadIdx.x] = b.z;
    }
    __syncthreads();
    uint32_t buf = 0;
    // one chunk; Both: its bodies are not the group's own and take their share
    // (a choice per chunk, so that the pair loop holds no branch)
    auto chunk = [&](auto both) {
        constexpr bool Both = decltype(both)::value;
        // the next chunk's bodies travel while this one is worked on
        float3 next;
        const bool more = c + kPairChunk < end;
        if (more && threadIdx.x < kPairChunk) next = pair_body(h, p, L, c + kPairChunk + threadIdx.x);
#pragma unroll 1
        for (uint32_t t = 0; t < kPairChunk; t += 32) {
            const float xj = s_x[buf][t + col], yj = s_y[buf][t + col], mj = s_m[buf][t + col];
            const f32x16 dx = __builtin_amdgcn_mfma_f32_32x32x2f32(ax, hi ? xj : 1.f, f32x16{}, 0, 0, 0);
            const f32x16 dy = __builtin_amdgcn_mfma_f32_32x32x2f32(ay, hi ? yj : 1.f, f32x16{}, 0, 0, 0);
            float jx = 0.f, jy = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float r2 = fmaf(dx[r], dx[r], fmaf(dy[r], dy[r], p.eps2));
                float inv = __frsqrt_rn(r2);
                if (kGuard) inv = r2 > 0.f ? inv : 0.f;
                // difference over distance before the inverse square: no
                // factor leaves float32's range where r2 and the term do not
                const float inv2 = inv * inv;
                const float wx = inv2 * (inv * dx[r]), wy = inv2 * (inv * dy[r]);
                sx[r] = fmaf(mj, wx, sx[r]);
                sy[r] = fmaf(mj, wy, sy[r]);
                if constexpr (Both) {
                    jx = fmaf(-mi[r], wx, jx);
                    jy = fmaf(-mi[r], wy, jy);
                }
            }
            if constexpr (Both) {
                jx += __shfl_xor(jx, 32);
                jy += __shfl_xor(jy, 32);
                if (!hi) s_a[buf][w][t + col] = make_float2(jx, jy);
            }
        }
        if (more && threadIdx.x < kPairChunk) {
            s_x[buf ^ 1][threadIdx.x] = next.x;
            s_y[buf ^ 1][threadIdx.x] = next.y;
            s_m[buf ^ 1][threadIdx.x] = next.z;
        }
        // one barrier a chunk: a buffer is written again only after the next
        // chunk's barrier, which follows the reads below
        __syncthreads();
        if (Both && threadIdx.x < kPairChunk && c + threadIdx.x < n) {
            float2 s = s_a[buf][0][threadIdx.x];
#pragma unroll
            for (int k = 1; k < W; ++k) {
                const float2 v = s_a[buf][k][threadIdx.x];
                s.x += v.x;
                s.y += v.y;
            }
            pl.part[(uint64_t)a * pl.stride + c + threadIdx.x] = s;
        }
        c += kPairChunk;
        buf ^= 1;
    };
    while (c < end && c < i0 + I) chunk(std::false_type{});
    while (c < end) chunk(std::true_type{});
    // the own bodies' sums over the 32 lanes of each half: every step halves
    // the values a lane keeps, until lane (comp, r) holds component comp of row r
    float v[32];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        v[r] = sx[r];
        v[16 + r] = sy[r];
    }
#pragma unroll
    for (int d = 16; d; d >>= 1) {
        const bool up = (lane & d) != 0;
#pragma unroll
        for (int r = 0; r < d; ++r) {
            const float keep = up ? v[r + d] : v[r], send = up ? v[r] : v[r + d];
            v[r] = keep + __shfl_xor(send, d);
        }
    }
    const uint32_t r = lane & 15, i = ib + 8 * (r / 4) + 4 * hi + r % 4;
    const uint32_t slot = a + seg - i0 / pl.J;
    reinterpret_cast<float *>(pl.part)[2 * ((uint64_t)slot * pl.stride + i) + ((lane >> 4) & 1)] = v[0];
}

// v += f / m dt; x += v dt (velocity first)
__device__ __forceinline__ void nbody_move(float dt, float fx, float fy, float m, float &vx, float &vy, float &x,
                                           float &y)
{
    vx += fx / m * dt;
    vy += fy / m * dt;
    x += vx * dt;
    y += vy * dt;
}

// Adds up each body's partial sums with Kahan compensation and stores its
// force: a work-group per listed block, whose four wavefronts take a quarter
// of the slots each, in order, eight rows in flight (one wavefront a block
// took 25 us over the 64 to 256 rows of 65,536 bodies: too few loads in
// flight).  kCaptured: also the forces of a list that is too long for the rows.
// kMove: also Body::update of the body, which no other work-group of the
// launch reads.  A step of a few thousand bodies is three launches near the
// launch floor (3,001 bodies: 9.0, 3.3 and 3.3 us and the gaps between them);
// this one saves the third: eight steps and their read-back 273 us with it and
// 247 without.
template <int W, bool kMove, bool kCaptured>
__global__ __launch_bounds__(256) void k_nbody_sum(HeapView h, NbodyK p, PairPlan pl)
{
    static_assert(!(kMove && kCaptured), "the walk reads positions that other work-groups would move");
    __shared__ float2 red[4][64];
    const uint32_t err = ald32(h.ctrl + CTRL_ERR);
    const BlockList L = block_list(h, p.cls);
    const uint32_t e = blockIdx.x, s = lane_id(), w = threadIdx.x >> 6;
    if constexpr (kCaptured) {
        __shared__ float4 tile[4][64];
        if (!err && 64 * L.r > pl.stride) {
            if (p.eps2 > 0.f) nbody_force_walk<false>(h, p, L, tile, red);
            else nbody_force_walk<true>(h, p, L, tile, red);
            return;
        }
    }
    if (err || e >= L.r || 64 * L.r > pl.stride) return;
    const uint32_t n = 64 * L.r, g = e * 64 / (32 * W), i = e * 64 + s;
    const uint32_t slots = g + (n + pl.J - 1) / pl.J - g * (32 * W) / pl.J;
    const uint32_t lo = slots * w / 4, hi = slots * (w + 1) / 4;
    const uint32_t bid = L.at(e);
    const uint32_t t = h.type[bid];
    const uint64_t bm = h.alloc_bm[bid];
    const float m = farr<float>(h, bid, p.o_m)[s];
    float vx = 0.f, vy = 0.f, x = 0.f, y = 0.f;
    if (kMove && w == 0) {
        vx = farr<float>(h, bid, p.o_vx)[s];
        vy = farr<float>(h, bid, p.o_vy)[s];
        x = farr<float>(h, bid, p.o_x)[s];
        y = farr<float>(h, bid, p.o_y)[s];
    }
    float ax = 0.f, ay = 0.f, cx = 0.f, cy = 0.f;
    for (uint32_t k = lo; k < hi; k += 8) {
        float2 v[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u)
            v[u] = k + u < hi ? pl.part[(uint64_t)(k + u) * pl.stride + i] : make_float2(0.f, 0.f);
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const float yx = v[u].x - cx, tx = ax + yx;
            cx = (tx - ax) - yx;
            ax = tx;
            const float yy = v[u].y - cy, ty = ay + yy;
            cy = (ty - ay) - yy;
            ay = ty;
        }
    }
    red[w][s] = make_float2(ax, ay);
    __syncthreads();
    if (w || t != p.cls || !((bm >> s) & 1)) return;
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        ax += red[k][s].x;
        ay += red[k][s].y;
    }
    const float gm = p.G * m, fx = gm * ax, fy = gm * ay;
    farr<float>(h, bid, p.o_fx)[s] = fx;
    farr<float>(h, bid, p.o_fy)[s] = fy;
    if (!kMove) return;
    nbody_move(p.dt, fx, fy, m, vx, vy, x, y);
    farr<float>(h, bid, p.o_vx)[s] = vx;
    farr<float>(h, bid, p.o_vy)[s] = vy;
    farr<float>(h, bid, p.o_x)[s] = x;
    farr<float>(h, bid, p.o_y)[s] = y;
}

// Body::update
__global__ __launch_bounds__(1024) void k_nbody_update(HeapView h, NbodyK p)
{
    for_each_block(h, p.cls, false, [&](uint32_t bid, uint64_t bm) {
        const uint32_t s = lane_id();
        if (!((bm >> s) & 1)) return;
        const float m = farr<float>(h, bid, p.o_m)[s];
        float vx = farr<float>(h, bid, p.o_vx)[s], vy = farr<float>(h, bid, p.o_vy)[s];
        float x = farr<float>(h, bid, p.o_x)[s], y = farr<float>(h, bid, p.o_y)[s];
        nbody_move(p.dt, farr<float>(h, bid, p.o_fx)[s], farr<float>(h, bid, p.o_fy)[s], m, vx, vy, x, y);
        farr<float>(h, bid, p.o_vx)[s] = vx;
        farr<float>(h, bid, p.o_vy)[s] = vy;
        farr<float>(h, bid, p.o_x)[s] = x;
        farr<float>(h, bid, p.o_y)[s] = y;
    });
}

smmo_status bind_nbody(smmo_heap *h, uint32_t cls, const smmo_nbody_args &a, NbodyK &k)
{
    if (!(a.eps >= 0.f) || !(a.dt == a.dt) || !(a.G == a.G)) return fail(SMMO_EINVAL, "nbody: bad parameters");
    k.cls = cls;
    BIND(cls, "pos_x", SMMO_F32, 1, &k.o_x, nullptr);
    BIND(cls, "pos_y", SMMO_F32, 1, &k.o_y, nullptr);
    BIND(cls, "vel_x", SMMO_F32, 1, &k.o_vx, nullptr);
    BIND(cls, "vel_y", SMMO_F32, 1, &k.o_vy, nullptr);
    BIND(cls, "force_x", SMMO_F32, 1, &k.o_fx, nullptr);
    BIND(cls, "force_y", SMMO_F32, 1, &k.o_fy, nullptr);
    BIND(cls, "mass", SMMO_F32, 1, &k.o_m, nullptr);
    k.G = a.G;
    k.eps2 = a.eps * a.eps;
    k.dt = a.dt;
    return SMMO_OK;
}

// The pair kernel's shape for a class of up to `blocks` blocks: wavefronts per
// group (W; 0: the class takes k_nbody_force) and slots per segment (J).
// Small segments fill the chip, large ones spend less on starting a
// work-group and on partial sums; the lines lie where two shapes cross
// (us a force pass): at 640 bodies k_nbody_force 8.2, W 4 J 128 8.2 (at 500:
// 6.7 and 8.2); at 6,000 J 128 18.0, J 256 19.2 (8,000: 24.6 and 23.6); at
// 16,000 J 256 66.2, J 512 65.9 (12,000: 42.1 and 44.5).  W 8 halves the
// partial sums' memory, which grows with the square of the class (134 MB for
// 65,536 bodies), for 1-2 % of the time (32,000: W 4 J 512 219, W 8 J 1024
// 225); past 98,000 bodies they would take over 300 MB and the class goes
// back to k_nbody_force.  `blocks` is the host's bound, which
// grows with every creation and never falls: a small class whose bodies are
// destroyed and created again drifts to the larger shapes and past the last.
struct PairShape {
    uint32_t W, J;
};

constexpr uint64_t kPairMostBlocks = 1536;

PairShape pair_shape(uint64_t blocks)
{
    if (blocks < 12 || blocks > kPairMostBlocks) return {0, 0};
    if (blocks <= 96) return {4, 128};
    if (blocks <= 224) return {4, 256};
    if (blocks <= 512) return {4, 512};
    return {8, 1024};
}

// Rows of partial sums: one per group before a body's own, and per segment from
// its own on (the largest over the groups), see k_nbody_pairs.
uint64_t pair_rows(uint64_t slots, const PairShape &s)
{
    const uint64_t I = 32 * s.W, groups = (slots + I - 1) / I, segs = (slots + s.J - 1) / s.J;
    uint64_t rows = 0;
    for (uint64_t g = 0; g < groups; ++g) rows = std::max(rows, g + segs - g * I / s.J);
    return rows;
}

template <int W, bool kCaptured>
void launch_pairs(smmo_heap *h, const NbodyK &k, const PairPlan &pl, uint64_t blocks, bool move, hipStream_t st)
{
    const uint64_t segs = (64 * blocks + pl.J - 1) / pl.J;
    const dim3 grid((uint32_t)(pl.J / (32 * W) * (segs * (segs + 1) / 2)));
    if (k.eps2 > 0.f) hipLaunchKernelGGL((k_nbody_pairs<W, false, kCaptured>), grid, dim3(64 * W), 0, st, h->v, k, pl);
    else hipLaunchKernelGGL((k_nbody_pairs<W, true, kCaptured>), grid, dim3(64 * W), 0, st, h->v, k, pl);
    const dim3 covered(pl.stride / 64);                 // the blocks of whole groups
    if (move) hipLaunchKernelGGL((k_nbody_sum<W, true, false>), covered, dim3(256), 0, st, h->v, k, pl);
    else hipLaunchKernelGGL((k_nbody_sum<W, false, kCaptured>), covered, dim3(256), 0, st, h->v, k, pl);
}

uint64_t pair_stride(uint64_t blocks, const PairShape &s)
{
    const uint64_t I = 32 * s.W;
    return (64 * blocks + I - 1) / I * I;
}

uint64_t pair_bytes(uint64_t blocks)
{
    const PairShape s = pair_shape(blocks);
    return pair_rows(64 * blocks, s) * pair_stride(blocks, s) * sizeof(float2);
}

// The pair kernel's plan for class cls, whose list is ready: whether it takes
// the pair form, and then the workspace that holds the partial sums.
bool pair_plan(smmo_heap *h, uint32_t cls, uint64_t blocks, PairShape &sh, PairPlan &pl, hipStream_t st)
{
    sh = pair_shape(blocks);
    if (!sh.W || h->replayed[cls] || ((h->v.direct >> cls) & 1)) return false;
    static const uint64_t most = pair_bytes(kPairMostBlocks);
    float2 *part = static_cast<float2 *>(class_workspace(h, cls, pair_bytes(blocks), most, st));
    pl = PairPlan{part, (uint32_t)pair_stride(blocks, sh), sh.J};
    return part != nullptr;
}

void run_pairs(smmo_heap *h, const NbodyK &k, const PairShape &sh, const PairPlan &pl, uint64_t blocks, bool move,
               hipStream_t st)
{
    if (stream_captured(st)) {                          // (never with `move`)
        if (sh.W == 4) launch_pairs<4, true>(h, k, pl, blocks, false, st);
        else launch_pairs<8, true>(h, k, pl, blocks, false, st);
    } else {
        if (sh.W == 4) launch_pairs<4, false>(h, k, pl, blocks, move, st);
        else launch_pairs<8, false>(h, k, pl, blocks, move, st);
    }
}

smmo_status nbody_force_launch(smmo_heap *h, uint32_t cls, const void *args, hipStream_t st)
{
    smmo_nbody_args a;
    memcpy(&a, args, sizeof a);
    NbodyK k;
    smmo_status s = cached_bind(h, (const void *)&nbody_force_launch, cls, a, k,
                                [&] { return bind_nbody(h, cls, a, k); });
    if (s) return s;
    if ((s = ensure_enumerated(h, cls, false, st))) return s;
    const uint64_t blocks = std::max<uint64_t>(1, h->ub_blocks[cls]);
    PairShape sh;
    PairPlan pl;
    if (pair_plan(h, cls, blocks, sh, pl, st)) {
        run_pairs(h, k, sh, pl, blocks, false, st);
        return launched("k_nbody_pairs");
    }
    const uint32_t grid = (uint32_t)std::min<uint64_t>(blocks, 8192);
    if (k.eps2 > 0.f)
        hipLaunchKernelGGL(k_nbody_force<false>, dim3(grid), dim3(256), 0, st, h->v, k);
    else
        hipLaunchKernelGGL(k_nbody_force<true>, dim3(grid), dim3(256), 0, st, h->v, k);
    return launched("k_nbody_force");
}

smmo_status nbody_update_launch(smmo_heap *h, uint32_t cls, const void *args, hipStream_t st)
{
    smmo_nbody_args a;
    memcpy(&a, args, sizeof a);
    NbodyK k;
    smmo_status s = cached_bind(h, (const void *)&nbody_update_launch, cls, a, k,
                                [&] { return bind_nbody(h, cls, a, k); });
    if (s) return s;
    if ((s = ensure_enumerated(h, cls, false, st))) return s;
    hipLaunchKernelGGL(k_nbody_update, method_shape(h, cls).grid, method_shape(h, cls).block, 0, st, h->v, k);
    return launched("k_nbody_update");
}

// nbody.steps on Body: `steps` times nbody.force and nbody.update, a body moved
// by the launch that adds up its force where the class takes the pair form, no
// snapshot taken ahead waits for one of the two do-alls and the launches are
// not captured (a replay may have to walk all pairs before any body moves).
smmo_status nbody_steps_launch(smmo_heap *h, uint32_t cls, const void *args, hipStream_t st)
{
    smmo_nbody_steps_args sa;
    memcpy(&sa, args, sizeof sa);
    const smmo_nbody_args a{sa.G, sa.eps, sa.dt, 0};
    NbodyK k;
    smmo_status s = cached_bind(h, (const void *)&nbody_steps_launch, cls, a, k,
                                [&] { return bind_nbody(h, cls, a, k); });
    if (s) return s;
    if (sa.steps == 0) return SMMO_OK;
    const uint64_t blocks = std::max<uint64_t>(1, h->ub_blocks[cls]);
    PairShape sh;
    PairPlan pl;
    if (!((h->v.snap >> cls) & 1) && !stream_captured(st)) {
        if ((s = ensure_enumerated(h, cls, false, st))) return s;
        if (pair_plan(h, cls, blocks, sh, pl, st)) {
            for (uint32_t t = 0; t < sa.steps; ++t) run_pairs(h, k, sh, pl, blocks, true, st);
            return launched("k_nbody_pairs");
        }
    }
    // as the two do-alls, with their launch shapes; a snapshot is the first one's
    uint32_t force = 0, update = 0;
    if ((s = smmo_method_id("nbody.force", &force)) || (s = smmo_method_id("nbody.update", &update))) return s;
    const uint32_t method = h->cur_method;
    for (uint32_t t = 0; t < sa.steps && !s; ++t) {
        h->cur_method = force;
        s = nbody_force_launch(h, cls, &a, st);
        h->v.snap &= ~(1u << cls);
        h->cur_method = update;
        if (!s) s = nbody_update_launch(h, cls, &a, st);
    }
    h->cur_method = method;
    return s;
}

} // namespace

namespace smmo {
smmo_status launch_nbody_force(smmo_heap *h, uint32_t c, const void *a, hipStream_t s) { return nbody_force_launch(h, c, a, s); }
smmo_status launch_nbody_update(smmo_heap *h, uint32_t c, const void *a, hipStream_t s) { return nbody_update_launch(h, c, a, s); }
smmo_status launch_nbody_steps(smmo_heap *h, uint32_t c, const void *a, hipStream_t s) { return nbody_steps_launch(h, c, a, s); }
} // namespace smmo
