// Spring-mass methods (thesis Ch.7 "structure", its compute steps):
// Spring::force, Node::update and the topology link; field contracts in
// include/smmo_methods.h.  These are the kernels of the spring step; the
// launch conventions are those of every method kernel (method_common.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "../../include/smmo_methods.h"
#include "method_common.hpp"

using namespace smmo;

namespace {

// ======================================================== spring-mass =====
struct SpringK {
    uint32_t node_cls, spring_cls;
    uint32_t s_a, s_b, s_k, s_L0, s_fx, s_fy, s_sa, s_sb;      // Spring fields
    uint32_t n_x, n_y, n_vx, n_vy, n_m, n_adj, n_adj_stride;   // Node fields
    float dt, limit;
    uint32_t tension_only;
    uint32_t wpg;             // wavefronts per work-group of this launch
};

// A load of a field that a do-all reads once per object (not one of the
// gathered fields): with NT it carries the non-temporal hint, so that these
// lines do not displace the gathered ones (node positions, spring forces,
// each read by several objects) from the L2 and the MALL.
template <bool NT, class T>
__device__ __forceinline__ T stream_ld(const T &r)
{
    if constexpr (NT) return __builtin_nontemporal_load(&r);
    else return r;
}

// The break decision is integer-valued, so it is evaluated in float32 with a
// fixed operation order (no contraction): dx, dy; l2 = fma(dx, dx, dy*dy);
// l = sqrt(l2) (correctly rounded); strain = (l - L0) / L0 (correctly rounded).
__device__ __forceinline__ bool spring_breaks(float dx, float dy, float L0, float limit, float &l)
{
#pragma clang fp contract(off)
    const float dy2 = dy * dy;
    const float l2 = __builtin_fmaf(dx, dx, dy2);
    l = __builtin_sqrtf(l2);
    const float strain = (l - L0) / L0;
    return strain > limit;
}

// the force of a live spring on its endpoint a, and whether the spring breaks
// (the force is then 0)
__device__ __forceinline__ bool spring_law(const SpringK &p, float dx, float dy, float k, float L0, float &fx,
                                           float &fy)
{
    float l;
    const bool brk = spring_breaks(dx, dy, L0, p.limit, l);
    fx = fy = 0.f;
    if (!brk && (!p.tension_only || l > L0)) {
        const float c = k * (l - L0) / l;
        fx = c * dx;
        fy = c * dy;
    }
    return brk;
}

// v += F/m dt, x += v dt
__device__ __forceinline__ void node_law(const SpringK &p, float Fx, float Fy, float m, float &x, float &y, float &vx,
                                         float &vy)
{
    vx += Fx / m * p.dt;
    vy += Fy / m * p.dt;
    x += vx * p.dt;
    y += vy * p.dt;
}

// Spring::compute_force (Ch.7 "structure"): Hooke's law on the length change;
// a spring strained past the limit empties its two adjacency slots and
// deletes itself (the thesis's remove_spring followed by destroy).  A
// wavefront works on U blocks at once: the spring fields of all U blocks are
// loaded, then all position gathers issued, then the forces computed.
template <int U, bool NT>
__device__ __forceinline__ void spring_force(const HeapView &h, const SpringK &p)
{
    const uint32_t s = lane_id();
    for_each_block_heads<U>(h, p.spring_cls, p.wpg, [&](const BlockHeads<U> &hd) {
        const uint32_t *bid = hd.bid;
        uint32_t a[U], b[U];
        float k[U], L0[U], xa[U], ya[U], xb[U], yb[U];
        bool live[U], own[U];
        // the blocks' own fields for all 64 slots (one contiguous run each),
        // issued before the headers are used
#pragma unroll
        for (int j = 0; j < U; ++j) {
            a[j] = stream_ld<NT>(farr<uint32_t>(h, bid[j], p.s_a)[s]);
            b[j] = stream_ld<NT>(farr<uint32_t>(h, bid[j], p.s_b)[s]);
            k[j] = stream_ld<NT>(farr<float>(h, bid[j], p.s_k)[s]);
            L0[j] = stream_ld<NT>(farr<float>(h, bid[j], p.s_L0)[s]);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            own[j] = hd.own(j);
            live[j] = (hd.bm(j) >> s) & 1;
        }
        // gathers through the node handles, live slots only
#pragma unroll
        for (int j = 0; j < U; ++j) {
            xa[j] = ya[j] = xb[j] = yb[j] = 0.f;
            if (live[j]) {
                xa[j] = fref<float>(h, a[j], p.n_x);
                ya[j] = fref<float>(h, a[j], p.n_y);
                xb[j] = fref<float>(h, b[j], p.n_x);
                yb[j] = fref<float>(h, b[j], p.n_y);
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if (!own[j]) continue;
            float fx = 0.f, fy = 0.f;
            bool brk = false;
            if (live[j]) brk = spring_law(p, xb[j] - xa[j], yb[j] - ya[j], k[j], L0[j], fx, fy);
            // full-width stores: dead and broken slots get 0, never read
            farr<float>(h, bid[j], p.s_fx)[s] = fx;
            farr<float>(h, bid[j], p.s_fy)[s] = fy;
            if (brk) {
                const uint32_t qa = farr<uint8_t>(h, bid[j], p.s_sa)[s];
                const uint32_t qb = farr<uint8_t>(h, bid[j], p.s_sb)[s];
                fref<uint32_t>(h, a[j], p.n_adj + qa * p.n_adj_stride) = kNull;
                fref<uint32_t>(h, b[j], p.n_adj + qb * p.n_adj_stride) = kNull;
            }
            wave_release_own_block(h, p.spring_cls, bid[j], __ballot(brk));
        }
    });
}

// One and two blocks per iteration: the registers are held to what eight
// wavefronts per SIMD allow (the rare release path of a breaking spring would
// otherwise raise the scalar registers past that), so one grid of 32
// wavefronts per CU stays resident.  Four blocks per iteration need more
// registers than that and keep the compiler's allocation.
template <int U, bool NT>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_spring_force(HeapView h,
                                                                                                 SpringK p)
{
    spring_force<U, NT>(h, p);
}

template <bool NT>
__global__ __launch_bounds__(1024) void k_spring_force4(HeapView h, SpringK p)
{
    spring_force<4, NT>(h, p);
}

// Node::update: sum the attached springs' forces in slot order (+f if this
// node is endpoint a, -f if b), then v += F/m dt, x += v dt.  U blocks at
// once, as in the force kernel.
template <int U, bool NT>
__device__ __forceinline__ void spring_node(const HeapView &h, const SpringK &p)
{
    const uint32_t s = lane_id();
    for_each_block_heads<U>(h, p.node_cls, p.wpg, [&](const BlockHeads<U> &hd) {
        const uint32_t *bid = hd.bid;
        uint32_t e[U][8];
        float m[U], x[U], y[U], vx[U], vy[U], Fx[U], Fy[U];
        bool live[U];
        // the blocks' fields, issued before the headers are used
#pragma unroll
        for (int j = 0; j < U; ++j) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
                e[j][q] = stream_ld<NT>(farr<uint32_t>(h, bid[j], p.n_adj + q * p.n_adj_stride)[s]);
            m[j] = stream_ld<NT>(farr<float>(h, bid[j], p.n_m)[s]);
            x[j] = stream_ld<NT>(farr<float>(h, bid[j], p.n_x)[s]);
            y[j] = stream_ld<NT>(farr<float>(h, bid[j], p.n_y)[s]);
            vx[j] = stream_ld<NT>(farr<float>(h, bid[j], p.n_vx)[s]);
            vy[j] = stream_ld<NT>(farr<float>(h, bid[j], p.n_vy)[s]);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) live[j] = (hd.bm(j) >> s) & 1;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            float gx[8], gy[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                gx[q] = 0.f;
                gy[q] = 0.f;
                if (live[j] && e[j][q] != kNull) {
                    const uint32_t sh = e[j][q] & 0x7FFFFFFFu;
                    gx[q] = fref<float>(h, sh, p.s_fx);
                    gy[q] = fref<float>(h, sh, p.s_fy);
                }
            }
            Fx[j] = 0.f;
            Fy[j] = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (e[j][q] == kNull) continue;
                if (e[j][q] >> 31) {
                    Fx[j] -= gx[q];
                    Fy[j] -= gy[q];
                } else {
                    Fx[j] += gx[q];
                    Fy[j] += gy[q];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if (!live[j]) continue;
            node_law(p, Fx[j], Fy[j], m[j], x[j], y[j], vx[j], vy[j]);
            farr<float>(h, bid[j], p.n_vx)[s] = vx[j];
            farr<float>(h, bid[j], p.n_vy)[s] = vy[j];
            farr<float>(h, bid[j], p.n_x)[s] = x[j];
            farr<float>(h, bid[j], p.n_y)[s] = y[j];
        }
    });
}

template <int U, bool NT>
__global__ __launch_bounds__(1024) void k_spring_node(HeapView h, SpringK p)
{
    spring_node<U, NT>(h, p);
}

// ---- several steps of a small mesh in one launch ----------------------------
// A mesh of a few dozen blocks spends its step on two launches and their
// chains of dependent loads (7.0 us for 957 nodes and 2,748 springs, of which
// the arithmetic is a fraction).  Here one work-group of 16 wavefronts runs
// `steps` of them: wavefront w owns entries w, w + 16, ... of both block
// lists, the fields of its springs and nodes stay in registers, positions and
// forces in LDS, and two barriers separate the passes of a step.  Bound by
// the arithmetic of one CU: 1.9 us a step there, 4.2 us for 1,936 nodes and
// 5,633 springs (6.5 as two launches in a graph); two steps of 957 nodes cost
// 8.9 us each in one launch, 12.1 as four.
// Same operations in the same order as the two do-alls.  A spring that breaks
// exerts no force from then on; its slots are emptied and released after the
// last step, which leaves the heap as the separate launches do.  A handle that
// names a block outside the two lists (a node or spring of another class with
// the same field offsets) is followed in memory at every step.
// A replay of a captured launch may find lists that have grown beyond the
// registers since: a second launch, captured with it, then walks the two
// do-alls' passes (in this kernel they would take its scalar registers).
constexpr uint32_t kStepsMaxBlocks = 4096;   // heap blocks: the table of list positions
// Steps of one launch, so that it ends within 17 ms at most (4.2 us a step):
// nothing else on the stream runs meanwhile.  A launch more costs 7 us.
constexpr uint32_t kStepsMost = 4096;
constexpr uint32_t kNone16 = 0x7FFF, kFar16 = 0x7FFE;

template <int SBW, int NBW, bool kCaptured>
__global__ __launch_bounds__(1024) void k_spring_steps(HeapView h, SpringK p, uint32_t steps)
{
    __shared__ float2 s_x[NBW * 1024], s_f[SBW * 1024];
    __shared__ uint16_t s_pos[kStepsMaxBlocks];   // list position of a block; springs' with bit 15
    const uint32_t s = lane_id(), w = threadIdx.x >> 6;
    const uint32_t err = ald32(h.ctrl + CTRL_ERR);
    const BlockList SL = block_list(h, p.spring_cls), NL = block_list(h, p.node_cls);
    if (err) return;
    if (SL.r > 16 * SBW || NL.r > 16 * NBW || h.M > kStepsMaxBlocks) {   // only a replay finds more than the host's bounds
        if (!kCaptured && threadIdx.x == 0) raise_error(h, ERR_INTERNAL);
        return;
    }
    for (uint32_t b = threadIdx.x; b < h.M; b += 1024) s_pos[b] = (uint16_t)kNone16;
    __syncthreads();
    // this wavefront's blocks (kNoBlock where there is none)
    uint32_t sbid[SBW], nbid[NBW];
    uint64_t live[SBW], nlive[NBW];
#pragma unroll
    for (int j = 0; j < SBW; ++j) {
        const uint32_t i = w + 16 * j;
        sbid[j] = __builtin_amdgcn_readfirstlane(i < SL.r ? SL.at(i) : kNoBlock);
        live[j] = 0;
        if (sbid[j] == kNoBlock) continue;
        if (h.type[sbid[j]] != p.spring_cls) {
            sbid[j] = kNoBlock;
            continue;
        }
        live[j] = uniform64(h.alloc_bm[sbid[j]]);
        if (s == 0) s_pos[sbid[j]] = (uint16_t)(0x8000u | i);
    }
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
        const uint32_t i = w + 16 * j;
        nbid[j] = __builtin_amdgcn_readfirstlane(i < NL.r ? NL.at(i) : kNoBlock);
        nlive[j] = 0;
        if (nbid[j] == kNoBlock) continue;
        if (h.type[nbid[j]] != p.node_cls) {
            nbid[j] = kNoBlock;
            continue;
        }
        nlive[j] = uniform64(h.alloc_bm[nbid[j]]);
        if (s == 0) s_pos[nbid[j]] = (uint16_t)i;
    }
    __syncthreads();
    // the LDS index of a handle's object among the nodes (tag 0) or springs
    // (tag 0x8000)
    auto index = [&](uint32_t handle, uint32_t tag) -> uint32_t {
        const uint32_t b = handle >> 6;
        const uint32_t pos = b < h.M ? s_pos[b] : kNone16;
        return pos != kNone16 && (pos & 0x8000u) == tag ? ((pos & 0x7FFu) << 6 | (handle & 63)) : kFar16;
    };
    uint32_t ab[SBW];
    float k[SBW], L0[SBW];
#pragma unroll
    for (int j = 0; j < SBW; ++j) {
        ab[j] = 0;
        k[j] = L0[j] = 0.f;
        if (!((live[j] >> s) & 1)) continue;
        k[j] = farr<float>(h, sbid[j], p.s_k)[s];
        L0[j] = farr<float>(h, sbid[j], p.s_L0)[s];
        ab[j] = index(farr<uint32_t>(h, sbid[j], p.s_a)[s], 0) | index(farr<uint32_t>(h, sbid[j], p.s_b)[s], 0) << 16;
    }
    uint32_t e[NBW][4];                    // two slots each: LDS index, bit 15: endpoint b
    float m[NBW], x[NBW], y[NBW], vx[NBW], vy[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) e[j][q] = kNone16 << 16 | kNone16;
        m[j] = x[j] = y[j] = vx[j] = vy[j] = 0.f;
        if (nbid[j] == kNoBlock) continue;
        // positions of free slots too, as a spring would read them
        x[j] = farr<float>(h, nbid[j], p.n_x)[s];
        y[j] = farr<float>(h, nbid[j], p.n_y)[s];
        s_x[(w + 16 * j) * 64 + s] = make_float2(x[j], y[j]);
        if (!((nlive[j] >> s) & 1)) continue;
        vx[j] = farr<float>(h, nbid[j], p.n_vx)[s];
        vy[j] = farr<float>(h, nbid[j], p.n_vy)[s];
        m[j] = farr<float>(h, nbid[j], p.n_m)[s];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint32_t hd = farr<uint32_t>(h, nbid[j], p.n_adj + q * p.n_adj_stride)[s];
            const uint32_t v = hd == kNull ? kNone16 : index(hd & 0x7FFFFFFFu, 0x8000u) | (hd >> 31) << 15;
            e[j][q / 2] = q % 2 ? (e[j][q / 2] & 0xFFFFu) | v << 16 : v;
        }
    }
    __syncthreads();
    auto node_at = [&](uint32_t i, int j, uint32_t field) {
        if (i != kFar16) return s_x[i];
        const uint32_t hd = farr<uint32_t>(h, sbid[j], field)[s];
        return make_float2(fref<float>(h, hd, p.n_x), fref<float>(h, hd, p.n_y));
    };
    for (uint32_t t = 0; t < steps; ++t) {
#pragma unroll
        for (int j = 0; j < SBW; ++j) {
            if (sbid[j] == kNoBlock) continue;
            float fx = 0.f, fy = 0.f;
            bool brk = false;
            if ((live[j] >> s) & 1) {
                const float2 a = node_at(ab[j] & 0xFFFFu, j, p.s_a), b = node_at(ab[j] >> 16, j, p.s_b);
                brk = spring_law(p, b.x - a.x, b.y - a.y, k[j], L0[j], fx, fy);
            }
            s_f[(w + 16 * j) * 64 + s] = make_float2(fx, fy);
            live[j] &= ~__ballot(brk);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NBW; ++j) {
            if (!((nlive[j] >> s) & 1)) continue;
            float Fx = 0.f, Fy = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t v = e[j][q / 2] >> 16 * (q % 2), i = v & 0x7FFFu;
                if (i == kNone16) continue;
                float2 f;
                if (i != kFar16) {
                    f = s_f[i];
                } else {
                    const uint32_t hd = farr<uint32_t>(h, nbid[j], p.n_adj + q * p.n_adj_stride)[s] & 0x7FFFFFFFu;
                    f = make_float2(fref<float>(h, hd, p.s_fx), fref<float>(h, hd, p.s_fy));
                }
                if (v & 0x8000u) {
                    Fx -= f.x;
                    Fy -= f.y;
                } else {
                    Fx += f.x;
                    Fy += f.y;
                }
            }
            node_law(p, Fx, Fy, m[j], x[j], y[j], vx[j], vy[j]);
            s_x[(w + 16 * j) * 64 + s] = make_float2(x[j], y[j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < NBW; ++j) {
        if (!((nlive[j] >> s) & 1)) continue;
        farr<float>(h, nbid[j], p.n_vx)[s] = vx[j];
        farr<float>(h, nbid[j], p.n_vy)[s] = vy[j];
        farr<float>(h, nbid[j], p.n_x)[s] = x[j];
        farr<float>(h, nbid[j], p.n_y)[s] = y[j];
    }
#pragma unroll
    for (int j = 0; j < SBW; ++j) {
        if (sbid[j] == kNoBlock) continue;
        const float2 f = s_f[(w + 16 * j) * 64 + s];
        farr<float>(h, sbid[j], p.s_fx)[s] = f.x;
        farr<float>(h, sbid[j], p.s_fy)[s] = f.y;
        const uint64_t broken = uniform64(h.alloc_bm[sbid[j]]) & ~live[j];
        if ((broken >> s) & 1) {
            const uint32_t a = farr<uint32_t>(h, sbid[j], p.s_a)[s], b = farr<uint32_t>(h, sbid[j], p.s_b)[s];
            const uint32_t qa = farr<uint8_t>(h, sbid[j], p.s_sa)[s], qb = farr<uint8_t>(h, sbid[j], p.s_sb)[s];
            fref<uint32_t>(h, a, p.n_adj + qa * p.n_adj_stride) = kNull;
            fref<uint32_t>(h, b, p.n_adj + qb * p.n_adj_stride) = kNull;
        }
        wave_release_own_block(h, p.spring_cls, sbid[j], broken);
    }
}

// The steps that k_spring_steps<SBW, NBW> left because a list was too long for
// it (nothing where it was not): one work-group, the passes of the do-alls.
template <int SBW, int NBW>
__global__ __launch_bounds__(1024) void k_spring_steps_grown(HeapView h, SpringK p, uint32_t steps)
{
    if (block_list(h, p.spring_cls).r <= 16 * SBW && block_list(h, p.node_cls).r <= 16 * NBW) return;
    for (uint32_t t = 0; t < steps; ++t) {
        spring_force<1, false>(h, p);
        __threadfence();                   // slots emptied and blocks released by the other wavefronts
        __syncthreads();
        spring_node<1, false>(h, p);
        __threadfence();
        __syncthreads();
    }
}

template <int SBW, int NBW>
void launch_spring_steps(smmo_heap *h, SpringK k, uint32_t steps, bool captured, hipStream_t st)
{
    k.wpg = 16;
    for (uint32_t left = steps, n; left; left -= n) {
        n = std::min(left, kStepsMost);
        if (captured) {
            hipLaunchKernelGGL((k_spring_steps<SBW, NBW, true>), dim3(1), dim3(1024), 0, st, h->v, k, n);
            hipLaunchKernelGGL((k_spring_steps_grown<SBW, NBW>), dim3(1), dim3(1024), 0, st, h->v, k, n);
        } else {
            hipLaunchKernelGGL((k_spring_steps<SBW, NBW, false>), dim3(1), dim3(1024), 0, st, h->v, k, n);
        }
    }
}

// Spring::link: registers the spring in its two nodes' adjacency slots
// (slot_a of a, slot_b of b, the latter flagged as endpoint b).  Builds a
// mesh's topology on the device after parallel_new of nodes and springs;
// every (node, slot) pair belongs to one spring, so the writes never collide.
__global__ __launch_bounds__(1024) void k_spring_link(HeapView h, SpringK p)
{
    for_each_block(h, p.spring_cls, false, [&](uint32_t bid, uint64_t bm) {
        const uint32_t s = lane_id();
        if (!((bm >> s) & 1)) return;
        const uint32_t self = (bid << 6) | s;
        const uint32_t a = farr<uint32_t>(h, bid, p.s_a)[s];
        const uint32_t b = farr<uint32_t>(h, bid, p.s_b)[s];
        const uint32_t qa = farr<uint8_t>(h, bid, p.s_sa)[s];
        const uint32_t qb = farr<uint8_t>(h, bid, p.s_sb)[s];
        if (qa >= 8 || qb >= 8) {
            raise_error(h, ERR_BADHANDLE);
            return;
        }
        fref<uint32_t>(h, a, p.n_adj + qa * p.n_adj_stride) = self;
        fref<uint32_t>(h, b, p.n_adj + qb * p.n_adj_stride) = self | 0x80000000u;
    });
}

smmo_status bind_spring(smmo_heap *h, const smmo_spring_args &a, SpringK &k)
{
    const uint32_t nc = h->schema->nclasses;
    if (a.node_class >= nc || a.spring_class >= nc || a.node_class == a.spring_class)
        return fail(SMMO_EINVAL, "spring: bad class ids");
    if (!(a.dt == a.dt) || !(a.strain_limit == a.strain_limit)) return fail(SMMO_EINVAL, "spring: NaN parameter");
    if (a.flags & ~SMMO_SPRING_TENSION_ONLY) return fail(SMMO_EINVAL, "spring: unknown flags");
    k.node_cls = a.node_class;
    k.spring_cls = a.spring_class;
    BIND(a.spring_class, "a", SMMO_HANDLE, 1, &k.s_a, nullptr);
    BIND(a.spring_class, "b", SMMO_HANDLE, 1, &k.s_b, nullptr);
    BIND(a.spring_class, "k", SMMO_F32, 1, &k.s_k, nullptr);
    BIND(a.spring_class, "L0", SMMO_F32, 1, &k.s_L0, nullptr);
    BIND(a.spring_class, "fx", SMMO_F32, 1, &k.s_fx, nullptr);
    BIND(a.spring_class, "fy", SMMO_F32, 1, &k.s_fy, nullptr);
    BIND(a.spring_class, "slot_a", SMMO_U8, 1, &k.s_sa, nullptr);
    BIND(a.spring_class, "slot_b", SMMO_U8, 1, &k.s_sb, nullptr);
    BIND(a.node_class, "x", SMMO_F32, 1, &k.n_x, nullptr);
    BIND(a.node_class, "y", SMMO_F32, 1, &k.n_y, nullptr);
    BIND(a.node_class, "vx", SMMO_F32, 1, &k.n_vx, nullptr);
    BIND(a.node_class, "vy", SMMO_F32, 1, &k.n_vy, nullptr);
    BIND(a.node_class, "m", SMMO_F32, 1, &k.n_m, nullptr);
    BIND(a.node_class, "adj", SMMO_HANDLE, 8, &k.n_adj, &k.n_adj_stride);
    k.dt = a.dt;
    k.limit = a.strain_limit;
    k.tension_only = (a.flags & SMMO_SPRING_TENSION_ONLY) ? 1u : 0u;
    return SMMO_OK;
}

// Default launch shapes (us a step, one do-all's shape varied; 1000 x 1000,
// 600 x 500 and 224 meshes of 3.5M nodes).  Both take work-groups of two
// wavefronts, which fill the last gaps of a CU better than four.  The force
// pass runs best with one grid that is resident all at once, 32 wavefronts per
// CU: 33.5, 14.7 and 132.8 against 34.8, 16.0 and 135.6 with 64.  The node
// pass keeps 64 (33.6, 15.6), and beyond the MALL, where its two rounds of
// loads wait longest, takes two blocks at a time: 125.9 against 135.6.
constexpr uint32_t kSpringWg = 128, kForceWaves = 32, kNodeWaves = 64;

// the MALL (Infinity Cache) of an MI355X, in front of HBM
constexpr uint64_t kMallBytes = 256ull << 20;

// whether the step's once-read fields get the non-temporal hint (the heap's
// streaming_loads; automatic: when the node and spring blocks exceed the
// MALL, so that a step's blocks cannot stay in it for the next step anyway)
bool streaming(const smmo_heap *h, const SpringK &k)
{
    if (h->cfg.streaming_loads) return h->cfg.streaming_loads == 2;
    return (h->ub_blocks[k.node_cls] + h->ub_blocks[k.spring_cls]) * (uint64_t)h->v.block_bytes > kMallBytes;
}

template <int U, bool NT>
void launch_force(const LaunchShape &ls, hipStream_t st, const HeapView &v, const SpringK &k)
{
    if constexpr (U == 4) hipLaunchKernelGGL(k_spring_force4<NT>, ls.grid, ls.block, 0, st, v, k);
    else hipLaunchKernelGGL((k_spring_force<U, NT>), ls.grid, ls.block, 0, st, v, k);
}

template <int Which>
smmo_status launch_spring(smmo_heap *h, uint32_t cls, const void *args, hipStream_t st)
{
    smmo_spring_args a;
    memcpy(&a, args, sizeof a);
    SpringK k;
    smmo_status s = cached_bind(h, (const void *)&launch_spring<Which>, cls, a, k,
                                [&] { return bind_spring(h, a, k); });
    if (s) return s;
    if (cls != (Which == 1 ? a.node_class : a.spring_class))
        return fail(SMMO_EINVAL, "spring: method runs on a different class");
    if ((s = ensure_enumerated(h, cls, false, st))) return s;
    const bool nt = Which != 2 && streaming(h, k);
    const LaunchShape ls = Which == 0 ? method_shape(h, cls, 1, kSpringWg, kForceWaves)
                                      : method_shape(h, cls, Which == 1 && nt ? 2 : 1, kSpringWg, kNodeWaves);
    k.wpg = ls.block.x / 64;
    if (Which == 0) {
        if (ls.group == 4) nt ? launch_force<4, true>(ls, st, h->v, k) : launch_force<4, false>(ls, st, h->v, k);
        else if (ls.group == 2) nt ? launch_force<2, true>(ls, st, h->v, k) : launch_force<2, false>(ls, st, h->v, k);
        else nt ? launch_force<1, true>(ls, st, h->v, k) : launch_force<1, false>(ls, st, h->v, k);
    }
    if (Which == 1) {
        if (ls.group == 4) {
            if (nt) hipLaunchKernelGGL((k_spring_node<4, true>), ls.grid, ls.block, 0, st, h->v, k);
            else hipLaunchKernelGGL((k_spring_node<4, false>), ls.grid, ls.block, 0, st, h->v, k);
        } else if (ls.group == 2) {
            if (nt) hipLaunchKernelGGL((k_spring_node<2, true>), ls.grid, ls.block, 0, st, h->v, k);
            else hipLaunchKernelGGL((k_spring_node<2, false>), ls.grid, ls.block, 0, st, h->v, k);
        } else {
            if (nt) hipLaunchKernelGGL((k_spring_node<1, true>), ls.grid, ls.block, 0, st, h->v, k);
            else hipLaunchKernelGGL((k_spring_node<1, false>), ls.grid, ls.block, 0, st, h->v, k);
        }
    }
    if (Which == 2) {
        const LaunchShape l1 = method_shape(h, cls);
        hipLaunchKernelGGL(k_spring_link, l1.grid, l1.block, 0, st, h->v, k);
    }
    return launched("spring kernel");
}

// spring.steps on Spring: `steps` times spring.force and spring.node_update.
// In one launch where the mesh fits one work-group's passes and no snapshot
// taken ahead waits for one of the two do-alls.  The line lies where the
// registers of 16 wavefronts end, at 96 and 32 blocks: one launch is still the
// faster there (4.2 against 6.5 us a step, see k_spring_steps).  The blocks are
// the host's bounds, which deletions do not lower.
smmo_status run_spring_steps(smmo_heap *h, uint32_t cls, const void *args, hipStream_t st)
{
    smmo_spring_steps_args sa;
    memcpy(&sa, args, sizeof sa);
    const smmo_spring_args a{sa.node_class, sa.spring_class, sa.dt, sa.strain_limit, sa.flags};
    SpringK k;
    smmo_status s = cached_bind(h, (const void *)&run_spring_steps, cls, a, k, [&] { return bind_spring(h, a, k); });
    if (s) return s;
    if (cls != a.spring_class) return fail(SMMO_EINVAL, "spring: method runs on a different class");
    if (sa.steps == 0) return SMMO_OK;
    const uint64_t sb = h->ub_blocks[a.spring_class], nb = h->ub_blocks[a.node_class];
    const uint32_t both = 1u << a.spring_class | 1u << a.node_class;
    if (sa.steps > 1 && sb <= 96 && nb <= 32 && h->v.M <= kStepsMaxBlocks && !(h->snap_pending & both) &&
        !h->replayed[a.spring_class] && !h->replayed[a.node_class]) {
        if ((s = ensure_enumerated(h, a.spring_class, false, st, false, false))) return s;
        if ((s = ensure_enumerated(h, a.node_class, false, st, false, false))) return s;
        const bool captured = stream_captured(st);
        if (sb <= 48 && nb <= 16) launch_spring_steps<3, 1>(h, k, sa.steps, captured, st);
        else launch_spring_steps<6, 2>(h, k, sa.steps, captured, st);
        return launched("k_spring_steps");
    }
    // through the do-alls themselves, with their launch shapes and snapshots
    uint32_t force = 0, node = 0;
    if ((s = smmo_method_id("spring.force", &force)) || (s = smmo_method_id("spring.node_update", &node))) return s;
    for (uint32_t t = 0; t < sa.steps; ++t) {
        if ((s = smmo_parallel_do(h, a.spring_class, force, &a, sizeof a, st))) return s;
        if ((s = smmo_parallel_do(h, a.node_class, node, &a, sizeof a, st))) return s;
    }
    return SMMO_OK;
}

} // namespace

namespace smmo {
smmo_status launch_spring_steps(smmo_heap *h, uint32_t c, const void *a, hipStream_t s) { return run_spring_steps(h, c, a, s); }
smmo_status launch_spring_force(smmo_heap *h, uint32_t c, const void *a, hipStream_t s) { return launch_spring<0>(h, c, a, s); }
smmo_status launch_spring_node_update(smmo_heap *h, uint32_t c, const void *a, hipStream_t s) { return launch_spring<1>(h, c, a, s); }
smmo_status launch_spring_link(smmo_heap *h, uint32_t c, const void *a, hipStream_t s) { return launch_spring<2>(h, c, a, s); }
} // namespace smmo
