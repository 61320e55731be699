// What csrc/smmo_device.hpp needs of HIP, for a host compiler and a wavefront
// of one lane.
#pragma once
#include <algorithm>
#include <cstdint>

#define __host__
#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0

struct Dim3 { uint32_t x = 1, y = 1, z = 1; };
static Dim3 blockDim;
static struct { uint32_t x = 0; } threadIdx, blockIdx;

template <class T, class V> T __hip_atomic_fetch_or(T *p, V v, int, int) { T o = *p; *p = o | (T)v; return o; }
template <class T, class V> T __hip_atomic_fetch_and(T *p, V v, int, int) { T o = *p; *p = o & (T)v; return o; }
template <class T, class V> T __hip_atomic_fetch_add(T *p, V v, int, int) { T o = *p; *p = o + (T)v; return o; }
template <class T> T __hip_atomic_load(const T *p, int, int) { return *p; }
template <class T, class V> void __hip_atomic_store(T *p, V v, int, int) { *p = (T)v; }

inline uint32_t __lane_id() { return 0; }
inline uint64_t __ballot(bool b) { return b ? 1 : 0; }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline int __ffsll(unsigned long long v) { return __builtin_ffsll((long long)v); }
inline int __clzll(long long v) { return v ? __builtin_clzll((unsigned long long)v) : 64; }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
inline int __shfl_xor(int v, int) { return v; }
inline uint32_t amdgcn_same(uint32_t v) { return v; }
inline uint32_t amdgcn_lane(uint32_t v, uint32_t) { return v; }
#define __builtin_amdgcn_readfirstlane amdgcn_same
#define __builtin_amdgcn_readlane amdgcn_lane
#define __builtin_amdgcn_ds_permute(to, v) (v)
#define __builtin_amdgcn_ds_bpermute(from, v) (v)
#define __builtin_amdgcn_s_sleep(n) ((void)0)
#define __builtin_amdgcn_s_waitcnt(n) ((void)0)
