// Device helpers shared by the single-instance and batched phase loops.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace prot {

template <class T>
__device__ inline T ld_agent(const T *p)
{
    return __hip_atomic_load(const_cast<T *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ inline void st_agent(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ inline T add_agent(T *p, T v)
{
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The XCD this wave runs on (hardware register XCC_ID, id 20, all 32 bits).
constexpr uint32_t kXcds = 8;
__device__ inline uint32_t xcd_id()
{
    return (uint32_t)__builtin_amdgcn_s_getreg(20 | (31 << 11)) % kXcds;
}

// bit e set iff lo <= col0 + e < hi, for e in [0, 8)
__device__ inline uint32_t range_mask(int col0, int lo, int hi)
{
    const int s = lo - col0, t = hi - col0;
    uint32_t m = 0xFFu;
    if (s > 0) m = s >= 8 ? 0u : (m << s) & 0xFFu;
    if (t < 8) m = t <= 0 ? 0u : m & (0xFFu >> (8 - t));
    return m;
}

// bit e set iff k[e] + t[e] == need, i.e. k + 1 == y(a) + y(b) with
// y(a) = -t and need = y(b) - 1.
__device__ inline uint32_t match_mask(uint4 kv, uint4 tv, int need)
{
    const uint32_t kw[4] = {kv.x, kv.y, kv.z, kv.w};
    const uint32_t tw[4] = {tv.x, tv.y, tv.z, tv.w};
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k0 = (int)(int16_t)(kw[i] & 0xFFFFu), k1 = (int)(int16_t)(kw[i] >> 16);
        const int t0 = (int)(tw[i] & 0xFFFFu), t1 = (int)(tw[i] >> 16);
        m |= (uint32_t)(k0 + t0 == need) << (2 * i);
        m |= (uint32_t)(k1 + t1 == need) << (2 * i + 1);
    }
    return m;
}

// Smallest k[e] + t[e] over the elements e whose bit is set in mask (a large
// value if none).
__device__ inline int min_sum_masked(uint4 kv, uint4 tv, uint32_t mask)
{
    const uint32_t kw[4] = {kv.x, kv.y, kv.z, kv.w};
    const uint32_t tw[4] = {tv.x, tv.y, tv.z, tv.w};
    int m = 0x7FFFFFFF;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int s0 = (int)(int16_t)(kw[i] & 0xFFFFu) + (int)(tw[i] & 0xFFFFu);
        const int s1 = (int)(int16_t)(kw[i] >> 16) + (int)(tw[i] >> 16);
        if ((mask >> (2 * i)) & 1u) m = min(m, s0);
        if ((mask >> (2 * i + 1)) & 1u) m = min(m, s1);
    }
    return m;
}

__device__ inline uint32_t lanes_below(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Wave-wide reductions and scans on the cross-lane paths of the vector ALU
// (DPP), a few cycles a step where a shuffle through LDS takes tens.
template <int kCtrl, int kRows = 0xF>
__device__ inline uint32_t dpp_u32(uint32_t identity, uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, kCtrl, kRows, 0xF, false);
}
constexpr int kDppShr1 = 0x111, kDppShr2 = 0x112, kDppShr4 = 0x114, kDppShr8 = 0x118;
constexpr int kDppBcast15 = 0x142, kDppBcast31 = 0x143;
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141,
              kDppMirror = 0x140;

// lane i: v(0) + ... + v(i)
__device__ inline uint32_t wave_inclusive_sum_u32(uint32_t v)
{
    v += dpp_u32<kDppShr1>(0u, v);
    v += dpp_u32<kDppShr2>(0u, v);
    v += dpp_u32<kDppShr4>(0u, v);
    v += dpp_u32<kDppShr8>(0u, v);
    v += dpp_u32<kDppBcast15, 0xA>(0u, v);
    v += dpp_u32<kDppBcast31, 0xC>(0u, v);
    return v;
}
__device__ inline uint32_t wave_sum_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum_u32(v), 63);
}
__device__ inline uint32_t wave_min_u32(uint32_t v)
{
    v = min(v, dpp_u32<kDppShr1>(0xFFFFFFFFu, v));
    v = min(v, dpp_u32<kDppShr2>(0xFFFFFFFFu, v));
    v = min(v, dpp_u32<kDppShr4>(0xFFFFFFFFu, v));
    v = min(v, dpp_u32<kDppShr8>(0xFFFFFFFFu, v));
    v = min(v, dpp_u32<kDppBcast15, 0xA>(0xFFFFFFFFu, v));
    v = min(v, dpp_u32<kDppBcast31, 0xC>(0xFFFFFFFFu, v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
// minimum over each group of N = 8 or 16 lanes, in all of them
template <int N>
__device__ inline uint32_t group_min_u32(uint32_t v)
{
    static_assert(N == 8 || N == 16, "lanes of a group");
    v = min(v, dpp_u32<kDppXor1>(0xFFFFFFFFu, v));
    v = min(v, dpp_u32<kDppXor2>(0xFFFFFFFFu, v));
    v = min(v, dpp_u32<kDppHalfMirror>(0xFFFFFFFFu, v));
    if constexpr (N >= 16) v = min(v, dpp_u32<kDppMirror>(0xFFFFFFFFu, v));
    return v;
}

struct Hit {
    int j;  // scan position of the hit, -1 if the row is exhausted
    int a;  // its column
};

}  // namespace prot
