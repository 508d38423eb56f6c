// Small helpers shared by the selection kernels (gfx950, wave64).
#pragma once
#include <hip/hip_ext.h>

#include "lgc_internal.h"

namespace lgc {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
// 16-byte accesses at any 4-byte address (the hardware takes them)
typedef f4 f4u __attribute__((aligned(4)));
typedef u4 u4u __attribute__((aligned(4)));

// ------------------------------------------------------------------ small helpers

__device__ __forceinline__ uint32_t key_of(float x) { return __float_as_uint(x) & 0x7fffffffu; }

__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Inclusive prefix sum over the lanes of a wavefront, register to register (DPP: four shifts inside rows of 16 lanes,
// two row broadcasts).  All 64 lanes must be active.  A shuffle through the LDS unit costs some 60 cycles a step.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t x) {
    x += __builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0u, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0u, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return x;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t x) { return __builtin_amdgcn_readlane(wave_prefix(x), 63); }

__device__ __forceinline__ unsigned long long ld_agent(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(unsigned long long *p, unsigned long long x) {
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_agent32(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void st_agent32(uint32_t *p, uint32_t x) {
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t mix32(uint32_t h) {
    h *= 0x9E3779B1u; h ^= h >> 15; h *= 0x85EBCA77u; h ^= h >> 13; h *= 0xC2B2AE3Du; h ^= h >> 16;
    return h;
}

// First element of the j-th group of 4 sampled neighbours.  Four groups make one 64-byte cluster of 16 elements; the clusters sit at
// jittered positions, one in each of kSampleGroups / 4 strata of the vector: stratum cl = clusters [cl * C / 4096, (cl + 1) * C / 4096) of
// the vector's C = n / 16 whole clusters (n >= kMinFastN makes none of them empty).
__device__ __forceinline__ uint32_t sample_place(const uint32_t j, const int node, const uint32_t n) {
    static_assert(kSampleGroups / 4 == 4096 && kMinFastN >= 16 * 4096, "4096 strata of at least one cluster");
    const uint32_t cl = j >> 2, clusters = n >> 4;
    const uint32_t s_lo = (uint32_t)(((unsigned long long)cl * clusters) >> 12);
    const uint32_t s_hi = (uint32_t)(((unsigned long long)(cl + 1) * clusters) >> 12);
    return ((s_lo + mix32(cl + 0x5bd1e995u * (uint32_t)node) % (s_hi - s_lo)) << 4) + ((j & 3u) << 2);
}

// accumulation step: three separately rounded fp32 operations, never contracted
__device__ __forceinline__ void accum1(float g, float &u, float &v, float m) {
    u = __fadd_rn(__fmul_rn(m, u), g);
    v = __fadd_rn(v, u);
}

// Block-wide search in a histogram held in LDS (16-byte aligned): finds the bin b such that
// count(bins > b) < rank <= count(bins >= b).  Every one of the T threads owns NB / T consecutive bins and reads them
// once, in 16-byte pieces (4-byte reads NB / T words apart meet in a few banks: 0.9 us for 8192 bins).
// Result through LDS: res[0] = b (or 0xffffffff if the histogram holds fewer than rank), res[1] =
// count(bins > b).  All threads must call; contains barriers.
template <int NB, int T>
__device__ __forceinline__ void find_rank_bin(const uint32_t *hist, uint32_t rank, uint32_t *wave_tmp, uint32_t *res) {
    constexpr int kPer = NB / T, kWavesHere = T / 64;
    static_assert(NB % T == 0 && kWavesHere <= 64, "bins per thread");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t h[kPer], part = 0;
    if constexpr (kPer % 4 == 0) {
#pragma unroll
        for (int i = 0; i < kPer / 4; ++i) {
            const u4 x = ((const u4 *)hist)[tid * (kPer / 4) + i];
#pragma unroll
            for (int c = 0; c < 4; ++c) h[4 * i + c] = x[c];
        }
    } else {
#pragma unroll
        for (int i = 0; i < kPer; ++i) h[i] = hist[tid * kPer + i];
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) part += h[i];
    const uint32_t incl = wave_prefix(part), all = __builtin_amdgcn_readlane(incl, 63);
    if (tid == 0) { res[0] = 0xffffffffu; res[1] = 0; }
    if (lane == 0) wave_tmp[wave] = all;
    __syncthreads();
    const uint32_t other = lane < kWavesHere ? wave_tmp[lane] : 0u;
    uint32_t acc = all - incl + wave_sum(lane > wave ? other : 0u);   // in the bins above this thread's
    if (acc < rank && rank <= acc + part) {
#pragma unroll
        for (int i = kPer - 1; i >= 0; --i) {
            const bool here = acc < rank && rank <= acc + h[i];
            if (here) { res[0] = tid * kPer + i; res[1] = acc; }
            acc += h[i];
        }
    }
    __syncthreads();
}

// Exclusive prefix sum over a block of 1024 threads; `total` receives the sum.  tmp: 16 words.
__device__ __forceinline__ uint32_t block_scan(const uint32_t x, uint32_t *tmp, uint32_t &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t incl = wave_prefix(x);
    __syncthreads();
    if (lane == 63) tmp[wave] = incl;
    __syncthreads();
    const uint32_t t = lane < 16 ? tmp[lane] : 0u;   // the wavefronts' sums go over the lanes
    total = wave_sum(t);
    return incl - x + wave_sum(lane < wave ? t : 0u);
}

// Candidates per kGroupRows rows of a node, in long vectors.  They lie where the exact path keeps its runs' counts: by the
// time a node falls back the gather has read them, and each 4096 elements have two words there.
__device__ __forceinline__ uint32_t *group_counts(const SelArgs &a, const int node) {
    return (uint32_t *)(a.status_exact + (size_t)node * a.status_exact_stride);
}

// An ordinary launch, or, with timing events, the launch form that stamps them itself.
template <typename K, typename... Args>
static void launch_timed(K kernel, dim3 grid, dim3 block, hipStream_t st, Bracket e, Args... args) {
    if (e.start || e.stop) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, e.start, e.stop, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
}

}  // namespace lgc
