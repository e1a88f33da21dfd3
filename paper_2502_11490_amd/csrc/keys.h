// Sorted 64-bit keys shared by the search kernels and the exhaustive search: the order-preserving key of a
// (relevance, id) pair, an LDS bitonic sort and a binary search.
#pragma once

#include "common.h"

namespace gmpgr {

// ---- order-preserving key: ascending uint64 == (score descending, id ascending) ----------
__device__ __forceinline__ uint64_t make_key(float score, int32_t id, uint32_t expanded) {
    uint32_t f = __float_as_uint(score);
    uint32_t asc = (f & 0x80000000u) ? ~f : (f | 0x80000000u);
    return ((uint64_t)(~asc) << 32) | ((uint64_t)(uint32_t)id << 1) | expanded;
}
__device__ __forceinline__ float key_score(uint64_t key) {
    uint32_t asc = ~(uint32_t)(key >> 32);
    uint32_t f = (asc & 0x80000000u) ? (asc ^ 0x80000000u) : ~asc;
    return __uint_as_float(f);
}
__device__ __forceinline__ int32_t key_id(uint64_t key) { return (int32_t)((uint32_t)key >> 1); }
__device__ __forceinline__ uint32_t key_expanded(uint64_t key) { return (uint32_t)key & 1u; }

// Ascending bitonic sort of keys[0..n) in LDS, n a power of two.  Thread t owns the t-th
// compare-exchange of every step (and t + BLOCK, ...): for strides up to 64 the 64 threads of a
// wave then touch one and the same 128-key segment step after step, so those steps need no
// workgroup barrier, only the wave's own program order (LDS executes a wave's operations in
// order); a barrier is needed around the steps with larger strides and at the end.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int BLK>
__device__ void bitonic_sort(uint64_t *keys, int n) {
    for (int k = 2; k <= n; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const bool across_waves = j > 64;
            if (across_waves) __syncthreads();
            for (int t = threadIdx.x; t < (n >> 1); t += BLK) {
                // t-th compare-exchange of this step: indices i < ixj
                int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                int ixj = i | j;
                bool up = ((i & k) == 0);
                uint64_t a = keys[i], b = keys[ixj];
                if ((a > b) == up) {
                    keys[i] = b;
                    keys[ixj] = a;
                }
            }
            if (across_waves) __syncthreads();
            else wave_lds_fence();
        }
    }
    __syncthreads();
}

// c0 += (a < k) + (c < k), c1 += (b < k) + (d < k), the two halves of a key in the words of a 16-byte piece.  Three full-rate
// instructions a comparison, where one on 64 bits is slow, and four carries at a time, so that none is waited for.
__device__ __forceinline__ void count_less4(uint32_t &c0, uint32_t &c1, const uint4 &ab, const uint4 &cd, uint64_t k) {
    uint32_t t0, t1, t2, t3;
    uint64_t v0, v1, v2, v3;
    asm("v_sub_co_u32 %2, %6, %10, %18\n\tv_sub_co_u32 %3, %7, %12, %18\n\t"
        "v_sub_co_u32 %4, %8, %14, %18\n\tv_sub_co_u32 %5, %9, %16, %18\n\t"
        "v_subb_co_u32 %2, %6, %11, %19, %6\n\tv_subb_co_u32 %3, %7, %13, %19, %7\n\t"
        "v_subb_co_u32 %4, %8, %15, %19, %8\n\tv_subb_co_u32 %5, %9, %17, %19, %9\n\t"
        "v_addc_co_u32 %0, %6, 0, %0, %6\n\tv_addc_co_u32 %1, %7, 0, %1, %7\n\t"
        "v_addc_co_u32 %0, %8, 0, %0, %8\n\tv_addc_co_u32 %1, %9, 0, %1, %9"
        : "+v"(c0), "+v"(c1), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3), "=&s"(v0), "=&s"(v1), "=&s"(v2), "=&s"(v3)
        : "v"(ab.x), "v"(ab.y), "v"(ab.z), "v"(ab.w), "v"(cd.x), "v"(cd.y), "v"(cd.z), "v"(cd.w), "v"((uint32_t)k),
          "v"((uint32_t)(k >> 32)));
}

// smaller[u] = how many of keys[0..n) are below key[u].  The keys are read as LDS broadcasts, eight at a time and eight ahead of
// their use.  keys: LDS, 16-byte aligned, sentinels behind it up to a multiple of eight, room for eight more to be read.
template <int PER>
__device__ __forceinline__ void count_smaller(const uint64_t *keys, int n, const uint64_t (&key)[PER], uint32_t (&smaller)[PER]) {
    const uint4 *k = (const uint4 *)keys;
    uint4 a[4];
    uint32_t odd[PER];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = k[i];
#pragma unroll
    for (int u = 0; u < PER; ++u) smaller[u] = odd[u] = 0;
#pragma unroll 1
    for (int c = 0; c < n; c += 8) {
        uint4 ahead[4];
        k += 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) ahead[i] = k[i];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            count_less4(smaller[u], odd[u], a[0], a[1], key[u]);
            count_less4(smaller[u], odd[u], a[2], a[3], key[u]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = ahead[i];
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) smaller[u] += odd[u];
}
constexpr int KEYS_SLACK = 16;  // keys behind the last one that count_smaller may read

// First index of the ascending a[0..n) whose key is not below `key`.
__device__ __forceinline__ int lower_bound_keys(const uint64_t *a, int n, uint64_t key) {
    int lo = 0, hi = n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (a[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

}  // namespace gmpgr
