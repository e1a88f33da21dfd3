// The relevance metric of Eq. 5-8 on the matrix cores for a tile of pairs whose activations lie in LDS: device
// code shared by the kernels for layer widths of the caller's own (mlp_any.hip) and by the search kernel that
// scores a query's candidates itself (search_fused.hip).
//
// All waves of a workgroup work on the same tile: a wave takes blocks of output units, reads the weights of a block
// from L2 in the order its lanes need them (1 KB a fragment, the next ones requested while one is used) and the
// activations from LDS, and leaves its block's activations in LDS in the order in which the next layer reads them,
// so that every LDS access is 16 bytes per lane without bank conflicts.
//
// 16-bit formats: v_mfma_f32_32x32x16, transposed as in mlp_mfma.hip (weights are the A operand, 32 units x 16
// inputs; activations the B operand, 16 inputs x 32 pairs).  A slab of activations is one B operand: 16 inputs x
// 32 pairs, lane l's 16 bytes at 16 l.  fp32 accumulation from the bias (or the query's share of layer 1), hidden
// units rounded to the format after the ReLU.
// fp32: everything is carried in fp64 by v_mfma_f64_16x16x4 (weights and inputs widened, exact), as the
// vector-ALU kernel carries it; one rounding at the end.  A slab is 16 inputs x 16 pairs of fp64 (2 KB).
#pragma once

#include "common.h"

namespace gmpgr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------- 16-bit formats
template <bool F16>
__device__ __forceinline__ f32x16 tile_mfma(const uint4 &a, const uint4 &b, const f32x16 &acc) {
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// ReLU and rounding (nearest even) of half a block of hidden units.  The integer maximum is the ReLU of the rounded
// value: it keeps a NaN with a clear sign bit, as the kernel for the widest metric does; otherwise NaN gives 0.
template <bool F16, bool INT_RELU>
__device__ __forceinline__ uint4 tile_relu(const f32x16 &acc, int half) {
    f32x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = INT_RELU ? acc[half * 8 + j] : relu_f32(acc[half * 8 + j]);
    s16x8 r;
    if constexpr (F16) r = __builtin_bit_cast(s16x8, __builtin_convertvector(v, f16x8));
    else r = __builtin_bit_cast(s16x8, __builtin_convertvector(v, bf16x8));
    if (INT_RELU) r = __builtin_elementwise_max(r, (s16x8)(short)0);
    return __builtin_bit_cast(uint4, r);
}

// acc[c] += W-block * slabs of column block c, over KS inputs-of-16.  `w` points at this lane's 16 bytes of the
// block's first fragment; fragment k lies (k >> 1) * step2 + (k & 1) fragments behind it (KS is even).
template <bool F16, int CB>
__device__ __forceinline__ void tile_contract(f32x16 (&acc)[CB], const uint4 *__restrict__ w, int step2, int KS,
                                              const uint4 *in, int in_slabs) {
    const int lane = threadIdx.x & 63;
    constexpr int DEPTH = 4;  // fragments in flight; 8 lost more by their registers than they hid (1,024 queries 6.1 -> 8.5 ms)
    uint4 a[DEPTH];
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
        const int k = u < KS ? u : KS - 1;
        a[u] = w[((size_t)(k >> 1) * step2 + (k & 1)) * 64];
    }
    int k0 = 0;
    for (; k0 + DEPTH < KS; k0 += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[c] = tile_mfma<F16>(a[u], in[((size_t)c * in_slabs + k0 + u) * 64 + lane], acc[c]);
            const int k = k0 + DEPTH + u < KS ? k0 + DEPTH + u : KS - 1;  // past the end: one that nobody uses
            a[u] = w[((size_t)(k >> 1) * step2 + (k & 1)) * 64];
        }
    }
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
        if (u >= 2 && k0 + u >= KS) break;  // KS is even and at least 2
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[c] = tile_mfma<F16>(a[u], in[((size_t)c * in_slabs + k0 + u) * 64 + lane], acc[c]);
    }
}

// A hidden layer of the tile: NB blocks of 32 units over the workgroup's waves.  init[unit]: what a unit's sum starts
// from.  out: 2 NB slabs per column block, unit 32 nb + 16 s2 + 8 (j / 4) + 4 g + j % 4 at byte j of lane (m, g) of
// slab 2 nb + s2 (the D layout of the instruction as it comes; the next layer's weights are stored to match).
template <bool F16, bool INT_RELU, int CB>
__device__ __forceinline__ void tile_hidden(const uint4 *__restrict__ frag, int64_t base, int stride_n, int step2, int KS,
                                            int NB, const float *init, const uint4 *in, int in_slabs, uint4 *out,
                                            int out_slabs, int n_waves) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5;
    for (int nb = wave; nb < NB; nb += n_waves) {
        f32x16 acc[CB];
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
            const f32x4 v = *(const f32x4 *)(init + nb * 32 + 8 * t4 + 4 * g);
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[c][4 * t4 + e] = v[e];
        }
        tile_contract<F16, CB>(acc, frag + (base + (int64_t)nb * stride_n) * 64 + lane, step2, KS, in, in_slabs);
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            out[((size_t)c * out_slabs + 2 * nb) * 64 + lane] = tile_relu<F16, INT_RELU>(acc[c], 0);
            out[((size_t)c * out_slabs + 2 * nb + 1) * 64 + lane] = tile_relu<F16, INT_RELU>(acc[c], 1);
        }
    }
}

// ---------------------------------------------------------------------------------------- fp32 carried in fp64
// acc[c] += W-block (16 units) * slabs of column block c (16 pairs), KS inputs-of-16.  w: this lane's four weights of
// the block's first fragment (unit lane % 16, inputs 16 k + 4 u + lane / 16); fragments follow one another.
template <int CB>
__device__ __forceinline__ void tile_contract64(f64x4 (&acc)[CB], const float4 *w, int KS, const f64x2 *in,
                                                int in_slabs) {
    const int lane = threadIdx.x & 63;
    float4 a = w[0];
    for (int k = 0; k < KS; ++k) {
        const float4 n = w[(size_t)(k + 1 < KS ? k + 1 : k) * 64];
        const double a0 = a.x, a1 = a.y, a2 = a.z, a3 = a.w;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const f64x2 *s = in + ((size_t)c * in_slabs + k) * 128 + lane;
            const f64x2 b0 = s[0], b1 = s[64];
            acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0[0], acc[c], 0, 0, 0);
            acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0[1], acc[c], 0, 0, 0);
            acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2, b1[0], acc[c], 0, 0, 0);
            acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a3, b1[1], acc[c], 0, 0, 0);
        }
        a = n;
    }
}

// A block of 16 units of a hidden layer for CB column blocks.  A lane's four results (units lane / 16 + 4 i of its pair) are
// its four operands of the next layer's fragment.  `in`, `out`: the first of the column blocks.
template <int CB>
__device__ __forceinline__ void tile_block64(const float4 *w, int KS, int nb, const float *bias, const f64x2 *in, int in_slabs,
                                             f64x2 *out, int out_slabs) {
    const int lane = threadIdx.x & 63, g = lane >> 4;
    f64x4 acc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[c][i] = (double)bias[nb * 16 + g + 4 * i];
    tile_contract64<CB>(acc, w, KS, in, in_slabs);
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        f64x2 lo, hi;
        lo[0] = acc[c][0] > 0.0 ? acc[c][0] : 0.0;
        lo[1] = acc[c][1] > 0.0 ? acc[c][1] : 0.0;
        hi[0] = acc[c][2] > 0.0 ? acc[c][2] : 0.0;
        hi[1] = acc[c][3] > 0.0 ? acc[c][3] : 0.0;
        f64x2 *s = out + ((size_t)c * out_slabs + nb) * 128 + lane;
        s[0] = lo;
        s[64] = hi;
    }
}

// A hidden layer: NB blocks of 16 units over the workgroup's waves.
template <int CB>
__device__ __forceinline__ void tile_hidden64(const float4 *__restrict__ frag, int64_t base, int KS, int NB,
                                              const float *__restrict__ bias, const f64x2 *in, int in_slabs, f64x2 *out,
                                              int out_slabs, int n_waves) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int nb = wave; nb < NB; nb += n_waves)
        tile_block64<CB>(frag + (base + (int64_t)nb * KS) * 64 + lane, KS, nb, bias, in, in_slabs, out, out_slabs);
}

}  // namespace gmpgr
