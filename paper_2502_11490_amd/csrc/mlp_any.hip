// Relevance metric of Sec. 3.1 (1), Eq. 5-8, on the matrix cores for layer widths of the caller's own, in the 16-bit
// formats and in fp32 (carried in fp64).
//
// A workgroup takes a batch of pairs of the dense pair list (Algorithm 2), lays x = concat(user, item) (Eq. 5) down in
// LDS and walks the layers over two LDS buffers (mlp_tile.h has the layers themselves).  Widths are rounded up to what
// the instruction takes (32 units and 32 inputs, fp32: 16 and 16) with weights of zero, so what a rounded-up unit
// holds is multiplied by zero; a unit that is NaN becomes zero in the ReLU, so this is exact for every finite weight.
//
// What bounds it: the weights, which a workgroup reads from L2 once per batch (hence as many pairs per batch as the
// LDS holds two or three times over), and for short lists the chain of trips to memory of one batch (hence
// small batches there, one per CU before any CU takes two).  Widths whose activations do not fit the LDS stay with the
// vector-ALU kernel.
//
// Measured against that kernel (which served all of these before): 100,003 bf16 pairs of 80 + 96 -> 192 -> 96 -> 2
// 5,509 -> 31 us (1.35 -> 240 TFLOP/s without the user's share of layer 1); one fp32 round of 64 queries, about
// 8,000 pairs of 64 -> 64 -> 3, 40 -> 7 us, so that a search with lists of 4,096 takes 7.9 instead of 16.5 ms.
#include <vector>

#include "mlp_tile.h"

namespace gmpgr {

constexpr int ANY_BLOCK = 256;
constexpr int ANY_WAVES = ANY_BLOCK / 64;

// Query and item of the batch's pairs, -1 where the pair is out of range or past the end.
__device__ __forceinline__ void tile_pairs(int32_t *row_q, int32_t *row_v, int P, int64_t row0, int64_t M, int64_t N,
                                           int32_t Q, const int32_t *__restrict__ pair_q,
                                           const int32_t *__restrict__ pair_id) {
    if ((int)threadIdx.x < P) {
        const int64_t row = row0 + threadIdx.x;
        int32_t q = row < M ? pair_q[row] : -1, v = row < M ? pair_id[row] : -1;
        if (q < 0 || q >= Q || v < 0 || (int64_t)v >= N) q = v = -1;
        row_q[threadIdx.x] = q;
        row_v[threadIdx.x] = v;
    }
}

// WIDE_LOADS: both tables have 16-byte aligned rows of whole 8-element pieces.
template <bool F16, int CB, bool WIDE_LOADS>
__global__ void __launch_bounds__(ANY_BLOCK)
mlp_any16_kernel(TileNet T, const uint4 *__restrict__ frag, const float *__restrict__ b,
                 const uint16_t *__restrict__ emb, int64_t N, const uint16_t *__restrict__ users, int32_t Q,
                 const int32_t *__restrict__ pair_q, const int32_t *__restrict__ pair_id,
                 const int32_t *__restrict__ M_dev, int64_t M_max, float *__restrict__ scores) {
    constexpr int P = 32 * CB;
    extern __shared__ __align__(16) uint4 lds[];
    uint4 *buf0 = lds, *buf1 = lds + (size_t)CB * T.slabs[0] * 64;
    int32_t *row_q = (int32_t *)(buf1 + (size_t)CB * T.slabs[1] * 64), *row_v = row_q + P;
    int64_t M = M_dev ? (int64_t)*M_dev : M_max;
    if (M > M_max) M = M_max;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5, col = lane & 31;
    const int n_in = T.d_user + T.d_item;
    for (int64_t row0 = (int64_t)blockIdx.x * P; row0 < M; row0 += (int64_t)gridDim.x * P) {
        tile_pairs(row_q, row_v, P, row0, M, N, Q, pair_q, pair_id);
        __syncthreads();
        for (int i = wave; i < CB * T.KS[0]; i += ANY_WAVES) {
            const int c = i % CB, s = i / CB, k0 = 16 * s + 8 * g;
            const int32_t q = row_q[c * 32 + col], v = row_v[c * 32 + col];
            uint4 x = make_uint4(0, 0, 0, 0);
            if (v >= 0) {
                const uint16_t *u = users + (size_t)q * T.d_user, *e = emb + (size_t)v * T.d_item;
                if (WIDE_LOADS) {
                    if (k0 < T.d_user) x = *(const uint4 *)(u + k0);
                    else if (k0 < n_in) x = *(const uint4 *)(e + (k0 - T.d_user));
                } else {
                    uint32_t h[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int k = k0 + j;
                        h[j] = k < T.d_user ? u[k] : k < n_in ? e[k - T.d_user] : 0;
                    }
                    x = make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
                }
            }
            buf0[((size_t)c * T.slabs[0] + s) * 64 + lane] = x;
        }
        __syncthreads();
        const int last = T.n_layers - 1;
        for (int l = 0; l < last; ++l) {
            tile_hidden<F16, false, CB>(frag, T.base[l], T.stride_n[l], T.step2[l], T.KS[l], T.NB[l], b + T.b_off[l],
                                        l & 1 ? buf1 : buf0, T.slabs[l & 1], l & 1 ? buf0 : buf1, T.slabs[1 - (l & 1)], ANY_WAVES);
            __syncthreads();
        }
        if (wave < CB) {  // heads: one block of units, one wave per 32 pairs
            f32x16 z[1];
#pragma unroll
            for (int i = 0; i < 16; ++i) z[0][i] = 0.f;
            const uint4 *in = (last & 1 ? buf1 : buf0) + (size_t)wave * T.slabs[last & 1] * 64;
            tile_contract<F16, 1>(z, frag + T.base[last] * 64 + lane, T.step2[last], T.KS[last], in, T.slabs[last & 1]);
            float part = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = 4 * g + i;
                if (j < T.J) part += T.head_w[j] * (1.0f / (1.0f + expf(-(z[0][i] + b[T.b_off[last] + j]))));
            }
            const float other = __shfl_xor(part, 32);
            const int64_t row = row0 + wave * 32 + col;
            if (g == 0 && row < M)
                scores[row] = row_v[wave * 32 + col] >= 0 ? part + other : __uint_as_float(0x7fc00000u);
        }
        __syncthreads();
    }
}

template <int CB>
__global__ void __launch_bounds__(ANY_BLOCK)
mlp_any64_kernel(TileNet T, const float4 *__restrict__ frag, const float *__restrict__ b, const float *__restrict__ emb,
                 int64_t N, const float *__restrict__ users, int32_t Q, const int32_t *__restrict__ pair_q,
                 const int32_t *__restrict__ pair_id, const int32_t *__restrict__ M_dev, int64_t M_max,
                 float *__restrict__ scores) {
    constexpr int P = 16 * CB;
    extern __shared__ __align__(16) uint4 lds[];
    f64x2 *buf0 = (f64x2 *)lds, *buf1 = buf0 + (size_t)CB * T.slabs[0] * 128;
    int32_t *row_q = (int32_t *)(buf1 + (size_t)CB * T.slabs[1] * 128), *row_v = row_q + P;
    int64_t M = M_dev ? (int64_t)*M_dev : M_max;
    if (M > M_max) M = M_max;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, col = lane & 15;
    for (int64_t row0 = (int64_t)blockIdx.x * P; row0 < M; row0 += (int64_t)gridDim.x * P) {
        tile_pairs(row_q, row_v, P, row0, M, N, Q, pair_q, pair_id);
        __syncthreads();
        for (int i = wave; i < CB * T.KS[0]; i += ANY_WAVES) {
            const int c = i % CB, s = i / CB;
            const int32_t q = row_q[c * 16 + col], v = row_v[c * 16 + col];
            f64x2 lo = {0.0, 0.0}, hi = {0.0, 0.0};
            if (v >= 0) {
                const float *u = users + (size_t)q * T.d_user, *e = emb + (size_t)v * T.d_item;
                float x[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = 16 * s + 4 * j + g;
                    x[j] = k < T.d_user ? u[k] : k < T.d_user + T.d_item ? e[k - T.d_user] : 0.f;
                }
                lo[0] = x[0], lo[1] = x[1], hi[0] = x[2], hi[1] = x[3];
            }
            f64x2 *to = buf0 + ((size_t)c * T.slabs[0] + s) * 128 + lane;
            to[0] = lo;
            to[64] = hi;
        }
        __syncthreads();
        const int last = T.n_layers - 1;
        for (int l = 0; l < last; ++l) {
            tile_hidden64<CB>(frag, T.base[l], T.KS[l], T.NB[l], b + T.b_off[l], l & 1 ? buf1 : buf0, T.slabs[l & 1],
                              l & 1 ? buf0 : buf1, T.slabs[1 - (l & 1)], ANY_WAVES);
            __syncthreads();
        }
        for (int c = wave; c < CB; c += ANY_WAVES) {
            f64x4 z[1] = {{0.0, 0.0, 0.0, 0.0}};
            tile_contract64<1>(z, frag + T.base[last] * 64 + lane, T.KS[last],
                               (last & 1 ? buf1 : buf0) + (size_t)c * T.slabs[last & 1] * 128, T.slabs[last & 1]);
            double part = 0.0;  // heads g and g + 4
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int j = g + 4 * i;
                if (j < T.J) part += (double)T.head_w[j] * (1.0 / (1.0 + exp(-(z[0][i] + (double)b[T.b_off[last] + j]))));
            }
            part += __shfl_xor(part, 16);
            part += __shfl_xor(part, 32);
            const int64_t row = row0 + c * 16 + col;
            if (g == 0 && row < M) scores[row] = row_v[c * 16 + col] >= 0 ? (float)part : __uint_as_float(0x7fc00000u);
        }
        __syncthreads();
    }
}

// LDS of a batch of `cb` column blocks
static size_t any_smem(const TileNet &T, bool f64, int cb) {
    return (size_t)cb * (T.slabs[0] + T.slabs[1]) * (f64 ? 2048 : 1024) + (size_t)cb * (f64 ? 16 : 32) * 8;
}
constexpr size_t ANY_LDS = 144 * 1024;

bool any_supported(const ann_mlp *m) { return m->any_dev != nullptr; }

// The weights in fragment order (see mlp_tile.h), the first layer's inputs as they are, the others' in the order in
// which the layer before leaves them.  Where the activations of the smallest batch do not fit the LDS nothing is built.
int build_any_fragments(ann_mlp *m, const void *const *W_host, hipStream_t stream) {
    TileNet &T = m->any;
    const bool f64 = m->dtype == ANN_F32;
    T.n_layers = m->n_layers;
    T.J = m->J;
    T.d_user = m->d_user;
    T.d_item = m->d_item;
    for (int j = 0; j < m->J; ++j) T.head_w[j] = m->head_w[j];
    int64_t n_frag = 0;
    for (int l = 0; l < m->n_layers; ++l) {
        const int unit = f64 ? 16 : 32;
        T.KS[l] = (m->dims[l] + unit - 1) / unit * (unit / 16);
        T.NB[l] = (m->dims[l + 1] + unit - 1) / unit;
        T.stride_n[l] = T.KS[l];
        T.step2[l] = 2;
        T.b_off[l] = m->b_off[l];
        T.base[l] = n_frag;
        n_frag += (int64_t)T.KS[l] * T.NB[l];
        if (T.KS[l] > T.slabs[l & 1]) T.slabs[l & 1] = T.KS[l];
    }
    if (any_smem(T, f64, 1) > ANY_LDS) return ANN_OK;
    std::vector<uint32_t> buf((size_t)n_frag * 256, 0);  // 1 KB per fragment
    for (int l = 0; l < m->n_layers; ++l) {
        const int n_in = m->dims[l], n_out = m->dims[l + 1];
        for (int nb = 0; nb < T.NB[l]; ++nb)
            for (int k = 0; k < T.KS[l]; ++k) {
                const size_t fr = (size_t)(T.base[l] + (int64_t)nb * T.KS[l] + k);
                for (int lane = 0; lane < 64; ++lane)
                    for (int j = 0; j < (f64 ? 4 : 8); ++j) {
                        const int o = f64 ? nb * 16 + (lane & 15) : nb * 32 + (lane & 31);
                        const int i = f64 ? 16 * k + 4 * j + (lane >> 4)
                                      : l == 0 ? 16 * k + 8 * (lane >> 5) + j
                                               : 16 * k + 8 * (j / 4) + 4 * (lane >> 5) + j % 4;
                        if (o >= n_out || i >= n_in) continue;
                        const size_t at = (size_t)o * n_in + i;
                        if (f64) ((float *)buf.data())[fr * 256 + lane * 4 + j] = ((const float *)W_host[l])[at];
                        else ((uint16_t *)buf.data())[fr * 512 + lane * 8 + j] = ((const uint16_t *)W_host[l])[at];
                    }
            }
    }
    ANN_HIP_TRY(hipMalloc(&m->any_dev, buf.size() * 4));
    ANN_HIP_TRY(hipMemcpyAsync(m->any_dev, buf.data(), buf.size() * 4, hipMemcpyHostToDevice, stream));
    ANN_HIP_TRY(hipStreamSynchronize(stream));  // buf is freed on return
    return ANN_OK;
}

int launch_mlp_any(const ann_graph *g, const ann_mlp *m, const void *queries, const int32_t *pair_q,
                   const int32_t *pair_id, const int32_t *M_dev, int64_t M_max, int32_t Q, float *scores,
                   int32_t tile_rows, hipStream_t stream) {
    if (M_max <= 0) return ANN_OK;
    const TileNet &T = m->any;
    const bool f64 = m->dtype == ANN_F32;
    const int unit = f64 ? 16 : 32;
    // Pairs per batch: as many as leave room for two workgroups on a CU, fewer while a CU would stay idle.  The caller's
    // own number is a limit instead, down to one block of columns (and the LDS one upwards).
    int cb = f64 ? 4 : 2;
    if (tile_rows > 0)
        while (cb > 1 && (any_smem(T, f64, cb) > ANY_LDS || unit * cb > tile_rows)) cb >>= 1;
    else
        while (cb > 1 && (any_smem(T, f64, cb) > 80 * 1024 || (M_max + unit * cb - 1) / (unit * cb) < 512)) cb >>= 1;
    const size_t smem = any_smem(T, f64, cb);
    const int64_t tiles = (M_max + unit * cb - 1) / (unit * cb);
    const int grid = (int)(tiles < 1024 ? tiles : 1024);
    if (f64) {
        auto fn = cb == 4 ? mlp_any64_kernel<4> : cb == 2 ? mlp_any64_kernel<2> : mlp_any64_kernel<1>;
        static std::atomic<uint32_t> raised[3];
        if (int rc = raise_lds_limit((const void *)fn, ANY_LDS, m->device, raised[cb >> 1]); rc != ANN_OK) return rc;
        hipLaunchKernelGGL(fn, dim3(grid), dim3(ANY_BLOCK), smem, stream, T, (const float4 *)m->any_dev, m->b_dev,
                           (const float *)g->emb, g->N, (const float *)queries, Q, pair_q, pair_id, M_dev, M_max, scores);
    } else {
        const bool f16 = m->dtype == ANN_F16;
        const bool wide = ((T.d_user | T.d_item) & 7) == 0 && (((uintptr_t)queries | (uintptr_t)g->emb) & 15) == 0;
        using Fn = decltype(&mlp_any16_kernel<false, 1, false>);
        static const Fn fns[8] = {mlp_any16_kernel<false, 1, false>, mlp_any16_kernel<false, 1, true>,
                                  mlp_any16_kernel<false, 2, false>, mlp_any16_kernel<false, 2, true>,
                                  mlp_any16_kernel<true, 1, false>,  mlp_any16_kernel<true, 1, true>,
                                  mlp_any16_kernel<true, 2, false>,  mlp_any16_kernel<true, 2, true>};
        const int which = (f16 ? 4 : 0) + (cb == 2 ? 2 : 0) + (wide ? 1 : 0);
        static std::atomic<uint32_t> raised[8];
        if (int rc = raise_lds_limit((const void *)fns[which], ANY_LDS, m->device, raised[which]); rc != ANN_OK) return rc;
        hipLaunchKernelGGL(fns[which], dim3(grid), dim3(ANY_BLOCK), smem, stream, T, (const uint4 *)m->any_dev, m->b_dev,
                           (const uint16_t *)g->emb, g->N, (const uint16_t *)queries, Q, pair_q, pair_id, M_dev, M_max,
                           scores);
    }
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

}  // namespace gmpgr
