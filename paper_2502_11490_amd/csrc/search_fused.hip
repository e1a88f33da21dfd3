// A whole search in one launch: one workgroup per query runs every round of the joint best-first search (Sec. 3.2,
// Algorithm 1), scoring included, without going back to the host or to another workgroup.
//
// The batch path spends three dependent launches per round, which is right while a round's pairs fill the chip
// with matrix work.  A small batch does not: its rounds are chains of trips to memory, launch turn-overs and (for the
// kernels that keep all weights in LDS) a reload of the weights.  Here the list, the survivors and their scores stay
// in LDS from the first round to the last, the user's share of layer 1 is the same for all pairs of the workgroup,
// the weights come from L2 in fragment order (mlp_tile.h), and queries do not wait for one another.
//
// Up to 256 queries, where a workgroup has its CU to itself, what a round waits for is kept closer still: the weights of the
// metrics of 64-wide items in the registers of eight waves (HeldNet), a small metric of the caller's own widths in LDS, the
// visited set in LDS too while it is short or the table small.
//
// What bounds it: the chain of a round, some 20,000 clocks for one query of a million items (gather and visited set 20 %,
// scoring 42, new keys and their sort 15, the merge 14, the choice of parents 8): trips to the L2 and the LDS, barriers and
// the instructions between them, one after the other.  For the widest metric scoring is 77 %: its weights come from L2.
//
// Measured against the batch path of its time: one query on a million items (lists of 64) 0.88 -> 0.46 ms, 64 fp32 queries
// with lists of 32 and 4,096 0.78 -> 0.33 and 7.9 -> 4.2 ms.  Each part that came closer, without it -> with it, us: weights in registers
// 385 -> 275 (64 queries, lists of 256, two layers 1,741 -> 1,220; 256, W = 8, lists of 512 2,213 -> 1,448); a small metric in LDS
// 340 -> 312 (64 fp32 queries, lists of 32; 16 with lists of 512 1,765 -> 1,620); the visited set in LDS 295 -> 275 and 327 -> 312 (the same
// for lists of 256 and more); the merge of short lists by binary search 300 -> 275 (1,394 -> 1,220, 1,574 -> 1,448).
//
// A pair's relevance is computed in the order of the batch path's kernels (same fragments, same sequence of MFMAs,
// same start values), so which path serves a call does not show in its results.
#include "mlp_tile.h"
#include "search_device.h"

namespace gmpgr {

struct FusedArgs {
    TileNet T;
    const void *frag;
    const float *b, *upre;      // upre: the users' shares of layer 1 [Q][H1], null = layer 1 contracts the user too
    const void *emb, *users;
    const int32_t *adj, *adj_rank, *rank, *entries;
    const int32_t *W_q, *L_q, *cap_q;
    uint32_t *table;
    int64_t *stats;
    Ctrl *ctrl;
    int32_t *out_ids;
    float *out_scores;
    uint64_t *mailbox;
    uint64_t mail_tag;
    // searches that the batch path began (resume): their state, list and survivors not yet scored
    QState *state;
    uint64_t *pool;
    int32_t *counts;
    const int32_t *cand, *slot_query;
    const int32_t *handed;      // searches that waves began: their numbers, ctrl->handed of them; results are written here
    int64_t N;
    int32_t seen_words, seen_bits;   // visited set in LDS (0: in memory): one bit per item, or slots of one id
    int32_t frag_words, bias_words;  // a metric kept in LDS, 0 = read from L2
    int32_t R, E, W, L, cap, W_max, L_max, cap_max, C, k, slots, new_cap, table_words, hash_cap, Q, rounds_max;
    int32_t wide_loads, int_relu;
};

// FUSED_TWO, FUSED_ONE (+ 1: fp16): 64 -> 256 (-> 128) with the weights in the registers of eight waves
enum { FUSED_F64 = 0, FUSED_BF16 = 1, FUSED_F16 = 2, FUSED_TWO = 3, FUSED_ONE = 5 };

// Relevances of the query's pairs surv[0..n) as list keys to keys[0..n).  All threads call; ends with a barrier.
template <int BLK, bool F16, int CB>
__device__ __forceinline__ void fused_score16(const FusedArgs &A, const uint4 *frag, const float *b, int q, const int32_t *surv,
                                              uint64_t *keys, int n, uint4 *buf0) {
    constexpr int P = 32 * CB, NW = BLK / 64;
    const TileNet &T = A.T;
    uint4 *buf1 = buf0 + (size_t)CB * T.slabs[0] * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5, col = lane & 31;
    const float *upre = A.upre ? A.upre + (size_t)q * (32 * T.NB[0]) : nullptr;
    const int n_user = A.upre ? 0 : T.d_user, n_in = n_user + T.d_item, last = T.n_layers - 1;
    const uint16_t *u = (const uint16_t *)A.users + (size_t)q * T.d_user;
    for (int base = 0; base < n; base += P) {
        for (int i = wave; i < CB * T.KS[0]; i += NW) {
            const int c = i % CB, s = i / CB, k0 = 16 * s + 8 * g, row = base + c * 32 + col;
            uint4 x = make_uint4(0, 0, 0, 0);
            if (row < n) {
                const uint16_t *e = (const uint16_t *)A.emb + (size_t)surv[row] * T.d_item;
                if (A.wide_loads) {
                    if (k0 < n_user) x = *(const uint4 *)(u + k0);
                    else if (k0 < n_in) x = *(const uint4 *)(e + (k0 - n_user));
                } else {
                    uint32_t h[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int kk = k0 + j;
                        h[j] = kk < n_user ? u[kk] : kk < n_in ? e[kk - n_user] : 0;
                    }
                    x = make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
                }
            }
            buf0[((size_t)c * T.slabs[0] + s) * 64 + lane] = x;
        }
        __syncthreads();
        for (int l = 0; l < last; ++l) {
            const float *init = l == 0 && upre ? upre : b + T.b_off[l];
            uint4 *in = l & 1 ? buf1 : buf0, *out = l & 1 ? buf0 : buf1;
            if (A.int_relu)
                tile_hidden<F16, true, CB>(frag, T.base[l], T.stride_n[l], T.step2[l], T.KS[l], T.NB[l], init, in,
                                           T.slabs[l & 1], out, T.slabs[1 - (l & 1)], NW);
            else
                tile_hidden<F16, false, CB>(frag, T.base[l], T.stride_n[l], T.step2[l], T.KS[l], T.NB[l], init, in,
                                            T.slabs[l & 1], out, T.slabs[1 - (l & 1)], NW);
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
                const float bias = j < T.J ? b[T.b_off[last] + j] : 0.f, w = j < T.J ? T.head_w[j] : 0.f;
                if (upre) part = fmaf(w, sigmoid_hw(z[0][i] + bias), part);
                else if (j < T.J) part += w * (1.0f / (1.0f + expf(-(z[0][i] + bias))));
            }
            const float other = __shfl_xor(part, 32);
            const int row = base + wave * 32 + col;
            if (g == 0 && row < n) keys[row] = make_key(part + other, surv[row], 0u);
        }
        __syncthreads();
    }
}

template <int BLK, int CB>
__device__ __forceinline__ void fused_score64(const FusedArgs &A, const float4 *frag, const float *b, int q, const int32_t *surv,
                                              uint64_t *keys, int n, f64x2 *buf0) {
    constexpr int P = 16 * CB, NW = BLK / 64;
    const TileNet &T = A.T;
    f64x2 *buf1 = buf0 + (size_t)CB * T.slabs[0] * 128;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, col = lane & 15, last = T.n_layers - 1;
    const float *u = (const float *)A.users + (size_t)q * T.d_user;
    for (int base = 0; base < n; base += P) {
        const int cols = min(CB, (n - base + 15) >> 4);  // column blocks with pairs
        for (int i = wave; i < cols * T.KS[0]; i += NW) {
            const int c = i % cols, s = i / cols, row = base + c * 16 + col;
            f64x2 lo = {0.0, 0.0}, hi = {0.0, 0.0};
            if (row < n) {
                const float *e = (const float *)A.emb + (size_t)surv[row] * T.d_item;
                float x[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int kk = 16 * s + 4 * j + g;
                    x[j] = kk < T.d_user ? u[kk] : kk < T.d_user + T.d_item ? e[kk - T.d_user] : 0.f;
                }
                lo[0] = x[0], lo[1] = x[1], hi[0] = x[2], hi[1] = x[3];
            }
            f64x2 *to = buf0 + ((size_t)c * T.slabs[0] + s) * 128 + lane;
            to[0] = lo;
            to[64] = hi;
        }
        __syncthreads();
        for (int l = 0; l < last; ++l) {
            // a wave takes a block of units for two column blocks: with few blocks more waves have work
            const f64x2 *in = l & 1 ? buf1 : buf0;
            f64x2 *out = l & 1 ? buf0 : buf1;
            const int si = T.slabs[l & 1], so = T.slabs[1 - (l & 1)];
            for (int i = wave; i < T.NB[l] * ((cols + 1) >> 1); i += NW) {
                const int nb = i % T.NB[l], c = 2 * (i / T.NB[l]);
                const float4 *w = frag + (T.base[l] + (int64_t)nb * T.KS[l]) * 64 + lane;
                if (CB > 1 && c + 1 < cols)
                    tile_block64<2>(w, T.KS[l], nb, b + T.b_off[l], in + (size_t)c * si * 128, si, out + (size_t)c * so * 128, so);
                else
                    tile_block64<1>(w, T.KS[l], nb, b + T.b_off[l], in + (size_t)c * si * 128, si, out + (size_t)c * so * 128, so);
            }
            __syncthreads();
        }
        for (int c = wave; c < cols; c += NW) {
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
            const int row = base + c * 16 + col;
            if (g == 0 && row < n) keys[row] = make_key((float)part, surv[row], 0u);
        }
        __syncthreads();
    }
}

// The weights of the metrics of 64-wide items and 256 first hidden units in the registers of a workgroup's eight waves, and
// what a wave's units start from: wave w holds block w of layer 1 and block w % 4 of layer 2 (for the first or the second
// half of the columns), every wave the heads.  Read once per search; from L2, a wave would wait for them four times a layer.
template <bool TWO>
struct HeldNet {
    uint4 w1[4], w2[TWO ? 16 : 1], w3[TWO ? 8 : 16];
    f32x4 u1[4], b2[TWO ? 4 : 1];
    __device__ __forceinline__ void load(const FusedArgs &A, int user) {
        constexpr int PER = TWO ? 12 : 6;  // fragments of a block of layer 1 with what takes its units
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5;
        const uint4 *f = (const uint4 *)A.frag + lane;
#pragma unroll
        for (int s = 0; s < 4; ++s) w1[s] = f[(wave * PER + s) * 64];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if constexpr (TWO) w2[k] = f[((k >> 1) * PER + 4 + 2 * (wave & 3) + (k & 1)) * 64];
            else w3[k] = f[((k >> 1) * PER + 4 + (k & 1)) * 64];
        }
        if constexpr (TWO)
#pragma unroll
            for (int k = 0; k < 8; ++k) w3[k] = f[(8 * PER + k) * 64];
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
            u1[t4] = *(const f32x4 *)(A.upre + (size_t)user * 256 + wave * 32 + 8 * t4 + 4 * g);
            if constexpr (TWO) b2[t4] = *(const f32x4 *)(A.b + A.T.b_off[1] + (wave & 3) * 32 + 8 * t4 + 4 * g);
        }
    }
};

// Relevances of the query's pairs surv[0..n) as list keys to keys[0..n) by eight waves, 128 pairs at a time: activations in LDS, 32 pairs a
// column block.  consts: head weights and bias, 8 each.  All threads call; ends with a barrier.
template <bool TWO, bool F16>
__device__ __forceinline__ void fused_score_held(const FusedArgs &A, const HeldNet<TWO> &H, const float *consts,
                                                 const int32_t *surv, uint64_t *keys, int n, uint4 *buf0) {
    constexpr int SLABS0 = TWO ? 8 : 4, SLABS1 = 16;
    uint4 *buf1 = buf0 + 4 * SLABS0 * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5, col = lane & 31;
    for (int base = 0; base < n; base += 128) {
        const int cols = min(4, (n - base + 31) >> 5);
        for (int i = wave; i < 4 * cols; i += 8) {
            const int c = i >> 2, s = i & 3, row = base + c * 32 + col;
            uint4 x = make_uint4(0, 0, 0, 0);
            if (row < n) x = *(const uint4 *)((const uint16_t *)A.emb + (size_t)surv[row] * 64 + 16 * s + 8 * g);
            buf0[(c * SLABS0 + s) * 64 + lane] = x;
        }
        __syncthreads();
#pragma unroll
        for (int c0 = 0; c0 < 4; c0 += 2) {  // layer 1: this wave's 32 units of all columns
            if (c0 >= cols) break;
            f32x16 acc[2];
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[c][i] = H.u1[i >> 2][i & 3];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[c] = tile_mfma<F16>(H.w1[s], buf0[((c0 + c) * SLABS0 + s) * 64 + lane], acc[c]);
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int h = 0; h < 2; ++h) buf1[((c0 + c) * SLABS1 + 2 * wave + h) * 64 + lane] = tile_relu<F16, false>(acc[c], h);
        }
        __syncthreads();
        if constexpr (TWO) {
            const int c0 = wave >> 2;  // layer 2: 32 units of every second column
            f32x16 acc[2];
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[c][i] = H.b2[i >> 2][i & 3];
            if (c0 + 2 < cols) {
#pragma unroll
                for (int k = 0; k < 16; ++k)
#pragma unroll
                    for (int c = 0; c < 2; ++c) acc[c] = tile_mfma<F16>(H.w2[k], buf1[((c0 + 2 * c) * SLABS1 + k) * 64 + lane], acc[c]);
            } else if (c0 < cols) {
#pragma unroll
                for (int k = 0; k < 16; ++k) acc[0] = tile_mfma<F16>(H.w2[k], buf1[(c0 * SLABS1 + k) * 64 + lane], acc[0]);
            }
#pragma unroll
            for (int c = 0; c < 2; ++c)
                if (c0 + 2 * c < cols)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        buf0[((c0 + 2 * c) * SLABS0 + 2 * (wave & 3) + h) * 64 + lane] = tile_relu<F16, false>(acc[c], h);
            __syncthreads();
        }
        if (wave < cols) {  // heads: one wave per column
            f32x16 z;
#pragma unroll
            for (int i = 0; i < 16; ++i) z[i] = 0.f;
#pragma unroll
            for (int k = 0; k < (TWO ? 8 : 16); ++k)
                z = tile_mfma<F16>(H.w3[k], (TWO ? buf0 + (wave * SLABS0 + k) * 64 : buf1 + (wave * SLABS1 + k) * 64)[lane], z);
            const f32x4 hw = *(const f32x4 *)(consts + 4 * g), bh = *(const f32x4 *)(consts + 8 + 4 * g);
            float part = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) part = fmaf(hw[i], sigmoid_hw(z[i] + bh[i]), part);
            const float other = __shfl_xor(part, 32);
            const int row = base + wave * 32 + col;
            if (g == 0 && row < n) keys[row] = make_key(part + other, surv[row], 0u);
        }
        __syncthreads();
    }
}

// Entries of the ascending a[0..n) in front of `key`: three probes a step, a chain of log4(n) trips to the LDS.  top: the
// largest power of four with 4 top > n.
__device__ __forceinline__ int entries_in_front(const uint64_t *a, int n, int top, uint64_t key) {
    int in_front = 0;
    for (int s = top; s > 0; s >>= 2) {
        int step = 0;
#pragma unroll
        for (int i = 1; i <= 3; ++i) {
            const int at = in_front + i * s;
            step += at <= n && a[max(min(at, n) - 1, 0)] < key ? s : 0;
        }
        in_front += step;
    }
    return in_front;
}
__device__ __forceinline__ int search_top(int n) {
    int top = 1;
    while (4 * top <= n) top *= 4;
    return top;
}

// Merges the m sorted keys into the sorted list, both in LDS, in place, where together they are at most two for every thread: an
// entry's new rank is its own plus the number of entries of the other sequence in front of it.  *first: the first
// insertion's rank.  (Counting the unsorted keys in front of every entry instead, without a sort: 280 us for one query on a
// million items either way, but 64 queries of the widest metric 3.25 -> 3.52 ms.)
template <int BLK>
__device__ __forceinline__ void fused_merge_short(uint64_t *list, int n_list, int C, const uint64_t *keys, int m, int *first) {
    uint64_t key[2];
    int to[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = threadIdx.x + u * BLK;
        to[u] = C;
        if (i < n_list) {
            key[u] = list[i];
            to[u] = i + lower_bound_keys(keys, m, key[u]);
        } else if (i < n_list + m) {
            key[u] = keys[i - n_list];
            to[u] = (i - n_list) + lower_bound_keys(list, n_list, key[u]);
            if (i == n_list) *first = to[u];
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (to[u] < C) list[to[u]] = key[u];
}

// Sum of x over the lanes up to this one.
__device__ __forceinline__ int wave_prefix_sum(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // from 1, 2, 4, 8 lanes down inside a row of 16
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // the last of row 0 (2) to row 1 (3)
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // the last of row 1 to rows 2 and 3
    return x;
}

// Merges the m sorted keys into the sorted list (n_list entries, capacity C), both in LDS, in place, as wave_merge does
// (search_wave.hip): bits of `taken` mark the ranks that new keys take, every other rank o holds the old entry o - (marked
// ranks in front of it); ranks are written from the end, 64 a wave and step.  *first: the first insertion's rank.  (Every
// old entry looking its rank up among the new keys instead: 64 fp32 queries with lists of 4,096 2.83 -> 3.25 ms.)
//   taken : LDS uint64[ceil(C / 64)], zero; left so.   marked : LDS int, zero; left so
template <int BLK>
__device__ __forceinline__ void fused_merge(uint64_t *list, int n_list, int C, const uint64_t *keys, int m, uint64_t *taken,
                                            int *first, int *marked) {
    constexpr int U = 4, PIECES = U * BLK / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_out = min(C, n_list + m), top = search_top(n_list);
    for (int j0 = 0; j0 < m; j0 += BLK) {
        const int j = j0 + threadIdx.x;
        int to = C;
        if (j < m) {
            to = j + entries_in_front(list, n_list, top, keys[j]);
            if (to < C) atomicOr((uint32_t *)taken + (to >> 5), 1u << (to & 31));
            if (j == 0) *first = to;
        }
        const unsigned long long in = __ballot(to < C);
        if (lane == 0 && in) atomicAdd(marked, __popcll(in));
    }
    __syncthreads();
    const int end = (n_out + 63) >> 6, begin = __builtin_amdgcn_readfirstlane(*first) >> 6;
    int before = __builtin_amdgcn_readfirstlane(*marked);  // marks in front of piece `hi`
    for (int hi = end; hi > begin; hi -= PIECES) {
        // marks in piece hi - 1 - lane and those behind it
        const int marks_from = wave_prefix_sum(hi - 1 - lane >= begin && lane < PIECES ? __popcll(taken[hi - 1 - lane]) : 0);
        uint64_t e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = u * (BLK / 64) + wave, c = hi - 1 - p;
            e[u] = 0;
            if (c >= begin) {
                const unsigned long long marks = taken[c];
                const int o = c * 64 + lane, k = before - __builtin_amdgcn_readlane(marks_from, p) + __popcll(marks & ((1ull << lane) - 1ull));
                if (o < n_out) e[u] = (marks >> lane) & 1ull ? keys[k] : list[o - k];
            }
        }
        before -= __builtin_amdgcn_readlane(marks_from, PIECES - 1);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = hi - 1 - (u * (BLK / 64) + wave), o = c * 64 + lane;
            if (c >= begin && o < n_out) list[o] = e[u];
        }
    }
    if (threadIdx.x == 0) *marked = 0;
    for (int c = begin + threadIdx.x; c < end; c += BLK) taken[c] = 0;
}

// LDS, in bytes: the list, its marks during a merge, the survivors' ids and keys, the visited set of a small search, the parents, the small words and head
// constants, a metric of the caller's own widths (weights and biases) where it fits, and one region used in turn by the scoring and the sort.
struct FusedLds {
    size_t taken, keyed, surv, seen, parents, small, net, scratch;
};
__host__ __device__ inline size_t up16(size_t v) { return (v + 15) & ~(size_t)15; }
__host__ __device__ inline void fused_lds(int C, int slots, int W_max, int seen_words, int net_words, FusedLds *o) {
    o->taken = up16((size_t)8 * C);
    o->keyed = up16(o->taken + (size_t)8 * ((C + 63) >> 6));
    o->surv = up16(o->keyed + (size_t)8 * slots);
    o->seen = up16(o->surv + (size_t)4 * slots);
    o->parents = up16(o->seen + (size_t)4 * seen_words);
    o->small = up16(o->parents + (size_t)4 * W_max);
    o->net = up16(o->small + 48 * 4);
    o->scratch = up16(o->net + (size_t)4 * net_words);
}

// RESUME: the slot's search goes on from where the batch path's last round left it (survivors chosen, not yet scored)
// and its list and state go back there, for the kernels that write the results; slots without a running search leave.
template <int BLK, bool BITMAP, int METRIC, int CB, bool RESUME>
__global__ void __launch_bounds__(BLK, CB == 4 ? 2 : 4) fused_search_kernel(FusedArgs A) {  // waves a SIMD: see fused_plan
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    int q = blockIdx.x;
    if (RESUME && A.handed) {
        if (q >= __builtin_amdgcn_readfirstlane(A.ctrl->handed)) return;
        q = __builtin_amdgcn_readfirstlane(A.handed[q]);
    }
    FusedLds at;
    fused_lds(A.C, A.slots, A.W_max, A.seen_words, A.frag_words + A.bias_words, &at);
    uint64_t *cur = (uint64_t *)smem, *taken = (uint64_t *)(smem + at.taken);
    int32_t *surv = (int32_t *)(smem + at.surv);
    uint64_t *keyed = (uint64_t *)(smem + at.keyed);
    uint32_t *seen = (uint32_t *)(smem + at.seen);
    int32_t *parents = (int32_t *)(smem + at.parents);
    int *wave_sums = (int *)(smem + at.small), *shared_i = wave_sums + 16;
    float *consts = (float *)(wave_sums + 32);
    unsigned char *scratch = smem + at.scratch;
    // the scratch region in its two roles (the other is the scoring's)
    uint64_t *newk = (uint64_t *)scratch;
    uint32_t *sort_cnt = (uint32_t *)(newk + A.new_cap);

    int n_list = 0, n_visited = 0, n_expanded = 0, first_open = 0, t = 0, n_cand = A.E, user = q, pending = 0;
    if (RESUME) {
        const QState *st = A.state + q;
        if (!A.handed) {
            pending = __builtin_amdgcn_readfirstlane(A.counts[q]);
            if (pending < 0) return;
            if (__builtin_amdgcn_readfirstlane(st->done)) return;
        }
        n_list = __builtin_amdgcn_readfirstlane(st->n_list);
        n_visited = __builtin_amdgcn_readfirstlane(st->n_visited);
        n_expanded = __builtin_amdgcn_readfirstlane(st->n_expanded);
        first_open = __builtin_amdgcn_readfirstlane(st->first_open);
        t = __builtin_amdgcn_readfirstlane(st->t);
        if (A.slot_query) user = __builtin_amdgcn_readfirstlane(A.slot_query[q]);
        for (int i = tid; i < n_list; i += BLK) cur[i] = A.pool[(size_t)q * A.C + i];
        for (int i = tid; i < pending; i += BLK) surv[i] = A.cand[(size_t)q * A.slots + i];
        n_cand = 0;
    }
    const int W = min(max(A.W_q ? A.W_q[user] : A.W, 1), A.W_max), L = min(max(A.L_q ? A.L_q[user] : A.L, 1), A.L_max);
    const int c_own = A.cap_q ? A.cap_q[user] : A.cap;
    const int cap = A.cap_max > 0 ? min(max(c_own, 1), A.cap_max) : max(c_own, 0);
    uint32_t *table = A.table + (size_t)q * A.table_words;
    for (int i = tid; i < (A.C + 63) >> 6; i += BLK) taken[i] = 0;
    if (tid == 0) shared_i[2] = 0;
    if (tid < 8) {
        consts[tid] = tid < A.T.J ? A.T.head_w[tid] : 0.f;
        consts[8 + tid] = tid < A.T.J ? A.b[A.T.b_off[A.T.n_layers - 1] + tid] : 0.f;
    }
    HeldNet<METRIC != FUSED_ONE && METRIC != FUSED_ONE + 1> held;
    if constexpr (METRIC >= FUSED_TWO) held.load(A, user);
    const uint4 *net = (const uint4 *)(smem + at.net);
    const float *net_b = (const float *)(net + A.frag_words / 4);
    if (METRIC < FUSED_TWO && A.frag_words) {
        for (int i = tid; i < A.frag_words / 4; i += BLK) ((uint4 *)net)[i] = ((const uint4 *)A.frag)[i];
        for (int i = tid; i < A.bias_words; i += BLK) ((float *)net_b)[i] = A.b[i];
    }
    auto clear_table = [&]() {
        const uint32_t e = BITMAP ? 0u : EMPTY_SLOT;
        for (int i = tid; i < A.table_words / 4; i += BLK) ((uint4 *)table)[i] = make_uint4(e, e, e, e);
        visited_cleared();
    };
    bool in_lds = !RESUME && A.seen_words > 0;
    if (in_lds) {
        for (int i = tid; i < A.seen_words; i += BLK) seen[i] = A.seen_bits ? 0u : EMPTY_SLOT;
        __syncthreads();
    } else if (!RESUME) {
        clear_table();
    } else {
        __syncthreads();
    }
    bool seeding = true, overflow = false;
    // bounded: a search cannot run more rounds than its cap or than ids fit its visited set
    for (int round = 0; round <= A.rounds_max; ++round) {
        // candidates (the seeds, later one adjacency row per parent) through the visited filter
        auto candidate = [&](int j, uint32_t *bit) {
            int32_t v;
            if (seeding) {
                v = A.entries[(size_t)q * A.E + j];
                if (BITMAP || A.seen_bits) *bit = BITMAP && A.rank && v >= 0 && (int64_t)v < A.N ? (uint32_t)A.rank[v] : (uint32_t)v;
            } else {
                const int p = j / A.R;
                const size_t from = (size_t)parents[p] * A.R + (j - p * A.R);
                v = A.adj[from];
                if (BITMAP || A.seen_bits) *bit = (uint32_t)(BITMAP && A.adj_rank ? A.adj_rank[from] : v);
            }
            return v;
        };
        if (!RESUME && in_lds && !A.seen_bits && n_visited + n_cand > A.seen_words / 8 * 5) {  // on to the table in memory
            clear_table();
            for (int i = tid; i < A.seen_words; i += BLK) {
                const int32_t v[1] = {(int32_t)seen[i]};
                uint32_t slot[1];
                bool fresh[1];
                visited_enter<false, false, 1>(v, slot, fresh, table, A.hash_cap, A.N, Nothing{});
            }
            in_lds = false;
            __syncthreads();
        }
        int n_new;
        if (RESUME || !in_lds) n_new = visit<BLK, BITMAP, false, 2>(candidate, n_cand, table, A.hash_cap, A.N, surv, wave_sums, Nothing{});
        else if (A.seen_bits) n_new = visit<BLK, true, false, 2>(candidate, n_cand, seen, 0, A.N, surv, wave_sums, Nothing{});
        else n_new = visit<BLK, false, false, 2>(candidate, n_cand, seen, A.seen_words, A.N, surv, wave_sums, Nothing{});
        n_visited += n_new;
        if (RESUME && round == 0) n_new = pending;  // counted by the round that found them
        if (tid == 0) shared_i[0] = 0x7fffffff;  // rank of the first inserted entry
        __syncthreads();
        uint32_t next = 0;  // a byte of a new item's adjacency row brings its line into the L2 slice while the item is scored
        if (CB == 4 && tid < n_new) next = ((const uint8_t *)A.adj)[(size_t)surv[tid] * A.R * 4];

        if constexpr (METRIC >= FUSED_ONE) {
            fused_score_held<false, METRIC == FUSED_ONE + 1>(A, held, consts, surv, keyed, n_new, (uint4 *)scratch);
        } else if constexpr (METRIC >= FUSED_TWO) {
            fused_score_held<true, METRIC == FUSED_TWO + 1>(A, held, consts, surv, keyed, n_new, (uint4 *)scratch);
        } else if constexpr (METRIC == FUSED_F64) {
            if (A.frag_words) fused_score64<BLK, CB>(A, (const float4 *)net, net_b, user, surv, keyed, n_new, (f64x2 *)scratch);
            else fused_score64<BLK, CB>(A, (const float4 *)A.frag, A.b, user, surv, keyed, n_new, (f64x2 *)scratch);
        } else {
            if (A.frag_words) fused_score16<BLK, METRIC == FUSED_F16, CB>(A, net, net_b, user, surv, keyed, n_new, (uint4 *)scratch);
            else fused_score16<BLK, METRIC == FUSED_F16, CB>(A, (const uint4 *)A.frag, A.b, user, surv, keyed, n_new, (uint4 *)scratch);
        }
        asm volatile("" ::"v"(next));  // here at the latest

        // merge: what can enter the list, sorted, into the list
        const uint64_t worst = n_list == A.C ? cur[A.C - 1] : KEY_SENTINEL;
        int m = 0;
        for (int j0 = 0; j0 < n_new; j0 += BLK) {
            const int j = j0 + tid;
            const uint64_t key = j < n_new ? keyed[j] : KEY_SENTINEL;
            const bool keep = j < n_new && key < worst;
            int tot;
            const int pos = block_excl_count<BLK>(keep, wave_sums, &tot);
            if (keep) newk[m + pos] = key;
            m += tot;
        }
        if (m > 0) {
            if (m <= BLK) {
                rank_sort<BLK>(newk, m, sort_cnt);
            } else {
                int m2 = 2;
                while (m2 < m) m2 <<= 1;
                for (int i = m + tid; i < m2; i += BLK) newk[i] = KEY_SENTINEL;
                __syncthreads();
                bitonic_sort<BLK>(newk, m2);
            }
            if (n_list + m <= 2 * BLK) fused_merge_short<BLK>(cur, n_list, A.C, newk, m, &shared_i[0]);
            else fused_merge<BLK>(cur, n_list, A.C, newk, m, taken, &shared_i[0], &shared_i[2]);
            n_list = min(A.C, n_list + m);
        }
        __syncthreads();

        // termination test and choice of the parents: the first <= W unexpanded entries among the first L ranks
        first_open = min(first_open, shared_i[0]);
        int n_par = 0;
        if (!(cap > 0 && t >= cap)) {
            const int lim = min(L, n_list);
            // First an entry a lane of one wave, with no barrier on the way, where that is mostly enough (one query, W = 4, L = 64 271 ->
            // 267 us, 64 with W = 1, L = 1,000 6,850 -> 6,671, W = 2, L = 300 1,766 -> 1,723); with W = 4, L = 1,000 it is behind, 2,567 -> 2,608,
            // and a wave that walks on, 256 entries a step, more so (2,624; 256 queries, W = 8, L = 512 1,385 -> 1,448).
            if (lim - first_open <= 64 || W <= 2) {
                if (tid < 64) {
                    const int i = first_open + tid;
                    const uint64_t e = i < lim ? cur[i] : 1ull;
                    const bool open = !key_expanded(e);
                    const unsigned long long b = __ballot(open);
                    const int pos = __popcll(b & ((1ull << tid) - 1ull)), tot = __popcll(b);
                    const bool take = open && pos < W;
                    if (take) {
                        parents[pos] = key_id(e);
                        cur[i] = e | 1ull;
                    }
                    const int behind = __ffsll(__ballot(take && pos == W - 1));  // the last parent's lane + 1
                    if (tid == 0) shared_i[1] = tot >= W ? first_open + behind : min(first_open + 64, lim), shared_i[3] = min(W, tot);
                }
                __syncthreads();
                first_open = __builtin_amdgcn_readfirstlane(shared_i[1]);
                n_par = __builtin_amdgcn_readfirstlane(shared_i[3]);
            }
            if (first_open < lim && n_par < W) {
                int i0 = first_open;
                bool filled = false;
                while (i0 < lim && !filled) {
                    const int i = i0 + tid;
                    const uint64_t e = i < lim ? cur[i] : KEY_SENTINEL;
                    const bool open = i < lim && !key_expanded(e);
                    int tot;
                    const int pos = block_excl_count<BLK>(open, wave_sums, &tot);
                    if (open && n_par + pos < W) {
                        parents[n_par + pos] = key_id(e);
                        cur[i] = e | 1ull;
                        if (n_par + pos == W - 1) shared_i[1] = i + 1;  // everything in front of it is expanded now
                    }
                    filled = n_par + tot >= W;
                    n_par = min(W, n_par + tot);
                    i0 += BLK;
                    first_open = min(i0, lim);
                }
                __syncthreads();
                if (filled) first_open = shared_i[1];
            }
        }
        if (!BITMAP && n_par > 0 && (int64_t)n_visited + (int64_t)n_par * A.R > (int64_t)(A.hash_cap / 2)) {
            overflow = true;
            n_par = 0;
        }
        if (n_par == 0) break;
        ++t;
        n_expanded += n_par;
        n_cand = n_par * A.R;
        seeding = false;
        // A sign of progress for the waiting host thread, after a query's first round and every eighth one: a store that
        // nobody waits for, but a thousand workgroups send theirs over one link.
        if (A.mailbox && tid == 0 && (t & 7) == 1)
            __hip_atomic_store(A.mailbox + MAIL_SIGN, A.mail_tag | (uint32_t)t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __syncthreads();
    }
    __syncthreads();
    if (RESUME && !A.handed) {
        for (int i = tid; i < n_list; i += BLK) A.pool[(size_t)q * A.C + i] = cur[i];
        if (tid == 0) {
            QState *st = A.state + q;
            st->n_list = n_list;
            st->n_visited = n_visited;
            st->n_expanded = n_expanded;
            st->first_open = first_open;
            st->t = t;
            st->done = overflow ? 3 : 1;
            A.counts[q] = -1;
            atomicAdd((unsigned long long *)&A.stats[7], 1ull);
        }
        return;
    }
    for (int i = tid; i < A.k; i += BLK) {
        const bool held = i < n_list;
        const uint64_t key = held ? cur[i] : 0;
        A.out_ids[(size_t)q * A.k + i] = held ? key_id(key) : -1;
        A.out_scores[(size_t)q * A.k + i] = held ? key_score(key) : -INFINITY;
    }
    if (tid == 0) {
        add_to_totals(A.stats, n_visited, n_expanded, t, overflow ? 1 : 0);
        if (RESUME) atomicAdd((unsigned long long *)&A.stats[7], 1ull);  // a batch that begins here has been counted
        if (A.mailbox) {
            // the last query to end reports
            __threadfence_system();
            if (atomicAdd(RESUME ? &A.ctrl->ended : &A.ctrl->next_query, 1) == A.Q - 1) report_end(A.stats, A.mailbox, A.mail_tag);
        }
    }
}

// The layers of a built-in shape over the fragments that its batch kernel keeps (see mlp_mfma.hip,
// mlp_mfma_stream.hip for the orders).
static void built_in_net(const ann_mlp *m, TileNet *T) {
    const int KS1 = m->d_item / 16, NB1 = m->dims[1] / 32, last = m->n_layers - 1;
    *T = TileNet{};
    T->n_layers = m->n_layers;
    T->J = m->J;
    T->d_user = m->d_user;
    T->d_item = m->d_item;
    for (int j = 0; j < m->J; ++j) T->head_w[j] = m->head_w[j];
    for (int l = 0; l < m->n_layers; ++l) {
        T->KS[l] = l == 0 ? KS1 : m->dims[l] / 16;
        T->NB[l] = l == last ? 1 : m->dims[l + 1] / 32;
        T->b_off[l] = m->b_off[l];
        T->step2[l] = 2;
        if (T->KS[l] > T->slabs[l & 1]) T->slabs[l & 1] = T->KS[l];
    }
    if (m->n_layers == 2) {  // block of units: layer 1, then the two head fragments that take it
        T->stride_n[0] = T->step2[1] = KS1 + 2;
        T->base[1] = KS1;
        return;
    }
    const int chunk = KS1 + 2 * T->NB[1];  // layer 1 of a block, then the fragments of layer 2 that take a block
    const int skew = mfma_stream_supported(m->d_item, m->dims[1], m->dims[2]) ? 1 : 0;  // ... the block before
    T->stride_n[0] = T->step2[1] = chunk;
    T->base[1] = (int64_t)skew * chunk + KS1;
    T->stride_n[1] = 2;
    T->base[2] = (int64_t)(NB1 + skew) * chunk;
}

static size_t fused_smem(const SearchArgs &a, const TileNet &T, bool f64, int cb, int new_cap, int blk, int net_words, int seen_words = 0) {
    FusedLds at;
    fused_lds(a.plan.C, a.plan.slots, a.plan.W_max, seen_words, net_words, &at);
    const size_t sort = (size_t)new_cap * 8 + (size_t)blk * 4;
    const size_t net = (size_t)cb * (T.slabs[0] + T.slabs[1]) * (f64 ? 2048 : 1024);
    return at.scratch + (net > sort ? net : sort);
}

template <int BLK, int METRIC, int CB, bool RESUME>
static int fused_launch(const SearchArgs &a, const FusedArgs &A, size_t smem, int grid) {
    const bool bm = a.plan.bitmap_words > 0;
    auto fn = bm ? fused_search_kernel<BLK, true, METRIC, CB, RESUME> : fused_search_kernel<BLK, false, METRIC, CB, RESUME>;
    static std::atomic<uint32_t> raised[2];
    if (int rc = raise_lds_limit((const void *)fn, FUSED_LDS, a.m->device, raised[bm ? 1 : 0]); rc != ANN_OK) return rc;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(BLK), smem, a.stream, A);
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

// Which searches run here, and with what workgroups.  Both sides measured, batch path (beyond 512 queries with its last
// queries in one launch) -> this one, lists of L, W nodes a round, 32 candidates a node:
//   - the whole batch is resident at once (a second turn of workgroups would start when the batch path is half
//     done).  64 -> 256 -> 128, 2,048 queries, W = 4, L = 256 6.4 -> 7.5 ms; 1,024 queries, W = 4, L = 64 1.9 -> 1.6,
//     L = 256 4.9 -> 4.9, L = 512 7.1 -> 6.2, W = 8, L = 512 5.4 -> 5.5, W = 1, L = 256 12.3 -> 7.6; 512 queries,
//     W = 4, L = 256 4.8 -> 3.2, W = 8, L = 512 4.5 -> 3.4.  64 -> 256, W = 4, L = 64: 2,048 queries 2.24 -> 2.25, 1,024
//     1.8 -> 1.4;
//   - a round's matrix work per CU stays small, at most FUSED_WORK operations (fp64 ones count 32 times), since a
//     query's pairs are scored by one CU while the batch path spreads them over the chip.  128 -> 512 -> 256, 64 queries,
//     W = 8 (0.10 GFLOP) 5.1 -> 4.2 ms, W = 16 5.2 -> 5.8; 256 queries, W = 8 6.2 -> 5.0, and W = 16, beyond the line,
//     8.2 -> 6.5 as well.  fp32 32 -> 64, 16 candidates a node: 64 queries, W = 16, L = 4,096 9.3 -> 6.4, and 1,024
//     queries, W = 8, L = 512, beyond the line, 4.3 -> 3.4;
//   - tiles of a single column block read all weights from L2 for 32 pairs: with more than one workgroup on a CU only
//     for weights of at most FUSED_WEIGHTS bytes (512 queries of the widest metric, W = 4 7.1 -> 8.6 ms; with W = 1,
//     where a round is mostly launches, 18.7 -> 12.1).
// The largest tile that leaves every query resident wins (fewer passes over the weights; 256 queries of 64 -> 256 -> 128
// 2.1 ms at 128 pairs, 2.6 at 64, 3.2 at 32), and 512 threads over 256 wherever two such workgroups suffice.
constexpr int64_t FUSED_WORK = 110 * 1000000, FUSED_WEIGHTS = 128 * 1024, FUSED_NET = 64 * 1024, FUSED_BITS = 128 * 1024;

struct FusedPlan {
    TileNet T;
    int blk, cb, new_cap, frag_words, bias_words, seen_words, seen_bits;
    bool held;
    size_t smem;
};

// The visited set in LDS, where that leaves as many workgroups on a CU: one bit per item of a small table, else slots for the
// ids of a short search (it goes on in memory when five eighths of them are taken).
static void fused_seen(const SearchArgs &a, int Q, FusedPlan *f) {
    const Plan &p = a.plan;
    f->seen_words = f->seen_bits = 0;
    auto fits = [&](int words) {
        const size_t smem = fused_smem(a, f->T, a.m->dtype == ANN_F32, f->cb, f->new_cap, f->blk, f->frag_words + f->bias_words, words);
        if (smem > FUSED_LDS || Q > 256 * (int)(160 * 1024 / smem)) return false;
        f->seen_words = words;
        f->smem = smem;
        return true;
    };
    if (a.g->N <= FUSED_BITS && fits((int)((a.g->N + 31) / 32))) f->seen_bits = 1;
    else if (p.bitmap_words == 0 && a.g->N > FUSED_BITS)
        for (int words = p.hash_cap < 8192 ? p.hash_cap & ~7 : 8192; words >= 2048 && !fits(words); words >>= 1) {}
}

static bool fused_plan(const SearchArgs &a, int Q, FusedPlan *f) {
    const Plan &p = a.plan;
    const ann_mlp *m = a.m;
    if (a.walkers || m->dtype == ANN_F8) return false;
    const bool built_in = m->kernel == MLP_MFMA2, f64 = m->dtype == ANN_F32;
    if (built_in) built_in_net(m, &f->T);
    else if (m->any_dev) f->T = m->any;
    else return false;
    int64_t weights = 0;
    for (int l = 0; l < m->n_layers; ++l)
        weights += (int64_t)m->dims[l + 1] * (l == 0 && built_in ? m->d_item : m->dims[l]);
    if ((int64_t)((Q + 255) / 256) * p.slots * 2 * weights * (f64 ? 32 : 1) > FUSED_WORK) return false;
    f->new_cap = 2;
    while (f->new_cap < p.slots) f->new_cap <<= 1;
    f->frag_words = f->bias_words = 0;
    f->held = Q <= 256 && built_in && m->d_item == 64 && m->dims[1] == 256 && ((uintptr_t)a.g->emb & 15) == 0;
    if (f->held) {
        f->cb = 4;
        f->blk = 512;
        f->smem = fused_smem(a, f->T, false, 4, f->new_cap, 512, 0);
        if (f->smem <= FUSED_LDS) {
            fused_seen(a, Q, f);
            return true;
        }
        f->held = false;
    }
    const int last = f->T.n_layers - 1;
    const int64_t frag_words = built_in ? 0 : (f->T.base[last] + (int64_t)f->T.KS[last] * f->T.NB[last]) * 256;
    for (f->cb = 4; f->cb >= 1; f->cb >>= 1) {
        if (f->cb > 1 && (f->cb >> 1) * (f64 ? 16 : 32) >= p.slots) continue;  // half of it holds every round's pairs
        if (f->cb == 1 && Q > 256 && weights * (f64 ? 4 : 2) > FUSED_WEIGHTS) continue;
        f->blk = f->cb > 1 ? 512 : 256;
        for (int in_lds = frag_words > 0 && frag_words * 4 <= FUSED_NET ? 1 : 0; in_lds >= 0; --in_lds) {
            f->frag_words = in_lds ? (int)frag_words : 0;
            f->bias_words = in_lds ? f->T.b_off[last] + 64 : 0;
            f->smem = fused_smem(a, f->T, f64, f->cb, f->new_cap, f->blk, f->frag_words + f->bias_words);
            if (f->smem > FUSED_LDS) continue;
            const int by_lds = (int)(160 * 1024 / f->smem), by_waves = f->cb == 4 ? 1 : 1024 / f->blk;  // registers: 168, 126, 107
            if (Q > 256 * (by_lds < by_waves ? by_lds : by_waves)) continue;
            fused_seen(a, Q, f);
            return true;
        }
    }
    return false;
}

static bool fused_takes(const SearchArgs &a, int Q) {
    FusedPlan f;
    return fused_plan(a, Q, &f);
}

bool fused_serves(const SearchArgs &a) { return a.Q_total == 0 && fused_takes(a, a.plan.Q); }

int fused_tail(const SearchArgs &a) {
    if (a.Q_total < 0) return 0;
    return fused_takes(a, 512) ? 512 : fused_takes(a, 256) ? 256 : 0;
}

static FusedArgs fused_args(const SearchArgs &a, const FusedPlan &f, int32_t rounds_max, bool resume) {
    const Plan &p = a.plan;
    const ann_mlp *m = a.m;
    FusedArgs A{};
    A.T = f.T;
    A.new_cap = f.new_cap;
    A.frag_words = f.frag_words, A.bias_words = f.bias_words;
    A.seen_words = resume ? 0 : f.seen_words, A.seen_bits = resume ? 0 : f.seen_bits;
    const bool built_in = m->kernel == MLP_MFMA2, f64 = m->dtype == ANN_F32, bm = p.bitmap_words > 0;
    A.frag = built_in ? m->frag_dev : m->any_dev;
    A.b = m->b_dev;
    A.upre = !built_in ? nullptr : a.upre_all ? a.upre_all : (const float *)(a.ws + p.off_upre);
    A.emb = a.g->emb;
    A.users = a.queries;
    A.adj = a.g->adj;
    A.adj_rank = bm ? a.g->adj_rank : nullptr;
    A.rank = bm ? a.g->rank : nullptr;
    A.entries = a.entries;
    A.W_q = a.W_q, A.L_q = a.L_q, A.cap_q = a.cap_q;
    A.table = (uint32_t *)(a.ws + p.off_hash);
    A.stats = (int64_t *)(a.ws + p.off_stats);
    A.ctrl = (Ctrl *)(a.ws + p.off_ctrl);
    A.out_ids = a.out_ids;
    A.out_scores = a.out_scores;
    A.mailbox = a.mailbox;
    A.mail_tag = a.mail_tag;
    A.state = (QState *)(a.ws + p.off_state);
    A.pool = (uint64_t *)(a.ws + p.off_pool);
    A.counts = (int32_t *)(a.ws + p.off_counts);
    A.cand = (const int32_t *)(a.ws + p.off_cand);
    A.slot_query = a.slot_query;
    A.N = a.g->N;
    A.R = p.R, A.E = p.E, A.W = a.W, A.L = a.L, A.cap = a.cap;
    A.W_max = p.W_max, A.L_max = p.L_max, A.cap_max = p.max_iters_max;
    A.C = p.C, A.k = p.k, A.slots = p.slots;
    A.table_words = bm ? p.bitmap_words : p.hash_cap;
    A.hash_cap = p.hash_cap;
    A.Q = p.Q;
    A.rounds_max = rounds_max;
    A.int_relu = built_in && m->n_layers == 3 && mfma_stream_supported(m->d_item, m->dims[1], m->dims[2]);
    A.wide_loads = ((uintptr_t)a.g->emb & 15) == 0 && (m->d_item & 7) == 0 &&
                   (built_in || ((m->d_user & 7) == 0 && ((uintptr_t)a.queries & 15) == 0));
    return A;
}

int launch_fused(const SearchArgs &a, int32_t rounds_max, int32_t tail) {
    const Plan &p = a.plan;
    const ann_mlp *m = a.m;
    FusedPlan f;
    if (!fused_plan(a, tail > 0 ? tail : p.Q, &f)) return ANN_EINVAL;
    const FusedArgs A = fused_args(a, f, rounds_max, tail > 0);
    const bool f64 = m->dtype == ANN_F32;
    if (tail <= 0)
        if (int rc = launch_zero_stats(a, p.Q); rc != ANN_OK) return rc;
#define FUSED_PICK(METRIC, RESUME)                                \
    (f.cb == 4   ? fused_launch<512, METRIC, 4, RESUME>(a, A, f.smem, p.Q)  \
     : f.cb == 2 ? fused_launch<512, METRIC, 2, RESUME>(a, A, f.smem, p.Q)  \
               : fused_launch<256, METRIC, 1, RESUME>(a, A, f.smem, p.Q))
    if (tail > 0)
        return f64                     ? FUSED_PICK(FUSED_F64, true)
               : m->dtype == ANN_F16   ? FUSED_PICK(FUSED_F16, true)
                                       : FUSED_PICK(FUSED_BF16, true);
    if (f.held && m->n_layers == 3)
        return m->dtype == ANN_F16 ? fused_launch<512, FUSED_TWO + 1, 4, false>(a, A, f.smem, p.Q) : fused_launch<512, FUSED_TWO, 4, false>(a, A, f.smem, p.Q);
    if (f.held) return m->dtype == ANN_F16 ? fused_launch<512, FUSED_ONE + 1, 4, false>(a, A, f.smem, p.Q) : fused_launch<512, FUSED_ONE, 4, false>(a, A, f.smem, p.Q);
    return f64 ? FUSED_PICK(FUSED_F64, false) : m->dtype == ANN_F16 ? FUSED_PICK(FUSED_F16, false) : FUSED_PICK(FUSED_BF16, false);
#undef FUSED_PICK
}

bool fused_goes_on(const SearchArgs &a, int32_t most) {
    FusedPlan f;
    return fused_plan(a, most, &f) && f.held;
}

int launch_fused_rest(const SearchArgs &a, int32_t rounds_max, int32_t most) {
    const ann_mlp *m = a.m;
    FusedPlan f;
    if (!fused_plan(a, most, &f) || !f.held) return ANN_EINVAL;
    FusedArgs A = fused_args(a, f, rounds_max, true);
    A.handed = (const int32_t *)(a.ws + a.plan.off_offsets);
    if (m->n_layers == 3)
        return m->dtype == ANN_F16 ? fused_launch<512, FUSED_TWO + 1, 4, true>(a, A, f.smem, most) : fused_launch<512, FUSED_TWO, 4, true>(a, A, f.smem, most);
    return m->dtype == ANN_F16 ? fused_launch<512, FUSED_ONE + 1, 4, true>(a, A, f.smem, most) : fused_launch<512, FUSED_ONE, 4, true>(a, A, f.smem, most);
}

}  // namespace gmpgr
