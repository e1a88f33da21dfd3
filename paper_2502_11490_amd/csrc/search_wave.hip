// A whole search by one wave: every wave of a persistent grid takes a query, runs all rounds of the joint best-first search
// (Sec. 3.2, Algorithm 1) on it, scoring included, writes its result and takes the next one.  For the metrics of 64-wide
// items and 256 first hidden units, whose weights stay in the LDS of a CU for the whole launch; its waves share
// nothing else, so no wave ever waits for another one: not at a barrier, not for a launch, not for the end of a round.
//
// The list, the round's new keys and the user's share of layer 1 are in the wave's part of the LDS, the visited set in
// memory, one atomic per candidate.  Pairs go through all layers in registers (wave_tile), in the order of the batch
// kernels (same fragments, same sequence of MFMAs, same start values), so which path serves a call does not show in its
// results.
//
// What bounds it.  Few queries (a wave alone on its SIMD): the chain of a round, 17 us for 75 new pairs: half is scoring, of
// which the matrix instructions are half, a fifth the way to the neighbours and through the visited set, a seventh the
// merge; and the slowest search, which runs half as many rounds again as the average one.  Full batches: two waves a SIMD
// take 22 us a round, and the scattered accesses of a round (128 visited words, 75 item rows, 75 dirty lines) share
// the memory's bandwidth.  The builds of eight waves for two hidden layers take all 256 registers and spill 10 to 18 of them
// (60 to 76 bytes of scratch; bitmaps 44 to 60); scalar registers spill to vector ones in all of them.
// Against the batch path and, up to 1,024 queries, the search by workgroups: 1,024 queries of 10^6 items, lists of 512
// 6.1 -> 3.3 ms; 16,384 queries of 2 10^7 items, one hidden layer, lists of 64 8.3 -> 4.7; 8,192 ragged capped queries
// 7.4 -> 4.6.
#include "mlp_tile.h"
#include "search_device.h"

namespace gmpgr {

// Running queries from which on a workgroup per query goes on with them (search_fused.hip): it takes half the time for a
// round, and the longest searches run half as many rounds again as the average one.  Both sides measured, ms: 1,024 queries
// with lists of 512 3.70 -> 3.26, 300 with W = 4, L = 64 1.02 -> 0.81, 2,048 with W = 16, L = 256 4.5 -> 3.9, 8,192 with
// W = 4, L = 512 17.3 -> 16.2; 16,384 with lists of 64 the same.  No more than there are waves.
constexpr int WAVE_HAND = 256;

// Ticks of the 100 MHz clock after which a wave of a search that is waited for says again that it goes on (4 ms): a store over
// the link takes 60 ns of it, and one a query every eighth round made 16,384 short queries 4.5 -> 7.6 ms.
constexpr uint32_t SIGN_TICKS = 400000;

struct WaveArgs {
    const uint4 *frag;
    const float *b2, *b_head, *upre;
    float head_w[MAX_HEADS];
    const uint16_t *emb;
    const int32_t *adj, *adj_rank, *rank, *entries;
    const int32_t *W_q, *L_q, *cap_q, *order;
    // from `hand_at` running queries on (0: never) a query's list and state go to memory and its number to `handed`
    QState *state;
    uint64_t *pool;
    int32_t *handed;
    int32_t hand_at;
    uint32_t *table;
    int64_t *stats;
    Ctrl *ctrl;
    int32_t *out_ids;
    float *out_scores;
    uint64_t *mailbox;
    uint64_t mail_tag;
    int64_t N;
    uint32_t R_magic;  // ceil(2^32 / R): the high half of j * R_magic is j / R for j < 4,096 (R = 1: unused)
    int32_t J, R, E, W, L, cap, W_max, L_max, cap_max, C, k, table_words, hash_cap, Q, rounds_max;
    int32_t wave_off, wave_bytes, at_keys, at_taken, at_ut, at_parents;  // LDS of a wave, in bytes
};

// Sorts keys[0..m), m <= 64 * PER, by counting: a key's rank is the number of smaller ones.
template <int PER>
__device__ __forceinline__ void wave_rank_sort(uint64_t *keys, int m, int lane) {
    uint64_t key[PER];
    uint32_t rank[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        key[u] = lane + 64 * u < m ? keys[lane + 64 * u] : KEY_SENTINEL;
    }
    if (lane < 8) keys[m + lane] = KEY_SENTINEL;
    wave_lds_fence();
    count_smaller<PER>(keys, m, key, rank);
    wave_lds_fence();
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (lane + 64 * u < m) keys[rank[u]] = key[u];
    wave_lds_fence();
}

// The item rows of pairs base .. base + 32 CB - 1 (those at n and beyond: the last one's) as layer-1 operands.
template <int CB>
__device__ __forceinline__ void wave_rows(uint4 (&x)[CB][4], const uint16_t *emb, const uint64_t *keys, int base, int n,
                                          int lane) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        const int32_t id = key_id(keys[min(base + c * 32 + (lane & 31), n - 1)]);
        const uint4 *src = (const uint4 *)(emb + (size_t)id * 64) + (lane >> 5);
#pragma unroll
        for (int s = 0; s < 4; ++s) x[c][s] = src[2 * s];
    }
}

// Relevances of 32 CB pairs whose item rows are in xf, as list keys in the place of their ids.  The wave carries the
// pairs through all layers in registers, as the batch kernels do (mlp_mfma.hip: same fragments, same sequence of MFMAs, same
// start values); weights, biases and head constants are read from LDS, the user's share of layer 1 from ut.
template <bool TWO, bool F16, int CB, bool AHEAD>
__device__ __forceinline__ void wave_tile(const uint4 (&xf)[CB][4], const uint4 *w, const float *consts, const float *ut,
                                          uint64_t *keys, int base, int n, int lane) {
    constexpr int KS1 = 4, NB1 = 8, NB2 = TWO ? 4 : 1, PER = KS1 + 2 * NB2;
    const int g = lane >> 5, col = lane & 31;
    f32x16 acc2[NB2][CB];  // TWO: layer 2; else the heads
#pragma unroll
    for (int n2 = 0; n2 < NB2; ++n2)
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
            const f32x4 v = TWO ? *(const f32x4 *)(consts + 16 + n2 * 32 + 8 * t4 + 4 * g) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc2[n2][c][4 * t4 + e] = v[e];
        }
    auto layer1 = [&](f32x16 (&acc)[CB], int nb) {
        const uint4 *wc = w + (size_t)nb * PER * 64 + lane;
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
            const f32x4 v = *(const f32x4 *)(ut + nb * 32 + 8 * t4 + 4 * g);
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[c][4 * t4 + e] = v[e];
        }
#pragma unroll
        for (int s = 0; s < KS1; ++s) {
            const uint4 a = wc[s * 64];
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[c] = tile_mfma<F16>(a, xf[c][s], acc[c]);
        }
    };
    auto layer2 = [&](const f32x16 (&acc)[CB], int nb) {
        const uint4 *wc = w + (size_t)nb * PER * 64 + lane;
        uint4 hf[CB][2];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            hf[c][0] = tile_relu<F16, false>(acc[c], 0);
            hf[c][1] = tile_relu<F16, false>(acc[c], 1);
        }
#pragma unroll
        for (int n2 = 0; n2 < NB2; ++n2)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                const uint4 a = wc[(KS1 + 2 * n2 + s2) * 64];
#pragma unroll
                for (int c = 0; c < CB; ++c) acc2[n2][c] = tile_mfma<F16>(a, hf[c][s2], acc2[n2][c]);
            }
    };
    if (AHEAD) {  // a wave alone on its SIMD: layer 1 of the next block runs under the rounding of this one
        f32x16 even[CB], odd[CB];
        layer1(even, 0);
#pragma unroll 1
        for (int nb = 0; nb < NB1; nb += 2) {
            layer1(odd, nb + 1);
            layer2(even, nb);
            if (nb + 2 < NB1) layer1(even, nb + 2);
            layer2(odd, nb + 1);
        }
    } else {
#pragma unroll 1
        for (int nb = 0; nb < NB1; ++nb) {
            f32x16 acc[CB];
            layer1(acc, nb);
            layer2(acc, nb);
        }
    }
    f32x16 z[CB];
    if constexpr (TWO) {
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) z[c][i] = 0.f;
        const uint4 *w3 = w + (size_t)NB1 * PER * 64 + lane;
#pragma unroll
        for (int n2 = 0; n2 < NB2; ++n2)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                const uint4 a = w3[(2 * n2 + s2) * 64];
#pragma unroll
                for (int c = 0; c < CB; ++c) z[c] = tile_mfma<F16>(a, tile_relu<F16, false>(acc2[n2][c], s2), z[c]);
            }
    } else {
#pragma unroll
        for (int c = 0; c < CB; ++c) z[c] = acc2[0][c];
    }
    const f32x4 hw = *(const f32x4 *)(consts + 4 * g), bh = *(const f32x4 *)(consts + 8 + 4 * g);
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        float part = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) part = fmaf(hw[i], sigmoid_hw(z[c][i] + bh[i]), part);
        const float other = __shfl_xor(part, 32);
        const int row = base + c * 32 + col;
        if (g == 0 && row < n) keys[row] = make_key(part + other, key_id(keys[row]), 0u);
    }
}

// Merges the m sorted keys into the sorted list (n_list entries, capacity C), both in LDS, in place.  A new key's
// rank in the merged list is its own plus the number of old entries in front of it; bits of `taken` mark those ranks, and
// every other rank o holds the old entry o - (marked ranks in front of it).  Ranks are written from the end, 64 U at a time,
// each from an old rank not behind it, so nothing is overwritten before it is read; the ranks in front of the first
// insertion stay as they are.  Returns the first insertion's rank.
//   taken : LDS uint64[ceil(C / 64)], zero; left so
__device__ __forceinline__ int wave_merge(uint64_t *list, int n_list, int C, const uint64_t *keys, int m, uint64_t *taken,
                                          int lane) {
    constexpr int U = 4;
    const int n_out = min(C, n_list + m);
    int top = 1, first = 0, n_in = 0;
    while (4 * top <= n_list) top *= 4;
#pragma unroll 1
    for (int j0 = 0; j0 < m; j0 += 64) {
        const int j = j0 + lane;
        int to = C;
        if (j < m) {
            const uint64_t key = keys[j];
            int in_front = 0;  // three probes a step: a chain of log4(n_list) trips to the LDS
            for (int s = top; s > 0; s >>= 2) {
                int step = 0;
#pragma unroll
                for (int i = 1; i <= 3; ++i) {
                    const int at = in_front + i * s;
                    step += at <= n_list && list[max(min(at, n_list) - 1, 0)] < key ? s : 0;
                }
                in_front += step;
            }
            to = j + in_front;
            if (to < C) atomicOr((uint32_t *)taken + (to >> 5), 1u << (to & 31));
        }
        if (j0 == 0) first = __builtin_amdgcn_readfirstlane(to);
        n_in += __popcll(__ballot(to < C));
    }
    wave_lds_fence();
    const int end = (n_out + 63) >> 6, begin = first >> 6;  // pieces of 64 ranks
    for (int hi = end; hi > begin; hi -= U) {
        uint64_t e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = hi - 1 - u;
            e[u] = 0;
            if (c >= begin) {
                const unsigned long long marks = taken[c];
                n_in -= __popcll(marks);
                const int o = c * 64 + lane, k = n_in + __popcll(marks & ((1ull << lane) - 1ull));
                if (o < n_out) e[u] = (marks >> lane) & 1ull ? keys[k] : list[o - k];
            }
        }
        wave_lds_fence();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = hi - 1 - u, o = c * 64 + lane;
            if (c >= begin && o < n_out) list[o] = e[u];
        }
        wave_lds_fence();
    }
    for (int c = begin + lane; c < end; c += 64) taken[c] = 0;
    wave_lds_fence();
    return first;
}

// MOST: waves of a workgroup at most (it may be launched with fewer), from which follow the registers of a wave.
template <bool TWO, bool F16, bool BITMAP, int MOST, int U>
__global__ void __launch_bounds__(64 * MOST) wave_search_kernel(WaveArgs A) {
    constexpr int NB2 = 4, FRAGS = TWO ? 104 : 48, CB = MOST <= 8 ? 2 : 1;
    constexpr bool PEEK = MOST > 4;  // see visited_enter: four waves a CU wait for trips to memory, more of them share its bandwidth
    extern __shared__ __align__(16) unsigned char smem[];
    uint4 *w = (uint4 *)smem;
    float *consts = (float *)(w + FRAGS * 64);  // head weights and bias [8] each, layer-2 bias
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int i = threadIdx.x; i < FRAGS * 64; i += blockDim.x) w[i] = A.frag[i];
    if (threadIdx.x < 8) {
        consts[threadIdx.x] = (int)threadIdx.x < A.J ? A.head_w[threadIdx.x] : 0.f;
        consts[8 + threadIdx.x] = (int)threadIdx.x < A.J ? A.b_head[threadIdx.x] : 0.f;
    }
    if (TWO)
        for (int i = threadIdx.x; i < NB2 * 32; i += blockDim.x) consts[16 + i] = A.b2[i];
    unsigned char *mine = smem + A.wave_off + (size_t)wave * A.wave_bytes;
    uint64_t *list = (uint64_t *)mine, *keys = (uint64_t *)(mine + A.at_keys), *taken = (uint64_t *)(mine + A.at_taken);
    float *ut = (float *)(mine + A.at_ut);
    int32_t *parents = (int32_t *)(mine + A.at_parents);
    for (int i = lane; i < (A.C + 63) >> 6; i += 64) taken[i] = 0;
    __syncthreads();

    const int slots = gridDim.x * (blockDim.x >> 6);
    const unsigned long long below = (1ull << lane) - 1ull;
    long long scored = 0, expanded = 0;
    int longest = 0, overflowed = 0, ended = 0;
    int turn = wave * gridDim.x + blockIdx.x;
    // signs of progress for the waiting host thread, stores that nobody waits for; the waves' first ones spread over 4 to 8 ms
    uint32_t signed_at = (uint32_t)__builtin_amdgcn_s_memrealtime() + (uint32_t)turn * (SIGN_TICKS / (uint32_t)slots);
    auto sign = [&]() {
        const uint32_t now = (uint32_t)__builtin_amdgcn_s_memrealtime();
        if ((int32_t)(now - signed_at) < (int32_t)SIGN_TICKS) return;
        signed_at = now;
        if (lane == 0) __hip_atomic_store(A.mailbox + MAIL_SIGN, A.mail_tag | now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };
    while (turn < A.Q) {
        const int q = A.order ? A.order[turn] : turn;
        const int W = min(max(A.W_q ? A.W_q[q] : A.W, 1), A.W_max), L = min(max(A.L_q ? A.L_q[q] : A.L, 1), A.L_max);
        const int c_own = A.cap_q ? A.cap_q[q] : A.cap;
        const int cap = A.cap_max > 0 ? min(max(c_own, 1), A.cap_max) : max(c_own, 0);
        uint32_t *table = A.table + (size_t)q * A.table_words;
        // A query with a cap of its own enters at most E + cap W R ids: it clears and uses no more of its table than that.
        int hash_cap = A.hash_cap;
        if (!BITMAP && A.cap_max > 0) {
            int64_t ids = (int64_t)A.E + (int64_t)cap * W * A.R;
            ids = 2 * ((ids < A.N ? ids : A.N) + (int64_t)W * A.R);
            if (ids < hash_cap) hash_cap = max((int)((ids + 63) & ~63ll), 64);
        }
        {
            const uint32_t e = BITMAP ? 0u : EMPTY_SLOT;
            const int n4 = (BITMAP ? A.table_words : hash_cap) / 4;
            for (int i = lane; i < n4; i += 64) ((uint4 *)table)[i] = make_uint4(e, e, e, e);
            ((float4 *)ut)[lane] = ((const float4 *)(A.upre + (size_t)q * 256))[lane];
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the cleared words, before this wave's atomics
            wave_lds_fence();
        }
        int n_list = 0, n_visited = 0, n_expanded = 0, first_open = 0, t = 0, n_cand = A.E;
        bool seeding = true, overflow = false, handed = false;
        // Rounds after which the number of ended queries is looked at: 4 once all queries have been taken, 32 before that (every
        // 4: 16,384 queries of some 20 rounds 4.38 -> 4.66 ms).  When hand_at <= slots are left, none waits.
        int poll = turn + slots >= A.Q ? 3 : 31;
        // bounded: a search cannot run more rounds than its cap or than ids fit its visited set
        for (int round = 0; round <= A.rounds_max; ++round) {
            int gone = 0;  // queries that have ended; looked at after the round's work
            if (A.hand_at > 0 && (round & poll) == poll)
                gone = __hip_atomic_load(&A.ctrl->next_query, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // the candidates (the seeds, later one adjacency row per parent) piece by piece through the visited set, the
            // metric and into the list; which of them the list keeps does not depend on how they are cut
            for (int p0 = 0; p0 < n_cand; p0 += 64 * U) {
                int32_t v[U];
                uint32_t at[U];
                bool fresh[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int j = p0 + u * 64 + lane;
                    v[u] = -1;
                    at[u] = 0;
                    if (j < n_cand) {
                        if (seeding) {
                            v[u] = A.entries[(size_t)q * A.E + j];
                            if (BITMAP) at[u] = A.rank && v[u] >= 0 && (int64_t)v[u] < A.N ? (uint32_t)A.rank[v[u]] : (uint32_t)v[u];
                        } else {
                            const int p = A.R == 1 ? j : (int)__umulhi((uint32_t)j, A.R_magic);
                            const size_t from = (size_t)parents[p] * A.R + (j - p * A.R);
                            v[u] = A.adj[from];
                            if (BITMAP) at[u] = (uint32_t)(A.adj_rank ? A.adj_rank[from] : v[u]);
                        }
                    }
                }
                // the item rows of what may be new are requested while the visited set answers: a word of a 128-byte row
                // brings its line nearer, for the gather below
                uint32_t touched[U];
                visited_enter<BITMAP, PEEK, U>(v, at, fresh, table, hash_cap, A.N, [&](int u, int32_t id, bool may_be_new) {
                    touched[u] = may_be_new ? *(const uint32_t *)(A.emb + (size_t)id * 64) : 0u;
                });
                int n = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const unsigned long long b = __ballot(fresh[u]);
                    if (fresh[u]) keys[n + __popcll(b & below)] = (uint64_t)(uint32_t)v[u] << 1;
                    n += __popcll(b);
                }
                if (n == 0) continue;
                n_visited += n;
                wave_lds_fence();

#pragma unroll 1
                for (int base = 0; base < n;) {
                    if (CB == 2 && n - base > 32) {
                        uint4 x[2][4];
                        wave_rows<2>(x, A.emb, keys, base, n, lane);
                        wave_tile<TWO, F16, 2, MOST == 4>(x, w, consts, ut, keys, base, n, lane);
                        base += 64;
                    } else {
                        uint4 x[1][4];
                        wave_rows<1>(x, A.emb, keys, base, n, lane);
                        wave_tile<TWO, F16, 1, MOST == 4>(x, w, consts, ut, keys, base, n, lane);
                        base += 32;
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) asm volatile("" ::"v"(touched[u]));  // here at the latest
                wave_lds_fence();

                // what can enter the list, sorted, into the list
                const uint64_t worst = n_list == A.C ? list[A.C - 1] : KEY_SENTINEL;
                int m = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int j = u * 64 + lane;
                    const uint64_t key = j < n ? keys[j] : KEY_SENTINEL;
                    const bool keep = j < n && key < worst;
                    const unsigned long long b = __ballot(keep);
                    if (keep) keys[m + __popcll(b & below)] = key;
                    m += __popcll(b);
                }
                if (m > 0) {
                    wave_lds_fence();
                    if (m <= 64) wave_rank_sort<1>(keys, m, lane);
                    else if (m <= 128) wave_rank_sort<2>(keys, m, lane);
                    else wave_rank_sort<U>(keys, m, lane);
                    first_open = min(first_open, wave_merge(list, n_list, A.C, keys, m, taken, lane));
                    n_list = min(A.C, n_list + m);
                }
            }

            if (A.hand_at > 0 && (round & poll) == poll) {
                const int left = A.Q - __builtin_amdgcn_readfirstlane(gone);
                if (left <= A.hand_at) {
                    handed = true;
                    break;
                }
                if (left <= slots) poll = 3;
            }

            // termination test and choice of the parents: the first <= W unexpanded entries among the first L ranks
            int n_par = 0;
            if (!(cap > 0 && t >= cap)) {
                const int lim = min(L, n_list);
                while (first_open < lim) {
                    const int i = first_open + lane;
                    const uint64_t e = i < lim ? list[i] : KEY_SENTINEL;
                    const bool open = i < lim && !key_expanded(e);
                    const unsigned long long b = __ballot(open);
                    const int pos = n_par + __popcll(b & below), tot = __popcll(b);
                    const bool take = open && pos < W;
                    if (take) {
                        parents[pos] = key_id(e);
                        list[i] = e | 1ull;
                    }
                    if (n_par + tot >= W) {  // everything in front of the last one taken is expanded now
                        first_open += __ffsll(__ballot(take && pos == W - 1));
                        n_par = W;
                        break;
                    }
                    n_par += tot;
                    first_open = min(first_open + 64, lim);
                }
                wave_lds_fence();
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
            if (A.mailbox && (t & 7) == 0) sign();
        }
        if (handed) {
            for (int i = lane; i < n_list; i += 64) A.pool[(size_t)q * A.C + i] = list[i];
            if (lane == 0) {
                QState *st = A.state + q;
                st->t = t;
                st->n_list = n_list;
                st->n_visited = n_visited;
                st->n_expanded = n_expanded;
                st->first_open = first_open;
                A.handed[atomicAdd(&A.ctrl->handed, 1)] = q;
            }
            break;  // nothing waits
        }
        for (int i = lane; i < A.k; i += 64) {
            const bool held = i < n_list;
            const uint64_t key = held ? list[i] : 0;
            A.out_ids[(size_t)q * A.k + i] = held ? key_id(key) : -1;
            A.out_scores[(size_t)q * A.k + i] = held ? key_score(key) : -INFINITY;
        }
        scored += n_visited;
        expanded += n_expanded;
        longest = max(longest, t);
        overflowed += overflow ? 1 : 0;
        ++ended;
        if (A.mailbox) sign();
        wave_lds_fence();
        if (A.Q <= slots && A.hand_at == 0) break;
        int next = 0;
        if (lane == 0) next = atomicAdd(&A.ctrl->next_query, 1);
        turn = slots + __builtin_amdgcn_readfirstlane(next);
    }
    if (ended > 0 && lane == 0) {
        add_to_totals(A.stats, scored, expanded, longest, overflowed);
        if (A.mailbox) {  // the last wave to end reports
            __threadfence_system();
            if (atomicAdd(&A.ctrl->ended, ended) + ended == A.Q) report_end(A.stats, A.mailbox, A.mail_tag);
        }
    }
}

// Queries with parameters of their own, the ones that are likely to run longest first: the launch ends with its last query,
// and a long one that is taken last has the chip to itself (8,192 ragged queries, whose longest takes as long as the
// others' share of a wave).  Only the order in which waves take queries depends on this.
__global__ void __launch_bounds__(1024) wave_order_kernel(WaveArgs A, int32_t *order) {
    __shared__ int count[256], start[256];
    if (threadIdx.x < 256) count[threadIdx.x] = 0;
    __syncthreads();
    auto bin = [&](int q) {
        const int W = min(max(A.W_q ? A.W_q[q] : A.W, 1), A.W_max), L = min(max(A.L_q ? A.L_q[q] : A.L, 1), A.L_max);
        const int c_own = A.cap_q ? A.cap_q[q] : A.cap, cap = A.cap_max > 0 ? min(max(c_own, 1), A.cap_max) : max(c_own, 0);
        float nodes = 1.5f * L + W;
        if (cap > 0) nodes = fminf(nodes, (float)cap * W);
        const float cost = nodes + 3.f * nodes / W;  // a round costs about as much as three nodes
        return min(max((int)(12.f * log2f(cost)), 0), 255);
    };
    for (int q = threadIdx.x; q < A.Q; q += 1024) atomicAdd(&count[bin(q)], 1);
    __syncthreads();
    if (threadIdx.x == 0)
        for (int b = 255, at = 0; b >= 0; --b) start[b] = at, at += count[b];
    __syncthreads();
    for (int q = threadIdx.x; q < A.Q; q += 1024) order[atomicAdd(&start[bin(q)], 1)] = q;
}

// Long lists leave room for nw waves a CU where the batch wants more: is it still ahead of the batch path (up to 1,024
// queries: of the workgroup per query, where that serves the call)?  Rounds of a wave get hardly faster when it has its CU to
// itself, so the batch goes through in turns of 256 nw queries, while the batch path spreads every round over the chip;
// that one pays three launches for every round, also for those in which few queries or none are left.  Measured on
// 2 10^6 items with 32 neighbours, without / here, > 1 is a gain; "two", "one": hidden layers:
//   nw = 4  8,192 queries, W = 4, L = 1,024 1.21 (L = 1,200 1.10 at 16,384), W = 8, L = 1,000 1.16, W = 16, L = 1,024 1.07; one
//           8,192, W = 4, L = 3,000 1.27, W = 16 1.09.  With a cap that ends most searches: two 8,192, W = 4, L = 1,200 0.98
//           (2,048 1.40, 4,096 1.18), W = 8, L = 1,000 1.01 (2,048 1.18), but W = 16, L = 1,000 0.91 (4,096 0.92; 2,048 0.97;
//           1,024 1.18, where all are resident; own parameters 1.07); nw = 5, W = 16, L = 900 1.05 (4,096 0.95)
//   nw = 3  two 1,024, W = 4, L = 2,048 1.52, L = 1,300 1.56, W = 8, L = 1,500 1.16, W = 16 1.02; 2,048, W = 4 1.14, W = 8 0.96, W = 16
//           0.86; 4,096, W = 1 1.19, W = 2 1.16, W = 4 0.95; 8,192, W = 1 0.91, W = 2 0.91, W = 4 0.84, W = 16 0.82 (L = 64 with
//           k = 2,000 0.94); one 1,024, W = 4, L = 4,096 1.70; 2,048, W = 4 1.13, W = 8 0.99, W = 16 0.83; 4,096, W = 2 1.24, W = 4 1.04,
//           W = 8 0.97; 8,192, W = 2 1.10, W = 4 1.02, W = 16 0.83; 16,384, W = 1 0.95.  Capped: 1,024, W = 4, L = 2,000 1.07,
//           W = 8, L = 1,500 0.83; 2,048, W = 4 0.98, W = 16 0.71; 4,096, W = 4 0.79; 8,192 0.75; one 2,048, W = 8 0.96; 8,192, W = 16 0.82
//   nw = 2  two 600 and 768, W = 4, L = 3,000 0.87 and 0.89 (W = 2 0.88, W = 8 0.95); 1,024, W = 4 1.19, W = 8 1.00; 2,048, W = 1 1.13,
//           W = 2 0.99, W = 4 0.81, W = 16 0.60; 8,192, W = 8 0.63; one 768, W = 4, L = 6,000 1.55, W = 8 1.24; 1,024, W = 2 1.68, W = 4
//           1.26, W = 8 1.01; 2,048, W = 2 1.06, W = 4 0.84; 8,192, W = 8 0.72.  Capped: two 768 0.68; 1,024, W = 8 0.89; 2,048 0.53 to 0.64
//   nw = 1  two 300 and 512, W = 4, L = 5,000 0.72; 2,048, W = 8 0.37; 8,192 0.34; one 300, W = 4, L = 9,000 1.00, W = 2 1.34; 512,
//           W = 1 1.78, W = 4 1.04; 768 0.75
// Queries with parameters of their own and no cap (the batch path runs all their rounds at the pace of the longest): nw = 3 two
// 4,096 and 8,192, W = 4, L = 2,000 1.74 and 1.43, one 8,192, W = 8, L = 4,000 1.61; nw = 2 two 768, W = 4, L = 3,000 1.06, 1,024, W = 8
// 1.35, 2,048, W = 4 1.48, W = 8 and 16, L = 2,000 1.43, 4,096, W = 8 1.18, 8,192 1.01, W = 16 0.95; nw = 1 512 0.95, 1,024, W = 8, L = 5,000 1.02,
// 2,048, W = 4 0.74.  A cap far beyond the list (the batch path launches all its rounds): nw = 3 two 1,024, W = 16, L = 1,500 1.30,
// 2,048, W = 4 1.44 to 1.70, 8,192, W = 4 1.00; nw = 2 1,024, W = 8, L = 2,000 1.82, 2,048, W = 4, L = 3,000 1.04, 4,096, W = 16 0.70, 8,192,
// W = 8 0.69.  On 2 10^5 and 10^7 items 21 of these points lie within 0.1 of their figures here (the others: two, nw = 4, 8,192, W = 16
// 0.95 and 1.04; 8,192 with own parameters, W = 8 0.99 and 1.06; 4,096 1.85).
static bool few_waves_ahead(const SearchArgs &a, int nw, int wide, bool two) {
    const Plan &p = a.plan;
    const bool own = a.W_q || a.L_q || a.cap_q, capped = p.max_iters_max > 0;
    const bool far_cap = capped && (int64_t)p.max_iters_max * p.W_max >= 2 * (int64_t)p.C, near_cap = capped && !far_cap;
    const int64_t work = (int64_t)p.Q * wide;  // candidates of a round of all queries
    if (nw >= 4) return !(nw == 4 && two && near_cap && !own && wide > 256 && p.Q > 1024);
    if (far_cap || (own && !capped)) return nw >= 2 && work <= (capped ? 1 << 19 : 1 << 21);
    if (nw <= 2 && (near_cap || fused_serves(a))) return false;
    const int more = nw == 3 && !two ? 2 : 1;
    return p.Q <= 512 * nw * nw * more && work <= (int64_t)(near_cap ? 256 : 384) * 256 * nw * more;
}

// Which searches run here, with how many waves a CU.  Both sides measured on 2 10^6 items with 32 neighbours, without ->
// here, ms; beyond 1,024 queries without is the batch path, up to there a workgroup per query (search_fused.hip):
//   64 -> 256 -> 128: 300 queries, W = 4, L = 64 0.94 -> 0.88; 512, W = 4 1.09 -> 0.90, W = 8, L = 512 3.53 -> 3.64; 1,024,
//     W = 1, L = 64 2.1 -> 1.7, W = 16, L = 1,024 6.6 -> 5.8, W = 32 6.4 -> 7.6; 2,048, W = 4, L = 64 2.4 -> 1.4, W = 16, L = 256
//     5.5 -> 4.5, W = 32, L = 1,024 10.4 -> 11.2; 4,096, W = 8, L = 600 13.6 -> 11.0; 8,192, W = 4, L = 512 22.9 -> 17.0;
//   64 -> 256: 512 queries, W = 8, L = 512 2.6 -> 2.8; 1,024, W = 4, L = 64 1.24 -> 0.85; 2,048, W = 4, L = 512 8.3 -> 4.3,
//     W = 8, L = 2,000 17.7 -> 12.4, W = 32 13.9 -> 12.6; 8,192, W = 32, L = 2,000 46.6 -> 42.0; 16,384, W = 4, L = 64
//     7.6 -> 4.5;
//   1,025 to 2,000 queries: W = 4, L = 64 1.9 -> 1.1, W = 1, L = 256 12.1 -> 5.3, W = 16, L = 1,200 11.5 -> 9.7, W = 32, L = 1,000 8.3
//     either way; one hidden layer, W = 4, L = 300 5.5 -> 2.7.
// So: a wave per query from 257 queries on (below, a workgroup per query has a CU to itself), unless a round's pairs are
// many for the number of queries (a wave scores them alone), or long lists leave room for four waves only and rounds are
// wide, or for fewer than the batch wants (few_waves_ahead).
static bool wave_plan(const SearchArgs &a, int *nw, int *piece, WaveArgs *A, size_t *smem) {
    const Plan &p = a.plan;
    const ann_mlp *m = a.m;
    if (a.walkers || a.Q_total != 0 || m->kernel != MLP_MFMA2 || (m->dtype != ANN_BF16 && m->dtype != ANN_F16)) return false;
    if (m->d_item != 64 || m->dims[1] != 256 || (m->n_layers == 3 && m->dims[2] != 128)) return false;
    const int wide = p.W_max * p.R;  // candidates of a round
    if (p.Q <= 256) return false;
    if (p.Q <= 1024 && p.Q <= 2 * wide && (p.Q <= 768 || wide > 512)) return false;
    if (((uintptr_t)a.g->emb & 15) != 0) return false;
    const bool two = m->n_layers == 3;
    const size_t weights = two ? 104 * 1024 + 576 : 48 * 1024 + 64;
    *piece = wide > 128 ? 256 : 128;
    auto up16 = [](size_t v) { return (v + 15) & ~(size_t)15; };
    const size_t at_keys = up16((size_t)p.C * 8), at_taken = at_keys + (size_t)(*piece + KEYS_SLACK) * 8, at_ut = at_taken + up16((size_t)((p.C + 63) >> 6) * 8),
                 at_parents = at_ut + 1024, bytes = at_parents + up16((size_t)p.W_max * 4);
    *nw = 0;
    const int fit = (int)((160 * 1024 - weights) / bytes), most = two ? 8 : 16, want = (p.Q + 255) / 256;
    *nw = fit < most ? fit : most;
    if (*nw > want) *nw = want;
    if (*nw < 1 || (*nw <= 4 && wide > 512)) return false;
    if (*nw < want && *nw < most && !few_waves_ahead(a, *nw, wide, two)) return false;
    A->wave_off = (int32_t)weights;
    A->wave_bytes = (int32_t)bytes;
    A->at_keys = (int32_t)at_keys;
    A->at_taken = (int32_t)at_taken;
    A->at_ut = (int32_t)at_ut;
    A->at_parents = (int32_t)at_parents;
    *smem = weights + *nw * bytes;
    return true;
}

bool wave_serves(const SearchArgs &a) {
    WaveArgs A{};
    int nw, piece;
    size_t smem;
    return wave_plan(a, &nw, &piece, &A, &smem);
}

template <bool TWO, bool F16, int MOST, int U>
static int wave_launch(const SearchArgs &a, const WaveArgs &A, int nw, size_t smem) {
    const bool bm = a.plan.bitmap_words > 0;
    auto fn = bm ? wave_search_kernel<TWO, F16, true, MOST, U> : wave_search_kernel<TWO, F16, false, MOST, U>;
    static std::atomic<uint32_t> raised[2];
    if (int rc = raise_lds_limit((const void *)fn, 160 * 1024, a.m->device, raised[bm ? 1 : 0]); rc != ANN_OK) return rc;
    hipLaunchKernelGGL(fn, dim3(256), dim3(64 * nw), smem, a.stream, A);
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

int launch_wave(const SearchArgs &a, int32_t rounds_max) {
    const Plan &p = a.plan;
    const ann_mlp *m = a.m;
    WaveArgs A{};
    int nw, piece;
    size_t smem;
    if (!wave_plan(a, &nw, &piece, &A, &smem)) return ANN_EINVAL;
    const bool two = m->n_layers == 3, f16 = m->dtype == ANN_F16, bm = p.bitmap_words > 0;
    A.frag = (const uint4 *)m->frag_dev;
    A.b2 = two ? m->b_dev + m->b_off[1] : nullptr;
    A.b_head = m->b_dev + m->b_off[m->n_layers - 1];
    A.upre = (const float *)(a.ws + p.off_upre);
    for (int j = 0; j < m->J; ++j) A.head_w[j] = m->head_w[j];
    A.emb = (const uint16_t *)a.g->emb;
    A.adj = a.g->adj;
    A.adj_rank = bm ? a.g->adj_rank : nullptr;
    A.rank = bm && a.g->adj_rank ? a.g->rank : nullptr;
    A.entries = a.entries;
    A.W_q = a.W_q, A.L_q = a.L_q, A.cap_q = a.cap_q;
    A.table = (uint32_t *)(a.ws + p.off_hash);
    A.stats = (int64_t *)(a.ws + p.off_stats);
    A.ctrl = (Ctrl *)(a.ws + p.off_ctrl);
    A.out_ids = a.out_ids;
    A.out_scores = a.out_scores;
    A.mailbox = a.mailbox;
    A.mail_tag = a.mail_tag;
    A.N = a.g->N;
    A.R_magic = (uint32_t)((0x100000000ull + (uint64_t)p.R - 1) / (uint64_t)p.R);
    A.J = m->J, A.R = p.R, A.E = p.E, A.W = a.W, A.L = a.L, A.cap = a.cap;
    A.W_max = p.W_max, A.L_max = p.L_max, A.cap_max = p.max_iters_max;
    A.C = p.C, A.k = p.k;
    A.table_words = bm ? p.bitmap_words : p.hash_cap;
    A.hash_cap = p.hash_cap;
    A.Q = p.Q;
    A.rounds_max = rounds_max;
    A.state = (QState *)(a.ws + p.off_state);
    A.pool = (uint64_t *)(a.ws + p.off_pool);
    A.handed = (int32_t *)(a.ws + p.off_offsets);  // [Q], unused by this path otherwise
    A.hand_at = p.max_iters_max == 0 && fused_goes_on(a, WAVE_HAND) ? WAVE_HAND : 0;
    if (int rc = launch_zero_stats(a, 0, p.Q); rc != ANN_OK) return rc;
    if (a.W_q || a.L_q || a.cap_q) {
        int32_t *order = (int32_t *)(a.ws + p.off_counts);  // [Q], unused by this path otherwise
        hipLaunchKernelGGL(wave_order_kernel, dim3(1), dim3(1024), 0, a.stream, A, order);
        ANN_HIP_TRY(hipGetLastError());
        A.order = order;
    }
#define WAVE_PICK(TWO, F16, MOST) (piece > 128 ? wave_launch<TWO, F16, MOST, 4>(a, A, nw, smem) : wave_launch<TWO, F16, MOST, 2>(a, A, nw, smem))
    int rc = ANN_OK;
    if (two && f16) rc = nw <= 4 ? WAVE_PICK(true, true, 4) : WAVE_PICK(true, true, 8);
    else if (two) rc = nw <= 4 ? WAVE_PICK(true, false, 4) : WAVE_PICK(true, false, 8);
    else if (f16) rc = nw <= 4 ? WAVE_PICK(false, true, 4) : nw <= 8 ? WAVE_PICK(false, true, 8) : WAVE_PICK(false, true, 16);
    else rc = nw <= 4 ? WAVE_PICK(false, false, 4) : nw <= 8 ? WAVE_PICK(false, false, 8) : WAVE_PICK(false, false, 16);
    if (rc != ANN_OK || A.hand_at == 0) return rc;
    return launch_fused_rest(a, rounds_max, WAVE_HAND);
#undef WAVE_PICK
}

}  // namespace gmpgr
