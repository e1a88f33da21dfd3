// Per-query search state machine of the joint best-first search (Sec. 3.2, Algorithm 1)
// and the packing of ragged survivor groups into one dense pair list (Algorithm 2).
//
// One workgroup owns one query in every kernel here: its sorted candidate list (the shared
// container of Algorithm 1), its exact visited table and its survivors of the current round.
// Per round:   scan_compact -> (MLP kernel) -> round
//   round       : merge the scores of the previous round into the list, test termination,
//                 pick <= W unexpanded entries among the first L ranks, read their adjacency
//                 rows, drop out-of-range / repeated / already scored ids, keep the rest as
//                 this query's survivors
//   scan_compact: exclusive prefix sum of the survivor counts over all queries and a stable
//                 copy of every group into the dense pair list (query-major, first-found
//                 first), which the MLP kernel cuts into fixed-size batches
#include "common.h"
#include "keys.h"
#include "search_device.h"

namespace gmpgr {

// Threads per query in the per-query kernels (seeding, round, output).
#ifndef QUERY_BLOCK
#define QUERY_BLOCK 256
#endif
constexpr int BLOCK = QUERY_BLOCK;     // largest workgroup of the per-query kernels (launch bound, LDS sizing)
constexpr int WAVES = BLOCK / 64;
// The functions below are templates over the workgroup size BLK: the round kernel is also built for
// half-size workgroups (see launch_round).
#ifndef ROUND_BIG_FROM
#define ROUND_BIG_FROM 512   // candidates per query and round above which the round kernel runs larger workgroups
#endif
#ifndef FILTER_CHUNK
#define FILTER_CHUNK 1024   // candidates of a round that pass an ordered visited filter together
#endif
#ifndef ROUND_TILE_MAX
#define ROUND_TILE_MAX 4096   // most list entries held in LDS at a time during the merge
#endif
#ifndef ROUND_WAVES_MIN
#define ROUND_WAVES_MIN 8     // waves per SIMD the round kernel is compiled for (8: at most 64 registers per lane)
#endif
#ifndef ROUND_BIG_BLOCK
#define ROUND_BIG_BLOCK 512
#endif
constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_WAVES = SCAN_BLOCK / 64;

// Phase timing of the round kernel for measurement builds (-DROUND_TIMING): thread 0 of every
// 64th workgroup adds the shader-clock ticks of each phase to counters 9..15 of the stats block
// (every workgroup doing so would serialise on those few addresses and distort what is measured).
#ifdef ROUND_TIMING
#define PHASE_MARK(k)                                                                          \
    do {                                                                                       \
        if (threadIdx.x == 0 && (blockIdx.x & 63) == 0) {                                      \
            long long now_ = clock64();                                                        \
            atomicAdd((unsigned long long *)&stats[9 + (k)], (unsigned long long)(now_ - t_)); \
            t_ = now_;                                                                         \
        }                                                                                      \
    } while (0)
#define PHASE_START long long t_ = clock64();
#else
#define PHASE_MARK(k)
#define PHASE_START
#endif

// Counters and control block start at zero (a kernel, not a memset, so that a caller may
// capture the launch sequence into a HIP graph).
// stats[5], stats[6]: bytes of one adjacency row and of one item row, from which ann_search_stats derives the
// algorithmic bytes of the gather stages.  stats[7]: queries that a workgroup ran to their end (search_fused.hip), stats[8]:
// queries that waves were given (search_wave.hip; the last ones of a batch may count in both).
__global__ void zero_stats_kernel(int64_t *stats, Ctrl *ctrl, int Q, int keep_stats, int adj_row_bytes,
                                  int item_row_bytes, int one_launch, int by_waves) {
    if (threadIdx.x < 16 && !keep_stats)
        stats[threadIdx.x] = threadIdx.x == 4 ? Q : threadIdx.x == 5 ? adj_row_bytes : threadIdx.x == 6 ? item_row_bytes : 0;
    if (threadIdx.x == 7) stats[7] += one_launch;  // the thread that has just cleared it
    if (threadIdx.x == 8) stats[8] += by_waves;
    if (threadIdx.x < 16) ((int32_t *)ctrl)[threadIdx.x] = 0;
}

// ------------------------------------------------------------------------------------------
// Seeding: clear the visited table, keep the distinct in-range entry ids as the survivors of
// "round 0" (they are scored by the first MLP launch and merged by the first round kernel).
// `slot` names the search state that is set up, `query` the row of entries / per-query parameters.
// WALKERS is compile-time: with both forms in one body the kernels took 120 registers and a spill, four waves a SIMD instead of eight
// (4,096 bitmaps of 10^7 items 912 us, now 896; admission to 2,047 slots 10.6 us, now 8.6).
template <int BLK, bool WALKERS>
__device__ void seed_slot(int slot, int query, const int32_t *__restrict__ entries, const int32_t *__restrict__ rank,
                          int E, int64_t N, QState *state, uint32_t *hash, int hash_cap, int32_t *cand_g, int slots,
                          int32_t *counts,
                          const int32_t *W_q, const int32_t *L_q, const int32_t *cap_q, int W, int L, int cap,
                          int W_max, int L_max, int cap_max, unsigned char *smem, uint16_t *tag_g) {
    const int table_words = hash_cap < 0 ? -hash_cap : hash_cap;  // a multiple of 64, the table 256-byte aligned
    uint32_t *table = hash + (size_t)slot * table_words;
    {
        uint4 *t4 = (uint4 *)table;
        const uint32_t e = hash_cap < 0 ? 0u : EMPTY_SLOT;  // bitmap: no bit set; hash table: every slot free
        const uint4 e4 = make_uint4(e, e, e, e);
        for (int i = threadIdx.x; i < table_words / 4; i += BLK) t4[i] = e4;
    }
    visited_cleared();
    int32_t *out = cand_g + (size_t)slot * slots;
    const int32_t *seeds = entries + (size_t)query * E;
    int n;
    if constexpr (WALKERS) {  // the first of equal seeds starts one (see filter_and_insert, filter_and_mark)
        int dd_n = 2;
        while (dd_n < 2 * E) dd_n <<= 1;
        int32_t *cand = (int32_t *)smem;                                // [E]
        int32_t *cand_rank = rank ? cand + ((E + 3) & ~3) : nullptr;    // [E] the seeds' places in the visited bitmap
        uint32_t *dd_key = (uint32_t *)(cand + (rank ? 2 : 1) * ((E + 3) & ~3));
        uint32_t *dd_pos = dd_key + dd_n, *bk_key = dd_pos + dd_n, *bk_cnt = bk_key + dd_n;
        int *wave_sums = (int *)(bk_cnt + dd_n);
        uint16_t *tag = tag_g + (size_t)slot * slots;
        for (int i = threadIdx.x; i < E; i += BLK) {
            const int32_t v = seeds[i];
            cand[i] = v;
            if (rank) cand_rank[i] = (v >= 0 && (int64_t)v < N) ? rank[v] : -1;
        }
        __syncthreads();
        if (hash_cap < 0)
            n = filter_and_mark<BLK>(cand, cand_rank, E, dd_key, dd_pos, bk_key, bk_cnt, dd_n, table, N, out, wave_sums, tag, 1, 0);
        else
            n = filter_and_insert<BLK>(cand, E, dd_key, dd_pos, bk_key, bk_cnt, dd_n, table, hash_cap, N, out, wave_sums, tag, 1, 0);
    } else {
        auto seed = [&](int p, uint32_t *bit) {
            const int32_t v = seeds[p];
            if (hash_cap < 0) *bit = rank && v >= 0 && (int64_t)v < N ? (uint32_t)rank[v] : (uint32_t)v;
            return v;
        };
        int *wave_sums = (int *)smem;
        n = hash_cap < 0 ? visit<BLK, true, false, 1>(seed, E, table, 0, N, out, wave_sums, Nothing{})
                         : visit<BLK, false, false, 1>(seed, E, table, hash_cap, N, out, wave_sums, Nothing{});
    }
    if (threadIdx.x == 0) {
        QState s;
        s.t = 0;
        s.done = 0;
        s.n_list = 0;
        s.n_visited = n;
        int w = W_q ? W_q[query] : W, l = L_q ? L_q[query] : L, c = cap_q ? cap_q[query] : cap;
        s.W = min(max(w, 1), W_max);
        s.L = min(max(l, 1), L_max);
        s.cap = cap_max > 0 ? min(max(c, 1), cap_max) : max(c, 0);
        s.n_expanded = 0;
        s.first_open = 0;
        s.pad[0] = s.pad[1] = s.pad[2] = 0;
        state[slot] = s;
        counts[slot] = n;
    }
}

template <bool WALKERS>
__global__ void __launch_bounds__(BLOCK)
init_kernel(const int32_t *__restrict__ entries, const int32_t *__restrict__ rank, int E, int64_t N, QState *state,
            uint32_t *hash,
            int hash_cap, int32_t *cand_g, int slots, int32_t *counts, const int32_t *W_q,
            const int32_t *L_q, const int32_t *cap_q, int W, int L, int cap, int W_max, int L_max,
            int cap_max, uint16_t *tag_g) {
    extern __shared__ __align__(16) unsigned char smem[];
    seed_slot<BLOCK, WALKERS>(blockIdx.x, blockIdx.x, entries, rank, E, N, state, hash, hash_cap, cand_g, slots, counts, W_q, L_q, cap_q, W,
              L, cap, W_max, L_max, cap_max, smem, tag_g);
}

// First k entries of a slot's list to row `row` of the outputs, padded with (-1, -inf).
template <int BLK>
__device__ void emit_row(const QState *state, const uint64_t *pool_g, int C, int k, int slot, int64_t row,
                         int32_t *out_ids, float *out_scores) {
    const int n = state[slot].n_list;
    const uint64_t *pool = pool_g + (size_t)slot * C;
    for (int i = threadIdx.x; i < k; i += BLK) {
        int32_t id = -1;
        float sc = -INFINITY;
        if (i < n) {
            uint64_t key = pool[i];
            id = key_id(key);
            sc = key_score(key);
        }
        out_ids[(size_t)row * k + i] = id;
        out_scores[(size_t)row * k + i] = sc;
    }
}

// ------------------------------------------------------------------------------------------
// Continuous batching (Sec. 3.2, Q-HiPANNS: requests arrive and finish at different times and are
// aggregated into common batches).  The search state lives in slots; a slot whose query has
// finished writes that query's result and takes the next waiting query, in index order (a
// counter is the queue).  Runs before the packing step of every round.
__global__ void stream_reset_kernel(int64_t *stats, Ctrl *ctrl, QState *state, int32_t *counts, int32_t *slot_query,
                                    int S, int Q_total, int adj_row_bytes, int item_row_bytes) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 16) {
        stats[i] = i == 4 ? max(Q_total, 0) : i == 5 ? adj_row_bytes : i == 6 ? item_row_bytes : 0;
        ((int32_t *)ctrl)[i] = 0;
    }
    if (i < S) {
        QState s = {};
        s.done = 1;
        state[i] = s;
        counts[i] = -1;
        slot_query[i] = -1;
    }
}

// Open stream: queries [0, avail) have arrived (their rows in the query, entry and user-term arrays are valid).
// A kernel, so that the word changes in stream order behind the work that made the rows valid.
__global__ void stream_publish_kernel(Ctrl *ctrl, int64_t *stats, int avail) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        ctrl->avail = avail;
        stats[4] = avail;
    }
}

__global__ void __launch_bounds__(BLOCK)
admit_kernel(const int32_t *__restrict__ entries, const int32_t *__restrict__ rank, int E, int64_t N, QState *state,
             uint32_t *hash, int hash_cap,
             int32_t *cand_g, int slots, int32_t *counts, const int32_t *W_q, const int32_t *L_q,
             const int32_t *cap_q, int W, int L, int cap, int W_max, int L_max, int cap_max, int64_t *stats,
             Ctrl *ctrl, int32_t *slot_query, int Q_total, const uint64_t *pool_g, int C, int k, int32_t *out_ids,
             float *out_scores) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int next_s;
    const int slot = blockIdx.x;
    if (!state[slot].done) return;  // still searching
    const int served = slot_query[slot];
    if (served >= 0) {
        emit_row<BLOCK>(state, pool_g, C, k, slot, served, out_ids, out_scores);
        if (threadIdx.x == 0) {
            const QState st = state[slot];
            add_to_totals(stats, st.n_visited, st.n_expanded, st.t, (st.done & 2) ? 1 : 0);
        }
    }
    __syncthreads();  // every wave has read which query the slot served before thread 0 names the next one
    if (threadIdx.x == 0) {
        int next;
        if (Q_total >= 0) {
            next = Q_total;
            // the counter only grows; once it has passed the total nobody needs to touch it again
            if (*(volatile int32_t *)&ctrl->next_query < Q_total) next = atomicAdd(&ctrl->next_query, 1);
            next = next < Q_total ? next : -1;
        } else {
            // open stream: the number of queries that have arrived (ctrl->avail) grows while the search runs, so
            // the counter must never pass it: a query index claimed before its query exists would be lost
            const int avail = *(volatile int32_t *)&ctrl->avail;
            int cur = *(volatile int32_t *)&ctrl->next_query;
            next = -1;
            while (cur < avail) {
                const int seen = atomicCAS(&ctrl->next_query, cur, cur + 1);
                if (seen == cur) {
                    next = cur;
                    break;
                }
                cur = seen;
            }
        }
        next_s = next;
        slot_query[slot] = next_s;
        if (next_s < 0) counts[slot] = -1;  // idle: contributes no pairs, is not counted as running
    }
    __syncthreads();  // also: the list of the served query has been read before the slot is re-seeded
    const int next = next_s;
    if (next < 0) return;
    seed_slot<BLOCK, false>(slot, next, entries, rank, E, N, state, hash, hash_cap, cand_g, slots, counts, W_q, L_q, cap_q, W, L, cap,
              W_max, L_max, cap_max, smem, nullptr);
}

// ------------------------------------------------------------------------------------------
// Exclusive scan of survivor counts + stable packing into the dense pair list (Algorithm 2).
// A workgroup owns SCAN_QPB consecutive queries (4 or 8: few, so that many workgroups share the
// copying).  It first sums the counts of all earlier queries (every workgroup re-reads them from
// L2: O(Q^2 / SCAN_QPB) four-byte reads in total, no waiting on other workgroups, the same result
// every run), then scans its own counts and copies its groups, one wave per query at a time.
template <int SCAN_QPB>  // queries per workgroup, a multiple of 4
__global__ void __launch_bounds__(SCAN_BLOCK)
scan_compact_kernel(const int32_t *__restrict__ counts, int Q, const int32_t *__restrict__ cand_g, int slots,
                    int32_t *offsets, int32_t *pair_q, int32_t *pair_id, Ctrl *ctrl,
                    const int32_t *__restrict__ slot_query, uint64_t *mailbox, uint64_t mail_word, int Q_total) {
    __shared__ int red[SCAN_WAVES];
    __shared__ int red_active[SCAN_WAVES];
    __shared__ int loc_off[SCAN_QPB + 1];
    __shared__ int loc_cnt[SCAN_QPB];
    const int q0 = blockIdx.x * SCAN_QPB;
    const bool last = (blockIdx.x == gridDim.x - 1);
    // pairs of all earlier queries (and, in the last workgroup, the number of running queries)
    int sum = 0, act = 0;
    const int lim = last ? Q : q0;
    // q0 is a multiple of 4 and the array is 256-byte aligned: four counts per load up to q0
    const int4 *counts4 = (const int4 *)counts;
    for (int i4 = threadIdx.x; i4 < (q0 >> 2); i4 += SCAN_BLOCK) {
        const int4 c = counts4[i4];
        sum += max(c.x, 0) + max(c.y, 0) + max(c.z, 0) + max(c.w, 0);
        act += (c.x >= 0) + (c.y >= 0) + (c.z >= 0) + (c.w >= 0);
    }
    for (int i = q0 + threadIdx.x; i < lim; i += SCAN_BLOCK) act += (counts[i] >= 0);  // last workgroup only
    for (int o = 32; o > 0; o >>= 1) {
        sum += __shfl_down(sum, o);
        act += __shfl_down(act, o);
    }
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = sum;
        red_active[threadIdx.x >> 6] = act;
    }
    __syncthreads();
    int prefix = 0, n_active = 0;
    for (int w = 0; w < SCAN_WAVES; ++w) {
        prefix += red[w];
        n_active += red_active[w];
    }
    if (threadIdx.x < 64) {
        int q = q0 + threadIdx.x;
        int c = (threadIdx.x < SCAN_QPB && q < Q) ? max(counts[q], 0) : 0;
        int inc = c;
        for (int o = 1; o < SCAN_QPB; o <<= 1) {
            int v = __shfl_up(inc, o);
            if ((int)threadIdx.x >= o) inc += v;
        }
        if (threadIdx.x < SCAN_QPB) {
            loc_cnt[threadIdx.x] = c;
            loc_off[threadIdx.x] = prefix + inc - c;
            if (threadIdx.x == SCAN_QPB - 1) loc_off[SCAN_QPB] = prefix + inc;
            if (q < Q) offsets[q] = prefix + inc - c;
        }
    }
    __syncthreads();
    if (last && threadIdx.x == 0) {
        ctrl->M = loc_off[SCAN_QPB];
        ctrl->n_active = n_active;
        if (mailbox) {
            // progress for the enqueuing host thread: one store to pinned host memory, nobody waits for it
            // nothing running and nothing waiting (open stream, Q_total < 0: nothing that has arrived so far)
            const int waiting_until = Q_total >= 0 ? Q_total : *(volatile int32_t *)&ctrl->avail;
            const bool finished = n_active == 0 && (Q_total == 0 || ctrl->next_query >= waiting_until);
            if (Q_total == 0 || (Q_total > 0 && ctrl->next_query >= Q_total))
                __hip_atomic_store(mailbox + MAIL_RUNNING, (mail_word >> 40 << 40) | (uint32_t)n_active, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(mailbox + MAIL_ROUNDS, mail_word | (finished ? 1ull : 0ull), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = wave; i < SCAN_QPB; i += SCAN_WAVES) {
        int q = q0 + i;
        if (q >= Q) break;
        int c = loc_cnt[i], off = loc_off[i];
        const int32_t *src = cand_g + (size_t)q * slots;
        const int32_t user = slot_query ? slot_query[q] : q;  // whose user vector scores this group
        for (int j = lane; j < c; j += 64) {
            pair_id[off + j] = src[j];
            pair_q[off + j] = user;
        }
    }
}

// ------------------------------------------------------------------------------------------
// One round of one query.
//
// The list (a6) lives in global memory, sorted; LDS holds only the new entries of the round and one
// tile of the list at a time, so the list may be as long as the workspace allows.
//
// Merge.  Only new entries that can enter the list are kept (better than the current worst entry once
// the list is full) and sorted on their own (<= W*R keys).  The list is then walked in tiles from its
// END towards the front: a tile of old entries is read into LDS, every old entry moves up by the number
// of new entries that precede it, every new entry that falls behind the tile's first entry goes to its
// own index plus the number of old entries that precede it (one binary search per entry in each
// direction), and the walk stops at the tile that takes the smallest new entry: the ranks in front of
// it do not change and are neither read nor written.  Moving entries towards the end while walking
// towards the front never overwrites an entry that has not been read yet, so the merge is in place.
// Keys are unique (an id is scored once per query), so the destinations are a permutation.
//
// Choice of parents.  The state keeps `first_open`, a rank below which every entry has been expanded
// (a lower bound of the first unexpanded rank: it falls to the first insertion point of a round and
// otherwise only grows).  The scan for the first <= W unexpanded entries among the first L ranks starts
// there, reading the list in pieces of one entry per thread (four per thread after the first piece).
// Eight workgroups of 256 threads fill a CU's wave slots; that needs no more than 64 registers per lane.
// BITMAP: the visited set is one bit per item (hash_cap < 0), else the hash table.  RESIDENT: the whole list fits one tile
// (C <= tile_keys); it is then requested at the very start, together with the state, merged into a second LDS copy, and
// the parents are chosen from that copy: two dependent trips to memory fewer per round than the tiled walk, which is what
// short lists are bound by.  FILTER: see filter_of.
enum { FILTER_ATOMIC = 0, FILTER_ORDERED = 1, FILTER_WALKERS = 2 };
template <int BLK, bool BITMAP, bool RESIDENT, int FILTER>
__global__ void __launch_bounds__(BLK) __attribute__((amdgpu_waves_per_eu(ROUND_WAVES_MIN, 8)))
round_kernel(const int32_t *__restrict__ adj, const int32_t *__restrict__ adj_rank, int R, int64_t N, QState *state,
             uint64_t *pool_g, int C,
             uint32_t *hash, int hash_cap, int32_t *cand_g, int slots, int32_t *counts,
             const int32_t *__restrict__ offsets, const float *__restrict__ scores, int new_cap,
             int W_max, int64_t *stats, uint16_t *tag_g, int tile_keys, int chunk) {
    constexpr bool WALKERS = FILTER == FILTER_WALKERS;
    extern __shared__ __align__(16) unsigned char smem[];
    const int q = blockIdx.x;
    PHASE_START
    // LDS: parents and scan scratch first; then one region used twice: by the new entries and the list
    // tile during the merge, by the candidate ids and the dedupe tables afterwards
    int32_t *parents = (int32_t *)smem;                       // [W_max]
    int *wave_sums = parents + ((W_max + 3) & ~3);            // [16] one per wave
    int *shared_i = wave_sums + 16;                           // [8] values one thread hands to all
    uint64_t *newk = (uint64_t *)(shared_i + 8);              // [new_cap]   new entries, sorted
    uint64_t *best = newk + new_cap;                          // [W_max]     walkers: best new child of each
    uint64_t *tile = best + ((W_max + 1) & ~1);               // [tile_keys] a piece of the stored list
    uint64_t *merged = tile + tile_keys;                      // [C]         RESIDENT only: the list after the merge
    uint64_t *pool = pool_g + (size_t)q * C;
    int32_t *cand_q = cand_g + (size_t)q * slots;
    uint16_t *tag_q = WALKERS ? tag_g + (size_t)q * slots : nullptr;

    // Everything the round needs first is requested at once, before any of it is looked at: the
    // workgroups of a launch start together, and every dependent trip to memory costs them all a few
    // microseconds.  (The worst entry is read whether or not the list is full: C >= 1.)
    const int n_prev = __builtin_amdgcn_readfirstlane(counts[q]);
    QState st = state[q];
    const int off = __builtin_amdgcn_readfirstlane(offsets[q]);
    const uint64_t stored_worst = RESIDENT ? 0 : pool[C - 1];
    if (n_prev < 0) return;  // finished or idle: counts[q] stays -1
    // the state is the same in every lane: kept in scalar registers, it leaves the vector registers to the filter
    st.t = __builtin_amdgcn_readfirstlane(st.t);
    st.done = __builtin_amdgcn_readfirstlane(st.done);
    st.n_list = __builtin_amdgcn_readfirstlane(st.n_list);
    st.n_visited = __builtin_amdgcn_readfirstlane(st.n_visited);
    st.W = __builtin_amdgcn_readfirstlane(st.W);
    st.L = __builtin_amdgcn_readfirstlane(st.L);
    st.cap = __builtin_amdgcn_readfirstlane(st.cap);
    st.n_expanded = __builtin_amdgcn_readfirstlane(st.n_expanded);
    st.first_open = __builtin_amdgcn_readfirstlane(st.first_open);
    if (RESIDENT) {  // the whole list, not only its n_list valid entries: requested before the state has arrived
#pragma unroll 4
        for (int i = threadIdx.x; i < C; i += BLK) tile[i] = pool[i];
    }
    if (st.done) {
        if (threadIdx.x == 0) counts[q] = -1;
        return;
    }
    if (WALKERS)
        for (int i = threadIdx.x; i < W_max; i += BLK) best[i] = KEY_SENTINEL;
    if (threadIdx.x == 0) shared_i[0] = 0x7fffffff;  // rank of the first inserted entry
    __syncthreads();
    PHASE_MARK(0);  // state load

    // 1. the scores of the previous round (or of the seeds) become keys; those that cannot enter are dropped
    const bool full = (st.n_list == C);
    const uint64_t worst = full ? (RESIDENT ? tile[C - 1] : stored_worst) : KEY_SENTINEL;
    int m = 0;
    for (int j0 = 0; j0 < n_prev; j0 += BLK) {
        int j = j0 + threadIdx.x;
        uint64_t key = KEY_SENTINEL;
        bool keep = false;
        if (j < n_prev) {
            key = make_key(scores[off + j], cand_q[j], 0u);
            keep = key < worst;
            // walkers: the best newly scored neighbour of each walker, whether it enters the list or not
            if (WALKERS) atomicMin((unsigned long long *)&best[tag_q[j]], (unsigned long long)key);
        }
        int tot;
        int pos = block_excl_count<BLK>(keep, wave_sums, &tot);
        if (keep) newk[m + pos] = key;
        m += tot;
    }
    PHASE_MARK(1);  // new keys: scores load + filter
    int n_list = st.n_list;
    if (m > 0) {
        if (m <= BLK && 2 * tile_keys >= BLK && (!RESIDENT || 2 * C >= BLK)) {
            // scratch: a buffer that is free until the merge below
            rank_sort<BLK>(newk, m, (uint32_t *)(RESIDENT ? merged : tile));
        } else {
            int m2 = 2;
            while (m2 < m) m2 <<= 1;
            for (int i = m + threadIdx.x; i < m2; i += BLK) newk[i] = KEY_SENTINEL;
            __syncthreads();
            bitonic_sort<BLK>(newk, m2);
        }
        PHASE_MARK(6);  // sort of the new keys
        // 1b. merge into the stored list
        if (RESIDENT) {
            // by rank, into the second copy: an entry's position is its index in its own sequence plus the number
            // of entries of the other sequence in front of it
            for (int i = threadIdx.x; i < st.n_list + m; i += BLK) {
                uint64_t key;
                int pos;
                if (i < st.n_list) {
                    key = tile[i];
                    pos = i + lower_bound_keys(newk, m, key);
                } else {
                    key = newk[i - st.n_list];
                    pos = (i - st.n_list) + lower_bound_keys(tile, st.n_list, key);
                    if (i == st.n_list) shared_i[0] = pos;  // rank of the first inserted entry
                }
                if (pos < C) merged[pos] = key;
            }
        }
        // tile by tile from the end
        int hi = st.n_list, rem = RESIDENT ? 0 : m;
        while (rem > 0) {
            const int lo = max(0, hi - tile_keys), cnt = hi - lo;
            for (int i = threadIdx.x; i < cnt; i += BLK) tile[i] = pool[lo + i];
            __syncthreads();
            // new entries [0, nlo) precede the tile's first entry: they belong to tiles further front
            const int nlo = (lo == 0) ? 0 : lower_bound_keys(newk, rem, tile[0]);
            for (int i = threadIdx.x; i < cnt; i += BLK) {
                const uint64_t key = tile[i];
                const int lb = nlo + lower_bound_keys(newk + nlo, rem - nlo, key);
                const int dest = lo + i + lb;
                if (lb > 0 && dest < C) pool[dest] = key;  // lb = 0: the entry stays where it is
            }
            for (int j = nlo + threadIdx.x; j < rem; j += BLK) {
                const uint64_t key = newk[j];
                const int dest = j + lo + lower_bound_keys(tile, cnt, key);
                if (dest < C) pool[dest] = key;
                if (j == 0) shared_i[0] = dest;
            }
            __syncthreads();  // the tile buffer is free again
            hi = lo;
            rem = nlo;
        }
        n_list = min(C, st.n_list + m);
        // the scan below reads entries this workgroup has just stored
        if (!RESIDENT) __threadfence_block();
        __syncthreads();
    }
    PHASE_MARK(2);  // rank merge
    // RESIDENT: the list as it stands now, in LDS
    uint64_t *lw = RESIDENT ? (m > 0 ? merged : tile) : nullptr;

    // 2. termination test and choice of the parents
    int n_par = 0, n_live = 0;
    const bool capped = (st.cap > 0 && st.t >= st.cap);
    const int lim = WALKERS ? 0 : min(st.L, n_list);
    int first_open = min(st.first_open, shared_i[0]);
    if (WALKERS && !capped) {
        // Paper-literal variant (Alg. 1 read as independent walkers): walker s moves to the best of the
        // neighbours it scored last round (round 0: to its seed); a walker without one is dead (-1) and
        // contributes R invalid candidates, so that candidate position / R keeps naming the walker.
        for (int s0 = 0; s0 < st.W; s0 += BLK) {
            const int sl = s0 + threadIdx.x;
            const bool live = sl < st.W && best[sl] != KEY_SENTINEL;
            if (sl < st.W) parents[sl] = live ? key_id(best[sl]) : -1;
            int tot;
            (void)block_excl_count<BLK>(live, wave_sums, &tot);
            n_live += tot;
        }
        n_par = n_live > 0 ? st.W : 0;
    }
    if (!capped && !WALKERS) {
        int i0 = first_open;
        bool first_piece = true;
        while (i0 < lim && n_par < st.W) {
            // one entry per thread in the first piece (the parents are nearly always found there), four in the
            // later ones: all four are requested before the first is looked at
            const int per = first_piece ? 1 : 4;
            uint64_t e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * BLK + (int)threadIdx.x;
                e[u] = (u < per && i < lim) ? (RESIDENT ? lw[i] : pool[i]) : KEY_SENTINEL;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (u >= per || i0 >= lim || n_par >= st.W) break;  // uniform over the workgroup
                const int i = i0 + (int)threadIdx.x;
                const bool open = (i < lim) && !key_expanded(e[u]);
                int tot;
                const int pos = block_excl_count<BLK>(open, wave_sums, &tot);
                if (open && n_par + pos < st.W) {
                    parents[n_par + pos] = key_id(e[u]);
                    pool[i] = e[u] | 1ull;
                    if (RESIDENT) lw[i] = e[u] | 1ull;  // the ranks from the first inserted entry on are stored below
                    if (n_par + pos == st.W - 1) shared_i[1] = i + 1;  // everything in front of it is expanded now
                }
                first_open = (n_par + tot >= st.W) ? -1 : min(i0 + BLK, lim);  // -1: taken from shared_i[1] below
                n_par = min(st.W, n_par + tot);
                i0 += BLK;
            }
            first_piece = false;
        }
    }
    __syncthreads();
    if (first_open < 0) first_open = shared_i[1];
    if (RESIDENT && m > 0)  // what the merge moved: the ranks from the first inserted entry on
        for (int i = shared_i[0] + threadIdx.x; i < n_list; i += BLK) pool[i] = lw[i];
    // a visited table that could not take this round's ids ends the query
    bool overflow = false;
    if (!BITMAP && n_par > 0 && (int64_t)st.n_visited + (int64_t)n_par * R > (int64_t)(hash_cap / 2)) {
        overflow = true;
        n_par = 0;
    }
    if (n_par == 0) {
        if (threadIdx.x == 0) {
            state[q].n_list = n_list;
            state[q].first_open = first_open;
            state[q].done = overflow ? 3 : 1;
            counts[q] = -1;
        }
        return;
    }

    // 3. neighbour gather: one adjacency row per parent, consecutive lanes read consecutive ids;
    // 4. visited filter, 5. survivors of this query for the next MLP launch.
    PHASE_MARK(3);  // selection
    const int n_cand = n_par * R;
    uint32_t *table = hash + (size_t)q * (size_t)(BITMAP ? -hash_cap : hash_cap);
    int n_new = 0;
    if (FILTER != FILTER_ATOMIC) {
        // In pieces of at most `chunk` (what the dedupe tables in LDS hold); the first of equal candidates is kept.  An id that
        // comes again in a later piece is dropped there because the earlier piece has entered it into the visited set.
        if (RESIDENT) __syncthreads();  // the LDS copies of the list are dead from here on; their space is reused
        int dd_n = 2;
        while (dd_n < 2 * chunk) dd_n <<= 1;
        int32_t *cand = (int32_t *)newk;  // [chunk], then their ranks where the bitmap goes by rank
        int32_t *cand_rank = (BITMAP && adj_rank) ? cand + ((chunk + 3) & ~3) : nullptr;
        uint32_t *dd_key = (uint32_t *)(cand + (cand_rank ? 2 : 1) * ((chunk + 3) & ~3));
        uint32_t *dd_pos = dd_key + dd_n, *bk_key = dd_pos + dd_n, *bk_cnt = bk_key + dd_n;
        for (int c0 = 0; c0 < n_cand; c0 += chunk) {
            const int nc = min(chunk, n_cand - c0);
            if (c0 > 0) {  // the table stores of the piece before must be seen by this piece's reads
                __threadfence_block();
                __syncthreads();
            }
            for (int j = threadIdx.x; j < nc; j += BLK) {
                const int p = (c0 + j) / R, s = (c0 + j) - p * R;
                cand[j] = parents[p] >= 0 ? adj[(size_t)parents[p] * R + s] : -1;
                if (BITMAP && cand_rank) cand_rank[j] = parents[p] >= 0 ? adj_rank[(size_t)parents[p] * R + s] : -1;
            }
            __syncthreads();
            if (BITMAP)
                n_new += filter_and_mark<BLK>(cand, cand_rank, nc, dd_key, dd_pos, bk_key, bk_cnt, dd_n, table, N,
                                              cand_q + n_new, wave_sums, WALKERS ? tag_q + n_new : nullptr, R, c0);
            else
                n_new += filter_and_insert<BLK>(cand, nc, dd_key, dd_pos, bk_key, bk_cnt, dd_n, table, hash_cap, N,
                                                cand_q + n_new, wave_sums, WALKERS ? tag_q + n_new : nullptr, R, c0);
        }
    } else {
        auto neighbour = [&](int j, uint32_t *bit) {
            const int p = j / R;
            const size_t from = (size_t)parents[p] * R + (j - p * R);
            const int32_t v = adj[from];
            if (BITMAP) *bit = (uint32_t)(adj_rank ? adj_rank[from] : v);
            return v;
        };
        n_new = visit<BLK, BITMAP, true, 4>(neighbour, n_cand, table, hash_cap, N, cand_q, wave_sums, Nothing{});
    }
    PHASE_MARK(5);  // adjacency gather, dedupe + visited table
    if (threadIdx.x == 0) {
        state[q].n_list = n_list;
        state[q].first_open = first_open;
        state[q].t = st.t + 1;
        state[q].n_visited = st.n_visited + n_new;
        state[q].n_expanded = st.n_expanded + (WALKERS ? n_live : n_par);
        counts[q] = n_new;
    }
}

// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(BLOCK)
emit_kernel(const QState *__restrict__ state, const uint64_t *__restrict__ pool_g, int C, int k,
            int32_t *out_ids, float *out_scores, int64_t *stats, int Q) {
    emit_row<BLOCK>(state, pool_g, C, k, blockIdx.x, blockIdx.x, out_ids, out_scores);
    // counters: every 64th workgroup sums those of 64 consecutive queries in its first wave
    if ((blockIdx.x & 63) == 0 && threadIdx.x < 64) {
        const int q = blockIdx.x + threadIdx.x;
        long long scored = 0, expanded = 0;
        int rounds = 0, overflowed = 0;
        if (q < Q) {
            const QState st = state[q];
            scored = st.n_visited, expanded = st.n_expanded, rounds = st.t, overflowed = (st.done & 2) ? 1 : 0;
        }
        for (int o = 32; o > 0; o >>= 1) {
            scored += __shfl_down(scored, o);
            expanded += __shfl_down(expanded, o);
            rounds = max(rounds, __shfl_down(rounds, o));
            overflowed += __shfl_down(overflowed, o);
        }
        if (threadIdx.x == 0) add_to_totals(stats, scored, expanded, rounds, overflowed);
    }
}

// ------------------------------------------------------------------------------------------
// What the kernels take as `hash_cap`: the hash table's entries, or minus the bitmap's words.
static int table_cap_arg(const Plan &p) { return p.bitmap_words > 0 ? -p.bitmap_words : p.hash_cap; }

static int item_row_bytes(const ann_graph *g) {
    return g->d * (g->dtype == ANN_F32 ? 4 : g->dtype == ANN_F8 ? 1 : 2);
}

static int new_cap_of(const Plan &p) {
    int n = 2;
    while (n < p.slots) n <<= 1;
    return n;
}

// Entries of the stored list that the round kernel holds in LDS at a time during the merge: the whole list
// when it is short, a quarter of a long one, at most 4,096 (32 KB).
static int tile_keys_of(const Plan &p) {
    int t = 1024;
    while (t < ROUND_TILE_MAX && 4 * t < p.C) t <<= 1;
    return t;
}

// Does the visited bitmap of this search go by the graph's locality order?
static bool ranked(const ann_graph *g, const Plan &p) { return p.bitmap_words > 0 && g->adj_rank != nullptr; }

// Candidates that go through an ordered filter together.
static int filter_chunk(const ann_graph *g, const Plan &p) {
    const int most = ranked(g, p) ? FILTER_CHUNK / 2 : FILTER_CHUNK;
    return p.slots < most ? p.slots : most;
}

// LDS of an ordered filter over n candidates, dedupe tables included
static size_t filter_smem(const ann_graph *g, const Plan &p, int n) {
    int dd_n = 2;
    while (dd_n < 2 * n) dd_n <<= 1;
    return (size_t)((n + 3) & ~3) * 4 * (ranked(g, p) ? 2 : 1) + (size_t)dd_n * 16;
}

// Workgroups of the round kernel on a CU: its LDS, eight waves a SIMD.
static int groups_of(size_t smem, int threads) {
    const int by_lds = (int)(160 * 1024 / smem), by_waves = 2048 / threads;
    return by_lds < by_waves ? by_lds : by_waves;
}

// list_keys: list entries held in LDS (0: one tile)
static size_t round_smem(const SearchArgs &a, int filter, int list_keys = 0) {
    const Plan &p = a.plan;
    const size_t lists = (size_t)(new_cap_of(p) + ((p.W_max + 1) & ~1) + (list_keys > 0 ? list_keys : tile_keys_of(p))) * 8;
    const size_t filt = filter != FILTER_ATOMIC ? filter_smem(a.g, p, filter_chunk(a.g, p)) : 0;
    return (size_t)((p.W_max + 3) & ~3) * 4 + 24 * 4 + (lists > filt ? lists : filt);
}

// Which visited filter a round uses.  The walkers' rule needs the first of equal candidates.  Atomics, one a candidate, with a
// hash table (time in the round kernel: 2,048 queries of 2 10^6 items, 64 to 2,048 candidates 3 to 17 % less, 16,384 queries
// 8.3 -> 8.1 ms a call, 6,001 in slots 30.0 -> 29.1).  On a bitmap the ordered filter, whose barriers a few queries wait for, but whose
// loads and plain stores are less traffic when the chip is full.  Time in the round kernel, ordered / atomics, bitmaps of 0.1 to 10
// million items by id or by rank, candidates of a round in brackets:
//   16 and 64 queries 1.13 to 1.29 throughout; 256 (512) 1.16 to 1.22, (2,048) 1.06; 300 (512) 1.12 to 1.18, (2,048) 1.02; 384 (1,024) 1.00
//   to 1.04, (2,048) 0.98; 512 (512) 1.06 to 1.17, (768) 0.99 to 1.03, (1,024) 0.95 to 1.01, (2,048) 0.90 to 1.02; 700 (512) 1.01 to
//   1.06, (768) 0.97; 1,024 (256) 1.02 to 1.11, (320) 1.00, (384) 0.99 to 1.04, (512) 0.97 to 1.01, (2,048) 0.77 to 0.92; 1,500 (256) 1.00;
//   2,048 (64) 1.11 to 1.16, (128) 1.04 to 1.14, (160) 1.00, (192) 0.98, (256) 0.96 to 1.00, (512) 0.84 to 1.00, (1,024) 0.86 to 0.98;
//   4,096 and 6,000 (64) 1.08 to 1.17, (128) 1.01 to 1.05; 8,192 and 16,384 with 128 threads (32) 1.05 to 1.09, (64) 1.01 to 1.05, (96)
//   and (128) 0.94 to 0.98.
// So: atomics for up to half a candidate a thread, for 256 queries or fewer, for fewer than 393,216 candidates of all queries, and where
// the ordered filter's tables in LDS cost a workgroup on the CU (512 candidates by rank, lists of 2,048: 2,048 queries, which
// are then all resident, 1.12, 4,096 1.04, 8,192 0.99, 1,024 1.00).
static int filter_of(const SearchArgs &a, int threads, int list_keys) {
    const Plan &p = a.plan;
    if (a.walkers) return FILTER_WALKERS;
    if (p.bitmap_words == 0 || 2 * p.slots <= threads || p.Q <= 256 || (int64_t)p.Q * p.slots < 3 << 17) return FILTER_ATOMIC;
    return groups_of(round_smem(a, FILTER_ORDERED, list_keys), threads) < groups_of(round_smem(a, FILTER_ATOMIC, list_keys), threads)
               ? FILTER_ATOMIC : FILTER_ORDERED;
}

static size_t seed_smem(const SearchArgs &a) {
    return (WAVES + 1) * 4 + (a.walkers ? filter_smem(a.g, a.plan, a.plan.E) : 0);
}

int launch_zero_stats(const SearchArgs &a, int32_t one_launch, int32_t by_waves) {
    const Plan &p = a.plan;
    hipLaunchKernelGGL(zero_stats_kernel, dim3(1), dim3(64), 0, a.stream, (int64_t *)(a.ws + p.off_stats),
                       (Ctrl *)(a.ws + p.off_ctrl), p.Q, a.keep_stats ? 1 : 0, p.R * 4, item_row_bytes(a.g), one_launch, by_waves);
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

int launch_init(const SearchArgs &a) {
    const Plan &p = a.plan;
    size_t smem = seed_smem(a);
    if (int rc = launch_zero_stats(a, 0); rc != ANN_OK) return rc;
    hipLaunchKernelGGL(a.walkers ? init_kernel<true> : init_kernel<false>, dim3(p.Q), dim3(BLOCK), smem, a.stream, a.entries,
                       ranked(a.g, p) ? a.g->rank : nullptr, p.E, a.g->N,
                       (QState *)(a.ws + p.off_state), (uint32_t *)(a.ws + p.off_hash), table_cap_arg(p),
                       (int32_t *)(a.ws + p.off_cand), p.slots, (int32_t *)(a.ws + p.off_counts), a.W_q,
                       a.L_q, a.cap_q, a.W, a.L, a.cap, p.W_max, p.L_max, p.max_iters_max,
                       a.walkers ? (uint16_t *)(a.ws + p.off_tag) : nullptr);
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

int launch_stream_reset(const SearchArgs &a) {
    const Plan &p = a.plan;
    const int n = p.Q > 16 ? p.Q : 16;
    hipLaunchKernelGGL(stream_reset_kernel, dim3((n + 255) / 256), dim3(256), 0, a.stream,
                       (int64_t *)(a.ws + p.off_stats), (Ctrl *)(a.ws + p.off_ctrl), (QState *)(a.ws + p.off_state),
                       (int32_t *)(a.ws + p.off_counts), a.slot_query, p.Q, a.Q_total, p.R * 4, item_row_bytes(a.g));
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

int launch_stream_publish(const SearchArgs &a, int avail) {
    const Plan &p = a.plan;
    hipLaunchKernelGGL(stream_publish_kernel, dim3(1), dim3(64), 0, a.stream, (Ctrl *)(a.ws + p.off_ctrl),
                       (int64_t *)(a.ws + p.off_stats), avail);
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

int launch_admit(const SearchArgs &a) {
    const Plan &p = a.plan;
    hipLaunchKernelGGL(admit_kernel, dim3(p.Q), dim3(BLOCK), seed_smem(a), a.stream, a.entries,
                       ranked(a.g, p) ? a.g->rank : nullptr, p.E, a.g->N,
                       (QState *)(a.ws + p.off_state), (uint32_t *)(a.ws + p.off_hash), table_cap_arg(p),
                       (int32_t *)(a.ws + p.off_cand), p.slots, (int32_t *)(a.ws + p.off_counts), a.W_q, a.L_q,
                       a.cap_q, a.W, a.L, a.cap, p.W_max, p.L_max, p.max_iters_max, (int64_t *)(a.ws + p.off_stats),
                       (Ctrl *)(a.ws + p.off_ctrl), a.slot_query, a.Q_total, (const uint64_t *)(a.ws + p.off_pool), p.C,
                       p.k, a.out_ids, a.out_scores);
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

int launch_scan_compact(const SearchArgs &a) {
    const Plan &p = a.plan;
    // every workgroup reads the counts of all earlier queries: with very many queries fewer, larger workgroups
    const int qpb = p.Q <= 8192 ? 4 : 8;
    const int blocks = (p.Q + qpb - 1) / qpb;
    auto fn = qpb == 4 ? scan_compact_kernel<4> : scan_compact_kernel<8>;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(SCAN_BLOCK), 0, a.stream,
                       (const int32_t *)(a.ws + p.off_counts), p.Q, (const int32_t *)(a.ws + p.off_cand),
                       p.slots, (int32_t *)(a.ws + p.off_offsets), (int32_t *)(a.ws + p.off_pair_q),
                       (int32_t *)(a.ws + p.off_pair_id), (Ctrl *)(a.ws + p.off_ctrl), a.slot_query, a.mailbox,
                       a.mail_tag | ((uint64_t)(uint32_t)(a.round_index + 1) << 1), a.Q_total);
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

int launch_round(const SearchArgs &a) {
    const Plan &p = a.plan;
    // Workgroups of 128 threads when a round has at most 128 candidates per query and the batch is far larger
    // than what a chip holds at once (2,048 workgroups of 256): twice as many queries are then resident, and
    // the candidates still go through the visited filter in one pass.  (C4: 33 -> 28 ms per step; with few
    // queries the shorter path of the larger workgroup wins: C2 3.9 against 4.2 ms.)  Walkers merge every survivor: with lists
    // of up to 768 entries (8,192 queries, 64 hops, k = 100, 300, 500, 700 and 1,000: 128 threads 9.9, 19.3, 19.7, 20.3 and 21.6 ms,
    // the first one with 32 hops; 256 threads 10.3, 19.7, 19.9, 20.3 and 20.8).
    // Workgroups of 512 threads when a round brings more than 512 candidates per query: the sort and the merge have half
    // of the work per thread.
    const bool big = p.slots > ROUND_BIG_FROM, half = p.slots <= 128 && p.Q >= 8192 && (!a.walkers || p.C <= 768);
    const int which = half ? 1 : big ? 2 : 0;
    const int threads = half ? 128 : big ? ROUND_BIG_BLOCK : BLOCK;
    const bool bm = p.bitmap_words > 0;
    const bool resident = !big && p.C <= tile_keys_of(p);
    const int tile_keys = resident ? ((p.C + 1) & ~1) : tile_keys_of(p);  // resident: the list itself, twice
    const int list_keys = resident ? tile_keys + p.C : 0, filter = filter_of(a, threads, list_keys);
    const size_t smem = round_smem(a, filter, list_keys);
    using Fn = decltype(&round_kernel<BLOCK, false, false, FILTER_ATOMIC>);
    Fn fn;
#define ROUND_SHARED(BLK, RESIDENT)                                                \
    (filter == FILTER_ORDERED ? round_kernel<BLK, true, RESIDENT, FILTER_ORDERED>  \
                              : (bm ? round_kernel<BLK, true, RESIDENT, FILTER_ATOMIC> : round_kernel<BLK, false, RESIDENT, FILTER_ATOMIC>))
#define ROUND_FN(BLK, RESIDENT)                                                                                                \
    (filter == FILTER_WALKERS ? (bm ? round_kernel<BLK, true, RESIDENT, FILTER_WALKERS> : round_kernel<BLK, false, RESIDENT, FILTER_WALKERS>) \
                              : ROUND_SHARED(BLK, RESIDENT))
    if (big) fn = ROUND_FN(ROUND_BIG_BLOCK, false);
    else if (half) fn = resident ? ROUND_FN(128, true) : ROUND_SHARED(128, false);  // walkers: up to 768 entries, resident
    else fn = resident ? ROUND_FN(BLOCK, true) : ROUND_FN(BLOCK, false);
#undef ROUND_FN
#undef ROUND_SHARED
    if (smem > 48 * 1024) {
        static std::atomic<uint32_t> raised[36];
        if (int rc = raise_lds_limit((const void *)fn, 128 * 1024, a.m->device,
                                     raised[12 * which + (bm ? 6 : 0) + 2 * filter + (resident ? 1 : 0)]);
            rc != ANN_OK)
            return rc;
    }
    hipLaunchKernelGGL(fn, dim3(p.Q), dim3(threads), smem, a.stream, a.g->adj,
                       ranked(a.g, p) ? a.g->adj_rank : nullptr, p.R, a.g->N,
                       (QState *)(a.ws + p.off_state), (uint64_t *)(a.ws + p.off_pool), p.C,
                       (uint32_t *)(a.ws + p.off_hash), table_cap_arg(p), (int32_t *)(a.ws + p.off_cand), p.slots,
                       (int32_t *)(a.ws + p.off_counts), (const int32_t *)(a.ws + p.off_offsets),
                       (const float *)(a.ws + p.off_scores), new_cap_of(p), p.W_max,
                       (int64_t *)(a.ws + p.off_stats), (uint16_t *)(a.ws + p.off_tag), tile_keys, filter_chunk(a.g, p));
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

int launch_emit(const SearchArgs &a) {
    const Plan &p = a.plan;
    hipLaunchKernelGGL(emit_kernel, dim3(p.Q), dim3(BLOCK), 0, a.stream, (const QState *)(a.ws + p.off_state),
                       (const uint64_t *)(a.ws + p.off_pool), p.C, p.k, a.out_ids, a.out_scores,
                       (int64_t *)(a.ws + p.off_stats), p.Q);
    ANN_HIP_TRY(hipGetLastError());
    return ANN_OK;
}

}  // namespace gmpgr
