// Device code of the joint best-first search shared by its kernels (search_kernels.hip, search_fused.hip): ordered
// counting over a workgroup, the sort of a round's new keys, the visited filters, the counters.
#pragma once

#include "common.h"
#include "keys.h"

namespace gmpgr {

__device__ __forceinline__ uint32_t hash_id(uint32_t id) { return id * 0x9E3779B1u; }

// Exclusive prefix count of `flag` over the workgroup in thread order; *total = block sum.
// wave_sums: LDS int[WAVES + 1].  Contains two barriers.
template <int BLK>
__device__ __forceinline__ int block_excl_count(bool flag, int *wave_sums, int *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long b = __ballot(flag);
    int excl = __popcll(b & ((1ull << lane) - 1ull));
    if (lane == 0) wave_sums[wave] = __popcll(b);
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < (BLK >> 6); ++w) {
        int c = wave_sums[w];
        if (w < wave) base += c;
        tot += c;
    }
    __syncthreads();
    *total = tot;
    return base + excl;
}

// Sorts keys[0..m), 1 <= m <= BLK, ascending, by counting: the keys are distinct, so the rank of a key is the
// number of smaller ones.  The count for key j is shared by BLK / m_pad threads (m_pad: m rounded up to a power
// of two), each over its share of the keys, which a wave reads as LDS broadcasts, one after the other without
// waiting; the shares meet in an LDS counter.  Three barriers and m * m_pad / BLK independent reads per
// thread, where the bitonic network makes log2(m)^2 / 2 dependent trips to the LDS with most threads idle.
//   cnt : LDS uint32[m_pad], any contents.   All threads of the workgroup call; ends with a barrier.
template <int BLK>
__device__ void rank_sort(uint64_t *keys, int m, uint32_t *cnt) {
    int shift = 0;
    while ((1 << shift) < m) ++shift;
    const int m_pad = 1 << shift, groups = BLK >> shift;
    const int j = threadIdx.x & (m_pad - 1), part = threadIdx.x >> shift;
    if ((int)threadIdx.x < m_pad) cnt[threadIdx.x] = 0;
    __syncthreads();  // the keys are all written, the counters are zero
    const uint64_t key = j < m ? keys[j] : 0;
    const int per = (m + groups - 1) / groups;
    const int i0 = part * per, i1 = min(m, i0 + per);
    uint32_t smaller = 0;
    for (int i = i0; i < i1; ++i) smaller += keys[i] < key ? 1u : 0u;
    if (j < m && smaller) atomicAdd(&cnt[j], smaller);
    __syncthreads();  // every count is complete and nobody reads the unsorted keys any more
    if (part == 0 && j < m) keys[cnt[j]] = key;
    __syncthreads();
}

// The ordered visited filters: the first of equal candidates wins.  The walkers need that (whose neighbour it is decides where
// a walker goes next); the bitmap's serves the batch path's rounds too where it is the faster one.
//
// Drops ids that are out of range, repeated inside cand[0..n_cand) (first occurrence kept)
// or already in this query's visited table; inserts the rest into the table and writes them,
// in their order of occurrence, to out[0..n_new).  Returns n_new (same in every thread).
//   cand          : LDS int32[n_cand]
//   dd_key/dd_pos : LDS uint32[dd_n] each, dd_n a power of two >= 2 * n_cand (dedupe by id)
//   bk_key/bk_cnt : LDS uint32[dd_n] each (arrivals per bucket in this pass)
//   out_tag       : null, or global uint16[n_new]: (tag_base + candidate position) / tag_div of every survivor
//   table         : global uint32[hash_cap]: hash_cap/16 buckets of 16 slots (one 64-byte line);
//                   a bucket is filled from slot 0 up, EMPTY_SLOT = free.  An id lives in its home
//                   bucket or, if that one is full, in the next ones up to the first bucket that
//                   is not full.  The caller guarantees n_visited + n_cand <= hash_cap / 2.
//
// The table of a query is touched by one workgroup only, so it needs no global atomics: every candidate reads its whole bucket once (one line),
// decides "seen / room / full" from that snapshot, and the candidates that arrive at the same
// bucket in the same pass take consecutive free slots by a rank drawn from an LDS counter.
// Stores of a pass become visible to the next pass through a workgroup-scope fence + barrier.
template <int BLK>
__device__ int filter_and_insert(const int32_t *cand, int n_cand, uint32_t *dd_key, uint32_t *dd_pos,
                                 uint32_t *bk_key, uint32_t *bk_cnt, int dd_n, uint32_t *table, int hash_cap,
                                 int64_t N, int32_t *out, int *wave_sums, uint16_t *out_tag, int tag_div,
                                 int tag_base = 0) {
    const uint32_t n_buckets = (uint32_t)hash_cap >> 4;
    for (int i = threadIdx.x; i < dd_n; i += BLK) {
        dd_key[i] = EMPTY_SLOT;
        dd_pos[i] = 0xFFFFFFFFu;
    }
    __syncthreads();
    const uint32_t dd_mask = (uint32_t)dd_n - 1u;
    // pass 1: smallest position of every distinct id
    for (int p = threadIdx.x; p < n_cand; p += BLK) {
        int32_t v = cand[p];
        if (v < 0 || (int64_t)v >= N) continue;
        uint32_t s = hash_id((uint32_t)v) & dd_mask;
        for (;;) {
            uint32_t old = atomicCAS(&dd_key[s], EMPTY_SLOT, (uint32_t)v);
            if (old == EMPTY_SLOT || old == (uint32_t)v) {
                atomicMin(&dd_pos[s], (uint32_t)p);
                break;
            }
            s = (s + 1u) & dd_mask;
        }
    }
    __syncthreads();
    // pass 2: first occurrences look themselves up in the visited table and enter it if absent
    int n_new = 0;
    for (int p0 = 0; p0 < n_cand; p0 += BLK) {
        const int p = p0 + threadIdx.x;
        bool fresh = false, active = false;
        int32_t v = -1;
        uint32_t bkt = 0;
        if (p < n_cand) {
            v = cand[p];
            if (v >= 0 && (int64_t)v < N) {
                uint32_t s = hash_id((uint32_t)v) & dd_mask;
                while (dd_key[s] != (uint32_t)v) s = (s + 1u) & dd_mask;
                active = (dd_pos[s] == (uint32_t)p);
                bkt = __umulhi(hash_id((uint32_t)v), n_buckets);  // the hash's place among the buckets
            }
        }
        for (;;) {
            for (int i = threadIdx.x; i < dd_n; i += BLK) {
                bk_key[i] = EMPTY_SLOT;
                bk_cnt[i] = 0u;
            }
            // snapshot of the bucket: every read of this pass completes before any store of it
            bool found = false;
            int cnt = 0;
            if (active) {
                // (Requesting the home buckets before the dedupe, so that the lines travel meanwhile, keeps 16
                // registers busy across it: in a kernel held to 64 they spill, which cost C4 a quarter of its time.)
                const uint4 *line = (const uint4 *)(table + (size_t)bkt * 16);
                const uint4 q0 = line[0], q1 = line[1], q2 = line[2], q3 = line[3];
                const uint32_t w[16] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w,
                                        q2.x, q2.y, q2.z, q2.w, q3.x, q3.y, q3.z, q3.w};
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    found |= (w[i] == (uint32_t)v);
                    cnt += (w[i] != EMPTY_SLOT);
                }
            }
            __syncthreads();
            if (active) {
                if (found) {
                    active = false;  // scored in an earlier round
                } else if (cnt == 16) {
                    bkt = bkt + 1u == n_buckets ? 0u : bkt + 1u;  // full: the id can only be further on
                } else {
                    uint32_t s = hash_id(bkt) & dd_mask;
                    for (;;) {
                        uint32_t old = atomicCAS(&bk_key[s], EMPTY_SLOT, bkt);
                        if (old == EMPTY_SLOT || old == bkt) break;
                        s = (s + 1u) & dd_mask;
                    }
                    const int slot = cnt + (int)atomicAdd(&bk_cnt[s], 1u);
                    if (slot < 16) {
                        table[(size_t)bkt * 16 + slot] = (uint32_t)v;
                        fresh = true;
                        active = false;
                    } else {
                        bkt = bkt + 1u == n_buckets ? 0u : bkt + 1u;  // filled up by this pass: try the next bucket
                    }
                }
            }
            const bool more = (p0 + BLK < n_cand);
            if (!__syncthreads_or(active ? 1 : 0)) {
                if (more) {
                    __threadfence_block();
                    __syncthreads();
                }
                break;
            }
            // This pass's stores must be seen by the next pass's bucket reads.  A table belongs to one workgroup,
            // whose waves share a compute unit and its vector cache: workgroup scope is enough, and a device-scope
            // fence would write the whole L2 slice back.
            __threadfence_block();
            __syncthreads();
        }
        int tot;
        int pos = block_excl_count<BLK>(fresh, wave_sums, &tot);
        if (fresh) {
            out[n_new + pos] = v;
            if (out_tag) out_tag[n_new + pos] = (uint16_t)((tag_base + p) / tag_div);  // the parent (or seed) it came from
        }
        n_new += tot;
    }
    return n_new;
}

// The same filter over a bitmap of the item ids (one bit per item, N / 8 bytes per query) instead of the hash
// table: chosen where the bitmap is the smaller of the two (long lists on a moderate item count), because the
// probes of all queries then fall into a much smaller address range and seeding has much less to clear.
//   bits : global uint32[ceil(N / 32) rounded up to 64 words], all zero at the start of a search
// Every first occurrence reads its word (4 bytes); the ones whose bit is clear are new.  New ids that share a
// word meet in an LDS table keyed by the word index, OR their bits together there, and the one that opened the
// entry stores word | bits: plain loads and stores, the bitmap belongs to this workgroup alone.
//   cand_rank : LDS int32[n_cand] or nullptr: the bit that stands for candidate p is cand_rank[p] instead of its id
//               (a permutation of the ids chosen so that ids the graph joins lie in the same 64-byte lines)
template <int BLK>
__device__ int filter_and_mark(const int32_t *cand, const int32_t *cand_rank, int n_cand, uint32_t *dd_key,
                               uint32_t *dd_pos, uint32_t *bk_key, uint32_t *bk_cnt, int dd_n, uint32_t *bits, int64_t N,
                               int32_t *out, int *wave_sums, uint16_t *out_tag, int tag_div, int tag_base) {
    uint32_t pre = 0;  // the first BLK candidates request their word right away (nothing is stored before pass 2)
    if ((int)threadIdx.x < n_cand) {
        const int32_t v = cand[threadIdx.x];
        if (v >= 0 && (int64_t)v < N) pre = bits[(uint32_t)(cand_rank ? cand_rank[threadIdx.x] : v) >> 5];
    }
    for (int i = threadIdx.x; i < dd_n; i += BLK) {
        dd_key[i] = EMPTY_SLOT;
        dd_pos[i] = 0xFFFFFFFFu;
        bk_key[i] = EMPTY_SLOT;
        bk_cnt[i] = 0u;
    }
    __syncthreads();
    const uint32_t dd_mask = (uint32_t)dd_n - 1u;
    // pass 1: smallest position of every distinct id
    for (int p = threadIdx.x; p < n_cand; p += BLK) {
        int32_t v = cand[p];
        if (v < 0 || (int64_t)v >= N) continue;
        uint32_t s = hash_id((uint32_t)v) & dd_mask;
        for (;;) {
            uint32_t old = atomicCAS(&dd_key[s], EMPTY_SLOT, (uint32_t)v);
            if (old == EMPTY_SLOT || old == (uint32_t)v) {
                atomicMin(&dd_pos[s], (uint32_t)p);
                break;
            }
            s = (s + 1u) & dd_mask;
        }
    }
    __syncthreads();
    // pass 2: first occurrences test their bit; the new ones set it
    int n_new = 0;
    for (int p0 = 0; p0 < n_cand; p0 += BLK) {
        const int p = p0 + threadIdx.x;
        bool fresh = false, owner = false;
        int32_t v = -1;
        uint32_t word = 0, old_word = 0, slot = 0, bit = 0;
        if (p < n_cand) {
            v = cand[p];
            if (v >= 0 && (int64_t)v < N) {
                uint32_t s = hash_id((uint32_t)v) & dd_mask;
                while (dd_key[s] != (uint32_t)v) s = (s + 1u) & dd_mask;
                if (dd_pos[s] == (uint32_t)p) {
                    bit = (uint32_t)(cand_rank ? cand_rank[p] : v);
                    word = bit >> 5;
                    old_word = (p0 == 0) ? pre : bits[word];
                    fresh = ((old_word >> (bit & 31)) & 1u) == 0u;
                }
            }
        }
        if (fresh) {
            slot = hash_id(word) & dd_mask;
            for (;;) {
                uint32_t old = atomicCAS(&bk_key[slot], EMPTY_SLOT, word);
                if (old == EMPTY_SLOT || old == word) {
                    owner = (old == EMPTY_SLOT);
                    break;
                }
                slot = (slot + 1u) & dd_mask;
            }
            atomicOr(&bk_cnt[slot], 1u << (bit & 31));
        }
        __syncthreads();  // every new bit of this pass has reached its LDS entry
        if (owner) bits[word] = old_word | bk_cnt[slot];
        int tot;
        const int pos = block_excl_count<BLK>(fresh, wave_sums, &tot);
        if (fresh) {
            out[n_new + pos] = v;
            if (out_tag) out_tag[n_new + pos] = (uint16_t)((tag_base + p) / tag_div);
        }
        n_new += tot;
        if (p0 + BLK < n_cand) {
            // the words stored above must be seen by the next pass; its ids open fresh LDS entries
            for (int i = threadIdx.x; i < dd_n; i += BLK) {
                bk_key[i] = EMPTY_SLOT;
                bk_cnt[i] = 0u;
            }
            __threadfence_block();
            __syncthreads();
        }
    }
    return n_new;
}

// The visited set of a search without walkers: enters the candidates v[u] that are in range and new to the query;
// fresh[u] says which.  One atomic per candidate decides "seen", "repeated in this round" and "new" at once: of equal
// candidates exactly one finds the id absent, whichever it is (what a search returns does not depend on the order of its
// survivors).  The UNROLL atomics of a thread are in flight together.
//   at[u] : BITMAP: the bit that stands for the candidate; else scratch
//   table : BITMAP: one bit per item; else hash_cap slots of one id each, EMPTY_SLOT = free, an id lies in the first free
//           slot from its home on.  The caller guarantees that slots stay free: n_visited + n_cand is at most hash_cap / 2 of a
//           table in memory, five eighths of one in LDS.
//   PEEK  : the word is read first, and the atomic left out where it shows the id, or another one in its slot: an atomic
//           makes its line dirty whatever it finds, and full batches are bound by that traffic.  (What was read may be
//           older than the set; it only ever grows, so the atomic has the last word.)
// A query's set belongs to one workgroup, so the atomics need no more than workgroup scope: they are carried out in
// the L2 slice, like a load or a store.  (At device scope, the default of atomicCAS, they go to the memory side and
// cost several times as much.)
// Against the filters above, which sort out repetitions in LDS tables first (five barriers, 16 KB of tables for 512
// candidates, 64-byte buckets read whole): one query in one launch 473 -> 412 us, 64 fp32 queries 335 -> 270 us (lists of
// 4,096: 4.18 -> 3.63 ms).  In full batches, with PEEK: 2,048 8-bit queries with lists of 2,048 29.7 -> 28.3 ms, 6,001 fp16
// queries in slots 30.0 -> 29.1, 8,192 ragged ones 7.39 -> 7.05; without it 31.9, 29.7 and 7.50, and 16,384 queries of a
// table of 20 million items 8.8 ms where they take 8.05 with it.
//   meanwhile(u, v, may_be_new) : called once per candidate v while the atomics travel
template <bool BITMAP, bool PEEK, int UNROLL, class Meanwhile>
__device__ __forceinline__ void visited_enter(const int32_t (&v)[UNROLL], uint32_t (&at)[UNROLL], bool (&fresh)[UNROLL],
                                              uint32_t *table, int hash_cap, int64_t N, Meanwhile meanwhile) {
    uint32_t old[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        fresh[u] = v[u] >= 0 && (int64_t)v[u] < N;
        old[u] = BITMAP ? 0u : EMPTY_SLOT;
        if (!BITMAP) at[u] = __umulhi(hash_id((uint32_t)v[u]), (uint32_t)hash_cap);
        if (BITMAP && PEEK && fresh[u]) old[u] = table[at[u] >> 5];
    }
    // The rest of the home's four slots in one trip, up to the id or a free slot (one slot instead: 16,384 queries of a table of
    // 20 million items 4.74 ms instead of 4.64, 8,192 ragged ones 4.64 instead of 4.56).
    if (!BITMAP && PEEK) {
        uint4 w[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            if (fresh[u]) w[u] = *(const uint4 *)(table + (at[u] & ~3u));
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            if (fresh[u]) {
                const uint32_t slot[4] = {w[u].x, w[u].y, w[u].z, w[u].w}, from = at[u] & 3;
                uint32_t to = 3;
                old[u] = slot[3];
#pragma unroll
                for (uint32_t i = 3; i-- > 0;)
                    if (i >= from && (slot[i] == (uint32_t)v[u] || slot[i] == EMPTY_SLOT)) to = i, old[u] = slot[i];
                at[u] = (at[u] & ~3u) + to;
            }
    }
    if (BITMAP) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint32_t bit = 1u << (at[u] & 31);
            fresh[u] = fresh[u] && !(old[u] & bit);
            if (fresh[u]) old[u] = __hip_atomic_fetch_or(&table[at[u] >> 5], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) meanwhile(u, v[u], fresh[u]);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) fresh[u] = fresh[u] && !((old[u] >> (at[u] & 31)) & 1u);
        return;
    }
    bool maybe[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) maybe[u] = fresh[u] && old[u] != (uint32_t)v[u];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u)
        if (fresh[u] && old[u] == EMPTY_SLOT)
            __hip_atomic_compare_exchange_strong(&table[at[u]], &old[u], (uint32_t)v[u], __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) meanwhile(u, v[u], maybe[u]);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        // another id in the slot: on to the next one.  Ends: some slots are free (see above)
        bool open = fresh[u] && old[u] != EMPTY_SLOT && old[u] != (uint32_t)v[u];
        fresh[u] = fresh[u] && old[u] == EMPTY_SLOT;
        while (open) {
            at[u] = at[u] + 1 == (uint32_t)hash_cap ? 0u : at[u] + 1;
            uint32_t seen = EMPTY_SLOT;
            if (PEEK) seen = table[at[u]];
            if (seen == EMPTY_SLOT)
                __hip_atomic_compare_exchange_strong(&table[at[u]], &seen, (uint32_t)v[u], __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP);
            fresh[u] = seen == EMPTY_SLOT;
            open = !fresh[u] && seen != (uint32_t)v[u];
        }
    }
}

struct Nothing {
    __device__ __forceinline__ void operator()(int, int32_t, bool) const {}
};

// The same for a workgroup: new candidates to out[0..n_new) in candidate order.  Returns n_new (same in every thread).
//   candidate(p, &bit) : the id of candidate p (p < n_cand) and, with a bitmap, the bit that stands for it
template <int BLK, bool BITMAP, bool PEEK, int UNROLL, class Candidate, class Meanwhile>
__device__ __forceinline__ int visit(Candidate candidate, int n_cand, uint32_t *table, int hash_cap, int64_t N,
                                     int32_t *out, int *wave_sums, Meanwhile meanwhile) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int n_new = 0;
    for (int p0 = 0; p0 < n_cand; p0 += BLK * UNROLL) {
        const int per = min(UNROLL, (n_cand - p0 + BLK - 1) / BLK);  // candidates of a wave follow one another
        int32_t v[UNROLL];
        uint32_t at[UNROLL];
        bool fresh[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int p = p0 + (wave * per + u) * 64 + lane;
            v[u] = -1;
            at[u] = 0;
            if (u < per && p < n_cand) v[u] = candidate(p, &at[u]);
        }
        visited_enter<BITMAP, PEEK, UNROLL>(v, at, fresh, table, hash_cap, N, meanwhile);
        int mine = 0, before = 0, total = 0;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) mine += __popcll(__ballot(fresh[u]));
        if (lane == 0) wave_sums[wave] = mine;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < BLK / 64; ++w) {
            const int c = wave_sums[w];
            if (w < wave) before += c;
            total += c;
        }
        __syncthreads();
        int32_t *to = out + n_new + before;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const unsigned long long b = __ballot(fresh[u]);
            if (fresh[u]) to[__popcll(b & ((1ull << lane) - 1ull))] = v[u];
            to += __popcll(b);
        }
        n_new += total;
    }
    return n_new;
}

// A table is filled by plain stores, then used by the atomics above, in one kernel: the stores have arrived.
__device__ __forceinline__ void visited_cleared() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// A query's counters join the totals once, when its result is written: every workgroup adding to the
// same few words in every round made those additions, which the memory side performs one after the
// other (about 10 ns each), the longest part of a round.  One lane calls this with sums over a
// group of queries.
__device__ __forceinline__ void add_to_totals(int64_t *stats, long long scored, long long expanded, int rounds,
                                              int overflowed) {
    atomicAdd((unsigned long long *)&stats[0], (unsigned long long)scored);
    atomicAdd((unsigned long long *)&stats[1], (unsigned long long)expanded);
    atomicMax((unsigned long long *)&stats[2], (unsigned long long)rounds);
    if (overflowed) atomicAdd((unsigned long long *)&stats[3], (unsigned long long)overflowed);
}

// The end of a search in one launch, by one thread once all queries have joined the totals: the number of those that filled
// their visited table, then the finished bit.
__device__ __forceinline__ void report_end(int64_t *stats, uint64_t *mailbox, uint64_t tag) {
    const uint64_t filled = atomicAdd((unsigned long long *)&stats[3], 0ull);
    __hip_atomic_store(mailbox + MAIL_FILLED, tag | filled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence_system();
    __hip_atomic_store(mailbox + MAIL_ROUNDS, tag | 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace gmpgr
