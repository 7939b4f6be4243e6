// The one-workgroup grouping of history ids (N <= kSmallN, and a second form up to kMediumN) as device functions: the kernel of its
// own runs it, and so does the kernel that goes on to the cache lookup in the same launch.
#pragma once

#include "device_utils.h"

namespace rnnlm {

constexpr uint64_t kEmpty = 0xFFFFFFFFFFFFFFFFull;   // marks a free slot; the key with this
                                                     // value lives in a slot of its own
constexpr int kSmallN = 4096;
constexpr int kSmallCap = 8192;                      // LDS slots of the small path
constexpr int kSmallThreads = 1024;

// Find or claim the slot of `key` in an open-addressing table of `cap` slots (+1 extra slot
// at index cap for the key that equals the free marker).
template <typename KeyPtr>
__device__ __forceinline__ int find_or_insert(KeyPtr tkeys, int cap, uint64_t key) {
    if (key == kEmpty) return cap;
    uint32_t h = id_hash(key) & (uint32_t)(cap - 1);
    // The table holds at most N <= cap/2 keys, so a free slot is always met.
    for (int probe = 0; probe < cap; ++probe) {
        unsigned long long old = atomicCAS(reinterpret_cast<unsigned long long *>(&tkeys[h]),
                                           (unsigned long long)kEmpty, (unsigned long long)key);
        if (old == kEmpty || old == key) return (int)h;
        h = (h + 1) & (uint32_t)(cap - 1);
    }
    return -1;   // unreachable for N <= cap/2
}

// The same for a table in LDS and PER keys of a thread.  The first probes, with which most end, are on their way together (all the
// further ones too was slower: a loop over PER keys is long).  What the insertion lasts is its longest chain, some 60 ns a probe, so the further
// slots of a key are an odd number apart that is its own: with a step of one 1024 different ids in 2048 slots made chains of 9 to 19, and a hidden
// update with them in front of it took 1 to 2 us more for the longer ones.  slot[i] = -1 where valid(i) is false.
template <int PER, typename KeyPtr, class Valid>
__device__ __forceinline__ void find_or_insert_lds(KeyPtr tkeys, int cap, const uint64_t (&key)[PER], int (&slot)[PER], Valid valid) {
    unsigned long long old[PER];
    int step[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        slot[i] = -1;
        old[i] = kEmpty;
        step[i] = 1;
        if (!valid(i)) continue;
        slot[i] = cap;
        if (key[i] == kEmpty) continue;
        const uint32_t h = id_hash(key[i]);
        slot[i] = (int)(h & (uint32_t)(cap - 1));
        step[i] = (int)(h >> 16) | 1;
        old[i] = atomicCAS(reinterpret_cast<unsigned long long *>(&tkeys[slot[i]]), (unsigned long long)kEmpty, (unsigned long long)key[i]);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        // The table holds at most half as many keys as it has slots, so a free slot is always met.
        for (int probe = 1; probe < cap && old[i] != kEmpty && old[i] != key[i]; ++probe) {
            slot[i] = (slot[i] + step[i]) & (cap - 1);
            old[i] = atomicCAS(reinterpret_cast<unsigned long long *>(&tkeys[slot[i]]), (unsigned long long)kEmpty, (unsigned long long)key[i]);
        }
    }
}

// The same for one key of a thread.
template <typename KeyPtr>
__device__ __forceinline__ int find_or_insert_lds(KeyPtr tkeys, int cap, uint64_t key) {
    if (key == kEmpty) return cap;
    const uint32_t h = id_hash(key);
    const int step = (int)(h >> 16) | 1;
    int slot = (int)(h & (uint32_t)(cap - 1));
    for (int probe = 0; probe < cap; ++probe) {
        const unsigned long long old = atomicCAS(reinterpret_cast<unsigned long long *>(&tkeys[slot]), (unsigned long long)kEmpty, (unsigned long long)key);
        if (old == kEmpty || old == key) return slot;
        slot = (slot + step) & (cap - 1);
    }
    return -1;   // unreachable: the table is at most half full
}

// How many of n things, side by side, a thread of `threads` takes: 1, 2 or 4 (more threads do nothing instead), so that what they
// read and write goes in whole vectors.  For n <= 4 * threads.
__device__ __forceinline__ int per_thread(int n, int threads) { return n > 2 * threads ? 4 : n > threads ? 2 : 1; }

// Elements at .. at + per - 1 (per <= CAP <= 4, a power of two, the same in all threads) of p[n], together where they all exist; 0
// in the others.
template <typename T, int CAP>
__device__ __forceinline__ void load_some(const T *p, int at, int per, int n, T (&v)[CAP]) {
#pragma unroll
    for (int i = 0; i < CAP; ++i) v[i] = 0;
    if (CAP == 4 && per == 4 && at + 4 <= n) {
        __builtin_memcpy(v, p + at, sizeof v);
    } else if (per == 2 && at + 2 <= n) {
        __builtin_memcpy(v, p + at, 2 * sizeof(T));
    } else {
#pragma unroll
        for (int i = 0; i < CAP; ++i)
            if (i < per && at + i < n) v[i] = p[at + i];
    }
}
template <int CAP>
__device__ __forceinline__ void store_some(int32_t *p, int at, int per, int n, const int (&v)[CAP]) {
    if (CAP == 4 && per == 4 && at + 4 <= n) {
        __builtin_memcpy(p + at, v, sizeof v);
    } else if (per == 2 && at + 2 <= n) {
        __builtin_memcpy(p + at, v, 2 * sizeof(int));
    } else {
#pragma unroll
        for (int i = 0; i < CAP; ++i)
            if (i < per && at + i < n) p[at + i] = v[i];
    }
}

// What the grouping leaves in LDS for a consumer in the same workgroup (valid after a barrier):
// representative and id of group u < total.  The arrays lie in the key table, which is free by then.
struct SmallGroups {
    int total;
    const int *rep;          // [total]
    const uint64_t *id;      // [total]
    int *spare;              // [kSmallCap] ints of LDS that are free from then on
};

// All kSmallThreads threads of the one workgroup call it; N <= kSmallN.
// What bounds it is what one compute unit can issue, sixteen waves on four SIMDs, and the LDS trips behind each other.  Us per launch of 4096 ids,
// 1229 distinct, before / with the short hash, whole vectors and first probes side by side 6.5 / 5.5; with the lookup behind it (cache.hip), 410
// distinct, some 41 of them new 8.3 / 7.0, 1229 distinct, all new 12.2 / 10.3.
__device__ __forceinline__ SmallGroups dedup_small_body(const uint64_t *__restrict__ keys, int N,
                                                        int32_t *__restrict__ rep, int32_t *__restrict__ inverse,
                                                        int32_t *__restrict__ n_unique) {
    constexpr int kPer = kSmallN / kSmallThreads;      // queries per thread at most
    static_assert(kPer == 4, "load_some, store_some");
    __shared__ __attribute__((aligned(16))) uint64_t tkeys[kSmallCap + 2];
    __shared__ __attribute__((aligned(16))) int tfirst[kSmallCap + 4];   // min raw index per slot, later the group number
    __shared__ int wsum[kSmallThreads / 64 + 1];
    static_assert(kSmallN * 4 + kSmallN * 8 <= kSmallCap * 8, "rep and id of every group fit the key table");
    int *const rep_lds = reinterpret_cast<int *>(tkeys);                 // [kSmallN] ints = kSmallN / 2 slots
    uint64_t *const id_lds = tkeys + kSmallN / 2;                        // [kSmallN]

    // Thread t owns the `per` contiguous queries from t * per on; contiguous ownership makes the scan below run over
    // raw-index order.  The keys are fetched first, all at once: an insertion is a loop around an
    // LDS atomic, and a load behind it would wait for it.
    const int per = per_thread(N, kSmallThreads), n0 = threadIdx.x * per;
    uint64_t key[kPer];
    load_some(keys, n0, per, N, key);
    constexpr u32x4 kFree = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, kNone = {0x7FFFFFFFu, 0x7FFFFFFFu, 0x7FFFFFFFu, 0x7FFFFFFFu};
    for (int i = threadIdx.x; i < (kSmallCap + 2) / 2; i += kSmallThreads) reinterpret_cast<u32x4 *>(tkeys)[i] = kFree;      // while the keys are on their way
    for (int i = threadIdx.x; i < (kSmallCap + 4) / 4; i += kSmallThreads) reinterpret_cast<u32x4 *>(tfirst)[i] = kNone;
    __syncthreads();
    int slot[kPer];
    find_or_insert_lds(tkeys, kSmallCap, key, slot, [&](int i) { return i < per && n0 + i < N; });
#pragma unroll
    for (int i = 0; i < kPer; ++i)
        if (slot[i] >= 0) atomicMin(&tfirst[slot[i]], n0 + i);
    __syncthreads();

    int is_first[kPer];
    int mine = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        is_first[i] = (slot[i] >= 0 && tfirst[slot[i]] == n0 + i) ? 1 : 0;
        mine += is_first[i];
    }
    int total;
    int u = block_exclusive_scan(mine, wsum, total);   // barriers inside: all tfirst reads done
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (is_first[i]) {
            rep[u] = n0 + i;
            rep_lds[u] = n0 + i;                       // (the key table is not read any more)
            id_lds[u] = key[i];
            tfirst[slot[i]] = u;                       // the slot now carries its group number
            ++u;
        }
    }
    __syncthreads();
    int group[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) group[i] = slot[i] >= 0 ? tfirst[slot[i]] : 0;
    store_some(inverse, n0, per, N, group);
    if (threadIdx.x == 0) *n_unique = total;
    return SmallGroups{total, rep_lds, id_lds, tfirst};
}

// ------------------------------------------------------------------------------ up to kMediumN ids
// The same grouping for more ids in the same LDS: the table keeps, per slot, the
// index of a raw query (4 bytes) instead of the key (8 bytes), and the keys themselves sit in LDS
// once, in raw order; a probe compares its key with the key of the query the slot points to.  A
// slot's index is only ever replaced by a smaller index of the SAME key (atomicMin after the
// comparison), so the key a slot stands for never changes, and after all insertions the slot holds
// the first raw index of its group.  No key value is special here.
// (7 ids per thread; with 8192 ids, half of the slots taken, the probe chains make the one workgroup
// slower than the launches of the grid-wide form: 16 to 30 us against 18 to 20, measured)
constexpr int kMediumN = 7168;
constexpr int kMediumCap = 16384;

struct MediumGroups {
    int total;
    const int *rep;          // [total]
    const uint64_t *key;     // [N] in raw order: id of group u = key[rep[u]]
    int *spare;              // [kMediumCap - kMediumN] ints of LDS that are free from then on
};

__device__ __forceinline__ MediumGroups dedup_medium_body(const uint64_t *__restrict__ keys, int N,
                                                          int32_t *__restrict__ rep, int32_t *__restrict__ inverse,
                                                          int32_t *__restrict__ n_unique) {
    __shared__ uint64_t lkey[kMediumN];
    __shared__ int table[kMediumCap];        // raw index, later the group number, last the representatives
    __shared__ int wsum[kSmallThreads / 64 + 1];
    constexpr int kPer = kMediumN / kSmallThreads;
    const int per = (N + kSmallThreads - 1) / kSmallThreads;
    uint64_t key[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int n = threadIdx.x * per + i;
        key[i] = (i < per && n < N) ? keys[n] : 0;
    }
    for (int i = threadIdx.x; i < kMediumCap; i += kSmallThreads) table[i] = -1;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int n = threadIdx.x * per + i;
        if (i < per && n < N) lkey[n] = key[i];
    }
    __syncthreads();
    int slot[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int n = threadIdx.x * per + i;
        slot[i] = -1;
        if (i < per && n < N) {
            const uint32_t hash = id_hash(key[i]), step = hash >> 16 | 1;      // as find_or_insert_lds
            uint32_t h = hash & (uint32_t)(kMediumCap - 1);
            // at most N <= kMediumCap / 2 slots are ever taken: a free one is always met
            for (int probe = 0; probe < kMediumCap; ++probe) {
                int cur = table[h];
                if (cur < 0) {
                    cur = atomicCAS(&table[h], -1, n);
                    if (cur < 0) { slot[i] = (int)h; break; }          // claimed
                }
                if (lkey[cur] == key[i]) {
                    atomicMin(&table[h], n);
                    slot[i] = (int)h;
                    break;
                }
                h = (h + step) & (uint32_t)(kMediumCap - 1);
            }
        }
    }
    __syncthreads();

    int is_first[kPer];
    int mine = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int n = threadIdx.x * per + i;
        is_first[i] = (slot[i] >= 0 && table[slot[i]] == n) ? 1 : 0;
        mine += is_first[i];
    }
    int total;
    const int u0 = block_exclusive_scan(mine, wsum, total);   // barriers inside: all reads of the first indices done
    int u = u0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (is_first[i]) {
            rep[u] = threadIdx.x * per + i;
            table[slot[i]] = u;                                // the slot now carries its group number
            ++u;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int n = threadIdx.x * per + i;
        if (slot[i] >= 0) inverse[n] = table[slot[i]];
    }
    if (threadIdx.x == 0) *n_unique = total;
    __syncthreads();                                           // the group numbers are read: the table is free
    u = u0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (is_first[i]) table[u++] = threadIdx.x * per + i;   // representatives, for a consumer in this workgroup
    }
    return MediumGroups{total, table, lkey, table + kMediumN};
}

}  // namespace rnnlm
