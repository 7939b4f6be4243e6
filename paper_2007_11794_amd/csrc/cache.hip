// The cache of RnnlmProb kept on the device between steps (Table 1 as a whole; Section 4.2:
// once-computed results are reused for the same context; Section 5.3: a size boundary).
//
// Key: the 8-byte history id (Section 3.2).  Value: what every answer for that history is
// made of -- its updated hidden vector h' (fp32) and its natural-log normaliser -- so a
// history found here skips the hidden update and the whole-vocabulary normalisation; only
// the H-long dot products of its queried words remain.  Entries are numbered in the order
// in which they were stored (Table 1 step 10) and never removed; the table is open
// addressing over 16-byte cells, at most half full.
//
// One step through the cache, after the grouping of the step's own ids:
//   lookup   probe every distinct history; the ones not found are numbered in order of
//            appearance by a prefix sum (row of the block that is computed now), get the next
//            entries while there is room, and their keys are inserted.  One workgroup in one
//            launch together with the grouping up to kMediumN raw queries, three launches of a full grid
//            (probe + counts, scan of the counts, numbering + insertion) for more;
//   (hidden update and output projection run on the numbered rows only)
//   commit   per distinct history: normaliser into lse_rows; new entries are written to the
//            stores, found ones copy their stored h' to the caller's h_out.
#include "dedup_small_body.h"
#include "device_utils.h"
#include "rnnlm_internal.h"

namespace rnnlm {

namespace {

constexpr int kLookupThreads = 1024;

__global__ __launch_bounds__(256) void cache_reset_kernel(CacheDev c, long long *errors) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < c.table_size) {
        CacheCell cell;
        cell.key = 0;
        cell.entry = -1;
        cell.pad = 0;
        c.table[i] = cell;
    }
    if (i == 0) *c.n_entries = 0;
    if (i < 4) c.totals[i] = 0;
    if (errors && i < 2) errors[i] = 0;
}

// One workgroup.  A round covers kLookupPer * 1024 distinct histories: every thread first
// requests the first table cell of all its up to kLookupPer histories (the usual probe ends there),
// then finishes the probes, then one prefix sum numbers the round's misses in order of
// u, and last the new keys are inserted.  Insertions happen only after every probe of the
// round is over (barriers of the scan in between), so no probe reads a half-written cell;
// the keys of one step are distinct, so a later round can never look for a key that an
// earlier round of the same step inserted.
constexpr int kLookupPer = 4;

// raw_of(u) / key_of(u, raw): representative and id of distinct history u < U.
//
// This workgroup is the only one that inserts, so who gets a free cell is settled in LDS: `claims` (claim_slots ints,
// more than there can be insertions) is a set of the cells given away in this launch, and a new cell is one
// 16-byte store.  (Compare-and-swaps on the table itself, one cache line each, were part of what the
// launch takes when every history is new: 4096 new contexts 33.5 us, now 30.0; 2048: 17.6, now 13.2.)  The set also makes a cell that an
// earlier round took, and that this compute unit may still read as free, unavailable.  (All the slots there are room for, not twice the
// histories: half full, their chains made 1229 new contexts 2.6 us slower.)
__device__ __forceinline__ bool claim_cell(int *claims, int claim_slots, uint32_t cell) {
    uint32_t s = (uint32_t)(((uint64_t)(cell * 0x9E3779B1u) * (uint32_t)claim_slots) >> 32);
    for (;;) {                                       // fewer claims than slots: a free one is always met
        const int old = atomicCAS(&claims[s], -1, (int)cell);
        if (old == -1) return true;
        if (old == (int)cell) return false;
        s = s + 1 == (uint32_t)claim_slots ? 0 : s + 1;
    }
}

// What the lookup adds to, requested in front of the grouping: the counters are a trip to memory at its beginning and, in the
// one thread that ends the launch, another one behind everything else (with the prefix sums in registers, 4096 ids, 410 distinct 9.0
// -> 8.2 us, 3631, 1089 distinct 11.3 -> 10.2).
struct CacheCounts {
    int entries;
    long long totals[4];                    // thread 0
    __device__ __forceinline__ explicit CacheCounts(const CacheDev &c) : entries(*c.n_entries) {
#pragma unroll
        for (int i = 0; i < 4; ++i) totals[i] = threadIdx.x == 0 ? c.totals[i] : 0;
    }
};

template <typename RawOf, typename KeyOf>
__device__ __forceinline__ void cache_lookup_body(const CacheDev &c, const CacheCounts &counts, int U, int32_t *__restrict__ step_stats,
                                                  int *claims, int claim_slots, RawOf raw_of, KeyOf key_of) {
    __shared__ int wsum[kLookupThreads / 64 + 1];
    const int base = counts.entries;        // read by everyone before thread 0 updates it below
    const uint32_t mask = (uint32_t)(c.table_size - 1);
    int n_miss = 0;                         // misses numbered so far (same in every thread)
    for (int i = threadIdx.x; i < claim_slots; i += kLookupThreads) claims[i] = -1;   // barriers before the first claim
    // Thread t takes the `per` distinct histories from u0 + t * per on: one prefix sum numbers a round's misses in order of u.
    const int per = per_thread(U, kLookupThreads);
    for (int u0 = 0; u0 < U; u0 += kLookupPer * kLookupThreads) {
        const int first = u0 + (int)threadIdx.x * per;
        uint64_t key[kLookupPer];
        int raw[kLookupPer], found[kLookupPer];
        uint32_t h[kLookupPer];
        CacheCell cell[kLookupPer];
#pragma unroll
        for (int i = 0; i < kLookupPer; ++i) {
            found[i] = 0;                               // (not a miss)
            if (i >= per || first >= U) continue;
            const int u = min(first + i, U - 1);
            raw[i] = raw_of(u);
            key[i] = key_of(u, raw[i]);
            h[i] = id_hash(key[i]) & mask;
            cell[i] = c.table[h[i]];
        }
        int mine = 0;
#pragma unroll
        for (int i = 0; i < kLookupPer; ++i) {
            if (i >= per || first >= U) continue;
            found[i] = -1;
            // At most capacity <= table_size / 2 cells are taken: a free cell is always met.
            for (int probe = 0; probe < c.table_size; ++probe) {
                if (cell[i].entry < 0) break;
                if (cell[i].key == key[i]) { found[i] = cell[i].entry; break; }
                h[i] = (h[i] + 1) & mask;
                cell[i] = c.table[h[i]];
            }
            mine += first + i < U && found[i] < 0 ? 1 : 0;
        }
        int total;
        int rank = n_miss + block_exclusive_scan(mine, wsum, total);
        n_miss += total;
        int entry[kLookupPer], row[kLookupPer];
#pragma unroll
        for (int i = 0; i < kLookupPer; ++i) {
            entry[i] = found[i];
            row[i] = -1;
            if (first + i < U && found[i] < 0) {        // (false beyond `per`)
                entry[i] = base + rank < c.capacity ? base + rank : -1;
                row[i] = rank;
                c.miss_src[rank] = raw[i];
                c.miss_dst[rank] = first + i;
                ++rank;
            }
        }
        store_some(c.miss_of, first, per, U, row);
        store_some(c.entry_of, first, per, U, entry);
        if (total == 0) continue;                       // uniform
        // Every probe of this round is done (the scan above contains barriers).  A probe that missed ended at
        // the first free cell of its chain, and cells are never given back: the insertion starts there.
#pragma unroll
        for (int i = 0; i < kLookupPer; ++i) {
            if (row[i] < 0 || entry[i] < 0) continue;
            while (!claim_cell(claims, claim_slots, h[i])) {
                do h[i] = (h[i] + 1) & mask;
                while (c.table[h[i]].entry >= 0);
            }
            CacheCell mine;
            mine.key = key[i];
            mine.entry = entry[i];
            mine.pad = 0;
            c.table[h[i]] = mine;
        }
        if (u0 + kLookupPer * kLookupThreads < U) {     // uniform: this round's insertions precede the next round's probes
            __threadfence_block();
            __syncthreads();
        }
    }
    if (threadIdx.x == 0) {
        const int stored = min(n_miss, max(c.capacity - base, 0));
        *c.n_miss = n_miss;
        *c.n_entries = base + stored;
        c.totals[0] = counts.totals[0] + U;
        c.totals[1] = counts.totals[1] + U - n_miss;
        c.totals[2] = counts.totals[2] + n_miss;
        c.totals[3] = counts.totals[3] + n_miss - stored;
        if (step_stats) {
            step_stats[0] = U;
            step_stats[1] = U - n_miss;
            step_stats[2] = n_miss;
            step_stats[3] = base + stored;
        }
    }
}

// The lookup is one workgroup.  The others of its launch bring what the output projection's workgroups read first into the L2s they
// read it through, for the case that few rows are left and the weights are streamed: a line read by one kernel is still there for the
// next one, and the workgroup of split s runs on XCD s % 8.  Bound by the lookup, which they hide behind; more bytes push each other out before
// they are used, or last longer than it.  A search's eight steps, us, none / 48 / 64 / 96 KB of every split: V = 65536, H = 512, 41 new
// histories of 4096 ids 303.7 / 294.3 / 294.6 / 298.2; V = 100000, H = 320 245.1 / 234.4 / 233.2 / 226.7; V = 200000, H = 1024 885 / 873 / 875 /
// 869; fp32 V = 65536, H = 512 410.6 / 404.1 / 403.5 / 400.2.  How many rows are left only the lookup finds out, too late to read ahead by it.
// One step, us, none / 64 KB:          few new (streamed)               all found                many new (not streamed)
//   V = 65536, H = 512    64 ids       4 new 28.9 / 28.7                12.4 / 13.5              64 new 29.9 / 28.8 (streamed)
//                         1024         10 new 30.4 / 29.1               13.5 / 14.2              100 new 32.0 / 32.2
//                         4096         41 new 35.7 / 35.2               18.0 / 18.8              410 new 46.7 / 47.0
//                         7000         60 new 45.2 / 44.5               27.4 / 28.4              2000 new 135.2 / 136.8
//   V = 100000, H = 320   1024         10 new 28.4 / 26.8               13.2 / 13.9              100 new 29.9 / 28.8 (69.7 / 70.0 for 1024)
//                         4096         41 new 33.6 / 32.0               17.8 / 18.3              410 new 45.7 / 45.9
//   V = 200000, H = 1024  1024         10 new 95.6 / 93.7               15.1 / 15.6              100 new 151.2 / 151.3
//   fp32 65536, 512       1024         10 new 43.9 / 42.0               14.3 / 14.4              100 new 51.4 / 50.8
//                         4096         41 new 56.1 / 55.9               21.3 / 21.8              410 new 114.0 / 114.4
// So at every number of ids it gives 0.2 to 1.9 us where few histories are new, the usual step, and takes 0.1 to 1.1 where none is.
// (In the shadow of the hidden update instead, on the compute units it leaves idle: 300 -> 324, it is the shorter launch.)
constexpr int kAheadGroups = 128, kAheadBytes = 64 * 1024;
__device__ __forceinline__ void read_ahead(const WeightsAhead &a) {
    constexpr int kWaves = kLookupThreads / 64, kSplits = kMaxSplits / kXcds, kPieces = kAheadBytes / 4096 * kSplits;
    constexpr int kWavesPerXcd = kAheadGroups / kXcds * kWaves, kEach = kPieces / kWavesPerXcd;
    static_assert(kEach * kWavesPerXcd == kPieces, "");
    if ((int)blockIdx.x < kXcds) return;
    const int xcd = blockIdx.x % kXcds, w = ((int)blockIdx.x / kXcds - 1) * kWaves + ((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    u32x4 v[kEach][4];
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const int t = w + k * kWavesPerXcd;              // every split's first piece, then every split's second
        const long long at = ahead_piece(a, xcd + kXcds * (t % kSplits), t / kSplits);
        const u32x4 *p = static_cast<const u32x4 *>(a.Ofrag) + (at > 0 ? at * 64 : 0) + lane;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[k][i] = p[i * 64];
    }
#pragma unroll
    for (int k = 0; k < kEach; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" ::"v"(v[k][i]));
}

// Grouping of the step's ids and the lookup of the distinct ones in one launch of one workgroup
// (N <= kSmallN): the lookup takes representatives and ids from LDS, where the grouping left them,
// so nothing is read back from memory between the two and one launch is saved.
static_assert(kLookupThreads == kSmallThreads, "");
__global__ __launch_bounds__(kLookupThreads) void dedup_lookup_kernel(
    CacheDev c, const uint64_t *__restrict__ ids, int N, int32_t *__restrict__ rep,
    int32_t *__restrict__ inverse, int32_t *__restrict__ n_unique, int32_t *__restrict__ step_stats,
    WeightsAhead ahead) {
    if (blockIdx.x != 0) {                  // uniform
        read_ahead(ahead);
        return;
    }
    const CacheCounts counts(c);
    const SmallGroups g = dedup_small_body(ids, N, rep, inverse, n_unique);
    __syncthreads();                        // the groups in LDS are complete
    cache_lookup_body(
        c, counts, g.total, step_stats, g.spare, kSmallCap, [&](int u) { return g.rep[u]; }, [&](int u, int) { return g.id[u]; });
}

// The same for up to kMediumN raw queries (the grouping keeps the keys in LDS in raw order).
__global__ __launch_bounds__(kLookupThreads) void dedup_lookup_medium_kernel(
    CacheDev c, const uint64_t *__restrict__ ids, int N, int32_t *__restrict__ rep,
    int32_t *__restrict__ inverse, int32_t *__restrict__ n_unique, int32_t *__restrict__ step_stats,
    WeightsAhead ahead) {
    if (blockIdx.x != 0) {                  // uniform
        read_ahead(ahead);
        return;
    }
    const CacheCounts counts(c);
    const MediumGroups g = dedup_medium_body(ids, N, rep, inverse, n_unique);
    __syncthreads();                        // the representatives in LDS are complete
    cache_lookup_body(
        c, counts, g.total, step_stats, g.spare, kMediumCap - kMediumN, [&](int u) { return g.rep[u]; },
        [&](int, int raw) { return g.key[raw]; });
}

// ---- the same lookup for many histories (more than one workgroup can number in one round):
// probe + per-workgroup miss counts, a scan of the counts, then numbering + insertion.  The
// launch boundaries put every probe before every insertion.
__device__ __forceinline__ int probe_table(const CacheDev &c, uint64_t key) {
    const uint32_t mask = (uint32_t)(c.table_size - 1);
    uint32_t h = id_hash(key) & mask;
    for (int probe = 0; probe < c.table_size; ++probe) {
        const CacheCell cell = c.table[h];
        if (cell.entry < 0) return -1;
        if (cell.key == key) return cell.entry;
        h = (h + 1) & mask;
    }
    return -1;
}

__global__ __launch_bounds__(kLookupThreads) void lookup_probe_kernel(
    CacheDev c, const uint64_t *__restrict__ ids, const int32_t *__restrict__ rep,
    const int32_t *__restrict__ n_unique) {
    __shared__ int wsum[kLookupThreads / 64 + 1];
    const int U = *n_unique;
    const int u = blockIdx.x * kLookupThreads + (int)threadIdx.x;
    int miss = 0;
    if (u < U) {
        const int found = probe_table(c, ids[rep[u]]);
        c.entry_of[u] = found;
        miss = found < 0 ? 1 : 0;
    }
    int total;
    (void)block_exclusive_scan(miss, wsum, total);
    if (threadIdx.x == 0) c.block_total[blockIdx.x] = total;
}

__global__ __launch_bounds__(kLookupThreads) void lookup_scan_kernel(CacheDev c, int blocks,
                                                                     const int32_t *__restrict__ n_unique,
                                                                     int32_t *__restrict__ step_stats) {
    __shared__ int wsum[kLookupThreads / 64 + 1];
    int carry = 0;
    for (int b0 = 0; b0 < blocks; b0 += kLookupThreads) {
        const int b = b0 + (int)threadIdx.x;
        const int v = (b < blocks) ? c.block_total[b] : 0;
        int total;
        const int excl = carry + block_exclusive_scan(v, wsum, total);
        if (b < blocks) c.block_total[b] = excl;
        carry += total;
    }
    if (threadIdx.x == 0) {
        const int U = *n_unique, n_miss = carry, base = *c.n_entries;
        const int stored = min(n_miss, max(c.capacity - base, 0));
        c.block_total[blocks] = base;               // entries before this call, for the numbering
        *c.n_miss = n_miss;
        *c.n_entries = base + stored;
        c.totals[0] += U;
        c.totals[1] += U - n_miss;
        c.totals[2] += n_miss;
        c.totals[3] += n_miss - stored;
        if (step_stats) {
            step_stats[0] = U;
            step_stats[1] = U - n_miss;
            step_stats[2] = n_miss;
            step_stats[3] = base + stored;
        }
    }
}

__global__ __launch_bounds__(kLookupThreads) void lookup_assign_kernel(
    CacheDev c, int blocks, const uint64_t *__restrict__ ids, const int32_t *__restrict__ rep,
    const int32_t *__restrict__ n_unique) {
    __shared__ int wsum[kLookupThreads / 64 + 1];
    const int U = *n_unique;
    const int base = c.block_total[blocks];
    const int u = blockIdx.x * kLookupThreads + (int)threadIdx.x;
    const bool active = u < U;
    const int miss = (active && c.entry_of[u] < 0) ? 1 : 0;
    int total;
    const int rank = c.block_total[blockIdx.x] + block_exclusive_scan(miss, wsum, total);
    if (miss) {
        const int raw = rep[u];
        const uint64_t key = ids[raw];
        const int entry = (base + rank < c.capacity) ? base + rank : -1;
        c.miss_of[u] = rank;
        c.miss_src[rank] = raw;
        c.miss_dst[rank] = u;
        c.entry_of[u] = entry;
        if (entry >= 0) {
            const uint32_t mask = (uint32_t)(c.table_size - 1);
            uint32_t h = id_hash(key) & mask;
            for (int probe = 0; probe < c.table_size; ++probe) {
                if (atomicCAS(&c.table[h].entry, -1, entry) == -1) {
                    c.table[h].key = key;
                    break;
                }
                h = (h + 1) & mask;
            }
        }
    } else if (active) {
        c.miss_of[u] = -1;
    }
}

__global__ __launch_bounds__(256) void cache_commit_kernel(CacheDev c, ModelDev m,
                                                            const int32_t *__restrict__ n_unique,
                                                            SplitInfo si, float *__restrict__ h_out) {
    const int u = blockIdx.x;
    if (u >= *n_unique) return;
    const int H = c.H;
    const int row = c.miss_of[u], entry = c.entry_of[u];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float *hrow = h_out + (size_t)u * H;
    if (row >= 0) {
        // computed in this step: its partials are in row `row` of the block of *n_miss rows
        // (a model with the hierarchical output layer has no normaliser: the hidden vector is all)
        if (wave == 0 && !m.hs) {
            const int splits = splits_of(si, *c.n_miss);
            const float lse = lse_from_partials(m.part + (size_t)row * kMaxSplits, splits, lane);
            if (lane == 0) {
                c.lse_rows[u] = lse;
                if (entry >= 0) c.store_lse[entry] = lse;
            }
        }
        if (entry >= 0) {
            float *dst = c.store_h + (size_t)entry * H;
            for (int j = threadIdx.x; j < H; j += 256) dst[j] = hrow[j];
        }
    } else {
        const float *src = c.store_h + (size_t)entry * H;
        for (int j = threadIdx.x; j < H; j += 256) hrow[j] = src[j];
        if (threadIdx.x == 0 && !m.hs) c.lse_rows[u] = c.store_lse[entry];
    }
}

__global__ __launch_bounds__(256) void pack_ids_kernel(const uint32_t *__restrict__ ctx,
                                                        const uint32_t *__restrict__ small_lm, int N,
                                                        uint64_t *__restrict__ ids) {
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n < N) ids[n] = ((uint64_t)ctx[n] << 32) | (uint64_t)small_lm[n];
}

}  // namespace

hipError_t launch_cache_reset(const CacheDev &c, long long *errors, hipStream_t stream) {
    const int n = c.table_size > 4 ? c.table_size : 4;
    hipLaunchKernelGGL(cache_reset_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, c, errors);
    return hipGetLastError();
}

hipError_t launch_cache_lookup(const CacheDev &c, int rows, const uint64_t *ids,
                               const int32_t *rep, const int32_t *n_unique, int32_t *step_stats,
                               hipStream_t stream) {
    if (rows <= 0) return hipSuccess;
    const int blocks = (rows + kLookupThreads - 1) / kLookupThreads;
    hipLaunchKernelGGL(lookup_probe_kernel, dim3(blocks), dim3(kLookupThreads), 0, stream, c, ids, rep, n_unique);
    hipLaunchKernelGGL(lookup_scan_kernel, dim3(1), dim3(kLookupThreads), 0, stream, c, blocks, n_unique,
                       step_stats);
    hipLaunchKernelGGL(lookup_assign_kernel, dim3(blocks), dim3(kLookupThreads), 0, stream, c, blocks, ids, rep,
                       n_unique);
    return hipGetLastError();
}

int dedup_lookup_max_rows() { return kMediumN; }

hipError_t launch_dedup_lookup(const CacheDev &c, const uint64_t *ids, int N, int32_t *rep, int32_t *inverse,
                               int32_t *n_unique, int32_t *step_stats, const WeightsAhead &ahead, hipStream_t stream) {
    if (N < 0 || N > kMediumN) return hipErrorInvalidValue;
    const dim3 grid(ahead.splits > 0 ? kXcds + kAheadGroups : 1);
    if (N <= kSmallN)
        hipLaunchKernelGGL(dedup_lookup_kernel, grid, dim3(kLookupThreads), 0, stream, c, ids, N, rep, inverse,
                           n_unique, step_stats, ahead);
    else
        hipLaunchKernelGGL(dedup_lookup_medium_kernel, grid, dim3(kLookupThreads), 0, stream, c, ids, N, rep,
                           inverse, n_unique, step_stats, ahead);
    return hipGetLastError();
}

hipError_t launch_cache_commit(const CacheDev &c, const ModelDev &m, int rows, const int32_t *n_unique,
                               SplitInfo splits, float *h_out, hipStream_t stream) {
    if (rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(cache_commit_kernel, dim3(rows), dim3(256), 0, stream, c, m, n_unique, splits, h_out);
    return hipGetLastError();
}

hipError_t launch_pack_ids(const uint32_t *ctx, const uint32_t *small_lm, int N, uint64_t *ids,
                           hipStream_t stream) {
    if (N <= 0) return hipSuccess;
    hipLaunchKernelGGL(pack_ids_kernel, dim3((N + 255) / 256), dim3(256), 0, stream, ctx, small_lm, N, ids);
    return hipGetLastError();
}

}  // namespace rnnlm
