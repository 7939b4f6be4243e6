// What the forms of the hidden update with a workgroup of eight waves share: where results go, the plain sum behind infinities,
// and the grouping of ids in front.
#pragma once

#include "dedup_small_body.h"
#include "recur_math.h"
#include "rnnlm_internal.h"

namespace rnnlm {

constexpr int kRecurThreads = 512;

struct Finish {                                       // where the results of one row go
    float *h_row;
    int b, H, Hp;
    bool word_ok;
};

// Four finished units je .. je + 3 of a row.  Padded units (zero weights, zero embedding) come out as
// sigmoid(0) - 1/2 = 0; either copy of the block is left out (null pointer) when the kernel that follows
// does not read it.
template <typename WT, bool VEC>
__device__ __forceinline__ void finish4(const ModelDev &m, const Finish &f, int je, const f32x4 &sum, const f32x4 &rs,
                                        const f32x4 &u) {
    f32x4 hp, dv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        hp[i] = f.word_ok ? sigmoid_f32(sum[i] + rs[i] + u[i]) : quiet_nan();
        dv[i] = hp[i] - 0.5f;
    }
    const size_t at = (size_t)f.b * f.Hp + je;
    const size_t frag = (size_t)(f.b >> 5) * (f.Hp >> 4) + (je >> 4);
    const int slot = (((je >> 3) & 1) * 32 + (f.b & 31)) * 8 + (je & 7);
    if constexpr (sizeof(WT) == 2) {
        if (m.d) {
            const uint2 pk = {pack_bf16x2(dv[0], dv[1]), pack_bf16x2(dv[2], dv[3])};
            *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(m.d) + at) = pk;
        }
        if (m.dfrag) {                                // (d_scale: log2(e) or 1)
            const uint2 pk = {pack_bf16x2(dv[0] * m.d_scale, dv[1] * m.d_scale), pack_bf16x2(dv[2] * m.d_scale, dv[3] * m.d_scale)};
            *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(m.dfrag) + frag * 512 + slot) = pk;
        }
    } else {
        if (m.d) *reinterpret_cast<f32x4 *>(static_cast<float *>(m.d) + at) = dv;
        if (m.dfrag) {                                // two fp16 terms
            uint16_t t[2][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) split2_f16(dv[i] * (float)(1 << kSplit2DExp), t[0][i], t[1][i]);
            uint16_t *dst = static_cast<uint16_t *>(m.dfrag) + frag * 1024 + slot;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint2 pk = {(uint32_t)t[k][0] | ((uint32_t)t[k][1] << 16), (uint32_t)t[k][2] | ((uint32_t)t[k][3] << 16)};
                *reinterpret_cast<uint2 *>(dst + k * 512) = pk;
            }
        }
    }
    if (VEC) {
        if (je + 4 <= f.H) *reinterpret_cast<f32x4 *>(f.h_row + je) = hp;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (je + i < f.H) f.h_row[je + i] = hp[i];
    }
}

// W (h - 1/2) of four units (rows w of Hp weights, `units` of them real) for one row of h_in, in plain fp32.  Only taken
// where the split of an fp32 operand into bf16 terms has no meaning: an infinity, or a number that rounds to one in bf16
// (beyond 3.389e38), leaves inf - inf in its lower terms, and the sum is NaN then.  Ends once nothing but NaN is left.
__device__ __forceinline__ f32x4 plain_sum4(const float *w, int Hp, int units, const float *h, int H) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < H; ++k) {
        const float d = h[k] - 0.5f;
        bool all_nan = true;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i < units) s[i] = fmaf(w[(size_t)i * Hp + k], d, s[i]);
            all_nan = all_nan && (i >= units || s[i] != s[i]);
        }
        if (all_nan) break;
    }
    return s;
}

// Grouping of the step's ids in front of the hidden update, by every workgroup for itself (N <= kGroupedMax): the same
// numbers as dedup_small_body.  Some two microseconds of LDS work in the place of a launch that does them on one compute
// unit and of the round trip of the count and the rows: step at V = 20000, H = 256, fp32, 256 ids 27.0 -> 25.2 us,
// V = 65536, H = 512, bf16, 1024 ids 67.4 -> 66.9.  Workgroup 0 leaves the result for the kernels behind.
// Returns the number of groups; representatives in LDS (valid until the ring is filled).
constexpr int kGroupLdsBytes = (4 * kGroupedMax + 4) * 12 + kGroupedMax * 4;

struct Nothing {
    __device__ __forceinline__ void operator()() const {}
};
// PER ids a thread, in code of its own for one: what is left out for the second is branches into lines of the program that are not there
// yet.  Grouped steps, hierarchical layer, us, one body for both / this: bf16, H = 94, 20 ids 10.22 / 10.00, H = 128, 40 10.24 / 9.89, H = 1200,
// 100 18.80 / 18.42, H = 512, 200 11.48 / 11.37; fp32, H = 256, 40 10.39 / 10.04; H = 512, 1000 ids 13.11 / 13.07.
// meanwhile(): requests that do not hang on the groups, once the ids are there.
template <int PER, class Meanwhile>
__device__ __forceinline__ int group_ids_of(const IdGroups &ids, int N, char *lds, int *wsum, const int *&rep_out, Meanwhile meanwhile) {
    constexpr int kCap = 4 * kGroupedMax;
    uint64_t *tkeys = reinterpret_cast<uint64_t *>(lds);                  // [kCap + 1]
    int *tfirst = reinterpret_cast<int *>(tkeys + kCap + 4);              // [kCap + 1] min raw index, later the group number
    int *rep = tfirst + kCap + 4;                                         // [kGroupedMax]
    const int tid = threadIdx.x, n0 = tid * PER;
    uint64_t key[PER];
    load_some(ids.key, n0, PER, N, key);
    int cap = 64;                                                         // a power of two, at most half full, many ids a quarter
    while (cap < (PER == 1 ? 2 : 4) * N) cap <<= 1;
    constexpr u32x4 kFree = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, kNone = {0x7FFFFFFFu, 0x7FFFFFFFu, 0x7FFFFFFFu, 0x7FFFFFFFu};
    for (int i = tid; i < (cap + 4) / 2; i += kRecurThreads) reinterpret_cast<u32x4 *>(tkeys)[i] = kFree;      // while the keys are on their way
    for (int i = tid; i < (cap + 4) / 4; i += kRecurThreads) reinterpret_cast<u32x4 *>(tfirst)[i] = kNone;
    __syncthreads();
    int slot[PER];
    if constexpr (PER == 1) {
        slot[0] = n0 < N ? find_or_insert_lds(tkeys, cap, key[0]) : -1;
    } else {
        find_or_insert_lds(tkeys, cap, key, slot, [&](int i) { return n0 + i < N; });
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (slot[i] >= 0) atomicMin(&tfirst[slot[i]], n0 + i);
    __builtin_amdgcn_sched_barrier(0);                                    // (loads are awaited in order, and the ids are there)
    meanwhile();
    __syncthreads();
    int is_first[PER], mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        is_first[i] = (slot[i] >= 0 && tfirst[slot[i]] == n0 + i) ? 1 : 0;
        mine += is_first[i];
    }
    int total;
    int u = block_exclusive_scan(mine, wsum, total);                      // barriers inside: all first indices are read
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (is_first[i]) {
            rep[u] = n0 + i;
            tfirst[slot[i]] = u;
            ++u;
        }
    }
    __syncthreads();
    if (blockIdx.x == 0) {
        int group[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) group[i] = slot[i] >= 0 ? tfirst[slot[i]] : 0;
        store_some(ids.inverse, n0, PER, N, group);
        for (int i = tid; i < total; i += kRecurThreads) ids.rep[i] = rep[i];
        if (tid == 0) *ids.n_unique = total;
    }
    rep_out = rep;
    return total;
}
template <class Meanwhile = Nothing>
__device__ __forceinline__ int group_ids(const IdGroups &ids, int N, char *lds, int *wsum, const int *&rep_out, Meanwhile meanwhile = Meanwhile()) {
    static_assert(kGroupedMax == 2 * kRecurThreads && kGroupLdsBytes <= 64 * 1024, "one or two ids a thread; fits the smallest ring");
    return N <= kRecurThreads ? group_ids_of<1>(ids, N, lds, wsum, rep_out, meanwhile) : group_ids_of<2>(ids, N, lds, wsum, rep_out, meanwhile);
}

}  // namespace rnnlm
