// Internal declarations shared by the translation units of librnnlm (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

#include "rnnlm.h"
#include "rnnlm_diag.h"

namespace rnnlm {

typedef uint16_t bf16_t;                       // bfloat16 bit pattern

constexpr int kMaxSplits = 256;                // most vocabulary splits of the output projection
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kSplit2Operand = 2048;           // bytes of one two-term fp16 operand, 32 words or rows x 16 units
constexpr int kSplit2DExp = 14;                // fp32 models: the centred hidden vector times 2^14 in dfrag
constexpr float kLn2 = 0.6931471805599453f;

// Device-side view of a loaded model (all pointers are device pointers).  It is an argument of every kernel, which fetches from it in front
// of everything else, by lines of 64 bytes: no holes but behind single floats, and the weights of the hidden update in the first line.  With a
// pointer more in front of half_rowsum_W, us: tree of 1000000 words, H = 128, 64 rows 7.72 -> 7.84; 109192 words, H = 92, 143 rows 7.31 -> 7.45.
struct ModelDev {
    int V, H;
    int Hp;            // H rounded up to a multiple of 64; padded weights are zero
    int Vp;            // V rounded up to a multiple of 256; padded rows of Ot are zero
    int dtype;
    int hs_max_len;    // hierarchical output layer: longest path
    const void *U;     // [V][Hp]
    const void *W;     // [Hp rounded up to 128][Hp], W[j][i]
    const void *Ot;    // [Vp][Hp], Ot[v][j] = O[j][v]
    // W in MFMA-operand order for the one-launch step (step_few_supported), else null.  bf16: [Hp / 32][Hp / 16][64 lanes][8], lane
    // 32 g + c of fragment (blk, ks) holds unit 32 blk + c, inputs 16 ks + 8 g .. + 7; fp32: [Hp / 32][Hp / 16][2][64 lanes][4], the
    // first and the last four of those eight.
    const void *Wfrag;
    const float *half_rowsum_W;   // [Hp]  0.5 * sum_i W[j][i]
    const float *bias;            // [V]
    const float *half_colsum_O;   // [V]   0.5 * sum_j O[j][v]
    // Additive constant of every base-2 logit, (bias[v] + 0.5*colsum_O[v]) * log2(e); -inf
    // for the padded words v >= V so they add nothing to the sum.
    const float *cvec2;           // [Vp]
    const float *cvec2_fixed;     // [Vp]  cvec2 - m2_fixed
    const float *cvec_fixed;      // [Vp]  cvec2_fixed / log2(e): kernels whose accumulators start from it
    float m2_fixed;    // upper bound of every base-2 logit z*log2(e), valid because |h' - 0.5| <= 0.5
    // A second copy of the output weights in MFMA-operand order.  bf16: [Vp / 32][Hp / 16][64 lanes][8],
    // lane 32 g + c of fragment (blk, ks) holds word 32 blk + c, units 16 ks + 8 g .. + 7 (one operand =
    // 1 KB contiguous).  fp32: two fp16 terms of the weights times a power of two of their word (the
    // largest weight of a word lies in [2^13, 2^14)), [Vp / 32][Hp / 16][2 terms][64 lanes][8].
    const void *Ofrag;
    const float *ofac;            // [Vp] fp32 models: log2(e) / (the word's power of two * 2^14)
    int infinite_O;               // fp32 models: some output weight is infinite or NaN (the two terms of an infinity add up to NaN)
    // hierarchical output layer (models loaded with rnnlm_hs_load; Ot .. cvec2_fixed are null then)
    int hs;                       // 1: hierarchical
    const void *Theta;            // [V-1][Hp] node vectors, weights' type, zero-padded
    const int32_t *path_off;      // [V+1]
    const int32_t *path_entry;    // [path_off[V]] node | code bit << 31, root first
    // W in MFMA-operand order as bf16 terms (one of bf16 models, the same as Wfrag there; three of fp32 models) for the whole form of the
    // hidden update (recur_whole_supported), else null: [Hp / 32][Hp / 16][terms][64 lanes][8].
    const void *Wops;
    // scratch
    void *d;           // [max_Bp][Hp]  h' - 0.5 in the weights' type
    // The same block in the order the output projection reads it as an MFMA operand.  bf16 models: times
    // d_scale, [max_Bp / 32][Hp / 16][64 lanes][8], lane 32 g + c of fragment (rb, ks) holds row
    // 32 rb + c, units 16 ks + 8 g .. + 7, so one operand of a wave is 1 KB contiguous.  fp32 models:
    // times 2^14 as two fp16 terms, [max_Bp / 32][Hp / 16][2 terms][64 lanes][8].
    void *dfrag;
    float d_scale;     // set for the hidden update only: outproj_d_scale of the output projection that follows
    float2 *part;      // [max_Bp][kMaxSplits]  (max, sum) partials of the base-2 log-sum-exp
    int *flag;         // sticky rnnlm_device_flag bits
    unsigned *done;    // workgroups of a one-launch step (step_few.hip) that have finished; wraps to 0 with the last one
};

// Device-side view of a cache kept between steps (cache.hip).
struct CacheCell {          // one slot of the open-addressing table
    uint64_t key;
    int32_t entry;          // index into the stores, -1 = free
    int32_t pad;
};
struct CacheDev {
    int capacity;           // entries the stores can hold
    int table_size;         // power of two >= 2 * capacity
    int H;
    CacheCell *table;       // [table_size]
    float *store_h;         // [capacity][H]  updated hidden vectors
    float *store_lse;       // [capacity]     natural-log normalisers
    int *n_entries;         // [1]
    long long *totals;      // [4] looked up, found, computed, computed but not kept
    // per-step scratch, each [max_B]
    int32_t *entry_of;      // distinct history u -> its entry (found or newly given), or -1
    int32_t *miss_of;       // u -> row of this step's computed block, or -1 when found
    int32_t *miss_src;      // computed row -> raw query that holds its prev word and h_in
    int32_t *miss_dst;      // computed row -> u
    float *lse_rows;        // [max_B] normaliser of every distinct history of the step
    int *n_miss;            // [1]
    int *block_total;       // [max_B / 1024 + 2] scan scratch of the many-workgroup lookup; last = entries before
};
// Device-side view of an index table (index_table.hip): contexts stored by value, found again
// by content.  The hash table, the counters and the per-call scratch are the cache's.
struct IndexDev {
    CacheDev c;             // c.store_h = hidden vectors [capacity][H]; c.store_lse, c.lse_rows unused
    int32_t *store_word;    // [capacity]
    uint64_t *keys;         // [max_N] content hashes of the call
    int32_t *rep, *inverse; // [max_N] grouping of the call's hashes
    int32_t *n_unique;      // [1]
    void *dedup_ws;
    long long *errors;      // [2] hash collisions caught by the full comparison, bad indices in fetch
};

}  // namespace rnnlm

struct rnnlm_index_table {
    rnnlm::IndexDev dev;
    int max_N;
};

struct rnnlm_cache {
    rnnlm::CacheDev dev;
    int max_B;
};

struct rnnlm_model {
    rnnlm::ModelDev dev;   // the weights' pointers may be another handle's (see owner); the scratch is this handle's
    int max_B, max_Bp;
    int fixed_ok;          // the fixed-offset log-sum-exp is usable for this model
    int lse_mode;          // RNNLM_OPT_LSE_MODE
    int outproj_kernel;    // RNNLM_OPT_OUTPROJ_KERNEL
    hipEvent_t ev0, ev1;
    // Handles made by rnnlm_model_share point at the handle that loaded the weights; that one counts
    // the handles alive on its weights (itself included until it is released) and frees the weights
    // with the last of them.  Both fields are guarded by one library-wide lock.
    rnnlm_model *owner;    // null: this handle loaded the weights
    int handles;           // owner only: handles alive on these weights
    int released;          // owner only: rnnlm_free was called on it, the struct lives on for the others
};

namespace rnnlm {

// A kernel's dynamic-LDS limit, raised once per device to the largest size asked for so far.  Safe
// when two host threads make the first launch at the same time (one static object per kernel).
class LdsLimit {
  public:
    hipError_t ensure(const void *kernel, size_t bytes) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kDevices) return hipErrorInvalidDevice;
        if (granted_[dev].load(std::memory_order_acquire) >= bytes) return hipSuccess;
        std::lock_guard<std::mutex> lock(mutex_);
        if (granted_[dev].load(std::memory_order_relaxed) >= bytes) return hipSuccess;
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e == hipSuccess) granted_[dev].store(bytes, std::memory_order_release);
        return e;
    }

  private:
    static constexpr int kDevices = 64;
    std::mutex mutex_;
    std::atomic<size_t> granted_[kDevices] = {};
};

// ---- launchers (each enqueues on `stream` and returns the hipGetLastError of the launch)

// Grouping of equal 64-bit keys.
size_t dedup_workspace_bytes(int N);
hipError_t launch_dedup(const uint64_t *keys, int N, int32_t *rep, int32_t *inverse,
                        int32_t *n_unique, void *workspace, hipStream_t stream);
// Looks the address of rnnlm_dedup_static's device array up for the current device (status code).
int dedup_static_prepare();

// Hidden update.  rows = number of rows the grid must cover (>= the true B); the true B is
// *B_dev when B_dev != nullptr, else rows.  row_src (nullable) maps row b to the raw row
// that holds its prev word and h_in; row_dst (nullable) maps it to its row of h_out (the
// operand block m.d always takes row b).
// ids.key set (recur_groups_ids(m, rows)): the launch groups the `rows` raw queries' ids first, as launch_dedup does,
// and takes rows and count from that (B_dev and row_src null).
struct IdGroups {
    const uint64_t *key;                       // [rows] or null
    int32_t *rep, *inverse, *n_unique;         // as launch_dedup leaves them
};
constexpr int kGroupedMax = 1024;          // most of them
bool recur_groups_ids(const ModelDev &m, int N);
hipError_t launch_recur(const ModelDev &m, int rows, const int *B_dev, const int32_t *row_src,
                        const int32_t *row_dst, const int32_t *prev_word, const float *h_in,
                        float *h_out, const IdGroups &ids, hipStream_t stream);
// Its whole form (recur_whole.hip): units per workgroup for these rows, 0 where the ring is taken.
bool recur_whole_supported(int dtype, int Hp);            // the model gets Wops
int recur_whole_units(const ModelDev &m, int rows, bool vec, bool grouped);
hipError_t launch_recur_whole(const ModelDev &m, int units, bool vec, int rows, const int *B_dev, const int32_t *row_src, const int32_t *row_dst,
                              const int32_t *prev_word, const float *h_in, float *h_out, const IdGroups &ids, hipStream_t stream);
constexpr int kXcds = 8;           // workgroup id modulo 8 = the XCD (L2 domain) it runs on
constexpr int kChipGroups = 256;   // workgroups in one round: one per compute unit
// Rows for which workgroups of 32 rows and `units` units fit the chip in `rounds` rounds, a row block on one XCD.
__host__ __device__ constexpr int whole_rows(int Hp, int units, int rounds) { return 32 * kXcds * (rounds * kChipGroups / kXcds / (Hp / units)); }
// The largest padded hidden size of the kernel that takes Hp.  In steps of 128: a kernel requests the weights of all its k-steps.  Us, hidden
// update of the next power of two or multiple of 256 / this, steps with the hierarchical layer: bf16, H = 384, 1000 rows 10.28 / 10.15, H = 640,
// 700 12.75 / 12.66; fp32, H = 384, 300 ids 12.34 / 12.00, 700 of 4096 distinct 21.73 / 21.45.
constexpr int recur_whole_top(int Hp) { return (Hp + 127) / 128 * 128; }
// Its kernels for hidden sizes up to `top`: where recur_whole_units, and the form for few units that comes in front of it, leave them any launch.
constexpr bool recur_whole_exists(bool bf16, int top, int units, bool vec, bool grouped) {
    if (units == 64 && !vec && top <= 512) return false;
    if (grouped) return top > (bf16 ? 128 : 64) && (units == 32 || whole_rows(top, 32, 1) < kGroupedMax);
    return bf16 || units == 64 || (!vec && top > 256);
}

constexpr int kStagedRows = 256;   // rows per workgroup of the staged kernel
constexpr int kStagedWords = 32;   // words per LDS stage
// Waves of the staged kernel's workgroups, its streaming form included: four where a row's two terms take the registers of two waves.
constexpr int staged_waves(bool f32, int Hp) { return f32 && Hp > 320 ? 4 : 8; }
constexpr size_t kAllL2s = (size_t)kXcds * 4 << 20;

// Work split of an output-projection kernel for B rows on a grid of kXcds * wg_per_xcd workgroups.
// The true B may be known on the device only (after the grouping of ids or the cache lookup), so the
// kernels derive the split there, and the kernels that read the partials afterwards derive the
// same: RG row groups of group_rows rows; the vocabulary is cut into S = kXcds * Sx splits, as
// many as the grid gives every row group (at most sx_cap: one per tile of words); split s is
// served by XCD s % kXcds, so the RG workgroups that stream the same weights share one L2.
struct RowPlan { int RG, Sx, S; };
__host__ __device__ inline RowPlan plan_rows(int B, int group_rows, int wg_per_xcd, int sx_cap) {
    RowPlan p;
    p.RG = (B + group_rows - 1) / group_rows;
    if (p.RG < 1) p.RG = 1;
    p.Sx = wg_per_xcd / p.RG;
    if (p.Sx > sx_cap) p.Sx = sx_cap;
    if (p.Sx > kMaxSplits / kXcds) p.Sx = kMaxSplits / kXcds;
    if (p.Sx < 1) p.Sx = 1;
    p.S = kXcds * p.Sx;
    return p;
}
// First unit of part `index` when `units` units are cut into `parts` nearly equal parts,
// floor(index * units / parts), for 0 <= index <= parts <= 256 and units < 2^31.  With q = units / parts
// and r = units % parts this is index * q + floor(index * r / parts), and index * r stays below 2^16: 32-bit
// arithmetic throughout (a 64-bit division costs a wave some hundred scalar instructions in front of
// its first load).
__host__ __device__ inline int part_begin(int index, int units, int parts) {
    const unsigned q = (unsigned)units / (unsigned)parts, r = (unsigned)units % (unsigned)parts;
    return (int)((unsigned)index * q + ((unsigned)index * r) / (unsigned)parts);
}
typedef RowPlan StagedPlan;
__host__ __device__ inline StagedPlan staged_plan(int B, int wg_per_xcd) {
    return plan_rows(B, kStagedRows, wg_per_xcd, kMaxSplits / kXcds);
}
// Groups of 128 rows that do not divide an XCD's workgroups leave some of them idle (12 groups: 24 of 32 busy): with up to three items per
// workgroup one after the other the vocabulary is cut finer and fewer are.  A further item costs its rows' way into the registers, some 3 us, which is taken as
// a tenth of the launch; vocabularies below 16384 words keep to one.  Us per launch, one item / this, fp32: V = 65536, H = 512, 1100 rows 181 / 177, 1300
// 229 / 219, 1500 248 / 237; V = 20000, H = 512, 1300 78 / 77; V = 17000, H = 512, 2100 116 / 102; V = 50000, H = 576, 2600 383 / 345.  800 rows (7
// groups, 28 of 32 busy) keep to one: V = 65536, H = 512 134.7 / 134.2, V = 20000 49.6 / 50.6.
// Beyond 32 groups one item for every group and XCD takes two rounds by itself, and is counted as that: one split per XCD / this, V = 17000,
// H = 512, 4200 rows 336 / 290, H = 384, 4600 247 / 211, V = 65536, H = 512, 4200 1096 / 908, 5200 1099 / 931, V = 40000, H = 576, 4100 776 / 642
// (whole steps, us).
__host__ __device__ inline RowPlan plan_rounds(int B, int group_rows, int wg_per_xcd, int Vp) {
    RowPlan p = plan_rows(B, group_rows, wg_per_xcd, kMaxSplits / kXcds);
    if (p.RG < 5 || Vp < 16384) return p;
    auto busy_48ths = [&](int Sx) {                          // of the rounds that the items take
        const int rounds = (p.RG * Sx + wg_per_xcd - 1) / wg_per_xcd;
        return 48 * p.RG * Sx / (rounds * wg_per_xcd) - 5 * (rounds - 1);
    };
    int best = busy_48ths(p.Sx);
    for (int r = 2; r <= 3; ++r) {
        const int Sx = r * wg_per_xcd / p.RG;
        if (Sx <= kMaxSplits / kXcds && Sx > 0 && busy_48ths(Sx) > best) {
            best = busy_48ths(Sx);
            p.Sx = Sx;
        }
    }
    p.S = kXcds * p.Sx;
    return p;
}
// The staged kernel's row groups: 256 rows.  Beyond Hp = 512, three groups of 128 (four of a workgroup's eight waves each, with a
// matrix pipe to itself) where two of 256 would leave one less than half full.  Us per launch, 256 / 128, V = 30011, H = 650: 257, 300, 384
// rows 17.4 / 16.3, 17.5 / 16.2, 18.8 / 17.1, running maximum 20.9 / 19.0, 21.1 / 18.6, 21.8 / 19.4.  Not for five groups instead of
// three (600 rows 24.3 / 24.2), not for fp32 models (V = 100000, H = 128, 300 rows 30.0 / 31.6; V = 60000, H = 192, 200 rows 18.7 / 20.5; V = 100000,
// H = 256, 300 rows 53.3 / 51.0) and not below (V = 65536, H = 512, 300 rows 23.1 / 22.7, 600 35.2 / 36.4; V = 20000, H = 256, 300 rows 6.6 / 6.8).
struct StagedSplit {
    StagedPlan plan;
    int rows;              // of a group
};
__host__ __device__ inline StagedSplit staged_split(int B, int wg_per_xcd, bool halves) {
    if (halves && B > kStagedRows && B <= 3 * kStagedRows / 2)
        return StagedSplit{plan_rows(B, kStagedRows / 2, wg_per_xcd, kMaxSplits / kXcds), kStagedRows / 2};
    return StagedSplit{staged_plan(B, wg_per_xcd), kStagedRows};
}

// How many (max, sum) partials per row the output projection left in m.part: a fixed number, or
// the S of plan_rows for the true number of rows; a kernel that streams the weights when at most
// stream_rows rows are left then leaves one partial per workgroup that does so.
struct SplitInfo {
    int fixed_splits;      // > 0: that many
    int wg_per_xcd;        // else plan_rows(B, group_rows, wg_per_xcd, sx_cap).S
    int group_rows;        // 0: staged_split(B, wg_per_xcd, true).plan.S
    int sx_cap;            // group_rows < 0: plan_rounds(B, -group_rows, wg_per_xcd, sx_cap).S
    int stream_rows;       // 0 < B <= stream_rows: stream_splits instead (0: every workgroup of the grid has one)
    int stream_splits;
};
__host__ __device__ inline int splits_of(const SplitInfo &si, int B) {
    if (si.fixed_splits > 0) return si.fixed_splits;
    if (B > 0 && B <= si.stream_rows) return si.stream_splits > 0 ? si.stream_splits : kXcds * si.wg_per_xcd;
    if (si.group_rows < 0) return plan_rounds(B, -si.group_rows, si.wg_per_xcd, si.sx_cap).S;
    if (si.group_rows == 0) return staged_split(B, si.wg_per_xcd, true).plan.S;
    return plan_rows(B, si.group_rows, si.wg_per_xcd, si.sx_cap).S;
}
__host__ inline SplitInfo fixed_split_info(int S) { return SplitInfo{S, 0, 1, 1, 0, 0}; }

// Output projection + log-sum-exp partials over the vocabulary, on the block m.d.
hipError_t launch_outproj(const ModelDev &m, int rows, const int *B_dev, bool fixed_offset,
                          int kernel_choice, SplitInfo *splits, hipStream_t stream);
// false: the kernel launch_outproj takes for these arguments reads only the fragment-ordered copy of
// the hidden block, and the hidden update may leave the row-ordered one (m.d) unwritten
bool outproj_reads_row_order(const ModelDev &m, int rows, bool fixed_offset, int kernel_choice);
// bf16 models: the factor the fragment-ordered copy carries.  log2(e): the accumulators are base-2 logits.  1, for the
// padded hidden sizes the staged kernel took over from the tiled one: units at their limits, h' - 1/2 = +-1/2, are
// exact in bf16 only unscaled, and models with large weights have many (V = 30011, H = 650, weights of 0.2: error of
// the log-probabilities 2.82e-5 unscaled, as in the tiled kernel, 3.70e-5 scaled).
constexpr bool staged_scaled_d(int Hp) { return Hp == 128 || Hp == 256 || Hp == 512; }
float outproj_d_scale(const ModelDev &m, int rows, bool fixed_offset, int kernel_choice);
const char *outproj_kernel_name(const ModelDev &m, int rows, bool fixed_offset, int kernel_choice);
bool outproj_staged_supported(const ModelDev &m);
bool outproj_rowstream_supported(const ModelDev &m);   // bf16 models
int outproj_stream_max_rows(const ModelDev &m);   // 0: the weight-streaming kernel cannot serve this model

// Query gather: logprob[n][k] = z[row(n)][query[n][k]] - lse[row(n)] - base_score[n][k].
// lse comes from lse_rows[row] when that is given, else from the partials in m.part;
// base_score may be null.
hipError_t launch_query(const ModelDev &m, int rows, const int *B_dev, int N, int K, SplitInfo splits,
                        const int32_t *query_word, const int32_t *row_of_query,
                        const float *h_out, const float *lse_rows, const float *base_score,
                        float *logprob, hipStream_t stream);

// Grouping of ids, hidden update, output projection and query gather of few rows in one launch.
struct FewStep {
    int rows;                                  // rows, or raw queries (ids.key set: the launch groups the ids)
    int N, K;
    IdGroups ids;
    const int32_t *prev_word;
    const float *h_in;
    const int32_t *query_word, *row_of_query;  // (row_of_query is not read with ids)
    const float *base_score;
    float *h_out, *logprob;
    bool vec;                                  // rows of h_in in 16-byte pieces
    uint32_t inverse_K;                        // ceil(2^32 / K), for K > 1
    // query that pair p (word p % K of query p / K) belongs to: exact while N * K * K < 2^32
    __host__ __device__ int query_of(int p) const { return K == 1 ? p : (int)(((uint64_t)(uint32_t)p * inverse_K) >> 32); }
};
bool step_few_supported(int dtype, int Hp);               // the model gets a Wfrag
bool step_few_chosen(const ModelDev &m, int rows, bool grouped, int N, int K);
hipError_t launch_step_few(const ModelDev &m, const FewStep &a, bool fixed_offset, hipStream_t stream);
// the output projection takes the weight-streaming kernel by itself, in one launch
bool outproj_streams_in_one_launch(const ModelDev &m, int rows, int kernel_choice);

// The same through a cache (after launch_cache_lookup and the computation of the histories not
// found): found histories take h' and lse from the stores, and the first raw query of every distinct
// history passes its h' on (to h_out when found, into the store with its lse when it got an entry),
// which is all that launch_cache_commit does otherwise.  rows / n_unique: distinct histories.
hipError_t launch_query_cached(const ModelDev &m, const CacheDev &c, int rows, const int32_t *n_unique, int N, int K,
                               SplitInfo splits, const int32_t *query_word, const int32_t *inverse,
                               const int32_t *rep, float *h_out, const float *base_score, float *score,
                               hipStream_t stream);

// ---- cache kept between steps (cache.hip)
// errors: an index table's two error counters, cleared along with it, or null
hipError_t launch_cache_reset(const CacheDev &c, long long *errors, hipStream_t stream);
// Looks the distinct histories ids[rep[u]], u < *n_unique, up; numbers the ones not found
// (in order of u), gives them entries while there is room and inserts their keys.
// rows = upper bound of *n_unique (sizes the grid).  Three launches of a full grid.
hipError_t launch_cache_lookup(const CacheDev &c, int rows, const uint64_t *ids,
                               const int32_t *rep, const int32_t *n_unique, int32_t *step_stats,
                               hipStream_t stream);
// Grouping of the ids (launch_dedup) and this lookup in ONE launch of one workgroup, for
// 0 <= N <= dedup_lookup_max_rows() raw queries (or contexts of an index table).
int dedup_lookup_max_rows();
// The output weights as a weight-streaming launch further on reads them; splits 0: nothing to read ahead.
struct WeightsAhead {
    const void *Ofrag;
    int blocks, block_kb;  // blocks of 32 words, kilobytes of each (a multiple of 4)
    int splits, waves;     // workgroups of that launch, waves of each
};
// Where piece number `piece` of four kilobytes, in the order the workgroup of `split` reads them (rounds of `waves` blocks side by
// side, a piece of each at a time), lies, in kilobytes; -1: that workgroup has no such piece.
__host__ __device__ inline long long ahead_piece(const WeightsAhead &a, int split, int piece) {
    const int per_round = a.block_kb / 4 * a.waves, round = piece / per_round, rest = piece % per_round;
    const int blk = part_begin(split, a.blocks, a.splits) + round * a.waves + rest % a.waves;
    return blk < part_begin(split + 1, a.blocks, a.splits) ? (long long)blk * a.block_kb + rest / a.waves * 4 : -1;
}
WeightsAhead outproj_weights_ahead(const ModelDev &m, int rows, bool fixed_offset, int kernel_choice);
hipError_t launch_dedup_lookup(const CacheDev &c, const uint64_t *ids, int N, int32_t *rep, int32_t *inverse,
                               int32_t *n_unique, int32_t *step_stats, const WeightsAhead &ahead, hipStream_t stream);
// After the computed block is done: normalisers of all distinct histories into c.lse_rows,
// new entries into the stores, stored hidden vectors of found histories into h_out.
hipError_t launch_cache_commit(const CacheDev &c, const ModelDev &m, int rows, const int32_t *n_unique,
                               SplitInfo splits, float *h_out, hipStream_t stream);
// Index table: content hashes of N contexts; after grouping and lookup, storage of the new
// contexts, full comparison of every context with the one it was identified with, and the
// indices; gather of stored contexts.
hipError_t launch_context_hash(const int32_t *word, const float *h, int N, int H, uint64_t *keys,
                               hipStream_t stream);
hipError_t launch_index_commit(const IndexDev &t, int N, const int32_t *word, const float *h, uint32_t *index,
                               hipStream_t stream);
hipError_t launch_index_fetch(const IndexDev &t, int N, const uint32_t *index, int32_t *word, float *h,
                              hipStream_t stream);
// Hierarchical output layer: logprob[n][k] = sum over the path of query[n][k] of
// log sigmoid(+-theta_node . h'[row(n)]) (- base_score[n][k]).
hipError_t launch_hs_query(const ModelDev &m, int rows, const int *B_dev, int N, int K,
                           const int32_t *query_word, const int32_t *row_of_query, const float *h_out,
                           const float *base_score, float *logprob, hipStream_t stream);
// The same with the hidden update in the launch (mapped: row_of_query is given).
bool hs_step_chosen(const ModelDev &m, int B, int N, int K, bool mapped);
hipError_t launch_hs_step(const ModelDev &m, int B, int N, int K, const int32_t *prev_word, const float *h_in, const int32_t *query_word,
                          const int32_t *row_of_query, float *h_out, const float *base_score, float *logprob, hipStream_t stream);
hipError_t launch_pack_ids(const uint32_t *ctx, const uint32_t *small_lm, int N, uint64_t *ids,
                           hipStream_t stream);

// Load-time helpers.
// [rows][H] -> [rows][Hp], zero-padded
hipError_t launch_pad_rows(const void *src, void *dst, int dtype, size_t rows, int H, int Hp, hipStream_t stream);
hipError_t launch_transpose_O(const void *O_dev /*[H][V]*/, void *Ot /*[Vp][Hp]*/, int dtype,
                              int H, int V, int Hp, int Vp, hipStream_t stream);
hipError_t launch_col_stats(const void *O_dev, const float *bias_or_null, int dtype, int H, int V,
                            float *half_colsum /*[V]*/, float *upper /*[V]*/, float *lower /*[V]*/,
                            hipStream_t stream);
hipError_t launch_frag_weights(const void *Ot /*[Vp][Hp] bf16*/, int Vp, int Hp, void *Ofrag, hipStream_t stream);
// W [Hp][Hp] in the order of Wfrag
hipError_t launch_frag_recurrent(const void *W, int dtype, int Hp, void *Wfrag, hipStream_t stream);
// fp32 W [Hp][Hp] in the order of Wops
hipError_t launch_recurrent_terms(const float *W, int Hp, void *Wops, hipStream_t stream);
hipError_t launch_split2_weights(const float *Ot /*[Vp][Hp]*/, int Vp, int Hp, void *Ofrag, float *ofac /*[Vp]*/,
                                 hipStream_t stream);
hipError_t launch_fill_cvec(const float *bias_or_null, const float *half_colsum, int V, int Vp,
                            float m2_fixed, float *bias_out, float *cvec2, float *cvec2_fixed, float *cvec_fixed,
                            hipStream_t stream);

}  // namespace rnnlm
