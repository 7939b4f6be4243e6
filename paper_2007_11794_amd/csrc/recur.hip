// Hidden update  h'[b][j] = sigmoid(U[prev[b]][j] + sum_i W[j][i] h_in[b][i])
// (the context update inside ComputeRnnlm, Table 1 step 6; Section 4.1: the context is the
// previous hidden layer plus the previous word).
//
// The activation enters the product centred: h_in = 1/2 + d, so
//     W h_in = 1/2 rowsum(W) + W d,
// with the first term precomputed at load time in fp64.  |d| <= 1/2 carries three times
// less rounding error than h_in when it is cut to bf16 for the matrix cores.  bf16 models: d = d1 + d2
// in bf16 terms, two MFMA passes, so that the hidden vector is accurate to fp32 level.  fp32 models: every
// fp32 number is the exact sum of three bf16 numbers, of the nine cross terms of a product the six with
// the largest weight are kept (w1 d1, w1 d2, w2 d1, w1 d3, w3 d1, w2 d2; the dropped ones are below 2^-24
// of the product): six MFMA passes, still a fraction of the time the operands take to arrive.  h_in is
// the caller's and need not lie in [0, 1]: sums that meet an infinity or a number beyond the largest bf16 one are done
// again in plain fp32 (plain_sum4).
//
// Besides h_out (fp32, caller's buffer) the kernel leaves d' = h' - 1/2 in the model's
// scratch blocks as the operand of the output projection: row-major in the weights' type;
// also in MFMA-operand order, for bf16 models times log2(e) where the following kernel wants that, for fp32
// models as two fp16 terms (see ModelDev).
//
// What bounds it is the way of the operands into LDS: a chain of dependent reads (row count and rows to
// take, side by side; then the rows; then the embedding rows), and after it the bytes a compute unit
// takes in.  There are two shapes of a workgroup of eight waves, picked by the true row count (which only
// the device may know), in one launch:
//   small  64 units x 32 rows, the reduction length split over four pairs of waves: while there are at most two
//          of its workgroups per compute unit (few bytes per workgroup, all units at work; see small_rows);
//   large  128 units x 64 rows, a wave owns 64 x 32 of them over half of the reduction: h_in is converted
//          once for two blocks of units, and reading, converting and multiplying overlap between the waves
//          (with 32 x 32 per wave over the whole reduction H = 1024, 3000 rows took 43 us instead of 30).
// Models of few units have a third, in kernels of its own (recur_few_units_f32_kernel, recur_few_units_bf16_kernel), and where the
// whole of a workgroup's operands fits registers and LDS and its workgroups the compute units there is a fourth (recur_whole.h), which of
// the sizes below has taken over bf16 H = 512, H = 650 and fp32 H = 512 with 1024 rows: what stands there are the ring's times.
// Launches of bf16 models that fit one small workgroup per compute unit use a whole unit's LDS as the ring (128 KB, all
// but one stage in flight), larger ones half of it, two workgroups per unit; fp32 models always the whole one.
// Measured, us per launch (rows in brackets), before and after, the kernels before being one tiled and one
// register-direct kernel for bf16 models and the fp32 matrix instruction for fp32 ones: bf16 H = 512 (1024)
// 9.6 -> 8.6, (41 of 4096) 8.3 -> 5.8, (1229 of 4096) 12.0 -> 11.2; H = 1024 (2048) 30.6 -> 22.6, (200 of 2048)
// 15.3 -> 10.8; H = 650 (317) 13.9 -> 10.7; H = 333 (1000) 14.7 -> 7.8; fp32 H = 512 (1024) 19.2 -> 12.8,
// (4000) 53.8 -> 29.7; H = 1024 (1024) 44.2 -> 32.9.  The error of fp32 models' h' against float64 went from
// 4.7e-8 to 4.3e-8 (H = 512), bf16 models' stayed.
#include <algorithm>

#include "dedup_small_body.h"
#include "device_utils.h"
#include "recur_whole.h"
#include "rnnlm_internal.h"

namespace rnnlm {

namespace {

constexpr int kThreads = kRecurThreads, kWaves = kThreads / 64;
constexpr int kGroups = kChipGroups;
constexpr int kFewUnitsBf16 = 128;                    // the only Hp of recur_few_units_bf16_kernel

// Tiles in LDS.  A half row is 128 bytes, eight pieces of 16; piece c of row r sits at c ^ ((r >> 1) & 7), so
// that the rows a ds_read_b128 takes together hit different banks.  A chunk is 64 units of the reduction:
// one half row per row of a bf16 tile, two (first all rows' lower halves, then the upper ones) of a
// float tile.  Direct global->LDS loads write LDS linearly, so the rotation is applied on the global side.
__device__ __forceinline__ int swizzle(int row) { return (row >> 1) & 7; }

// Eight floats (units 16 ks + 8 g .. + 7 of a chunk) of row r of a float tile of R rows.
template <int R>
__device__ __forceinline__ void read8(const char *tile, int r, int ks, int g, float (&x)[8]) {
    const char *half_row = tile + ((ks >> 1) * R + r) * 128;
    const int c = 4 * (ks & 1) + 2 * g;
    const f32x4 lo = *reinterpret_cast<const f32x4 *>(half_row + ((c ^ swizzle(r)) * 16));
    const f32x4 hi = *reinterpret_cast<const f32x4 *>(half_row + (((c + 1) ^ swizzle(r)) * 16));
#pragma unroll
    for (int i = 0; i < 4; ++i) { x[i] = lo[i]; x[4 + i] = hi[i]; }
}

// One shape: TU units x TB rows per workgroup; a wave owns 32 MB units x 32 rows, the reduction is split over
// WK groups of waves; stages of SUB chunks in RING bytes.  VEC: rows of h_in in 16-byte pieces (H a multiple
// of 4, aligned buffers), else in single floats.
template <typename WT, int TU, int TB, int MB, int WK, int SUB, int RING, bool VEC>
struct Shape {
    static constexpr bool kF32 = sizeof(WT) == 4;
    static constexpr int kWBytes = TU * 64 * (int)sizeof(WT), kHBytes = TB * 256, kChunkBytes = kWBytes + kHBytes;
    static constexpr int kStages = RING / (SUB * kChunkBytes);
    static constexpr int kWLoads = kWBytes / 16 / kThreads, kHLoads = kHBytes / (VEC ? 16 : 4) / kThreads;
    static constexpr int kLoads = SUB * (kWLoads + kHLoads);       // per thread and stage
    static constexpr int kSums = 4 * MB;                           // four-unit results of a lane's accumulators
    static_assert(TU / (32 * MB) * (TB / 32) * WK == kWaves && kWLoads * 16 * kThreads == kWBytes && kStages >= 2, "");
    static_assert((kStages - 2) * kLoads < 64, "vmcnt");
    static_assert(kWaves * kSums * 1024 <= kStages * SUB * kChunkBytes, "partial sums fit the stages");
    static_assert(kSums % WK == 0 && SUB * 4 % WK == 0, "");
};

// Wait until at most `later` (0 .. MAX) stages of L loads each are outstanding.
template <int MAX, int L>
__device__ __forceinline__ void wait_stages(int later) {
    if constexpr (MAX == 0) wait_vmcnt<0>();
    else if (later >= MAX) wait_vmcnt<MAX * L>();
    else wait_stages<MAX - 1, L>(later);
}

// rows b0 .. b0 + TB - 1, units j0 .. j0 + TU - 1; source: the row of h_in / prev_word that lane tid of the
// first TB threads holds for row b0 + tid (rows beyond B are dropped).
template <typename WT, int TU, int TB, int MB, int WK, int SUB, int RING, bool VEC>
__device__ __forceinline__ void recur_body(const ModelDev &m, int B, int b0, int j0, int source,
                                           const int32_t *__restrict__ row_dst, const int32_t *__restrict__ prev_word,
                                           const float *__restrict__ h_in, float *__restrict__ h_out, char *lds, int *srcs, int *prevs) {
    using C = Shape<WT, TU, TB, MB, WK, SUB, RING, VEC>;
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int WJ = TU / (32 * MB), WB = TB / 32;
    const int wj = wave % WJ, wb = wave / WJ % WB, wk = wave / (WJ * WB);
    const int H = m.H, Hp = m.Hp;
    const WT *W = static_cast<const WT *>(m.W), *U = static_cast<const WT *>(m.U);
    if (tid < TB) srcs[tid] = source;
    __syncthreads();
    const int last = B - 1 - b0;                       // rows beyond B repeat the last one; dropped later

    // loader
    uint32_t woff[C::kWLoads];
#pragma unroll
    for (int q = 0; q < C::kWLoads; ++q) {
        const int f = q * kThreads + tid, hr = f >> 3, r = hr % TU, c = (f & 7) ^ swizzle(r);
        woff[q] = (uint32_t)(r * Hp * (int)sizeof(WT) + (hr / TU) * 128 + c * 16);
    }
    const float *hrow[C::kHLoads];
    int hk[C::kHLoads];                                // unit of the chunk
#pragma unroll
    for (int q = 0; q < C::kHLoads; ++q) {
        const int f = q * kThreads + tid, e = VEC ? 0 : f & 3, p = VEC ? f : f >> 2;
        const int hr = p >> 3, r = hr % TB, c = (p & 7) ^ swizzle(r);
        hrow[q] = h_in + (size_t)srcs[min(r, last)] * H;
        hk[q] = (hr / TB) * 32 + 4 * c + e;
    }
    const uint32_t lds0 = lds_address(lds) + wave * (VEC ? 1024 : 256);
    const uint32_t ldsw = lds_address(lds) + wave * 1024;
    const int nk = Hp / (64 * SUB);                    // stage-chunks (the caller checks divisibility)
    auto issue = [&](int sc, int stage) {             // the SUB chunks of stage-chunk sc
#pragma unroll
        for (int sub = 0; sub < SUB; ++sub) {
            const int k0 = (sc * SUB + sub) * 64;
            const uint32_t base = (stage * SUB + sub) * C::kChunkBytes;
            const WT *wsrc = W + (size_t)j0 * Hp + k0;
#pragma unroll
            for (int q = 0; q < C::kWLoads; ++q) lds_dma_16(wsrc, woff[q], ldsw + base + q * (kThreads * 16));
#pragma unroll
            for (int q = 0; q < C::kHLoads; ++q) {
                // past the end of the row the weights are zero: fetch the row's beginning
                const int k = k0 + hk[q];
                if (VEC)
                    lds_dma_16_ptr(hrow[q] + (k + 4 <= H ? k : 0), lds0 + base + C::kWBytes + q * (kThreads * 16));
                else
                    lds_dma_4_ptr(hrow[q] + (k < H ? k : 0), lds0 + base + C::kWBytes + q * (kThreads * 4));
            }
        }
    };
    const int rb = 32 * wb + col, b = b0 + rb;
    // The previous words travel through LDS as well: as an ordinary load the compiler would await them with
    // everything that is on its way to LDS.
    if (wave == 0) lds_dma_4_ptr(prev_word + srcs[min(lane % TB, last)], lds_address(prevs));
#pragma unroll
    for (int c = 0; c < C::kStages - 1; ++c)
        if (c < nk) issue(c, c);
    // Of the 4 MB four-unit results in a lane's accumulators (number r: units 8 r + 4 g .. + 3 of the wave's
    // 32 MB) wave group wk finishes kMine from wk kMine on.
    constexpr int kMine = C::kSums / WK;
    const int je = j0 + 32 * MB * wj + 8 * kMine * wk + 4 * g;
    const bool units_ok = je - 4 * g < Hp;             // wave-uniform; a large tile may reach past Hp
    const bool row_ok = b < B;
    const int dst = row_dst ? row_dst[min(b, B - 1)] : min(b, B - 1);
    bool w_ok = false;
    f32x4 rs[kMine], u[kMine];
#pragma unroll
    for (int q = 0; q < kMine; ++q) rs[q] = load4(m.half_rowsum_W + (units_ok ? je + 8 * q : 0));

    f32x16 acc[MB] = {}, rest[MB] = {};
    int stage = 0, into = C::kStages - 1;
    for (int sc = 0; sc < nk; ++sc) {
        // my loads of this stage have landed once only those of the later ones requested are outstanding
        wait_stages<C::kStages - 2, C::kLoads>(nk - 1 - sc);
        __syncthreads();                               // everybody's; the stage before this one is free
        if (sc == 0) {                                 // the previous words are there as well: the embedding rows
            const int w = prevs[rb];
            w_ok = w >= 0 && w < m.V;
#pragma unroll
            for (int q = 0; q < kMine; ++q)
                u[q] = load4(U + (size_t)(w_ok ? w : 0) * Hp + (units_ok ? je + 8 * q : 0));
        }
        if (sc + C::kStages - 1 < nk) issue(sc + C::kStages - 1, into);
        into = into == C::kStages - 1 ? 0 : into + 1;
        const char *st = lds + stage * SUB * C::kChunkBytes;
        stage = stage == C::kStages - 1 ? 0 : stage + 1;
        constexpr int kSteps = SUB * 4 / WK;           // this wave's k-steps of the stage
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
            const int step = wk * kSteps + i, ks = step & 3;
            const char *tile = st + (step >> 2) * C::kChunkBytes;
            float x[8];
            read8<TB>(tile + C::kWBytes, rb, ks, g, x);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] -= 0.5f;
            u32x4 d[C::kF32 ? 3 : 2];
            bf16_terms(x, d);
#pragma unroll
            for (int a = 0; a < MB; ++a) {
                const int ra = 32 * (MB * wj + a) + col;
                if constexpr (C::kF32) {
                    float y[8];
                    read8<TU>(tile, ra, ks, g, y);
                    u32x4 w[3];
                    bf16_terms(y, w);
                    // the small cross terms in a sum of their own: what rounds is the large one, once per step
                    rest[a] = mma(w[1], d[1], rest[a]);
                    rest[a] = mma(w[2], d[0], rest[a]);
                    rest[a] = mma(w[0], d[2], rest[a]);
                    rest[a] = mma(w[1], d[0], rest[a]);
                    rest[a] = mma(w[0], d[1], rest[a]);
                    acc[a] = mma(w[0], d[0], acc[a]);
                } else {
                    const u32x4 w = *reinterpret_cast<const u32x4 *>(tile + ra * 128 + (((2 * ks + g) ^ swizzle(ra)) * 16));
                    acc[a] = mma(w, d[0], acc[a]);
                    acc[a] = mma(w, d[1], acc[a]);
                }
            }
        }
    }
    if constexpr (C::kF32) {
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][i] += rest[a][i];
    }
    if (row_ok && !w_ok && lane < 32 && wj == 0 && wk == 0 && j0 == 0) atomicOr(m.flag, RNNLM_FLAG_BAD_PREV_WORD);
    const Finish f = {h_out + (size_t)dst * H, b, H, Hp, w_ok};
    auto result = [&](int r) { return f32x4{acc[r / 4][4 * (r % 4)], acc[r / 4][4 * (r % 4) + 1], acc[r / 4][4 * (r % 4) + 2],
                                            acc[r / 4][4 * (r % 4) + 3]}; };
    // the partial sums of a block meet in LDS (the stages are free)
    f32x4 *red = reinterpret_cast<f32x4 *>(lds);   // [wave][result][lane]
    __syncthreads();
#pragma unroll
    for (int r = 0; r < C::kSums; ++r) red[(wave * C::kSums + r) * 64 + lane] = result(r);
    __syncthreads();
    if (!row_ok || !units_ok) return;
#pragma unroll
    for (int q = 0; q < kMine; ++q) {
        const f32x4 *mine = red + ((wave % (WJ * WB)) * C::kSums + wk * kMine + q) * 64 + lane;
        f32x4 sum = mine[0];
#pragma unroll
        for (int other = 1; other < WK; ++other) { // fixed order: deterministic
            const f32x4 t = mine[other * (WJ * WB) * C::kSums * 64];
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[i] += t[i];
        }
        if constexpr (C::kF32) {
            if (sum[0] != sum[0] || sum[1] != sum[1] || sum[2] != sum[2] || sum[3] != sum[3])
                sum = plain_sum4(W + (size_t)(je + 8 * q) * Hp, Hp, H - (je + 8 * q), h_in + (size_t)srcs[rb] * H, H);
        }
        finish4<WT, VEC>(m, f, je + 8 * q, sum, rs[q], u[q]);
    }
}

// Few units, fp32 models first: 32 units x 32 rows per workgroup of four waves, a quarter of the reduction each, every operand
// straight into registers in one go (no ring, no split into terms) and products on the fp32 matrix instruction.  While its
// workgroups fit the compute units in one round the chain of loads is all there is to it, and the shorter one wins.  Us per
// launch, the ring above / this: H = 64, 73 rows 4.1 / 3.6, 3000 4.7 / 3.9; H = 99, 172 rows 5.9 / 4.7; H = 204, 674 rows 6.9 / 5.6; H = 256,
// 1000 rows (one round) 7.2 / 6.5, 1500 7.4 / 8.7, 3000 13.7 / 12.5; H = 128, 2048 rows (one round) 5.6 / 4.8, 3000 5.7 / 5.9.
// MFMA 32x32x2 operand layout: lane l holds k = l / 32 of row (column) l % 32; here a lane takes four consecutive k, and
// instruction e of a group multiplies the k pair {k0 + e, k0 + 4 + e}.
// bf16 models the same with the products of the ring form, where rows are not 16-byte aligned and Hp = 128: steps of 172 rows at
// H = 69 with the hierarchical layer 10.1 / 9.8, 20 rows 9.3 / 8.9, 600 rows at H = 117 10.5 / 10.4 (H = 226, 60 rows 10.8 / 11.4).
template <typename WT, bool VEC>
struct FewUnits {
    f32x4 (*red)[4][64];                               // LDS: [source wave][result][lane]
    int wave, lane, col, g, j0, b, src, je;
    bool row_ok, w_ok;
    f32x4 rs, u;

    __device__ __forceinline__ FewUnits(const ModelDev &m, int B, f32x4 (*lds)[4][64], const int32_t *row_src) : red(lds) {
        wave = threadIdx.x >> 6; lane = threadIdx.x & 63; col = lane & 31; g = lane >> 5;
        j0 = blockIdx.x * 32;
        b = blockIdx.y * 32 + col;
        row_ok = b < B;
        const int last = min(b, B - 1);                // rows beyond B repeat the last one; dropped later
        src = row_src ? row_src[last] : last;
        je = j0 + 8 * wave + 4 * g;                    // the four units this lane finishes
        rs = load4(m.half_rowsum_W + je);
    }
    // the embedding row hangs on the previous word: requested behind the operands
    __device__ __forceinline__ void word(const ModelDev &m, int w) {
        w_ok = w >= 0 && w < m.V;
        u = load4(static_cast<const WT *>(m.U) + (size_t)(w_ok ? w : 0) * m.Hp + je);
    }
    __device__ __forceinline__ void finish(const ModelDev &m, const f32x16 &acc, const int32_t *row_dst, float *h_out) const {
#pragma unroll
        for (int q = 0; q < 4; ++q) red[wave][q][lane] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        __syncthreads();
        if (!row_ok) return;
        if (!w_ok && g == 0 && wave == 0 && blockIdx.x == 0) atomicOr(m.flag, RNNLM_FLAG_BAD_PREV_WORD);
        f32x4 sum = red[0][wave][lane];
#pragma unroll
        for (int other = 1; other < 4; ++other) {      // fixed order: deterministic
            const f32x4 t = red[other][wave][lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[i] += t[i];
        }
        if (sizeof(WT) == 4 && m.H != m.Hp) {          // units beyond H are 0, an infinity in h_in times zero weights is not
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[i] = je + i < m.H ? sum[i] : 0.f;
        }
        const Finish f = {h_out + (size_t)(row_dst ? row_dst[b] : b) * m.H, b, m.H, m.Hp, w_ok};
        finish4<WT, VEC>(m, f, je, sum, rs, u);
    }
};

// GROUPS of eight k are in flight together; longer reductions go in several passes.
template <bool VEC, int GROUPS>
__global__ __launch_bounds__(256) void recur_few_units_f32_kernel(
    ModelDev m, int rows, const int *__restrict__ B_dev, const int32_t *__restrict__ row_src,
    const int32_t *__restrict__ row_dst, const int32_t *__restrict__ prev_word, const float *__restrict__ h_in,
    float *__restrict__ h_out) {
    const int B = B_dev ? *B_dev : rows;
    if ((int)blockIdx.y * 32 >= B) return;             // uniform
    __shared__ f32x4 red[4][4][64];
    FewUnits<float, VEC> t(m, B, red, row_src);
    const int H = m.H, Hp = m.Hp;
    const float *hrow = h_in + (size_t)t.src * H, *wrow = static_cast<const float *>(m.W) + (size_t)(t.j0 + t.col) * Hp;
    const int w = prev_word[t.src];
    const int kq = Hp / 4, k_begin = t.wave * kq + 4 * t.g;
    f32x4 wf[GROUPS], hf[GROUPS];
    f32x16 acc = {};
    auto request = [&](int k_first) {
#pragma unroll
        for (int u = 0; u < GROUPS; ++u) {
            const int k0 = k_begin + k_first + 8 * u;
            if (k_first + 8 * u < kq) {
                wf[u] = load4(wrow + k0);
                if (VEC) {                             // past the end of the row the weights are zero
                    hf[u] = k0 + 4 <= H ? load4(hrow + k0) : f32x4{0.5f, 0.5f, 0.5f, 0.5f};
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) hf[u][i] = k0 + i < H ? hrow[k0 + i] : 0.5f;
                }
            }
        }
    };
    auto multiply = [&](int k_first) {
#pragma unroll
        for (int u = 0; u < GROUPS; ++u) {
            if (k_first + 8 * u < kq) {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[u][e], hf[u][e] - 0.5f, acc, 0, 0, 0);
            }
        }
    };
    request(0);
    t.word(m, w);
    multiply(0);
    for (int k = 8 * GROUPS; k < kq; k += 8 * GROUPS) {
        request(k);
        multiply(k);
    }
    t.finish(m, acc, row_dst, h_out);
}

__global__ __launch_bounds__(256) void recur_few_units_bf16_kernel(
    ModelDev m, int rows, const int *__restrict__ B_dev, const int32_t *__restrict__ row_src,
    const int32_t *__restrict__ row_dst, const int32_t *__restrict__ prev_word, const float *__restrict__ h_in,
    float *__restrict__ h_out) {
    const int B = B_dev ? *B_dev : rows;
    if ((int)blockIdx.y * 32 >= B) return;             // uniform
    __shared__ f32x4 red[4][4][64];
    FewUnits<bf16_t, false> t(m, B, red, row_src);
    const int H = m.H;
    const float *hrow = h_in + (size_t)t.src * H;
    const bf16_t *wrow = static_cast<const bf16_t *>(m.W) + (size_t)(t.j0 + t.col) * kFewUnitsBf16;
    const int w = prev_word[t.src];
    constexpr int kSteps = kFewUnitsBf16 / 64;         // of 16 units each, this wave's
    const int k_begin = t.wave * (16 * kSteps) + 8 * t.g;
    u32x4 wf[kSteps];
    float x[kSteps][8];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int k0 = k_begin + 16 * u;
        wf[u] = *reinterpret_cast<const u32x4 *>(wrow + k0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {                  // past the end of the row the weights are zero
            const float h = hrow[min(k0 + i, H - 1)];
            x[u][i] = k0 + i < H ? h - 0.5f : 0.f;
        }
    }
    t.word(m, w);
    f32x16 acc = {};
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        u32x4 d[2];
        bf16_terms(x[u], d);
        acc = mma(wf[u], d[0], acc);
        acc = mma(wf[u], d[1], acc);
    }
    t.finish(m, acc, row_dst, h_out);
}

// Row counts up to here take the small shape: at most `per_unit` of its workgroups for every compute unit of an XCD
// (row block rb, with all its blocks of units, belongs to XCD rb % 8).  bf16 models: one with the whole ring, two at a time with
// half of it; fp32 models: two, one after the other.  Us per launch, small / large shape, the limit in brackets: bf16
// Hp = 704 (512 and 1280 rows), 600 rows with half a ring 10.6 / 14.5, with the whole one, in two rounds, 14.7; Hp = 512 (2048), 2048
// rows 13.1 / 15.4, 2300 16.9 / 16.3; Hp = 1344 (768), 1000 rows 24.4 / 22.9; fp32 Hp = 512 (2048), 1025 rows 18.8 / 22.9, 2048 21.3
// / 23.8, 2300 28.8 / 23.9; Hp = 1344 (768), 520 rows 37.4 / 45.7, 1000 56.3 / 48.6.
__host__ __device__ inline int small_rows(int Hp, int per_unit) {
    return 32 * kXcds * (per_unit * (kGroups / kXcds) / (Hp / 64));
}

constexpr int ring_bytes(int elem, bool half) { return (half ? 64 : elem == 2 ? 128 : 144) * 1024; }

// UNITS > 0 (the count is known on the device only, Hp <= UNITS): the whole form where it would be taken for a count known on the host, 32
// units a workgroup while those fit the compute units in one round, then 64, bf16 models two workgroups of them side by side.
template <typename WT, int UNITS, int UB, bool VEC>
__device__ __forceinline__ void whole_body(const ModelDev &m, int B, int b0, int j0, const int32_t *row_src, const int32_t *row_dst,
                                           const int32_t *prev_word, const float *h_in, float *h_out, char *lds) {
    if (b0 >= B) return;                               // uniform
    RecurWhole<WT, UNITS, UB, VEC> t(b0, j0);
    int source = min(b0 + t.col, B - 1);
    if (row_src) source = row_src[source];
    __builtin_amdgcn_sched_barrier(0);                 // (loads are awaited in order)
    t.request_weights(m);
    t.request_rows(m, prev_word, h_in, source, B);
    t.run(m, B, row_dst, h_in, h_out, lds);
}

template <typename WT, bool VEC, bool HALF, int UNITS>
__global__ __launch_bounds__(kThreads) void recur_kernel(
    ModelDev m, int rows, const int *__restrict__ B_dev, const int32_t *__restrict__ row_src,
    const int32_t *__restrict__ row_dst, const int32_t *__restrict__ prev_word, const float *__restrict__ h_in,
    float *__restrict__ h_out, IdGroups ids) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    __shared__ int wsum[kWaves + 1];
    __shared__ int srcs[64], prevs[64];                // rows to take, their previous words
    // Workgroup id modulo 8 is the XCD (L2 domain).  Row block rb runs on XCD rb % 8 with all
    // its unit blocks, so h_in (the larger operand) is fetched into one L2 only.
    // the arguments fetched together, not one by one where they are used
    asm volatile("" ::"s"(m.W), "s"(m.U), "s"(m.half_rowsum_W), "s"(m.d), "s"(m.dfrag), "s"(m.Hp), "s"(m.H), "s"(m.V), "s"(prev_word), "s"(h_in), "s"(h_out), "s"(row_dst));
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds, tid = threadIdx.x;
    const int JS = m.Hp / 64, JL = (m.Hp + 127) / 128;
    const int bs = (xcd + kXcds * (local / JS)) * 32, bl = (xcd + kXcds * (local / JL)) * 64;
    // The ring's rows to take are requested for both shapes beside the row count, not behind it (entries
    // between the true count and `rows` are read and not used).  The whole form asks for its own behind it: asked by every wave beside
    // the count, for 32 and 64 units a workgroup, the same launches took as long or longer (steps with the hierarchical layer, us, behind /
    // beside: 4096 ids, bf16, H = 512, 1229 distinct 21.63 / 21.58, 410 17.35 / 17.41; H = 256, 1229 16.71 / 16.80, fp32 19.12 / 19.27).
    int source_s = bs + tid, source_l = bl + tid, B;
    if (UNITS == 0 && ids.key) {                       // uniform (with the count on the device the ids are grouped already)
        const int *rep;
        B = __builtin_amdgcn_readfirstlane(group_ids(ids, rows, lds, wsum, rep));
        if (tid < 64) {                                // (read before the barrier in front of the first load into the ring)
            source_s = rep[min(bs + tid, B - 1)];
            source_l = rep[min(bl + tid, B - 1)];
        }
    } else {
        if (row_src && tid < 64) {
            source_s = row_src[min(bs + tid, rows - 1)];
            source_l = row_src[min(bl + tid, rows - 1)];
        }
        B = B_dev ? *B_dev : rows;
    }
    if constexpr (UNITS > 0) {
        if (B <= whole_rows(m.Hp, 32, 1)) {            // uniform
            const int JW = m.Hp / 32;
            whole_body<WT, UNITS, 1, VEC>(m, B, (xcd + kXcds * (local / JW)) * 32, local % JW * 32, row_src, row_dst, prev_word, h_in, h_out, lds);
            return;
        }
        if (VEC && B <= whole_rows(m.Hp, 64, sizeof(WT) == 2 ? 2 : 1)) {
            whole_body<WT, UNITS, 2, VEC>(m, B, bs, local % JS * 64, row_src, row_dst, prev_word, h_in, h_out, lds);
            return;
        }
    }
    constexpr int kRing = ring_bytes(sizeof(WT), HALF);
    constexpr bool kSmallOnly = sizeof(WT) == 2 && !HALF;          // launches of at most small_rows(Hp, 1) rows
    constexpr bool kLargeOnly = sizeof(WT) == 2 && VEC && UNITS > 0;               // small_rows(Hp, 2) is whole_rows(Hp, 64, 2)
    static_assert(!(kSmallOnly && kLargeOnly), "all rows have the whole form");
    if (kSmallOnly || (!kLargeOnly && B <= small_rows(m.Hp, 2))) {                 // uniform
        if (bs >= B) return;
        const int j0 = (local % JS) * 64;
        if (m.Hp % 128 == 0)
            recur_body<WT, 64, 32, 1, 4, 2, kRing, VEC>(m, B, bs, j0, source_s, row_dst, prev_word, h_in, h_out, lds, srcs, prevs);
        else
            recur_body<WT, 64, 32, 1, 4, 1, kRing, VEC>(m, B, bs, j0, source_s, row_dst, prev_word, h_in, h_out, lds, srcs, prevs);
    } else {
        if (bl >= B) return;
        recur_body<WT, 128, 64, 2, 2, 1, kRing, VEC>(m, B, bl, (local % JL) * 128, source_l, row_dst, prev_word, h_in, h_out, lds,
                                                     srcs, prevs);
    }
}

template <typename WT, bool VEC, bool HALF, int UNITS>
hipError_t launch_ring(const ModelDev &m, int rows, const int *B_dev, const int32_t *row_src, const int32_t *row_dst,
                       const int32_t *prev_word, const float *h_in, float *h_out, const IdGroups &ids, hipStream_t stream) {
    int lds_bytes = ring_bytes(sizeof(WT), HALF);
    if constexpr (UNITS > 0) lds_bytes = std::max(lds_bytes, RecurWhole<WT, UNITS, 1, VEC>::lds_bytes(m.Hp));
    static LdsLimit limit;
    if (hipError_t e = limit.ensure(reinterpret_cast<const void *>(recur_kernel<WT, VEC, HALF, UNITS>), lds_bytes); e != hipSuccess)
        return e;
    auto slots = [](int blocks) { return kXcds * ((blocks + kXcds - 1) / kXcds); };   // row blocks, spread over the XCDs
    // With the count on the device only, the grid covers both shapes: the small one up to its limit, the
    // large one up to `rows`.
    const int few = std::min(rows, small_rows(m.Hp, sizeof(WT) == 2 && !HALF ? 1 : 2));
    const bool on_device = B_dev || ids.key;
    int grid = rows <= few || on_device ? slots((few + 31) / 32) * (m.Hp / 64) : 0;
    if (rows > few) grid = std::max(grid, slots((rows + 63) / 64) * ((m.Hp + 127) / 128));
    if (UNITS > 0) {
        grid = std::max(grid, slots((std::min(rows, whole_rows(m.Hp, 32, 1)) + 31) / 32) * (m.Hp / 32));
        grid = std::max(grid, slots((std::min(rows, whole_rows(m.Hp, 64, sizeof(WT) == 2 ? 2 : 1)) + 31) / 32) * (m.Hp / 64));
    }
    hipLaunchKernelGGL((recur_kernel<WT, VEC, HALF, UNITS>), dim3(grid), dim3(kThreads), lds_bytes, stream, m, rows, B_dev, row_src,
                       row_dst, prev_word, h_in, h_out, ids);
    return hipGetLastError();
}

// The whole form beside the ring: where its LDS leaves room for two workgroups of half a ring.
template <typename WT, bool VEC, bool HALF>
hipError_t launch(const ModelDev &m, int rows, const int *B_dev, const int32_t *row_src, const int32_t *row_dst,
                  const int32_t *prev_word, const float *h_in, float *h_out, const IdGroups &ids, hipStream_t stream) {
    auto go = [&](auto fn) { return fn(m, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out, ids, stream); };
    if constexpr (sizeof(WT) == 4 || HALF || !VEC) {          // (else all of a launch's rows have the whole form, in a kernel of its own)
        if (B_dev && m.Wops && m.Hp <= 512 && (VEC || m.H >= 4)) {
            switch (recur_whole_top(m.Hp)) {
                case 128: return go(launch_ring<WT, VEC, HALF, 128>);
                case 256: return go(launch_ring<WT, VEC, HALF, 256>);
                case 384: return go(launch_ring<WT, VEC, HALF, 384>);
                default: return go(launch_ring<WT, VEC, HALF, 512>);
            }
        }
    }
    return go(launch_ring<WT, VEC, HALF, 0>);
}

template <bool VEC>
hipError_t launch_type(const ModelDev &m, int rows, const int *B_dev, const int32_t *row_src, const int32_t *row_dst,
                       const int32_t *prev_word, const float *h_in, float *h_out, const IdGroups &ids,
                       hipStream_t stream) {
    if (m.dtype != RNNLM_BF16)
        return launch<float, VEC, false>(m, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out, ids, stream);
    // half a ring beyond one round of small workgroups: H = 512, 1229 rows 12.5 -> 10.4 us, H = 1024, 3000 rows
    // 37 -> 30, H = 1024, 2048 rows 22.2 -> 22.6
    if (rows <= small_rows(m.Hp, 1))
        return launch<bf16_t, VEC, false>(m, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out, ids, stream);
    return launch<bf16_t, VEC, true>(m, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out, ids, stream);
}

}  // namespace

// Every workgroup repeats the grouping, so they must be few: up to Hp = 2048 the grid for kGroupedMax rows is at most 512 of
// them, two per compute unit (side by side, or for fp32 models in turn).  Steps of 1024 distinct ids with the grouping here / in a
// launch of its own, V = 4000, us: bf16 H = 64 16.2 / 17.3, 512 23.0 / 24.2, 1600 59.7 / 59.2, 2048 70.7 / 71.9; fp32 H = 512 37.8 /
// 39.0, 1600 112.1 / 111.8, 2048 143.9 / 144.9; 102 distinct of 1024: 1.5 to 2.6 less everywhere.  A table for 2048 ids made the same
// launch 0.2 slower at up to 1024 and gained 1.1 to 2.0 at 1100, 0.3 to 1.9 at 1536, nothing at 2048 (-0.8 to +3 when all are distinct).
bool recur_groups_ids(const ModelDev &m, int N) { return N > 0 && N <= kGroupedMax && m.Hp <= 2048; }

// Steps with the hierarchical layer, V = 5000, fp32, us, ring / short form (the kernel of before the ring in brackets): H = 320, 7 rows
// 10.7 / 9.7 (9.9), 512 rows 11.7 / 11.0; H = 512, 7 rows 12.6 / 11.5 (11.7), 512 rows 13.6 / 13.4; unaligned rows H = 333, 7 rows 12.3 /
// 11.4, 30 rows 13.2 / 13.4, H = 1022, 7 rows 23.6 / 22.2, 16 rows 23.9 / 23.1; H = 1024, 7 rows 20.2 / 17.9 (18.0), 256 rows (one round)
// 22.1 / 20.6 (21.6); H = 2048, 1 row 33.2 / 27.0 (27.8), 64 rows (one round) 36.6 / 34.2 (34.6).  Where the ring's stages are single chunks
// (Hp no multiple of 128) it catches up: H = 960, 64 rows 19.1 / 19.1 (19.1), 256 rows 21.2 / 22.1 (23.3), H = 832, 200 rows 18.5 (20.1).
static bool few_units(int dtype, int Hp, bool vec, int rows) {
    if (dtype == RNNLM_BF16) return Hp == kFewUnitsBf16 && !vec;
    if (Hp <= 256) return true;
    if (!vec) return rows <= 16;
    return Hp <= 512 || Hp % 128 == 0 || rows <= 64;
}

hipError_t launch_recur(const ModelDev &m, int rows, const int *B_dev, const int32_t *row_src,
                        const int32_t *row_dst, const int32_t *prev_word, const float *h_in,
                        float *h_out, const IdGroups &ids, hipStream_t stream) {
    if (rows <= 0) return hipSuccess;
    const bool vec = m.H % 4 == 0 && (reinterpret_cast<uintptr_t>(h_in) & 15) == 0 &&
                     (reinterpret_cast<uintptr_t>(h_out) & 15) == 0;
    const dim3 grid(m.Hp / 32, (rows + 31) / 32), block(256);
    if (!ids.key && grid.x * grid.y <= (unsigned)kGroups && few_units(m.dtype, m.Hp, vec, rows)) {
        auto few = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, 0, stream, m, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out);
        };
        if (m.dtype == RNNLM_BF16) few(recur_few_units_bf16_kernel);
        else if (m.Hp <= 256 && vec) few(recur_few_units_f32_kernel<true, 8>);
        else if (m.Hp <= 256) few(recur_few_units_f32_kernel<false, 8>);
        else if (vec) few(recur_few_units_f32_kernel<true, 16>);
        else few(recur_few_units_f32_kernel<false, 16>);
        return hipGetLastError();
    }
    if (const int units = recur_whole_units(m, rows, vec, ids.key != nullptr); units > 0)
        return launch_recur_whole(m, units, vec, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out, ids, stream);
    return vec ? launch_type<true>(m, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out, ids, stream)
               : launch_type<false>(m, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out, ids, stream);
}

}  // namespace rnnlm
