// Output projection + log-sum-exp for fp32 models on the fp16 matrix cores, at fp32 accuracy.
//
// Same result as the other output-projection kernels (normalising over all words of the
// vocabulary, Section 2.1 of the paper; the paper's models are fp32).  Every fp32 operand is
// brought into the range of fp16 by a power of two (one per word for the weights, 2^14 for the
// centred hidden vector, |d| <= 1/2) and cut into two fp16 terms x = x1 + x2 (11 + 12 mantissa bits with the
// second one's sign: 2^-23 of x at worst); of the four cross terms three are kept (w2 d1, w1 d2, w1 d1; the
// dropped one is below 2^-22 of the product) and added in the fp32 accumulators of the matrix instruction.  So a
// product is off by 2^-21 of itself at worst, where three exact bf16 terms and six products (which this
// kernel replaced) were off by 3 2^-24; but it takes half as many roundings of the accumulator, and those are
// where the error of a sum comes from.  Log-sum-exp against float64, root mean square / 99.9th percentile / largest of 16
// to 40 models, six products -> three: V = 30011, H = 1000, 511 rows, weights of 0.2 1.43e-6 / 8.5e-6 / 1.19e-5 -> 1.15e-6 / 7.3e-6 /
// 9.9e-6, of 0.05 7.98e-7 / 1.77e-6 / 1.81e-6 -> 7.94e-7 / 1.78e-6 / 1.81e-6; V = 65536, H = 512, 300 rows, 0.05 4.90e-7 / 1.25e-6 /
// 1.33e-6 -> 4.89e-7 / 1.25e-6 / 1.30e-6.  Where one weight of every word is a hundred or a thousand times the others, so that
// few roundings matter, it is the other way round for short sums: H = 64 2.77e-6 / 9.7e-6 / 1.19e-5 -> 3.01e-6 / 1.09e-5 / 1.26e-5,
// H = 1000 1.56e-5 / 6.4e-5 / 8.6e-5 -> 1.61e-5 / 6.1e-5 / 8.4e-5 (log-sum-exp around 50 and 130).
// Bound by the matrix pipe at the clock the chip holds under it: 308 -> 163 to 173 us,
// as the clock allows (1.26 PFLOP/s of fp16 products), V = 20000, H = 256, 256 rows 20.5 -> 12.3 us.
//
// Padded hidden sizes of 128 to 576 take the form in outproj_staged.hip, rows in registers (figures there); this one on request, so
// the figures of such sizes here and below are of option 4.
//
// Layout: both operands are kept as MFMA operands (ModelDev::Ofrag, dfrag), so 32 words x 16 units x 2
// terms are 2 KB contiguous, global memory -> LDS -> register without any rearrangement, and every LDS
// read of a wave is one contiguous kilobyte (no bank conflicts).
//   - a workgroup of 2 x 2 waves owns 128 rows and walks the tiles of 64 MB words of its vocabulary
//     split; a wave owns 32 MB words x 64 rows = MB x 2 accumulators of 32x32;
//   - a stage of LDS holds one k-step (16 units), three stages, filled by direct global->LDS loads
//     two k-steps ahead;
//   - per k-step a wave reads 2 MB + 4 operands and issues 6 MB MFMA 32x32x16 (MB = 4: half a kilobyte
//     of LDS per MFMA, 64 of the 128 bytes a clock);
//   - two workgroups share a compute unit and are not synchronised with each other: one's barriers,
//     LDS latencies and exp-and-add (a third as many VALU cycles as MFMA cycles at Hp = 128, a twelfth
//     at 512) run under the other's MFMAs; with the 256-word tile a wave inside its MFMA chain goes
//     first (s_setprio: 177 -> 173 us at V = 65536, H = 512, 1024 rows; the 128-word tile gains nothing);
//   - MFMA roles as in the other kernels (A = words, B = rows): a lane holds sixteen logits of ONE
//     row per accumulator, the sum over words stays in the lane.
#include "device_utils.h"
#include "outproj_stream_body.h"
#include "rnnlm_internal.h"

namespace rnnlm {

namespace {

constexpr int kThreads = 256, kRows = 128, kStages = 3;
constexpr int kMaxLds = 80 * 1024;                             // two workgroups per compute unit

// Do both terms of a hidden block of 32 rb rows fit that much LDS (else the streaming form keeps the first one only)?
__host__ __device__ inline bool block_fits(int rb, int Hp) {
    return stream_lds_bytes(2, rb, Hp >> 4, kThreads / 64) <= (size_t)kMaxLds;
}

template <int MB>
struct Split2Cfg {
    static constexpr int kWords = 64 * MB;
    static constexpr int kWordBytes = 2 * MB * kSplit2Operand, kRowBytes = 4 * kSplit2Operand;
    static constexpr int kStageBytes = kWordBytes + kRowBytes;
    static constexpr int kLoads = MB + 2;                       // 1 KB loads per wave and k-step
    static constexpr int kConstBytes = 2 * kWords * 4;          // constants and factors of one tile
    static constexpr int kConstAt = kStages * kStageBytes, kRedAt = kConstAt + 2 * kConstBytes;
    static constexpr int kLdsBytes = kRedAt + 2 * kRows * 8;    // + final cross-wave reduction
    static_assert(kLdsBytes <= kMaxLds, "");
};

template <bool FIXED, int MB>
__global__ __launch_bounds__(kThreads, 2) void outproj_split2_kernel(ModelDev m, int rows,
                                                                     const int *__restrict__ B_dev, int wg_per_xcd,
                                                                     int sx_cap, int stream_rows, int stream_splits) {
    using C = Split2Cfg<MB>;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    // The arguments fetched together with the row count, not one by one where they are used (V = 20000, H = 256, 256 rows
    // 13.1 -> 12.9 us); not in the long-running shape, where it had the compiler await LDS in front of every barrier
    // (V = 65536, H = 512, 1024 rows 160 -> 172).
    if constexpr (MB == 2) asm volatile("" ::"s"(m.Ofrag), "s"(m.dfrag), "s"(m.ofac), "s"(FIXED ? m.cvec2_fixed : m.cvec2), "s"(m.Hp), "s"(m.Vp), "s"(m.part));
    // The split follows the TRUE number of rows (after the grouping of ids or the cache lookup only the device knows it):
    // few rows get many vocabulary splits, 256 at most, which up to 128 rows is one workgroup per compute unit of the grid's two.
    const int B = B_dev ? *B_dev : rows;
    if (B <= 0) return;                                       // uniform: no barrier is met
    // Few rows after all (the count known on the device only): the time is then the time to read the weights once, and
    // one workgroup per compute unit streams its share of them; the tiles would keep two k-steps of weights per workgroup
    // on their way, at most one workgroup per unit having any.  Us per launch, tiles / streaming (three-term kernel before
    // both, which streamed too): V = 20000, H = 256, 32 rows 13.7 / 5.0 (9.0), 64 rows 13.9 / 6.5 (11.8); V = 65536, H = 512,
    // 32 rows 31.6 / 24.2 (29.9); V = 100000, H = 128, 32 rows 16.5 / 10.3 (13.6); V = 20000, H = 768, 32 rows 34.2 / 12.4
    // (21.0).  A step at V = 20000, H = 256 with 32 of 4096 distinct 32.3 / 23.7 (27.8).
    if (__builtin_expect(B <= stream_rows, 0)) {              // (out of the way of the code below)
        constexpr int kWaves = kThreads / 64;
        if ((int)blockIdx.x >= stream_splits) return;
        if (!block_fits(1, m.Hp)) outproj_stream_f32_body<1, FIXED, kWaves, true>(m, B, 0, (int)blockIdx.x, stream_splits, lds);
        else if (B <= 32) outproj_stream_f32_body<1, FIXED, kWaves>(m, B, 0, (int)blockIdx.x, stream_splits, lds);
        else outproj_stream_f32_body<2, FIXED, kWaves>(m, B, 0, (int)blockIdx.x, stream_splits, lds);
        return;
    }
    const RowPlan plan = plan_rows(B, kRows, wg_per_xcd, sx_cap);
    const int S = plan.S, items = plan.RG * plan.Sx;
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;                  // word half, 64-row half of the tile
    const int KS = m.Hp >> 4;                                 // k-steps per tile, at least 4
    const char *Of = static_cast<const char *>(m.Ofrag);
    const char *Df = static_cast<const char *>(m.dfrag);
    const float *cvec = FIXED ? m.cvec2_fixed : m.cvec2;
    const int ntiles = m.Vp / C::kWords;
    const uint32_t lds0 = lds_address(lds);
    const size_t blk_bytes = (size_t)KS * kSplit2Operand;     // one block of 32 words or rows
    const uint32_t voff = lane * 16;

    for (int item = local; item < items; item += wg_per_xcd) {
    const int rg = item % plan.RG, split = xcd + kXcds * (item / plan.RG);
    const int b0 = rg * kRows;
    const int t_begin = part_begin(split, ntiles, S), t_end = part_begin(split + 1, ntiles, S);
    const int nchunks = (t_end - t_begin) * KS;
    const bool active = b0 + 64 * wn < B;                     // wave-uniform: any valid row in this wave's half

    // loader: piece p = 4 q + wave of a stage's word (row) part is term wave % 2 of block 2 q + wave / 2
    const char *wsrc = Of + ((size_t)t_begin * 2 * MB + (wave >> 1)) * blk_bytes + (wave & 1) * 1024;
    const char *dsrc = Df + ((size_t)(b0 >> 5) + (wave >> 1)) * blk_bytes + (wave & 1) * 1024;
    int in_tile = t_begin, in_ks = 0, in_stage = 0;
    auto issue = [&]() {
        if (in_ks == 0 && wave < 2) {                         // the tile's constants (wave 0) and factors (wave 1)
            const float *src = (wave ? m.ofac : cvec) + (size_t)in_tile * C::kWords;
            const uint32_t at = lds0 + C::kConstAt + (in_tile & 1) * C::kConstBytes + wave * (C::kWords * 4);
            if (lane < C::kWords / 4) lds_dma_16(src, voff, at);
        }
        const uint32_t base = lds0 + in_stage * C::kStageBytes + wave * 1024;
#pragma unroll
        for (int q = 0; q < MB; ++q) lds_dma_16(wsrc + 2 * q * blk_bytes, voff, base + q * 4096);
#pragma unroll
        for (int q = 0; q < 2; ++q) lds_dma_16(dsrc + 2 * q * blk_bytes, voff, base + C::kWordBytes + q * 4096);
        wsrc += kSplit2Operand;
        dsrc += kSplit2Operand;
        in_stage = in_stage == kStages - 1 ? 0 : in_stage + 1;
        if (++in_ks == KS) {                                  // next tile: the same rows again
            in_ks = 0;
            ++in_tile;
            wsrc += (2 * MB - 1) * blk_bytes;
            dsrc -= blk_bytes;
        }
    };

    float mrun[2], srun[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) { mrun[h] = FIXED ? m.m2_fixed : -INFINITY; srun[h] = 0.f; }
    f32x16 acc[MB][2];

    if (nchunks > 0) issue();
    if (nchunks > 1) issue();
    int ks = 0, tile = t_begin, stage = 0;
    for (int chunk = 0; chunk < nchunks; ++chunk) {
        // my loads of this k-step have landed once only those of the next one are outstanding
        // (constants requested with the next one make the wait stricter, never weaker)
        if (chunk + 1 < nchunks) wait_vmcnt<C::kLoads>();
        else wait_vmcnt<0>();
        __syncthreads();                                       // everybody's; the stage of chunk - 1 is free
        if (chunk + 2 < nchunks) issue();
        if (ks == 0) {
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
        }
        if (active) {
            const char *st = lds + stage * C::kStageBytes + lane * 16;
            const char *sw = st + wm * (MB * kSplit2Operand), *sd = st + C::kWordBytes + wn * (2 * kSplit2Operand);
            f16x8 w[MB][2], d[2][2];
#pragma unroll
            for (int t = 1; t >= 0; --t) {
#pragma unroll
                for (int a = 0; a < MB; ++a) w[a][t] = *reinterpret_cast<const f16x8 *>(sw + a * kSplit2Operand + t * 1024);
#pragma unroll
                for (int b = 0; b < 2; ++b) d[b][1 - t] = *reinterpret_cast<const f16x8 *>(sd + b * kSplit2Operand + (1 - t) * 1024);
            }
            // smallest cross terms first: (2,1) (1,2) (1,1)
            if constexpr (MB == 4) __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                constexpr int tw[3] = {1, 0, 0}, td[3] = {0, 1, 0};
#pragma unroll
                for (int a = 0; a < MB; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[a][tw[p]], d[b][td[p]], acc[a][b], 0, 0, 0);
            }
            if constexpr (MB == 4) __builtin_amdgcn_s_setprio(0);
            if (ks == KS - 1) {                                // the tile is complete: exp-and-add
                const f32x4 *cl = reinterpret_cast<const f32x4 *>(lds + C::kConstAt + (tile & 1) * C::kConstBytes) + wm * (8 * MB) + g;
#pragma unroll
                for (int a = 0; a < MB; ++a) {
                    f32x4 c[4], f[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        c[q] = cl[a * 8 + 2 * q];
                        f[q] = cl[C::kWords / 4 + a * 8 + 2 * q];
                    }
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        float x[16];
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int i = 0; i < 4; ++i) x[4 * q + i] = fmaf(acc[a][b][4 * q + i], f[q][i], c[q][i]);
                        lse2_fold16<FIXED>(x, mrun[b], srun[b]);
                    }
                }
            }
        }
        if (++ks == KS) { ks = 0; ++tile; }
        stage = stage == kStages - 1 ? 0 : stage + 1;
    }
    // (an item without tiles meets no barrier above: the partials of the item before are read by then)
    __syncthreads();
    // lanes l and l+32 hold two halves of a row; waves wm = 0, 1 hold the two word halves
    float2 *red = reinterpret_cast<float2 *>(lds + C::kRedAt);             // [2 (wm)][rows of the tile]
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float m2 = __shfl_xor(mrun[h], 32, 64), s2 = __shfl_xor(srun[h], 32, 64);
        if (FIXED) srun[h] += s2;
        else lse2_merge(mrun[h], srun[h], m2, s2);
        if (g == 0) red[wm * kRows + wn * 64 + h * 32 + col] = make_float2(mrun[h], srun[h]);
    }
    __syncthreads();                                           // also: every stage has been read
    if (tid < kRows && b0 + tid < B) {
        float2 p = red[tid], q = red[kRows + tid];
        if (FIXED) p.y += q.y;
        else lse2_merge(p.x, p.y, q.x, q.y);
        m.part[(size_t)(b0 + tid) * kMaxSplits + split] = p;
    }
    }   // items
}

template <int MB>
hipError_t launch_split2_shape(const ModelDev &m, int rows, const int *B_dev, bool fixed_offset, SplitInfo *splits,
                               hipStream_t stream) {
    using C = Split2Cfg<MB>;
    static LdsLimit limit[2];
    const void *fn = fixed_offset ? reinterpret_cast<const void *>(outproj_split2_kernel<true, MB>)
                                  : reinterpret_cast<const void *>(outproj_split2_kernel<false, MB>);
    // two workgroups per compute unit; at most one split per tile of words, rounded UP to a multiple of
    // 8 so that no split gets two tiles while the others have one
    const int wg_per_xcd = 64, ntiles = m.Vp / C::kWords, sx_cap = (ntiles + kXcds - 1) / kXcds;
    // Rows the streaming form takes, when the count is on the device: 64 (Hp <= 256) or 32 (Hp <= 576) with both terms
    // of the block in half a compute unit's LDS; 32 with one term where that needs no more LDS than the tiles do.
    int stream_rows = 0, lds_bytes = C::kLdsBytes;
    if (B_dev) {
        const int rb = block_fits(2, m.Hp) ? 2 : 1, terms = block_fits(1, m.Hp) ? 2 : 1;
        const int need = (int)stream_lds_bytes(terms, rb, m.Hp >> 4, kThreads / 64);
        if (terms == 2 || need <= lds_bytes) {
            stream_rows = 32 * rb;
            if (need > lds_bytes) lds_bytes = need;
        }
    }
    const int stream_splits = m.Vp / 32 < kMaxSplits ? m.Vp / 32 : kMaxSplits;
    if (hipError_t e = limit[fixed_offset ? 1 : 0].ensure(fn, kMaxLds); e != hipSuccess) return e;
    *splits = SplitInfo{0, wg_per_xcd, kRows, sx_cap, stream_rows, stream_splits};
    dim3 grid(kXcds * wg_per_xcd), block(kThreads);
    if (fixed_offset)
        hipLaunchKernelGGL((outproj_split2_kernel<true, MB>), grid, block, lds_bytes, stream, m, rows, B_dev,
                           wg_per_xcd, sx_cap, stream_rows, stream_splits);
    else
        hipLaunchKernelGGL((outproj_split2_kernel<false, MB>), grid, block, lds_bytes, stream, m, rows, B_dev,
                           wg_per_xcd, sx_cap, stream_rows, stream_splits);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_outproj_split2(const ModelDev &m, int rows, const int *B_dev, bool fixed_offset,
                                 SplitInfo *splits, hipStream_t stream) {
    if (m.dtype != RNNLM_F32 || !m.Ofrag || !m.dfrag || !m.ofac) return hipErrorInvalidValue;
    // 256-word tiles once they give every workgroup of the grid two, 128-word tiles below.  Measured, us,
    // 256 / 128 words: 2048 tiles (V = 65536, H = 512, 1024 rows) 173 / 184; 1024 tiles (512 rows) 88 / 92;
    // 944 tiles (V = 30000, H = 1000, 511 rows) 78 / 83 and 768 (V = 65536, H = 512, 384 rows) 74 / 82, which the line leaves
    // on the slower side; 942 tiles (V = 40000, H = 300, 700 rows) 54.7 / 55.6; 588 (V = 50000, H = 650, 300 rows) 85 / 76;
    // 158 (V = 20000, H = 256, 256 rows) 15.0 / 12.1.
    const long long tiles = (long long)((rows + kRows - 1) / kRows) * (m.Vp / 256);
    if (tiles >= 1024) return launch_split2_shape<4>(m, rows, B_dev, fixed_offset, splits, stream);
    return launch_split2_shape<2>(m, rows, B_dev, fixed_offset, splits, stream);
}

}  // namespace rnnlm
