// The weight-streaming output projection as device functions (bf16 models, then fp32 models): the
// kernels of its own (few rows known on the host) and the staged, tiled, row-streaming and two-term kernels (few
// rows known only on the device) run them.  See outproj_stream.hip for the design.
#pragma once

#include "device_utils.h"
#include "rnnlm_internal.h"

namespace rnnlm {

constexpr int kStreamThreads = 512;
constexpr int kStreamWaves = kStreamThreads / 64;
constexpr int kStreamGroup = 4;          // MFMA operands (k-steps) per group of loads; Hp is a multiple of 64
constexpr int kStreamRing = 5;           // groups per wave: one being consumed, four in flight

template <int WAVES>
struct StreamCursorOf {                  // walks the groups of the blocks blk, blk + WAVES, ... of one wave
    int blk, part;
    __device__ __forceinline__ void advance(int groups_per_block) {
        if (++part == groups_per_block) { part = 0; blk += WAVES; }
    }
};
typedef StreamCursorOf<kStreamWaves> StreamCursor;

// The hidden block (`pieces` kilobytes at `src`) into LDS, in front of the loop over the weights.  More than two
// kilobytes per wave go straight to LDS, all of it on its way at once, requested before the weights (stream_block_begin)
// and awaited after the first of them have been requested (stream_block_end): 64 rows at H = 512 16.4 -> 14.5 us per
// launch, V = 200000, H = 1024, 32 rows 73 -> 70, fp32 V = 100000, H = 512, 64 rows 40.6 -> 36.9.  Smaller blocks are
// requested into registers in the same place and written to LDS behind the first weights' requests (V = 20000, H = 128, 20
// rows: bf16 4.0 us, copied in front of the weights 4.1, fp32, copied behind them, 5.2 -> 4.9; a step at V = 1000000, H = 128, 64
// rows 51.6 -> 50.8).
// At the wait at least 16 younger loads of a wave with weights of its own are outstanding (four groups of the ring, which the memory
// clobbers keep between request and wait); operations complete in order, so the block has landed once no more than 12 are.
// A wave without any requests none and goes round the loop (before, it fetched the first sixteen kilobytes of the weights, for the count's
// sake, through the same 64 bytes a clock as the others' weights): bf16 V = 20000, H = 256, 32 rows 4.44 -> 3.74 us, 64 rows 4.99 -> 4.36, V =
// 12000, H = 128, 20 rows 3.95 -> 3.14, V = 5000, H = 512, 40 rows 5.9 -> 5.0; fp32 5.8 -> 5.1, 7.55 -> 6.8, 4.87 -> 3.9, 9.85 -> 8.7; from eight blocks
// of words per workgroup on no change.  Round it, not past the loads in it: a ring that may not have been requested is awaited whole.
constexpr int kStreamCopyPieces = 2;                // per wave

// What a lane holds of a small block between its request and its way into LDS.
struct StreamPieces {
    u32x4 at[kStreamCopyPieces];
};
// (pieces `stride` bytes apart, if there are more than kStreamCopyPieces per wave)
template <int WAVES = kStreamWaves>
__device__ __forceinline__ void stream_block_begin(const char *src, int pieces, char *lds, int wave, int lane, StreamPieces &held, int stride = 1024) {
    if (pieces <= kStreamCopyPieces * WAVES) {                // uniform
#pragma unroll
        for (int k = 0; k < kStreamCopyPieces; ++k)
            if (wave + k * WAVES < pieces) held.at[k] = *reinterpret_cast<const u32x4 *>(src + (size_t)(wave + k * WAVES) * 1024 + lane * 16);
        return;
    }
    for (int p = wave; p < pieces; p += WAVES) lds_dma_16(src + (size_t)p * stride, lane * 16, lds_address(lds) + p * 1024);
}
template <bool WEIGHTS, int WAVES = kStreamWaves>
__device__ __forceinline__ void stream_block_end(int pieces, char *lds, int wave, int lane, const StreamPieces &held) {
    if (pieces > kStreamCopyPieces * WAVES) {
        if constexpr (WEIGHTS) asm volatile("s_waitcnt vmcnt(12) ; hidden block" ::: "memory");
        else wait_vmcnt<0>();
    } else {
#pragma unroll
        for (int k = 0; k < kStreamCopyPieces; ++k)
            if (wave + k * WAVES < pieces) *reinterpret_cast<u32x4 *>(lds + (wave + k * WAVES) * 1024 + lane * 16) = held.at[k];
    }
    __syncthreads();                                          // hidden block visible to all waves
}

// Where the hidden block in LDS comes from: the copy a launch in front of this one left in memory.  (The other source:
// HiddenHere in step_few.hip, which computes it between the same two calls.)
template <int WAVES = kStreamWaves>
struct StoredBlock {
    const char *src;
    int pieces, stride;
    int B;                                            // rows of it that are valid, > 0
    StreamPieces held;
    __device__ __forceinline__ void begin(char *lds, int wave, int lane) { stream_block_begin<WAVES>(src, pieces, lds, wave, lane, held, stride); }
    // its wait counts the loads of the weights behind it: a wave that has none calls end_without_weights
    static constexpr bool kCountsLoads = true;
    __device__ __forceinline__ void end(char *lds, int wave, int lane) { stream_block_end<true, WAVES>(pieces, lds, wave, lane, held); }
    __device__ __forceinline__ void end_without_weights(char *lds, int wave, int lane) { stream_block_end<false, WAVES>(pieces, lds, wave, lane, held); }
    __device__ __forceinline__ static void put(float2 *at, float2 v) { *at = v; }             // a partial
};

// One launch's worth of streaming for the workgroup `split` of `S`: rows row0 .. row0 + 32 RB - 1 of
// the hidden block (block.B valid ones among them, known once block.begin has run), partials into m.part.  SCALED: the
// block carries log2(e) (outproj_d_scale).  Needs
// stream_lds_bytes(1, RB, Hp / 16) bytes of LDS at `lds` and kStreamThreads threads; contains two
// workgroup barriers, so all threads of the workgroup must call it.
template <int RB, bool FIXED, bool SCALED, class Block>
__device__ __forceinline__ void outproj_stream_block(const ModelDev &m, Block &block, int row0, int split, int S, char *lds) {
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KS = m.Hp >> 4, GPB = KS / kStreamGroup;
    const int T = m.Vp / 32;
    const int blk1 = part_begin(split + 1, T, S);
    const int blk0 = part_begin(split, T, S);
    const bf16x8 *Of = static_cast<const bf16x8 *>(m.Ofrag) + lane;
    const float *cvec = FIXED ? m.cvec2_fixed : m.cvec2;
    const float m2_fixed = m.m2_fixed;
    asm volatile("" ::"s"(m2_fixed), "s"(m.Ofrag), "s"(cvec));   // fetched together, here, not one by one where they are used
    bf16x8 *dl = reinterpret_cast<bf16x8 *>(lds);
    float2 *red = reinterpret_cast<float2 *>(lds + (size_t)RB * KS * 1024);    // [kStreamWaves][RB * 32]

    block.begin(lds, wave, lane);
    auto merge = [&]() {
        __syncthreads();
        if (tid < RB * 32) {
            float mm = red[tid].x, ss = red[tid].y;
            for (int w = 1; w < kStreamWaves; ++w) {
                const float2 p = red[w * (RB * 32) + tid];
                if (FIXED) ss += p.y;
                else lse2_merge(mm, ss, p.x, p.y);
            }
            if (tid < block.B) block.put(&m.part[(size_t)(row0 + tid) * kMaxSplits + split], make_float2(mm, ss));
        }
    };
    if constexpr (Block::kCountsLoads) {
        if (blk0 + wave >= blk1) {
            block.end_without_weights(lds, wave, lane);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                if (g == 0) red[wave * (RB * 32) + rb * 32 + col] = make_float2(FIXED ? m2_fixed : -INFINITY, 0.f);
            merge();
            return;
        }
    }
    bf16x8 ring[kStreamRing][kStreamGroup];
    StreamCursor in = {blk0 + wave, 0};
    // Always kStreamGroup loads, so that the number of younger loads behind any operand is the same on
    // every path and the waits for the ring stay partial; past the end of the wave's blocks the
    // loads go to the first kilobytes of the weights (cache hits, results unused).
    auto issue = [&](bf16x8(&dst)[kStreamGroup]) {
        const bf16x8 *p = Of + (in.blk < blk1 ? ((size_t)in.blk * KS + in.part * kStreamGroup) * 64 : (size_t)0);
#pragma unroll
        for (int i = 0; i < kStreamGroup; ++i) dst[i] = p[i * 64];
        in.advance(GPB);
    };
    const bool any = Block::kCountsLoads || blk0 + wave < blk1;
    if (any) {
#pragma unroll
        for (int st = 0; st < kStreamRing - 1; ++st) issue(ring[st]);
    }
    StreamCursor out = {blk0 + wave, 0};
    f32x4 cc[4];
    auto load_constants = [&]() {
        const int blk = out.blk < blk1 ? out.blk : blk0;
#pragma unroll
        for (int q = 0; q < 4; ++q) cc[q] = *reinterpret_cast<const f32x4 *>(cvec + blk * 32 + 8 * q + 4 * g);
    };
    if (any) load_constants();
    block.end(lds, wave, lane);

    f32x16 acc[RB];
    float mrun[RB], srun[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        mrun[rb] = FIXED ? m2_fixed : -INFINITY;
        srun[rb] = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[rb][i] = 0.f;
    }
    // The wave leaves the unrolled ring loop from wherever its last group falls (a return out of
    // the lambda, never a skip that rejoins the loop: the compiler sizes each wait by the path
    // with the fewest younger loads).
    [&]() {
        for (;;) {
#pragma unroll
            for (int st = 0; st < kStreamRing; ++st) {
                if (out.blk >= blk1) return;
                issue(ring[(st + kStreamRing - 1) % kStreamRing]);
#pragma unroll
                for (int i = 0; i < kStreamGroup; ++i) {
                    const int ks = out.part * kStreamGroup + i;
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[st][i], dl[(rb * KS + ks) * 64 + lane],
                                                                          acc[rb], 0, 0, 0);
                }
                if (out.part == GPB - 1) {                    // block complete: exp-and-add, next block
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        float x[16];
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int i = 0; i < 4; ++i) x[4 * q + i] = SCALED ? acc[rb][4 * q + i] + cc[q][i] : fmaf(acc[rb][4 * q + i], kLog2e, cc[q][i]);
                        lse2_fold16<FIXED>(x, mrun[rb], srun[rb]);
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[rb][i] = 0.f;
                    }
                    out.advance(GPB);
                    load_constants();
                } else {
                    out.advance(GPB);
                }
            }
        }
    }();
    // lanes l and l + 32 hold the two halves of a row; then the eight waves of the workgroup
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const float m2 = __shfl_xor(mrun[rb], 32, 64), s2 = __shfl_xor(srun[rb], 32, 64);
        if (FIXED) srun[rb] += s2;
        else lse2_merge(mrun[rb], srun[rb], m2, s2);
        if (g == 0) red[wave * (RB * 32) + rb * 32 + col] = make_float2(mrun[rb], srun[rb]);
    }
    merge();
}

template <int RB, bool FIXED, bool SCALED>
__device__ __forceinline__ void outproj_stream_body(const ModelDev &m, int B, int row0, int split, int S, char *lds) {
    const int KS = m.Hp >> 4;
    StoredBlock<> block = {static_cast<const char *>(m.dfrag) + (size_t)(row0 >> 5) * KS * 1024, RB * KS, 1024, B, {}};
    outproj_stream_block<RB, FIXED, SCALED>(m, block, row0, split, S, lds);
}

// ------------------------------------------------------------------------------ fp32 models
// The same streaming for fp32 weights, at fp32 accuracy on the fp16 matrix cores: weights and hidden
// block come as two fp16 terms in operand order (see outproj_split2.hip for the split), four bytes per
// weight as in fp32, and three MFMAs per operand add the cross terms.  The small ones (2.1, 1.2) have a sum of their own
// (up to 64 rows, while the registers last): what rounds is the large one, once per k-step.  Error of the log-sum-exp against
// float64, in one sum / apart / three-term kernel or plain one of before: V = 17612, H = 865, 6 rows, weights of 0.05 5.58e-7 /
// 5.46e-7 / 5.37e-7; V = 20000, H = 512, 64 rows, 0.2 5.62e-7 / 5.40e-7 / 5.86e-7; the same times (V = 100000, H = 512, 64 rows
// 36.7 us, 36.6; V = 20000, H = 576, 60 rows 13.1, 13.5).
constexpr int kStreamGroup32 = 2;        // operands per group (two terms each: four loads, as above)

// The fp32 form of outproj_stream_block, for a workgroup of WAVES waves: needs stream_lds_bytes(2, RB, Hp / 16, WAVES) bytes
// of LDS.  ONE_TERM (a StoredBlock only): stream_lds_bytes(1, ...) bytes (and more than kStreamCopyPieces kilobytes of block
// per wave): only the first term of the hidden block is kept there, the second comes from the caches beside the weights.
template <int RB, bool FIXED, int WAVES, bool ONE_TERM, class Block>
__device__ __forceinline__ void outproj_stream_f32_block(const ModelDev &m, Block &block, int row0, int split, int S, char *lds) {
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KS = m.Hp >> 4, GPB = KS / kStreamGroup32;
    const int T = m.Vp / 32;
    const int blk1 = part_begin(split + 1, T, S);
    const int blk0 = part_begin(split, T, S);
    const f16x8 *Of = static_cast<const f16x8 *>(m.Ofrag) + lane;           // [blk][ks][term][64]
    const float *cvec = FIXED ? m.cvec2_fixed : m.cvec2;
    const float m2_fixed = m.m2_fixed;
    asm volatile("" ::"s"(m2_fixed), "s"(m.Ofrag), "s"(cvec), "s"(m.ofac));  // as above
    constexpr int kTerms = ONE_TERM ? 1 : 2;
    f16x8 *dl = reinterpret_cast<f16x8 *>(lds);                             // [RB][KS][term][64]
    float2 *red = reinterpret_cast<float2 *>(lds + (size_t)kTerms * RB * KS * 1024);

    block.begin(lds, wave, lane);
    auto merge = [&]() {
        __syncthreads();
        if (tid < RB * 32) {
            float mm = red[tid].x, ss = red[tid].y;
            for (int w = 1; w < WAVES; ++w) {
                const float2 p = red[w * (RB * 32) + tid];
                if (FIXED) ss += p.y;
                else lse2_merge(mm, ss, p.x, p.y);
            }
            if (tid < block.B) block.put(&m.part[(size_t)(row0 + tid) * kMaxSplits + split], make_float2(mm, ss));
        }
    };
    if constexpr (Block::kCountsLoads) {
        if (blk0 + wave >= blk1) {
            block.end_without_weights(lds, wave, lane);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                if (g == 0) red[wave * (RB * 32) + rb * 32 + col] = make_float2(FIXED ? m2_fixed : -INFINITY, 0.f);
            merge();
            return;
        }
    }
    f16x8 ring[kStreamRing][2 * kStreamGroup32], second[kStreamRing][ONE_TERM ? RB * kStreamGroup32 : 1];
    StreamCursorOf<WAVES> in = {blk0 + wave, 0};
    auto issue = [&](int slot) __attribute__((always_inline)) {                  // always as many loads (see above)
        const f16x8 *p = Of + (in.blk < blk1 ? ((size_t)in.blk * KS + in.part * kStreamGroup32) * 128 : (size_t)0);
#pragma unroll
        for (int i = 0; i < 2 * kStreamGroup32; ++i) ring[slot][i] = p[i * 64];
        if constexpr (ONE_TERM) {
            const f16x8 *d2 = reinterpret_cast<const f16x8 *>(block.src) + in.part * (kStreamGroup32 * 128) + 64 + lane;
#pragma unroll
            for (int i = 0; i < RB * kStreamGroup32; ++i) second[slot][i] = d2[(i / kStreamGroup32 * KS + i % kStreamGroup32) * 128];
        }
        in.advance(GPB);
    };
    const bool any = Block::kCountsLoads || blk0 + wave < blk1;
    if (any) {
#pragma unroll
        for (int st = 0; st < kStreamRing - 1; ++st) issue(st);
    }
    StreamCursorOf<WAVES> out = {blk0 + wave, 0};
    f32x4 cc[4], ff[4];
    auto load_constants = [&]() {
        const int blk = out.blk < blk1 ? out.blk : blk0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            cc[q] = *reinterpret_cast<const f32x4 *>(cvec + blk * 32 + 8 * q + 4 * g);
            ff[q] = *reinterpret_cast<const f32x4 *>(m.ofac + blk * 32 + 8 * q + 4 * g);
        }
    };
    if (any) load_constants();
    block.end(lds, wave, lane);

    constexpr bool kApart = RB <= 2;
    f32x16 acc[RB], rest[kApart ? RB : 1];
    float mrun[RB], srun[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        mrun[rb] = FIXED ? m2_fixed : -INFINITY;
        srun[rb] = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[rb][i] = rest[kApart ? rb : 0][i] = 0.f;
    }
    [&]() {
        for (;;) {
#pragma unroll
            for (int st = 0; st < kStreamRing; ++st) {
                if (out.blk >= blk1) return;
                issue((st + kStreamRing - 1) % kStreamRing);
#pragma unroll
                for (int i = 0; i < kStreamGroup32; ++i) {
                    const int ks = out.part * kStreamGroup32 + i;
                    const f16x8 w1 = ring[st][2 * i], w2 = ring[st][2 * i + 1];
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        const int at = (rb * KS + ks) * (64 * kTerms) + lane;
                        const f16x8 d1 = dl[at], d2 = ONE_TERM ? second[st][rb * kStreamGroup32 + i] : dl[at + 64];
                        // smallest terms first
                        f32x16 &small = kApart ? rest[kApart ? rb : 0] : acc[rb];
                        small = __builtin_amdgcn_mfma_f32_32x32x16_f16(w2, d1, small, 0, 0, 0);
                        small = __builtin_amdgcn_mfma_f32_32x32x16_f16(w1, d2, small, 0, 0, 0);
                        acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w1, d1, acc[rb], 0, 0, 0);
                    }
                }
                if (out.part == GPB - 1) {                    // block complete: exp-and-add, next block
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        float x[16];
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const float sum = kApart ? acc[rb][4 * q + i] + rest[kApart ? rb : 0][4 * q + i] : acc[rb][4 * q + i];
                                x[4 * q + i] = fmaf(sum, ff[q][i], cc[q][i]);
                            }
                        lse2_fold16<FIXED>(x, mrun[rb], srun[rb]);
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[rb][i] = rest[kApart ? rb : 0][i] = 0.f;
                    }
                    out.advance(GPB);
                    load_constants();
                } else {
                    out.advance(GPB);
                }
            }
        }
    }();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const float m2 = __shfl_xor(mrun[rb], 32, 64), s2 = __shfl_xor(srun[rb], 32, 64);
        if (FIXED) srun[rb] += s2;
        else lse2_merge(mrun[rb], srun[rb], m2, s2);
        if (g == 0) red[wave * (RB * 32) + rb * 32 + col] = make_float2(mrun[rb], srun[rb]);
    }
    merge();
}

template <int RB, bool FIXED, int WAVES = kStreamWaves, bool ONE_TERM = false>
__device__ __forceinline__ void outproj_stream_f32_body(const ModelDev &m, int B, int row0, int split, int S, char *lds) {
    const int KS = m.Hp >> 4, terms = ONE_TERM ? 1 : 2;
    StoredBlock<WAVES> block = {static_cast<const char *>(m.dfrag) + (size_t)(row0 >> 5) * KS * 2048, terms * RB * KS, 2048 / terms, B, {}};
    outproj_stream_f32_block<RB, FIXED, WAVES, ONE_TERM>(m, block, row0, split, S, lds);
}

// terms = copies of the hidden block kept in LDS: 1 (bf16 models) or 2 (fp32 models)
__host__ __device__ inline size_t stream_lds_bytes(int terms, int RB, int KS, int waves = kStreamWaves) {
    return (size_t)terms * RB * KS * 1024 + (size_t)waves * RB * 32 * sizeof(float2);
}

}  // namespace rnnlm
