// Output projection + log-sum-exp, LDS-staged MFMA kernel: bf16 models with Hp <= 704, fp32 models with Hp <= 576 (multiples of 64 from 128 on).
//
// What is computed is the same as in the plain kernel (normalising over all words of the
// vocabulary, Section 2.1 of the paper); this is the fast form for batches of >= 128 rows (fp32 models: >= 64).
//
// Shape of the work.  The hidden block d = h' - 1/2 is tiny (rows x Hp bf16, 1 MB at
// 1024 x 512) and the output weights are large (64 MB at V = 65536), so the
// weights are streamed exactly once per row group and the hidden block never moves:
//   - a workgroup (8 waves; fp32 models beyond Hp = 320 four, and half of the rows) owns 256 rows; each wave keeps ITS 32 rows of d for the whole
//     reduction length in registers (Hp/16 MFMA B-operands, 128 VGPRs at Hp = 512), loaded from
//     the fragment-ordered copy of the block (one operand = 1 KB contiguous);
//   - the weights of 32 words (32 x Hp bf16, 32 KB at Hp = 512) form one LDS stage; four
//     stages (three beyond Hp = 512) are filled round-robin by direct global->LDS loads (no VGPR round trip), two to
//     three blocks ahead of use;
//   - per block a wave issues Hp/16 chained MFMA 32x32x16: A = 32 words x 16 k from LDS
//     (read four steps ahead), B = 16 k x 32 rows from registers, so lane l holds 16 logits
//     of ONE row and the sum over words stays inside the lane;
//   - the exp-and-add of block i is interleaved, instruction by instruction, with the MFMAs
//     of block i+1, so the vector ALU works in the shadow of the matrix core (the unrolled
//     block body is kept free of branches for that: see staged_block);
//   - one workgroup barrier per block.  It publishes the landing of block i+1 while block i
//     is being computed, so no wave ever waits at a barrier for data it is about to use, and
//     the first operands of block i+1 are already in registers when block i ends.
// Nothing at all happens at the boundary
// between two blocks: the barrier sits in the MIDDLE of a block's MFMA chain (a wave that waits
// there has its last MFMA in the pipe, and the chain goes on without any hand-over), the loads of
// block i+3 are issued one by one between the MFMAs of the block's second half instead of in a
// burst behind the barrier, two accumulator sets alternate (no copy between blocks, the next chain
// does not wait for the last MFMA of this one), and the constants a chain starts from (fixed log-sum-exp offset, the usual
// case) are read from LDS into the resting accumulator set half a block before they are needed.  With the running maximum a
// chain starts from zero and the constants are added in front of the exponentials.
// Where the weights come from.  Hp a multiple of 128 up to 512: from Ot, row by row; LDS rows are XOR-swizzled in 16-byte
// chunks (chunk c of word r sits at c ^ (r & 15)) so that the 16 lanes served together by one ds_read_b128 hit 16
// different bank groups.  The direct loads write LDS linearly (lane i -> base + 16 i), so the swizzle is applied on
// the global side: lane i fetches the chunk that belongs at position i.  Other multiples of 64 (and 640: the
// offsets of the swizzle would not fit the registers): from the copy in
// MFMA-operand order (Ofrag), where a block is Hp / 16 operands of one contiguous kilobyte each and a stage a straight
// copy of it; the upper four waves' share of the last 8 KB is a dummy load, and stages are whole 8 KB.  (Ot where it
// can be: the words the queries ask for are then in the L2s when the query kernel reads them from the same copy;
// the headline step 68.0 us, against 68.9 with Ofrag.)
// Padded sizes other than 128, 256 and 512 took the row-streaming and tiled kernels before.  Us per launch:
//   V = 65536: H = 192, 1024 rows 30.9 -> 26.6; 320, 1024 rows 44.3 -> 38.3; 384, 700 rows 45.5 -> 34.3; 448, 300
//   rows 31.3 -> 26.6; V = 100000: H = 576, 1000 rows 113 -> 89 (running maximum 126 -> 91); 704, 2048 rows
//   263 -> 210; 700, 200 rows 48 -> 35; V = 30011, H = 650, 317 rows, running maximum 25.2 -> 19.3.  H = 512 and
//   below at multiples of 128: as before (54 us at V = 65536, H = 512, 1024 rows).
// Beyond 704 the hidden block and the accumulators do not fit the 256 registers of a wave.
//
// The last row group is rarely full.  A wave without rows takes part in the loads and barriers only, so the others have the matrix
// pipes to themselves: alone on its SIMD a wave is nearly twice as fast.  Us per launch, all waves multiplying / this: V = 65536,
// H = 512, 70, 128, 300, 384, 600, 1229 rows 20.5 / 15.0, 18.5 / 15.3, 26.2 / 21.7, 26.4 / 23.3, 38.2 / 33.7, 61.3 / 60.3; V = 100390, H = 448,
// 100 rows 21.2 / 17.0, 513 51.8 / 43.2; V = 30011, H = 650, running maximum, 97, 317 rows 15.6 / 11.9, 21.8 / 20.4 (18.7 as groups of 128:
// staged_split).  Full groups: the same.
//
// fp32 models.  Weights and rows as two fp16 terms in operand order, three products (outproj_split2.hip, whose sums these are); an operand is two
// kilobytes, a k-step three MFMAs, and a word has a factor beside its constant.  A row's two terms fit 256 registers up to Hp = 320, and 512 up to
// Hp = 576, with four waves and 128 rows per workgroup; a block of weights then comes in two chunks, so that three are on their way.  The
// tiles of outproj_split2.hip, which take rows through LDS too, had two k-steps of 16 units on their way and a barrier for each.  Us per
// launch, tiles / this: V = 20000, H = 256, 100 rows 10.2 / 7.8, 256 12.7 / 11.3, 300 13.8 / 13.9, 2000 58.6 / 49.6; V = 100000, H = 256, 128 rows
// 34.2 / 22.6, 1024 136 / 113 (running maximum 139 / 115); H = 128, 80 rows 19.9 / 12.7, 500 43.8 / 35.2; V = 60000, H = 192, 200 rows 20.2 /
// 18.0, 1500 93.5 / 78.8; V = 50000, H = 300, 128 rows 22.4 / 17.0, 1024 94.5 / 71.9; V = 1000, H = 200, 200 rows 9.4 / 5.8;
// V = 65536, H = 512, 100 rows 36.0 / 28.2, 300 75 / 60, 1024 162.9 / 158.7; V = 20000, H = 512, 256 rows 21.6 / 18.9; V = 100000, H = 384, 700 155 / 134;
// V = 60000, H = 448, 4000 566 / 499; V = 50000, H = 570, 300 63 / 53; V = 3000, H = 512, 1000 17.7 / 12.6.  Beyond 576 registers spill.  Up to 64 rows, known on the
// device only, the streaming body has eight waves here, four there: V = 20000, H = 256, 32 rows 5.1 / 5.4, 64 6.8 / 7.3; V = 50000, H = 300, 50
// rows 17.7 / 14.7; V = 3000, H = 128, 32 rows 3.9 / 3.7;
// V = 65536, H = 512, 32 rows 23.9 / 23.8, 64 31.4 / 26.0; V = 20000, H = 512, 20 rows 9.3 / 9.5.  (Beyond the L2s at Hp = 128 too: whole steps of 130
// ids, 4 of them distinct, V = 80000 19.6 / 20.0, V = 150000 25.2 / 25.5.  With four of the eight waves here it was the same or slower.)
//
// When the batch turns out to hold at most 64 rows (the count may be known on the device only),
// the kernel runs the weight-streaming body instead (outproj_stream_body.h): see the top of
// the kernel.
//
// Work split (staged_plan): workgroup id modulo 8 is the XCD; vocabulary split s runs on
// XCD s % 8, with all row groups of that split next to each other, so the row groups that
// stream the same weights hit in the same 4 MB L2 and HBM is read once.
#include <type_traits>

#include "device_utils.h"
#include "outproj_stream_body.h"
#include "rnnlm_internal.h"

namespace rnnlm {

namespace {

constexpr int kStagedF32Hp = 576;               // largest padded hidden size of fp32 models whose rows' two terms fit the registers
constexpr int kCSlots = 8;                       // ring of per-block constants (32 floats each; fp32 models: and 32 factors)

// T: type of the weights.  An operand of one k-step (32 words or rows x 16 units) is a kilobyte of bf16, or two of fp16: the two terms.
template <typename T, int HP>
struct StagedCfg {
    static constexpr int kTerms = sizeof(T) / 2;
    using Operand = std::conditional_t<kTerms == 1, bf16x8, f16x8>;
    static constexpr int KS = HP / 16;                       // MFMA k-steps per block
    // A block's weights go through LDS in chunks of KC k-steps: one, or two where a wave needs the registers of two for its rows, so that
    // a workgroup has four waves and 128 rows.
    static constexpr int kWaves = staged_waves(kTerms == 2, HP), kChunks = 8 / kWaves, KC = KS / kChunks;
    static constexpr int kThreads = 64 * kWaves, kRows = 32 * kWaves;
    static constexpr bool kRowOrder = kTerms == 1 && HP % 128 == 0 && HP <= 512;       // weights from Ot, else from Ofrag
    static constexpr bool kScaledD = kTerms == 1 && staged_scaled_d(HP);
    static constexpr bool kHalves = kTerms == 1 && HP > 512;            // groups of 128 rows where they pay (staged_split)
    static constexpr int CPR = HP / 8;                                  // 16-byte chunks per word row
    static constexpr int kStages = kTerms * HP / kChunks <= (kChunks == 1 ? 512 : 576) ? 4 : 3;      // as LDS allows
    static constexpr int kPrefetch = 4 / kTerms;                        // A operands read this many k-steps ahead
    static constexpr int kLoadsPerThread = (kTerms * KC + kWaves - 1) / kWaves;      // weight loads per chunk: a kilobyte per wave each
    static constexpr int kStageBytes = kLoadsPerThread * kWaves * 1024;
    static constexpr int kLoadsPerChunk = kLoadsPerThread + kTerms;     // + one for the constants (+ one for the factors)
    static constexpr int kSlotBytes = kTerms * kStagedWords * 4;
    static constexpr int kLdsBytes = kStages * kStageBytes + kCSlots * kSlotBytes;
    static_assert(HP % 64 == 0 && KC >= 8 && (kChunks == 1 || kTerms * KC % kWaves == 0), "");
    static_assert(kLdsBytes <= 160 * 1024, "");
};
// Do the logits start from their constants?  Fixed offset, and no factor per word.
template <typename T, bool FIXED>
constexpr bool kStartsAtConstants = FIXED && sizeof(T) == 2;

// The block loader.
template <typename T, int HP>
struct Loader {
    using C = StagedCfg<T, HP>;
    const char *weights;
    const float *cvec, *factors;                             // of the words (factors: fp32 models)
    uint32_t wave;                                           // wave index, in an SGPR
    uint32_t voff[C::kRowOrder ? C::kLoadsPerThread : 1];    // this lane's bytes of a piece (row order: of a block)
    int lane;
    __device__ __forceinline__ void init() {
        const int tid = threadIdx.x;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        lane = tid & 63;
        if constexpr (C::kRowOrder) {
#pragma unroll
            for (int q = 0; q < C::kLoadsPerThread; ++q) {
                const int f = q * C::kThreads + tid;            // physical chunk this lane fills
                const int r = f / C::CPR, p = f % C::CPR;
                const int c = p ^ (r & 15);                  // logical chunk that belongs there
                voff[q] = (uint32_t)(r * HP * 2 + c * 16);
            }
        } else {
            voff[0] = (uint32_t)lane * 16;
        }
    }
    // (a block is 64 HP bytes in either order, times the terms)
    __device__ __forceinline__ const char *chunk_of(int chunk) const {
        return weights + (size_t)chunk * (64 * HP * C::kTerms / C::kChunks);
    }
    // The loads of a 32-word block into a stage and a slot of constants, in pieces and without branches (the block body is one
    // basic block): weight load q of the block, and its constants.  real = false turns the load into a dummy
    // that counts like a real one for vmcnt but fetches the first bytes of the weights (always
    // there, one cache line for the whole wave) into the same, free, LDS stage.
    __device__ __forceinline__ void issue_weights(const char *src, int q, bool real, uint32_t stage_lds) const {
        const uint32_t to = stage_lds + (q * C::kWaves + wave) * 1024;
        if constexpr (C::kRowOrder) {
            lds_dma_16(src, real ? voff[q] : 0u, to);
        } else {
            const bool mine = real && (C::kTerms * C::KC % C::kWaves == 0 || q + 1 < C::kLoadsPerThread || wave < 4);
            lds_dma_16(mine ? src + (q * C::kWaves + wave) * 1024 : src, mine ? voff[0] : 0u, to);
        }
    }
    // (0: the constants of the chunk's words, 1: their factors; 128 bytes, from one or two lanes of each wave)
    template <int WHICH>
    __device__ __forceinline__ void issue_words(int chunk, uint32_t cslot_lds) const {
        const float *src = (WHICH ? factors : cvec) + (size_t)(chunk / C::kChunks) * kStagedWords;
        const uint32_t to = cslot_lds + WHICH * (kStagedWords * 4) + wave * (128 / C::kWaves);
        if constexpr (C::kWaves == 8) lds_dma_16_lane0(src, wave * 16, to);
        else lds_dma_16_lanes01(src, wave * 32 + voff[0], to);
    }
    __device__ __forceinline__ void issue_consts(int chunk, uint32_t cslot_lds) const {
        issue_words<0>(chunk, cslot_lds);
        if constexpr (C::kTerms == 2) issue_words<1>(chunk, cslot_lds);
    }
    __device__ __forceinline__ void issue_all(int chunk, uint32_t stage_lds, uint32_t cslot_lds) const {
        const char *src = chunk_of(chunk);
#pragma unroll
        for (int q = 0; q < C::kLoadsPerThread; ++q) issue_weights(src, q, true, stage_lds);
        issue_consts(chunk, cslot_lds);
    }
};

// A hidden block that carries log2(e) (SCALED, see outproj_d_scale) makes the accumulators base-2; otherwise one
// multiplication per logit does.  Fixed offset: the accumulators START at the block's constants, and a finished
// accumulator IS the logit (|constant| < 100 there, so accumulating on top of it costs nothing the tolerance
// would notice).  Running maximum (constants of any size): the constants are added at the end.
template <bool SCALED>
__device__ __forceinline__ float base2(float acc) { return SCALED ? acc : acc * kLog2e; }
// fp32 models: f is the word's factor, which brings its powers of two and log2(e) back.
template <typename T, bool SCALED>
__device__ __forceinline__ float base2_plus(float acc, float f, float c) { return sizeof(T) == 4 ? fmaf(acc, f, c) : SCALED ? acc + c : fmaf(acc, kLog2e, c); }

// This lane's part of an A operand.  Row order: chunk (2 ks + g) of word `col`, swizzled; only the low 4 bits
// of the chunk index take part in the swizzle, so eight per-lane offsets plus compile-time constants cover
// all k-steps.  Operand order: one offset.
template <typename T, int HP>
struct FragOffsets {
    using C = StagedCfg<T, HP>;
    int at[C::kRowOrder ? 8 : 1];
    __device__ __forceinline__ void init(int lane) {
        if constexpr (C::kRowOrder) {
            const int col = lane & 31, g = lane >> 5;
#pragma unroll
            for (int j = 0; j < 8; ++j) at[j] = col * (HP * 2) + ((((2 * j) | g) ^ (col & 15)) * 16);
        } else {
            at[0] = lane * 16;
        }
    }
    __device__ __forceinline__ int operator()(int ks) const {
        if constexpr (C::kRowOrder) return at[ks & 7] + (ks >> 3) * 256;
        else return at[0] + ks * (C::kTerms * 1024);
    }
    // read the A operand of k-step ks
    __device__ __forceinline__ void read(const char *stage, int ks, typename C::Operand (&a)[C::kTerms]) const {
#pragma unroll
        for (int t = 0; t < C::kTerms; ++t) a[t] = *reinterpret_cast<const typename C::Operand *>(stage + (*this)(ks) + t * 1024);
    }
};

// fn(std::integral_constant<int, I>) for I = BEGIN .. END - 1, in order.
template <int BEGIN, int END, typename Fn>
__device__ __forceinline__ void static_for(Fn &&fn) {
    if constexpr (BEGIN < END) {
        fn(std::integral_constant<int, BEGIN>{});
        static_for<BEGIN + 1, END>(fn);
    }
}

// One MFMA B operand (this lane's 16 bytes of a 1 KB fragment) requested WITHOUT the compiler
// knowing that a load is in flight: the register is defined for it at once, and the caller keeps
// it unread until await_d_operand has waited for the data.  (A load the compiler can see makes
// it guard the operand with vmcnt waits of its own inside the block loop, and those drain the
// direct-to-LDS loads, which it cannot see.)
template <int OFFSET, typename Operand>
__device__ __forceinline__ void load_d_operand(Operand &dst, const bf16_t *lane_ptr) {
    static_assert(OFFSET >= 0 && OFFSET < 4096, "immediate offset of a global load");
    asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=v"(dst) : "v"(lane_ptr), "n"(OFFSET) : "memory");
}
// Wait until at most `younger` of this wave's vector-memory operations are outstanding; the
// operand goes in and out so that its first use cannot move in front of the wait.
template <int YOUNGER, typename Operand>
__device__ __forceinline__ void await_d_operand(Operand (&op)[1]) {
    static_assert(YOUNGER >= 0 && YOUNGER < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%1)" : "+v"(op[0]) : "n"(YOUNGER));
}
template <int YOUNGER, typename Operand>
__device__ __forceinline__ void await_d_operand(Operand (&op)[2]) {
    static_assert(YOUNGER >= 0 && YOUNGER < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%2)" : "+v"(op[0]), "+v"(op[1]) : "n"(YOUNGER));
}
// Dispatch of load_d_operand on a compile-time k-step: the kilobytes of a wave's operands lie one behind
// the other; one pointer every 4 KB, immediate offsets in between.
template <int KSTEP, typename Operand, int TERMS>
__device__ __forceinline__ void load_d_operand_at(Operand (&dst)[TERMS], const bf16_t *dfr) {
    static_for<0, TERMS>([&](auto t) __attribute__((always_inline)) {
        constexpr int J = KSTEP * TERMS + decltype(t)::value;
        load_d_operand<(J % 4) * 1024>(dst[decltype(t)::value], dfr + (size_t)(J / 4) * 2048);
    });
}

// In which k-steps of a chunk's second half its NW weight loads of the chunk kStages - 1 ahead are issued: evenly apart, several in
// one only if there are more loads than k-steps.
template <int KS, int NW>
struct LoadSchedule {
    static constexpr int HALF = KS / 2, kApart = (HALF - 2) / NW;
    static constexpr int at(int q) { return HALF + 1 + (kApart ? q * kApart : q * (KS - HALF - 2) / NW); }
};

// What block 0 of an item issues besides its own work (staged_block<HP, FIXED, true>): the part of
// d that the prologue has not requested, and blocks 1 and 2.  All loads of a wave are issued in
// one fixed program order, so the number of loads younger than any given one is a compile-time
// figure: that is what the vmcnt immediates of block 0 are computed from.
template <typename T, int HP>
struct FirstBlockSchedule {
    using C = StagedCfg<T, HP>;
    static constexpr int KS = C::KS, HALF = KS / 2, L = C::kLoadsPerChunk, NW = C::kLoadsPerThread, TERMS = C::kTerms;
    static constexpr int D0 = 8 / TERMS;                       // operands of d requested by the prologue
    static constexpr int kAhead = C::kStages - 2;              // blocks requested in the first half of block 0: 1 and, with four stages, 2
    static_assert(C::kChunks > 1 || kAhead * L <= HALF * TERMS, "");
    // loads issued in k-step k: before its MFMAs an operand of d (e1) and as many loads of block 1 or 2 (e2),
    // after them the regular loads of the block behind them (e3)
    static constexpr int e1(int k) { return k + D0 < KS ? TERMS : 0; }
    static constexpr int e2(int k) {
        const int left = kAhead * L - k * TERMS;
        return left <= 0 ? 0 : left < TERMS ? left : TERMS;
    }
    static constexpr int e3(int k) {
        int n = (k == KS - 2) ? TERMS : 0;                     // (constants and factors)
        for (int q = 0; q < NW; ++q)
            if (k == LoadSchedule<KS, NW>::at(q)) ++n;
        return n;
    }
    // loads younger than operand ks of d when the MFMA of k-step ks is about to be issued
    static constexpr int younger_than_d(int ks) {
        int n = 0;
        if (ks < D0) {
            n = (D0 - 1 - ks) * TERMS;
            for (int k = 0; k <= ks; ++k) n += e1(k) + e2(k);
            for (int k = 0; k < ks; ++k) n += e3(k);
        } else {
            const int j0 = ks - D0;                             // the k-step that requested it
            n = e2(j0);
            for (int k = j0 + 1; k <= ks; ++k) n += e1(k) + e2(k);
            for (int k = j0; k < ks; ++k) n += e3(k);
        }
        return n;
    }
    // loads younger than the last load of block 1 at the barrier on top of k-step HALF
    static constexpr int younger_than_block1() {
        const int last = (L - 1) / TERMS;                      // the k-step that issues it
        int n = e2(last) - 1 - (L - 1) % TERMS;
        for (int k = last + 1; k < HALF; ++k) n += e1(k) + e2(k);
        for (int k = last; k < HALF; ++k) n += e3(k);
        return n;
    }
    static constexpr int worst() {
        int w = younger_than_block1();
        for (int ks = 0; ks < KS; ++ks)
            if (younger_than_d(ks) > w) w = younger_than_d(ks);
        return w;
    }
    static_assert(C::kChunks > 1 || worst() < 64, "vmcnt is a 6-bit counter");
};
// The operands a wave holds: its rows of d for the whole reduction length, and the words' next ones.
template <typename T, int HP>
struct StagedOperands {
    using C = StagedCfg<T, HP>;
    typename C::Operand d[C::KS][C::kTerms], a[C::kPrefetch][C::kTerms];
};
struct FirstBlockLoads {
    const bf16_t *dfr;          // this lane's 16 bytes of operand 0 of its wave's rows
    const char *blk[2];         // weights of blocks 1 and 2 (or the dummy source)
    int block[2];               // their numbers (0)
    bool real[2];
    uint32_t stage[2], cslot[2];
};

// Where in a block's KS k-steps the running maximum takes in the previous block: its constants are read and added, four logits at
// a time, in the first quarter; then the new maximum; then one term after the other.  Up front, in one piece, in front of the chain
// the same instructions were in nobody's shadow.  Us per launch, up front / spread: V = 30011, H = 650, 317 rows 21.0 / 19.3, 511 25.6 /
// 24.3; V = 100000, H = 576, 1000 rows 98.8 / 90.9; V = 65536, H = 512, 1024 rows 63.5 / 57.4 (fixed offset 54), 300 31.7 / 27.9; H = 320, 1229
// rows 55.7 / 50.1; V = 200000, H = 128, 1000 rows 73.8 / 68.6; with two or three blocks in all V = 20000, H = 192, 200 rows 6.0 / 6.2.
template <int KS>
struct FoldSchedule {
    static constexpr int constants(int q) { return q * KS / 16; }
    static constexpr int kRead = KS < 12 ? 1 : KS < 16 ? 2 : 3;    // k-steps for an LDS read
    static constexpr int logits(int q) { return constants(q) + kRead; }
    static constexpr int kMaximum = logits(3) + 1;
    static constexpr int term(int e) { return kMaximum + 1 + e * (KS / 2) / 16; }
    static_assert(term(15) < KS, "");
};
// (max, sum) of a lane's logits so far; of the block being taken in its largest logit, then what its terms are taken from, and their
// sum.  The fixed offset needs the first sum alone.
struct RunningLse {
    float m, s, offset, terms;
};

// One 32-word block for this wave's 32 rows, as ONE basic block.
//   acc     on entry the block's constants (fixed offset: the logits start from them) or zero, on return the finished
//           logits of the block (running maximum: without their constants)
//   other   on entry the same of the previous block (unused in front of the first): their
//           exp-and-add is spread over the k-steps (fixed offset: of the first half); on return the start of
//           block bi+1 (constants read from the ring in the second half; after the last block: a landed
//           slot, unused)
// Half way through, the barrier publishes block bi+1 (everybody's loads of it have landed: the
// only younger loads of a wave are those of block bi+2) and frees the stage of block bi-1, which
// takes block bi+3 (past the end of the split: dummy loads, so that every wave always has the same
// number of loads in flight and the vmcnt immediates hold).  On return a[] holds the first
// kPrefetch A operands of block bi+1.
//
// FIRST (block 0 of an item): the prologue has requested block 0 and the first operands of d only,
// so that the chain starts early; the rest of d is requested here, one operand per k-step eight
// k-steps ahead of its use, and blocks 1 and 2 load by load in the first half.  Every MFMA waits
// for ITS operand of d alone, and the barrier for block 1 alone (FirstBlockSchedule has the
// counts): the chain runs at the pace at which d arrives instead of starting after all of it.
template <typename T, int HP, bool FIXED, bool FIRST, int CHUNK = 0>
__device__ __forceinline__ void staged_block(const char *lds, const char *cring, uint32_t lds0, uint32_t cring0,
                                             const Loader<T, HP> &loader, int blk0, int nblk, int bi,
                                             const FragOffsets<T, HP> &aoff, StagedOperands<T, HP> &op, int g, f32x16 &acc,
                                             f32x16 &other, RunningLse &lse, const FirstBlockLoads &first) {
    using C = StagedCfg<T, HP>;
    using F = FirstBlockSchedule<T, HP>;
    constexpr int KS = C::KC, HALF = KS / 2, NW = C::kLoadsPerThread, kPrefetch = C::kPrefetch, TERMS = C::kTerms;
    constexpr bool kAtConstants = kStartsAtConstants<T, FIXED>;
    using W = LoadSchedule<KS, NW>;
    constexpr bool kLoadsRows = FIRST && C::kChunks == 1;
    static_assert(KS >= 2 * kPrefetch && W::at(NW - 1) <= KS - 2, "");
    constexpr int NS = C::kStages;
    const char *stage = lds + bi % NS * C::kStageBytes;
    const char *next_stage = lds + ((bi + 1 < nblk) ? bi + 1 : bi) % NS * C::kStageBytes;
    // the constants the next block starts from, or those of the previous one
    const f32x4 *cn = reinterpret_cast<const f32x4 *>(cring + ((kAtConstants ? bi + 1 : bi - 1) & 7) * C::kSlotBytes);
    using R = FoldSchedule<KS>;
    f32x4 c4[4], f4[4];                                        // (those of the previous block: one or two of them in use at a time)
    const bool real = bi + NS - 1 < nblk;
    const int block3 = real ? blk0 + bi + NS - 1 : 0;
    const char *src3 = loader.chunk_of(block3);
    const uint32_t stage3 = lds0 + (bi + NS - 1) % NS * C::kStageBytes, cslot3 = cring0 + ((bi + NS - 1) & 7) * C::kSlotBytes;
    // the k-steps as a compile-time loop: every condition below is a constant, and so are the vmcnt
    // immediates
    static_for<0, KS>([&](auto step) __attribute__((always_inline)) {
        constexpr int ks = decltype(step)::value;
        if constexpr (ks == HALF) {
            if constexpr (kLoadsRows) wait_vmcnt<F::younger_than_block1()>();
            else wait_vmcnt<(NS - 3) * C::kLoadsPerChunk>();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        typename C::Operand cur[TERMS];
#pragma unroll
        for (int t = 0; t < TERMS; ++t) cur[t] = op.a[ks % kPrefetch][t];
        if constexpr (ks + kPrefetch < KS) aoff.read(stage, ks + kPrefetch, op.a[ks % kPrefetch]);
        else aoff.read(next_stage, ks + kPrefetch - KS, op.a[ks % kPrefetch]);
        if constexpr (kLoadsRows) {
            if constexpr (ks + F::D0 < KS) load_d_operand_at<ks + F::D0>(op.d[ks + F::D0], first.dfr);
            static_for<ks * TERMS, ks * TERMS + F::e2(ks)>([&](auto load) __attribute__((always_inline)) {
                constexpr int b = decltype(load)::value / F::L, q = decltype(load)::value % F::L;
                if constexpr (q < NW) loader.issue_weights(first.blk[b], q, first.real[b], first.stage[b]);
                else loader.template issue_words<q - NW>(first.block[b], first.cslot[b]);
            });
            await_d_operand<F::younger_than_d(ks)>(op.d[ks]);
        }
        if constexpr (TERMS == 1) {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur[0], op.d[ks][0], acc, 0, 0, 0);
        } else {                                               // smallest cross terms first
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(cur[1], op.d[CHUNK * KS + ks][0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(cur[0], op.d[CHUNK * KS + ks][1], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(cur[0], op.d[CHUNK * KS + ks][0], acc, 0, 0, 0);
        }
        if constexpr (!FIRST && CHUNK == 0 && kAtConstants) {
            // the previous block's sixteen logits, over k-steps 1 .. HALF
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (1 + (e * HALF) / 16 == ks) lse.s += fast_exp2(base2<C::kScaledD>(other[e]));
        } else if constexpr (!FIRST && CHUNK == 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (ks == R::logits(q)) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        other[4 * q + i] = base2_plus<T, C::kScaledD>(other[4 * q + i], f4[q][i], c4[q][i]);
                        if (!FIXED) lse.offset = q + i == 0 ? other[0] : fmaxf(lse.offset, other[4 * q + i]);
                    }
                }
                if (ks == R::constants(q)) {
                    c4[q] = cn[2 * q + g];
                    if constexpr (TERMS == 2) f4[q] = cn[kStagedWords / 4 + 2 * q + g];
                }
            }
            if constexpr (!FIXED && ks == R::kMaximum) {
                const float mn = fmaxf(lse.m, lse.offset);
                lse.offset = mn == -INFINITY ? 0.f : mn;       // (nothing but -inf so far: the terms below are 2^-inf)
                lse.s *= fast_exp2(lse.m - lse.offset);
                lse.m = mn;
                lse.terms = 0.f;
            }
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (R::term(e) == ks) {
                    if constexpr (FIXED) lse.s += fast_exp2(other[e]);             // (the offset is in the constants)
                    else lse.terms += fast_exp2(other[e] - lse.offset);
                }
            if constexpr (!FIXED && ks == KS - 1) lse.s += lse.terms;
        }
        if constexpr (!kAtConstants && CHUNK == 0 && ks == KS - 1) {
#pragma unroll
            for (int i = 0; i < 16; ++i) other[i] = 0.f;
        }
        // second half: loads of block bi+3, with the fixed offset the constants of block bi+1 into the resting accumulators
#pragma unroll
        for (int q = 0; q < NW; ++q)
            if (ks == W::at(q)) loader.issue_weights(src3, q, real, stage3);
        if constexpr (ks == KS - 2) loader.issue_consts(block3, cslot3);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (kAtConstants && ks == HALF + 1 + (q * (HALF - 1)) / 4) {
                const f32x4 c = cn[2 * q + g];
#pragma unroll
                for (int i = 0; i < 4; ++i) other[4 * q + i] = c[i];
            }
        // keep this order: the compiler's scheduler would otherwise sink every LDS read to
        // just before its MFMA and expose the LDS latency on each step
        __builtin_amdgcn_sched_barrier(0);
    });
}

// The exp-and-add of an item's last block.
template <typename T, int HP, bool FIXED>
__device__ __forceinline__ void fold_last_block(const f32x16 &acc, const char *cring, int bi, int g, RunningLse &lse) {
    using C = StagedCfg<T, HP>;
    if constexpr (kStartsAtConstants<T, FIXED>) {
#pragma unroll
        for (int e = 0; e < 16; ++e) lse.s += fast_exp2(base2<C::kScaledD>(acc[e]));
    } else {
        const f32x4 *cn = reinterpret_cast<const f32x4 *>(cring + (bi & 7) * C::kSlotBytes);
        float x[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 c = cn[2 * q + g], f = C::kTerms == 2 ? cn[kStagedWords / 4 + 2 * q + g] : c;
#pragma unroll
            for (int i = 0; i < 4; ++i) x[4 * q + i] = base2_plus<T, C::kScaledD>(acc[4 * q + i], f[i], c[i]);
        }
        lse2_fold16<FIXED>(x, lse.m, lse.s);
    }
}

// All blocks of one (row group, split) item for this wave's rows: the item's words' part of the log-sum-exp for this lane's half of
// its row, as (lse.m, lse.s); with the fixed offset the sum of 2^(logit - offset) alone.
template <typename T, int HP, bool FIXED>
__device__ __forceinline__ void staged_item(const ModelDev &m, char *lds, char *cring, const Loader<T, HP> &loader,
                                            const FragOffsets<T, HP> &aoff, int row0, int blk0, int nblk, int wave,
                                            int lane, int g, RunningLse &lse) {
    using C = StagedCfg<T, HP>;
    constexpr int KS = C::KS;
    const uint32_t lds0 = lds_address(lds), cring0 = lds_address(cring);
    // Block 0 and the first operands of this wave's rows of d (all k of 32 rows are MFMA B operands
    // held in registers; rows beyond B hold stale scratch: rows are independent and those lanes'
    // results are dropped).  The rest of d and blocks 1 and 2 are requested by block 0 itself.
    StagedOperands<T, HP> op;
    FirstBlockLoads first;
    if constexpr (C::kChunks == 1) {
        using F = FirstBlockSchedule<T, HP>;
        loader.issue_all(blk0, lds0, cring0);
        // fragment (row block, ks) of the fragment-ordered copy: 64 lanes x 16 bytes in a row, a term behind the other
        first.dfr = static_cast<const bf16_t *>(m.dfrag) + ((size_t)(row0 / 32 + wave) * KS * C::kTerms * 64 + lane) * 8;
        static_for<0, F::D0>([&](auto j) __attribute__((always_inline)) {
            load_d_operand_at<decltype(j)::value>(op.d[decltype(j)::value], first.dfr);
        });
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            first.real[i] = i + 1 < nblk;
            first.block[i] = first.real[i] ? blk0 + i + 1 : 0;
            first.blk[i] = loader.chunk_of(first.block[i]);
            first.stage[i] = lds0 + (i + 1) % C::kStages * C::kStageBytes;
            first.cslot[i] = cring0 + (i + 1) * C::kSlotBytes;
        }
        // Block 0 has landed once only the younger loads are outstanding: the first operands of d.
        wait_vmcnt<F::D0 * C::kTerms>();
    } else {
        // the first chunks, then the rows by loads the compiler sees, which may put them into either half of the 512 registers; the
        // wait is one it sees as well, so that it adds none inside the loop
#pragma unroll
        for (int i = 0; i < C::kStages - 1; ++i) {
            const int chunk = i < nblk ? blk0 + i : 0;
            const char *src = loader.chunk_of(chunk);
#pragma unroll
            for (int q = 0; q < C::kLoadsPerThread; ++q) loader.issue_weights(src, q, i < nblk, lds0 + i * C::kStageBytes);
            loader.issue_consts(chunk, cring0 + i * C::kSlotBytes);
        }
        const auto *dfr = static_cast<const typename C::Operand *>(m.dfrag) + (size_t)(row0 / 32 + wave) * KS * C::kTerms * 64 + lane;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int t = 0; t < C::kTerms; ++t) op.d[ks][t] = dfr[(ks * C::kTerms + t) * 64];
        __builtin_amdgcn_s_waitcnt(0x0f70);                   // vmcnt(0)
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();                             // block 0 is published
    asm volatile("" ::: "memory");
    // From block 1 on every wave has, at the barrier in the middle of block bi, the loads of blocks
    // bi+1 and bi+2 in flight at most.
#pragma unroll
    for (int i = 0; i < C::kPrefetch; ++i) aoff.read(lds, i, op.a[i]);
    f32x16 acc0, acc1;
    {
        const f32x4 *c0 = reinterpret_cast<const f32x4 *>(cring);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 c = c0[2 * q + g];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc0[4 * q + i] = kStartsAtConstants<T, FIXED> ? c[i] : 0.f;
        }
    }
    lse.m = -INFINITY;
    lse.s = 0.f;
    auto block = [&](auto first_block, int bi, f32x16 &acc, f32x16 &other) __attribute__((always_inline)) {
        static_for<0, C::kChunks>([&](auto chunk) __attribute__((always_inline)) {
            constexpr int c = decltype(chunk)::value;
            staged_block<T, HP, FIXED, decltype(first_block)::value, c>(lds, cring, lds0, cring0, loader, blk0, nblk, C::kChunks * bi + c, aoff, op, g, acc, other, lse, first);
        });
    };
    const int blocks = nblk / C::kChunks;
    block(std::true_type{}, 0, acc0, acc1);
    int bi = 1;
    for (; bi + 1 < blocks; bi += 2) {
        block(std::false_type{}, bi, acc1, acc0);
        block(std::false_type{}, bi + 1, acc0, acc1);
    }
    if (bi < blocks) {
        block(std::false_type{}, bi, acc1, acc0);
        fold_last_block<T, HP, FIXED>(acc1, cring, nblk - 1, g, lse);
    } else {
        fold_last_block<T, HP, FIXED>(acc0, cring, nblk - 1, g, lse);
    }
    // dummy loads may still be in flight into stages the next item fills first
    wait_vmcnt<0>();
}

// A wave without rows in an item: its share of the loads and all barriers, as staged_item has them (block 0 is published by the
// first barrier; the barrier of block bi publishes block bi + 1 and frees the stage of block bi - 1), and nothing else.  The matrix
// pipes are left to the waves that have rows: with up to four of them each has one to itself.
template <typename T, int HP>
__device__ __forceinline__ void staged_item_loads(uint32_t lds0, uint32_t cring0, const Loader<T, HP> &loader, int blk0, int nblk) {
    using C = StagedCfg<T, HP>;
    constexpr int NS = C::kStages;
    auto issue = [&](int bi) __attribute__((always_inline)) {            // always as many loads
        const bool real = bi < nblk;
        const int block = real ? blk0 + bi : 0;
        const char *src = loader.chunk_of(block);
#pragma unroll
        for (int q = 0; q < C::kLoadsPerThread; ++q) loader.issue_weights(src, q, real, lds0 + bi % NS * C::kStageBytes);
        loader.issue_consts(block, cring0 + (bi & 7) * C::kSlotBytes);
    };
    issue(0);
    wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 1; i < NS - 1; ++i) issue(i);
    for (int bi = 0; bi < nblk; ++bi) {
        wait_vmcnt<(NS - 3) * C::kLoadsPerChunk>();                      // block bi + 1 has landed
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(bi + NS - 1);
    }
    wait_vmcnt<0>();                                                     // (dummies: the next item fills these stages)
}

template <typename T, int HP, bool FIXED>
__device__ __forceinline__ void staged_kernel(const ModelDev &m, int rows, const int *__restrict__ B_dev, int wg_per_xcd) {
    using C = StagedCfg<T, HP>;
    constexpr int KS = C::KS;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    char *const cring = lds + C::kStages * C::kStageBytes;
    const int B = B_dev ? *B_dev : rows;
    if (B <= 0) return;                                       // uniform: nothing to do, no barrier met
    // Few rows after all (after the grouping or the cache lookup only the device knows how many
    // are left): the time is then the time to read the weights once, and the workgroup streams
    // them instead.  Same grid, and the same partials come out: with one row group the vocabulary
    // is cut into as many splits as there are workgroups (kMaxSplits), split = workgroup index.
    static_assert(C::kLdsBytes >= C::kTerms * 2 * KS * 1024 + C::kWaves * 64 * 8, "LDS for two row blocks of the streaming form");
    if (B <= 64) {
        if constexpr (C::kTerms == 2) {
            if (B <= 32) outproj_stream_f32_body<1, FIXED, C::kWaves>(m, B, 0, (int)blockIdx.x, kMaxSplits, lds);
            else outproj_stream_f32_body<2, FIXED, C::kWaves>(m, B, 0, (int)blockIdx.x, kMaxSplits, lds);
        } else {
            if (B <= 32) outproj_stream_body<1, FIXED, C::kScaledD>(m, B, 0, (int)blockIdx.x, kMaxSplits, lds);
            else outproj_stream_body<2, FIXED, C::kScaledD>(m, B, 0, (int)blockIdx.x, kMaxSplits, lds);
        }
        return;
    }
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5;
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
    const int blocks = m.Vp / kStagedWords;                  // 32-word blocks in the vocabulary
    const StagedSplit split_of = C::kRows == kStagedRows ? staged_split(B, wg_per_xcd, C::kHalves) : StagedSplit{plan_rounds(B, C::kRows, wg_per_xcd, m.Vp), C::kRows};
    const StagedPlan plan = split_of.plan;
    const int items = plan.RG * plan.Sx;
    const uint32_t lds0 = lds_address(lds), cring0 = lds_address(cring);
    Loader<T, HP> loader;
    loader.init();
    loader.weights = static_cast<const char *>(C::kRowOrder ? m.Ot : m.Ofrag);
    loader.cvec = !FIXED ? m.cvec2 : C::kTerms == 2 || C::kScaledD ? m.cvec2_fixed : m.cvec_fixed;
    loader.factors = m.ofac;
    FragOffsets<T, HP> aoff;
    aoff.init(lane);

    for (int item = local; item < items; item += wg_per_xcd) {
        const int rg = item % plan.RG, split = xcd + kXcds * (item / plan.RG);
        const int blk0 = part_begin(split, blocks, plan.S) * C::kChunks;               // (in chunks, from here on)
        const int nblk = part_begin(split + 1, blocks, plan.S) * C::kChunks - blk0;
        const int row0 = rg * split_of.rows;
        const bool has_rows = (int)loader.wave * 32 < min(split_of.rows, B - row0);       // (wave-uniform)
        if (!has_rows) {
            if (nblk > 0) staged_item_loads<T, HP>(lds0, cring0, loader, blk0, nblk);
            __syncthreads();
            continue;
        }
        RunningLse lse;
        lse.m = -INFINITY;
        lse.s = 0.f;
        if (nblk > 0) staged_item<T, HP, FIXED>(m, lds, cring, loader, aoff, row0, blk0, nblk, wave, lane, g, lse);
        // lanes l and l+32 hold the two halves of a row (the lane asked for anew: with Hp = 704 there is no register to keep it in)
        const int lane_now = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        const int b = row0 + (int)loader.wave * 32 + (lane_now & 31);                        // this lane's row
        const float s2 = __shfl_xor(lse.s, 32, 64);
        if (FIXED) {
            lse.m = m.m2_fixed;
            lse.s += s2;
        } else {
            lse2_merge(lse.m, lse.s, __shfl_xor(lse.m, 32, 64), s2);
        }
        if (lane_now < 32 && b < B) m.part[(size_t)b * kMaxSplits + split] = make_float2(lse.m, lse.s);
        __syncthreads();                                      // LDS is reused by the next item
    }
}

template <int HP, bool FIXED>
__global__ __launch_bounds__((StagedCfg<bf16_t, HP>::kThreads)) void outproj_staged_kernel(ModelDev m, int rows, const int *__restrict__ B_dev, int wg_per_xcd) {
    staged_kernel<bf16_t, HP, FIXED>(m, rows, B_dev, wg_per_xcd);
}
template <int HP, bool FIXED>
__global__ __launch_bounds__((StagedCfg<float, HP>::kThreads)) void outproj_staged_f32_kernel(ModelDev m, int rows, const int *__restrict__ B_dev, int wg_per_xcd) {
    staged_kernel<float, HP, FIXED>(m, rows, B_dev, wg_per_xcd);
}

template <typename T, int HP>
hipError_t launch_hp(const ModelDev &m, int rows, const int *B_dev, bool fixed_offset, int wg_per_xcd,
                     hipStream_t stream) {
    using C = StagedCfg<T, HP>;
    static LdsLimit limit[2];
    auto launch = [&](auto kernel, LdsLimit &l) -> hipError_t {
        if (hipError_t e = l.ensure(reinterpret_cast<const void *>(kernel), C::kLdsBytes); e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(kXcds * wg_per_xcd), dim3(C::kThreads), C::kLdsBytes, stream, m, rows, B_dev, wg_per_xcd);
        return hipGetLastError();
    };
    if constexpr (C::kTerms == 2)
        return fixed_offset ? launch(outproj_staged_f32_kernel<HP, true>, limit[1]) : launch(outproj_staged_f32_kernel<HP, false>, limit[0]);
    else
        return fixed_offset ? launch(outproj_staged_kernel<HP, true>, limit[1]) : launch(outproj_staged_kernel<HP, false>, limit[0]);
}

}  // namespace

bool outproj_staged_supported(const ModelDev &m) {
    if (m.dtype != RNNLM_BF16) return m.ofac && m.Ofrag && m.Hp >= 128 && m.Hp <= kStagedF32Hp && m.Hp % 64 == 0;
    return m.Ofrag && m.Hp >= 128 && m.Hp <= 704 && m.Hp % 64 == 0;
}

hipError_t launch_outproj_staged(const ModelDev &m, int rows, const int *B_dev, bool fixed_offset,
                                 SplitInfo *splits, hipStream_t stream) {
    // One workgroup per compute unit: 256 CUs in 8 XCDs.
    constexpr int wg_per_xcd = 32;
    static_assert(kXcds * wg_per_xcd == kMaxSplits, "splits of the streaming form");
    *splits = SplitInfo{0, wg_per_xcd, m.Hp > 512 ? 0 : kStagedRows, kMaxSplits / kXcds, 0, 0};
    if (m.dtype != RNNLM_BF16) {
        *splits = staged_waves(true, m.Hp) == 4 ? SplitInfo{0, wg_per_xcd, -kStagedRows / 2, m.Vp, 0, 0} : SplitInfo{0, wg_per_xcd, kStagedRows, kMaxSplits / kXcds, 0, 0};
        switch (m.Hp) {
            case 128: return launch_hp<float, 128>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
            case 192: return launch_hp<float, 192>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
            case 256: return launch_hp<float, 256>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
            case 320: return launch_hp<float, 320>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
            case 384: return launch_hp<float, 384>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
            case 448: return launch_hp<float, 448>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
            case 512: return launch_hp<float, 512>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
            case 576: return launch_hp<float, 576>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
            default: return hipErrorInvalidValue;
        }
    }
    switch (m.Hp) {
        case 128: return launch_hp<bf16_t, 128>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        case 192: return launch_hp<bf16_t, 192>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        case 256: return launch_hp<bf16_t, 256>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        case 320: return launch_hp<bf16_t, 320>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        case 384: return launch_hp<bf16_t, 384>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        case 448: return launch_hp<bf16_t, 448>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        case 512: return launch_hp<bf16_t, 512>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        case 576: return launch_hp<bf16_t, 576>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        case 640: return launch_hp<bf16_t, 640>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        case 704: return launch_hp<bf16_t, 704>(m, rows, B_dev, fixed_offset, wg_per_xcd, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rnnlm
