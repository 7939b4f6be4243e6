// Hidden update of 32 rows x 32 UB units by a workgroup of eight waves with all operands on their way at once ("whole" form,
// recur.hip has the one with a ring of stages).
//
// What a workgroup of the ring form waits for is not bytes but turns: H = 512, 1024 rows, its first stage has landed 1.7 us after
// the rows are known, and four stages, each a wait, a barrier, LDS reads, a conversion and a few MFMAs behind each other, take
// 2.4 us more.  Here
//   - the weights come in operand order (ModelDev::Wops: one operand of a wave is 1 KB contiguous) straight into matrix
//     registers, requested in front of everything that the rows hang on;
//   - a wave requests four rows of h_in, as wide loads whatever the rows' alignment, converts them once to bf16 terms and leaves
//     them in LDS in operand order; then there is one barrier, and a chain of LDS reads and MFMAs without another wait.
// A wave owns 32 units and every (8 / UB)-th k-step of 16; the partial sums of a block meet in LDS in a fixed order.
// What bounds it now: trips to memory behind each other (count, rows, previous words, embeddings: some 1 us each) and, with a
// workgroup on every compute unit, the 128 KB each of them takes in (H = 512; 0.95 us at 64 bytes a clock).
// Replayed steps with the hierarchical layer (one word a query; path kernel and launches some 6 us of them), us, ring / this:
//   bf16   H = 512, 8, 200, 512, 1024, 2048 rows 9.7 / 9.0, 11.0 / 10.2, 11.4 / 10.7, 12.0 / 11.7, 15.8 / 15.3;  H = 256, 200 rows 9.9 / 9.5
//          H = 650 (unaligned), 8, 200, 512 rows 14.8 / 13.4, 17.9 / 15.9, 18.7 / 17.7;  H = 1024, 64, 512 15.0 / 13.9, 16.8 / 16.3
//          41 of 4096 ids left by a cache, H = 512 (launch) 5.6 / 4.7;  1229 of 4096 distinct 23.3 / 22.0
//   fp32   grouped by the launch, H = 256, 40, 300, 1024 ids 12.9 / 11.3, 13.7 / 11.8, 15.2 / 12.7;  H = 512 14.7 / 12.3, 15.9 / 13.6, 19.5 / 17.1
// The sums are those of the ring in another order: error of h' against float64 as there.
#pragma once

#include "recur_parts.h"

namespace rnnlm {

// One operand (32 rows x 16 units) in LDS: 16 bytes more than it holds, so that the four-unit pieces of one row, which a wave
// writes together, lie in different banks.
constexpr int kOperandStride = 1040;

// UNITS: Hp at most (a multiple of 128).  VEC: rows of h_in are 16-byte aligned; otherwise H >= 4.
template <typename WT, int UNITS, int UB, bool VEC>
struct RecurWhole {
    static constexpr bool kF32 = sizeof(WT) == 4;
    static constexpr int kWTerms = kF32 ? 3 : 1, kTerms = kF32 ? 3 : 2;
    static constexpr int kGroupsOfWaves = 8 / UB;                        // that share a reduction
    static constexpr int kSteps = UNITS / 16 / kGroupsOfWaves;           // k-steps of a wave at most
    static constexpr int kPieces = (UNITS + 255) / 256;                  // loads of a lane per row
    static constexpr int kRows = 4;                                      // of a wave: wave, wave + 8, ...
    static __host__ __device__ constexpr int lds_bytes(int Hp) {
        const int operands = kTerms * (Hp / 16) * kOperandStride, sums = 8 * 4 * 1024;
        return operands > sums ? operands : sums;
    }

    const int wave, lane, col, g, wj, wk, b0, j0;
    u32x4 w[kSteps][kWTerms];
    f32x4 x[kRows][kPieces];
    f32x4 rs;
    int prev, src;                                                       // of row b0 + col
    int je;                                                              // the four units this lane finishes (if wk < 4)

    __device__ __forceinline__ RecurWhole(int b0_, int j0_)
        : wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)), lane(threadIdx.x & 63), col(lane & 31), g(lane >> 5), wj(wave % UB), wk(wave / UB), b0(b0_), j0(j0_) {
        je = j0 + 32 * wj + 8 * (wk & 3) + 4 * g;
    }

    __device__ __forceinline__ void request_weights(const ModelDev &m) {
        const int KS = m.Hp >> 4;
        const u32x4 *frag = static_cast<const u32x4 *>(m.Wops) + (size_t)(((j0 >> 5) + wj) * KS) * (kWTerms * 64) + lane;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int ks = min(wk + s * kGroupsOfWaves, KS - 1);         // (steps past the end are not multiplied)
#pragma unroll
            for (int t = 0; t < kWTerms; ++t) w[s][t] = frag[(ks * kWTerms + t) * 64];
        }
        rs = load4(m.half_rowsum_W + je);
    }

    __device__ __forceinline__ void request_row(const ModelDev &m, const float *h_in, int r) {
        const float *row = h_in + (size_t)__builtin_amdgcn_readlane(src, wave + 8 * r) * m.H;
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
            const int k = 256 * q + 4 * lane;
            if (256 * q < m.H) {                                         // uniform
                if (VEC) x[r][q] = *reinterpret_cast<const f32x4 *>(row + (k < m.H ? k : 0));
                else __builtin_memcpy(&x[r][q], row + min(k, m.H - 4), 16);
            }
        }
    }
    // source: the row of h_in and prev_word to take for row b0 + col, of B > b0.  Rows that are not there are not requested: a request
    // takes its time on the compute unit's way to its caches, whatever it hits.  Us, 32 rows requested / those there are, steps with the
    // hierarchical layer, bf16, 1 row: H = 256 7.05 / 6.93, 384 7.74 / 7.41, 512 8.59 / 8.32, 640 10.44 / 9.75, 768 10.60 / 9.99, 1024 11.44 / 10.77; 8
    // rows, H = 512 9.11 / 8.86.
    __device__ __forceinline__ void request_rows(const ModelDev &m, const int32_t *prev_word, const float *h_in, int source, int B) {
        src = source;
        prev = prev_word[src];
        if (b0 + wave + 8 * (kRows - 1) < B) {                                                // uniform
#pragma unroll
            for (int r = 0; r < kRows; ++r) request_row(m, h_in, r);
        } else {
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
#pragma unroll
                for (int q = 0; q < kPieces; ++q) x[r][q] = f32x4{};
                if (b0 + wave + 8 * r < B) request_row(m, h_in, r);
            }
            __builtin_amdgcn_s_waitcnt(0x0f70);                          // vmcnt(0), seen by the compiler: what it counts below are the loads above
        }
    }

    // The rows' terms in operand order, in LDS.
    __device__ __forceinline__ void stage(const ModelDev &m, char *lds) const {
        const int plane = (m.Hp >> 4) * kOperandStride;
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int q = 0; q < kPieces; ++q) {
                const int k = 256 * q + 4 * lane;
                if (k < m.Hp) {
                    float d[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) d[i] = x[r][q][i];
                    if (!VEC) {                                          // the row's last piece was fetched from H - 4 on
                        const int s = k - min(k, m.H - 4);
                        d[0] = s == 0 ? d[0] : s == 1 ? d[1] : s == 2 ? d[2] : d[3];
                        d[1] = s == 0 ? d[1] : s == 1 ? d[2] : d[3];
                        d[2] = s == 0 ? d[2] : d[3];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) d[i] = (VEC ? k < m.H : k + i < m.H) ? d[i] - 0.5f : 0.f;
                    char *at = lds + (k >> 4) * kOperandStride + (32 * ((k >> 3) & 1) + wave + 8 * r) * 16 + (k & 7) * 2;
#pragma unroll
                    for (int t = 0; t < kTerms; ++t) {
                        const uint2 pk = {pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3])};
                        *reinterpret_cast<uint2 *>(at + t * plane) = pk;
                        d[0] -= __uint_as_float(pk.x << 16);
                        d[1] -= __uint_as_float(pk.x & 0xFFFF0000u);
                        d[2] -= __uint_as_float(pk.y << 16);
                        d[3] -= __uint_as_float(pk.y & 0xFFFF0000u);
                    }
                }
            }
    }

    // To be called by all waves behind request_weights and request_rows, with B > b0; all LDS of the workgroup is free.
    __device__ __forceinline__ void run(const ModelDev &m, int B, const int32_t *row_dst, const float *h_in, float *h_out, char *lds) {
        const int KS = m.Hp >> 4, plane = KS * kOperandStride, b = b0 + col;
        const bool w_ok = prev >= 0 && prev < m.V;
        const f32x4 u = load4(static_cast<const WT *>(m.U) + (size_t)(w_ok ? prev : 0) * m.Hp + je);
        const int dst = row_dst ? row_dst[min(b, B - 1)] : min(b, B - 1);
        stage(m, lds);
        __syncthreads();
        f32x16 acc = {}, rest = {};
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int ks = wk + s * kGroupsOfWaves;
            if (ks < KS) {                                               // uniform
                u32x4 d[kTerms];
#pragma unroll
                for (int t = 0; t < kTerms; ++t) d[t] = *reinterpret_cast<const u32x4 *>(lds + t * plane + ks * kOperandStride + lane * 16);
                if constexpr (kF32) {
                    // the small cross terms in a sum of their own: what rounds is the large one, once per step
                    rest = mma(w[s][1], d[1], rest);
                    rest = mma(w[s][2], d[0], rest);
                    rest = mma(w[s][0], d[2], rest);
                    rest = mma(w[s][1], d[0], rest);
                    rest = mma(w[s][0], d[1], rest);
                    acc = mma(w[s][0], d[0], acc);
                } else {
                    acc = mma(w[s][0], d[0], acc);
                    acc = mma(w[s][0], d[1], acc);
                }
            }
        }
        if constexpr (kF32) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] += rest[i];
        }
        f32x4 *red = reinterpret_cast<f32x4 *>(lds);                     // [wave][result][lane]
        __syncthreads();                                                 // the operands are read
#pragma unroll
        for (int q = 0; q < 4; ++q) red[(wave * 4 + q) * 64 + lane] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        __syncthreads();
        if (wk >= 4 || b >= B) return;
        if (!w_ok && g == 0 && wave == 0 && j0 == 0) atomicOr(m.flag, RNNLM_FLAG_BAD_PREV_WORD);
        const f32x4 *mine = red + (wj * 4 + wk) * 64 + lane;
        f32x4 sum = mine[0];
#pragma unroll
        for (int other = 1; other < kGroupsOfWaves; ++other) {           // fixed order: deterministic
            const f32x4 t = mine[other * UB * 4 * 64];
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[i] += t[i];
        }
        if constexpr (kF32) {
            if (sum[0] != sum[0] || sum[1] != sum[1] || sum[2] != sum[2] || sum[3] != sum[3])
                sum = plain_sum4(static_cast<const float *>(m.W) + (size_t)je * m.Hp, m.Hp, m.H - je, h_in + (size_t)src * m.H, m.H);
        }
        const Finish f = {h_out + (size_t)dst * m.H, b, m.H, m.Hp, w_ok};
        finish4<WT, VEC>(m, f, je, sum, rs, u);
    }
};

}  // namespace rnnlm
