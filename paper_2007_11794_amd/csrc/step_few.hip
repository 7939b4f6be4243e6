// A whole step of few rows in one launch (full softmax): grouping of the ids, hidden update, weight streaming, the words
// asked for, and the log-sum-exp.
//
// With a handful of rows a step is launches and chains of dependent loads: hidden update, streaming and query kernel of 8
// rows at V = 1000, H = 64 take 5, 5 and 3.5 us, an empty launch 2.5, and the host needs 2.5 to 3 us for each.  So
//   - while the recurrent weights are small (few_here), every workgroup of the streaming kernel groups the ids and computes
//     the hidden block for itself, straight into LDS, while its first weights are on their way;
//   - the dot products of the words asked for are spread over all waves, behind their share of the stream, and the unnormalised
//     logits go where the answers belong;
//   - the workgroup that finishes last merges the partials and subtracts the normalisers.  It is found with a counter in the
//     handle's scratch (ModelDev::done, left at zero); nobody waits for another workgroup.  The order of every sum is fixed:
//     which workgroup is the last one makes no difference to the result.
#include <algorithm>

#include "device_utils.h"
#include "outproj_stream_body.h"
#include "recur_math.h"
#include "rnnlm_internal.h"

namespace rnnlm {

namespace {

constexpr int kThreads = kStreamThreads, kWaves = kStreamWaves;
constexpr int kHereRows = 32;                         // most rows (or raw queries, grouped here)
constexpr int kMostPairs = 8192;                      // most words asked for (FewStep::query_of)

// LDS behind what the streaming needs: fp32 rows (h_in, then the hidden vectors) and the sums of the matrix products,
// [wave][result][half][row], both with 16 bytes between them that spread them over the banks.
__host__ __device__ inline int row_stride(int Hp) { return Hp + 4; }
__host__ __device__ inline int wave_parts(int Hp) { return Hp == 64 ? 4 : Hp == 128 ? 2 : 1; }
constexpr int kSumStride = kHereRows + 1;
__host__ __device__ inline size_t few_lds_bytes(int terms, int Hp) {
    return stream_lds_bytes(terms, 1, Hp >> 4) + (size_t)kHereRows * row_stride(Hp) * 4 + (size_t)kWaves * 8 * kSumStride * 16;
}

struct FewLds {
    int first[64], rep[64], inverse[64];
    float lse[kHereRows];
    int last;
};

// The words asked for: pair p = word p % K of query p / K.  2^lg lanes per dot product, 4 * 64 / 2^lg of them per wave at a time;
// the batches go round over the workgroups.  The logit without the normaliser goes to logprob[p].  The words of a wave's first batch
// are requested in front of everything else, their weight rows (fetch) beside the first weights of the stream.
template <typename T>
struct Pairs {
    static constexpr int U = 4;
    int lg, batch, word[U], row[U];
    float bias[U];
    u32x4 raw[U][sizeof(T) / 2];                      // eight weights of a lane
    __device__ __forceinline__ explicit Pairs(int Hp) : lg(Hp <= 128 ? 4 : 5) {}
    __device__ __forceinline__ int per_batch() const { return U * (64 >> lg); }
    __device__ __forceinline__ int pair(int u, int lane) const { return batch * per_batch() + u * (64 >> lg) + (lane >> lg); }
    // groups: of this launch's own grouping, in LDS (not there yet), or null
    __device__ __forceinline__ void request(const FewStep &a, int lane, const int *groups) {
        const int P = a.N * a.K;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = min(pair(u, lane), P - 1), n = a.query_of(p);
            word[u] = a.query_word[p];
            row[u] = !groups && a.row_of_query ? a.row_of_query[n] : n;
        }
    }
    __device__ __forceinline__ bool word_ok(const ModelDev &m, int u) const { return word[u] >= 0 && word[u] < m.V; }
    __device__ __forceinline__ float weight(int u, int i) const {
        if (sizeof(T) == 4) return __uint_as_float(raw[u][i / 4 % (sizeof(T) / 2)][i % 4]);
        return __uint_as_float(i & 1 ? raw[u][0][i / 2] & 0xFFFF0000u : raw[u][0][i / 2] << 16);
    }
    __device__ __forceinline__ int lane_units(int lane) const { return 8 * (lane & ((1 << lg) - 1)); }
    __device__ __forceinline__ void fetch(const ModelDev &m, int lane) {
#pragma unroll
        for (int u = 0; u < U; ++u) bias[u] = m.bias[word_ok(m, u) ? word[u] : 0];
        const int j0 = lane_units(lane);                                 // (lanes beyond the row do not use theirs)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T *w = static_cast<const T *>(m.Ot) + (size_t)(word_ok(m, u) ? word[u] : 0) * m.Hp + (j0 < m.Hp ? j0 : 0);
#pragma unroll
            for (int i = 0; i < (int)sizeof(T) / 2; ++i) raw[u][i] = reinterpret_cast<const u32x4 *>(w)[i];
        }
    }
    __device__ __forceinline__ void finish(const ModelDev &m, const FewStep &a, int lane, int B, const int *groups, const float *hidden) {
        const int P = a.N * a.K, j0 = lane_units(lane);
        float acc[U];
        bool r_ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = groups ? groups[row[u]] : row[u];
            r_ok[u] = r >= 0 && r < B;
            acc[u] = 0.f;
            if (j0 < m.Hp) {
                const float *h = hidden + (r_ok[u] ? r : 0) * row_stride(m.Hp) + j0;
                const f32x4 lo = *reinterpret_cast<const f32x4 *>(h), hi = *reinterpret_cast<const f32x4 *>(h + 4);
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[u] = fmaf(weight(u, i), i < 4 ? lo[i % 4] : hi[i % 4], acc[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (lg == 5) {                                               // uniform
                float x, y;
                row_pair(acc[u], acc[u], x, y); acc[u] = x + y;
            }
            acc[u] += lane_xor<8>(acc[u]);
            acc[u] += lane_xor<4>(acc[u]);
            acc[u] += lane_xor<2>(acc[u]);
            acc[u] += lane_xor<1>(acc[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = pair(u, lane);
            if (j0 == 0 && p < P) {
                const bool ok = word_ok(m, u) && r_ok[u];
                if (!ok) atomicOr(m.flag, r_ok[u] ? RNNLM_FLAG_BAD_QUERY_WORD : RNNLM_FLAG_BAD_ROW);
                store_seen(a.logprob + p, ok ? acc[u] + bias[u] : quiet_nan());
            }
        }
    }
};

// Hidden block of up to kHereRows rows, computed where outproj_stream_block wants it: the operands are requested in begin, in
// front of the weights, and multiplied in end, behind the first weights' requests.  A wave takes a block of 32 units (W goes
// straight into matrix registers) for all rows (h_in through LDS, the waves share it); with fewer than eight blocks the waves
// share the reductions.  bf16 models: two bf16 terms of h_in; fp32 models: the fp32 instruction (as recur_few_units_*).
// The sums go through LDS to the threads that finish them, so that this costs by the rows there are, not by 32: all of it
// happens in every workgroup, and instructions are what it takes (B = 32, Hp = 128: 1.4 us, row by lane).
template <typename WT>
struct HiddenHere {
    static constexpr bool kF32 = sizeof(WT) == 4;
    static constexpr int kSteps = kF32 ? 4 : 16;      // k-steps of 16 units a wave may have (Hp <= 128, 256)
    static constexpr int kPieces = kF32 ? 2 : 4;      // 16-byte pieces of rows per thread
    static constexpr bool kCountsLoads = false;
    const ModelDev &m;
    const FewStep &a;
    FewLds &s;
    float *rows;                                      // [kHereRows][row_stride(Hp)]
    f32x4 *sums;                                      // [wave][result][half][kSumStride]
    bool leader;                                      // this workgroup reports mistakes
    Pairs<WT> &pairs;
    int B;
    int parts, part, unit, steps, lg;                 // this wave: units unit .. unit + 31, its share of the reduction; lanes of a row: 2^lg
    u32x4 wf[kSteps][kF32 ? 2 : 1];
    f32x4 x[kPieces], u[kPieces], rs;
    int w[kPieces];

    __device__ __forceinline__ HiddenHere(const ModelDev &m_, const FewStep &a_, FewLds &s_, float *rows_, f32x4 *sums_, bool leader_, Pairs<WT> &pairs_)
        : m(m_), a(a_), s(s_), rows(rows_), sums(sums_), leader(leader_), pairs(pairs_), B(a_.rows) {}

    // Piece i of a thread: units 4 k .. 4 k + 3 of row r, 2^lg lanes per row (Hp = 192: those beyond it idle).
    __device__ __forceinline__ int piece_row(int i, int tid) const { return (i * kThreads + tid) >> lg; }
    __device__ __forceinline__ bool pieces(int i) const { return i * kThreads < B << lg; }        // uniform
    __device__ __forceinline__ int source(int b) const { return a.ids.key ? s.rep[min(b, B - 1)] : min(b, B - 1); }

    // The ids' groups, in every workgroup: wave w compares each id with ids 4 w .. 4 w + 3, the first equal one stands for it.
    __device__ __forceinline__ void group(int wave, int lane) {
        const int N = a.rows;
        const uint64_t id = lane < N ? a.ids.key[lane] : 0;
        if (wave == 0) s.first[lane] = lane;
        __syncthreads();
        int f = lane;
#pragma unroll
        for (int i = kHereRows / kWaves - 1; i >= 0; --i) {
            const int j = wave * (kHereRows / kWaves) + i;
            const uint64_t other = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(id >> 32), j) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)id, j);
            if (other == id && j < f) f = j;                             // (a lane of an id: j < lane < N)
        }
        if (lane < N && f < lane) atomicMin(&s.first[lane], f);
        __syncthreads();
        const int first = s.first[lane];
        const uint64_t firsts = __ballot(lane < N && first == lane);
        B = __popcll(firsts);
        if (wave == 0) {
            const int mine = __popcll(firsts & ((1ull << first) - 1));
            s.inverse[lane] = mine;
            if (lane < N && first == lane) s.rep[mine] = lane;
        }
        __syncthreads();
    }

    __device__ __forceinline__ void begin(char *, int wave, int lane) {
        const int Hp = m.Hp, H = m.H, tid = wave * 64 + lane;
        parts = wave_parts(Hp);
        part = wave & (parts - 1);
        unit = (parts == 4 ? wave >> 2 : parts == 2 ? wave >> 1 : wave) * 32;
        steps = parts == 1 ? Hp >> 4 : Hp == 128 ? 4 : 1;
        lg = Hp <= 64 ? 4 : Hp <= 128 ? 5 : 6;
        if (a.ids.key) group(wave, lane);
        const int k = 4 * (lane & ((1 << lg) - 1));
#pragma unroll
        for (int i = 0; i < kPieces; ++i)
            if (pieces(i)) w[i] = a.prev_word[source(piece_row(i, tid))];
        if (a.vec) {
#pragma unroll
            for (int i = 0; i < kPieces; ++i)
                if (pieces(i)) x[i] = *reinterpret_cast<const f32x4 *>(a.h_in + (size_t)source(piece_row(i, tid)) * H + (k < H ? k : 0));
        } else {
#pragma unroll
            for (int i = 0; i < kPieces; ++i)
                if (pieces(i)) {
                    const float *row = a.h_in + (size_t)source(piece_row(i, tid)) * H;
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[i][e] = row[min(k + e, H - 1)];
                }
        }
        if (unit < Hp) {                                                 // uniform
            const u32x4 *frag = static_cast<const u32x4 *>(m.Wfrag) + (size_t)((unit >> 5) * (Hp >> 4) + part * steps) * (64 * sizeof(WT) / 2) + lane;
#pragma unroll
            for (int i = 0; i < kSteps; ++i)
                if (i < steps) {
                    wf[i][0] = frag[i * (64 * sizeof(WT) / 2)];
                    if (kF32) wf[i][kF32 ? 1 : 0] = frag[i * (64 * sizeof(WT) / 2) + 64];
                }
        }
        rs = load4(m.half_rowsum_W + (k < Hp ? k : 0));
#pragma unroll
        for (int i = 0; i < kPieces; ++i)
            if (pieces(i)) u[i] = load4(static_cast<const WT *>(m.U) + (size_t)((uint32_t)w[i] < (uint32_t)m.V ? w[i] : 0) * Hp + (k < Hp ? k : 0));
        pairs.fetch(m, lane);
    }

    __device__ __forceinline__ static void put(float2 *at, float2 v) { store_seen(at, v); }

    // Four finished units k .. k + 3 of row b: fp32, and as operand of the output projection.
    __device__ __forceinline__ void store4(char *lds, int b, int k, const f32x4 &sum, const f32x4 &emb, bool ok) const {
        f32x4 hp, dv;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            hp[i] = ok ? sigmoid_f32(sum[i] + rs[i] + emb[i]) : quiet_nan();
            dv[i] = hp[i] - 0.5f;
        }
        *reinterpret_cast<f32x4 *>(rows + b * row_stride(m.Hp) + k) = hp;
        const int frag = k >> 4, slot = (((k >> 3) & 1) * 32 + b) * 8 + (k & 7);
        uint16_t *dl = reinterpret_cast<uint16_t *>(lds);
        if constexpr (kF32) {
            uint16_t t[2][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) split2_f16(dv[i] * (float)(1 << kSplit2DExp), t[0][i], t[1][i]);
#pragma unroll
            for (int c = 0; c < 2; ++c)
                *reinterpret_cast<uint2 *>(dl + frag * 1024 + c * 512 + slot) =
                    uint2{(uint32_t)t[c][0] | ((uint32_t)t[c][1] << 16), (uint32_t)t[c][2] | ((uint32_t)t[c][3] << 16)};
        } else {
            *reinterpret_cast<uint2 *>(dl + frag * 512 + slot) =
                uint2{pack_bf16x2(dv[0] * kLog2e, dv[1] * kLog2e), pack_bf16x2(dv[2] * kLog2e, dv[3] * kLog2e)};
        }
    }

    // (rows from B on hold whatever was there: a column of the products is its row's own, and theirs are dropped)
    __device__ __forceinline__ void end(char *lds, int wave, int lane) {
        const int Hp = m.Hp, H = m.H, tid = wave * 64 + lane, k = 4 * (lane & ((1 << lg) - 1));
#pragma unroll
        for (int i = 0; i < kPieces; ++i)
            if (pieces(i) && k < Hp && piece_row(i, tid) < B) {
                f32x4 d;                                                 // past the end of a row the weights are zero
#pragma unroll
                for (int e = 0; e < 4; ++e) d[e] = k + e < H ? x[i][e] - 0.5f : 0.f;
                *reinterpret_cast<f32x4 *>(rows + piece_row(i, tid) * row_stride(Hp) + k) = d;
            }
        __syncthreads();
        if (unit < Hp) {                                                 // uniform
            f32x16 acc = {};
            const float *row = rows + (lane & 31) * row_stride(Hp) + 16 * part * steps + 8 * (lane >> 5);
#pragma unroll
            for (int i = 0; i < kSteps; ++i)
                if (i < steps) {
                    const f32x4 lo = *reinterpret_cast<const f32x4 *>(row + 16 * i), hi = *reinterpret_cast<const f32x4 *>(row + 16 * i + 4);
                    const float d[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    if constexpr (kF32) {
#pragma unroll
                        for (int e = 0; e < 8; ++e)                      // instruction e: units 16 i + e and 16 i + 8 + e
                            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(wf[i][e / 4][e % 4]), d[e], acc, 0, 0, 0);
                    } else {
                        u32x4 t[2];
                        bf16_terms(d, t);
                        acc = mma(wf[i][0], t[0], acc);
                        acc = mma(wf[i][0], t[1], acc);
                    }
                }
#pragma unroll
            for (int q = 0; q < 4; ++q)                                  // units 8 q + 4 half .. + 3
                sums[((wave * 4 + q) * 2 + (lane >> 5)) * kSumStride + (lane & 31)] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        }
        __syncthreads();                                                 // h_in is read, the sums are there
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int b = piece_row(i, tid);
            if (pieces(i) && k < Hp && b < B) {
                const f32x4 *from = sums + (((k >> 5) * parts * 4 + ((k >> 3) & 3)) * 2 + ((k >> 2) & 1)) * kSumStride + b;
                f32x4 sum = from[0];
                for (int other = 1; other < parts; ++other) {            // fixed order
                    const f32x4 t = from[other * 8 * kSumStride];
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] += t[e];
                }
                if (kF32 && H != Hp) {                                   // units beyond H are 0, an infinity in h_in times zero weights is not
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] = k + e < H ? sum[e] : 0.f;
                }
                const bool ok = (uint32_t)w[i] < (uint32_t)m.V;
                if (leader && !ok && k == 0) atomicOr(m.flag, RNNLM_FLAG_BAD_PREV_WORD);
                store4(lds, b, k, sum, u[i], ok);
            }
        }
        __syncthreads();
        // the words' rows came in front of the weights: multiplied while those are on their way
        if (pairs.batch * pairs.per_batch() < a.N * a.K) pairs.finish(m, a, lane, B, a.ids.key ? s.inverse : nullptr, rows);
    }
};

// Normalisers of rows 0 .. B - 1 from the partials of this launch: a wave per row, four rows of a wave on their way together,
// merged as lse_from_partials merges them.
__device__ __forceinline__ void normalisers(const float2 *part, int S, int B, float *lse, int wave, int lane) {
    constexpr int kPer = kMaxSplits / 64, kTogether = 4;
    for (int r0 = wave; r0 < B; r0 += kWaves * kTogether) {
        float2 v[kTogether][kPer];
#pragma unroll
        for (int i = 0; i < kTogether; ++i)
#pragma unroll
            for (int c = 0; c < kPer; ++c) {
                v[i][c] = make_float2(-INFINITY, 0.f);
                if (r0 + i * kWaves < B && 64 * c < S && 64 * c + lane < S) v[i][c] = load_seen(part + (size_t)(r0 + i * kWaves) * kMaxSplits + 64 * c + lane);
            }
#pragma unroll
        for (int i = 0; i < kTogether; ++i)
            if (r0 + i * kWaves < B) {
                float pm = -INFINITY, ps = 0.f;
#pragma unroll
                for (int c = 0; c < kPer; ++c) lse2_merge(pm, ps, v[i][c].x, v[i][c].y);
                const float mm = wave_max(pm), ss = wave_sum(mm == -INFINITY ? 0.f : ps * fast_exp2(pm - mm));
                if (lane == 0) lse[r0 + i * kWaves] = (mm + fast_log2(ss)) * kLn2;
            }
    }
}

template <typename T, bool FIXED>
__global__ __launch_bounds__(kThreads) void step_few_kernel(ModelDev m, FewStep a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ FewLds s;
    // the arguments the first loads hang on, fetched together, not one by one where they are used
    asm volatile("" ::"s"(m.Hp), "s"(m.H), "s"(m.V), "s"(m.Vp), "s"(m.Wfrag), "s"(m.U), "s"(m.half_rowsum_W), "s"(m.Ot), "s"(m.bias), "s"(m.Ofrag));
    asm volatile("" ::"s"(a.rows), "s"(a.N), "s"(a.K), "s"(a.ids.key), "s"(a.prev_word), "s"(a.h_in), "s"(a.query_word), "s"(a.row_of_query));
    constexpr bool kF32 = sizeof(T) == 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int split = blockIdx.x, S = gridDim.x, P = a.N * a.K;
    float *rows = reinterpret_cast<float *>(lds + stream_lds_bytes(kF32 ? 2 : 1, 1, m.Hp >> 4));
    Pairs<T> pairs(m.Hp);
    const int *groups = a.ids.key ? s.inverse : nullptr;
    pairs.batch = split + S * (kWaves - 1 - wave);                       // (the first waves have most of the stream)
    pairs.request(a, lane, groups);
    HiddenHere<T> block(m, a, s, rows, reinterpret_cast<f32x4 *>(rows + kHereRows * row_stride(m.Hp)), split == 0, pairs);
    if constexpr (kF32) outproj_stream_f32_block<1, FIXED, kWaves, false>(m, block, 0, split, S, lds);
    else outproj_stream_block<1, FIXED, true>(m, block, 0, split, S, lds);
    const int B = block.B;
    for (int r = split; r < B; r += S)                                   // the hidden vectors, a row here, a row there
        for (int j = tid; j < m.H; j += kThreads) a.h_out[(size_t)r * m.H + j] = rows[r * row_stride(m.Hp) + j];
    if (a.ids.key && split == S - 1) {
        if (tid < a.rows) a.ids.inverse[tid] = s.inverse[tid];
        if (tid < B) a.ids.rep[tid] = s.rep[tid];
        if (tid == 0) *a.ids.n_unique = B;
    }
    for (pairs.batch += S * kWaves; pairs.batch * pairs.per_batch() < P; pairs.batch += S * kWaves) {
        pairs.request(a, lane, groups);
        pairs.fetch(m, lane);
        pairs.finish(m, a, lane, B, groups, rows);
    }
    // The workgroup that comes last has all partials and logits before it.
    seen_by_all();
    __syncthreads();
    // The count wraps at S, the same for every launch on a handle, so it is 0 again behind any number of whole launches: two that
    // a caller let overlap, against the rules, may spoil each other's answers but not those of later ones.
    if (tid == 0) s.last = atomicInc(m.done, S - 1) == (unsigned)S - 1;
    __syncthreads();
    if (!s.last) return;
    constexpr int kHeld = 4;                                             // answers of a thread, beside the partials
    float z[kHeld], base[kHeld];
    int row[kHeld];
    auto request = [&](int first) {
#pragma unroll
        for (int i = 0; i < kHeld; ++i) {
            const int p = min(first + i * kThreads, P - 1), n = a.query_of(p);
            z[i] = load_seen(a.logprob + p);
            row[i] = !groups && a.row_of_query ? a.row_of_query[n] : n;
            base[i] = a.base_score ? a.base_score[p] : 0.f;
        }
    };
    request(tid);
    normalisers(m.part, S, B, s.lse, wave, lane);
    __syncthreads();
    for (int first = tid; first < P; first += kHeld * kThreads) {
        if (first != tid) request(first);
#pragma unroll
        for (int i = 0; i < kHeld; ++i) {
            const int r = groups ? groups[row[i]] : row[i];
            const float lp = r >= 0 && r < B ? z[i] - s.lse[r] : z[i];   // (z is NaN where the row is none)
            if (first + i * kThreads < P) a.logprob[first + i * kThreads] = a.base_score ? lp - base[i] : lp;
        }
    }
}

}  // namespace

bool step_few_supported(int dtype, int Hp) { return dtype == RNNLM_BF16 ? Hp <= 256 : Hp <= 128; }

// Workgroups: one per block of 32 words up to 40 of them, then one per six blocks, between 40 and 160.  More of them share the stream,
// but each repeats the hidden update and leaves partials to the last one (bf16, Hp = 128, 16 rows, 256 / 160 / 105 / 79 workgroups:
// V = 20000 11.5 / 10.5 / 10.2 / 10.5 us, V = 80000 12.8 / 12.3 / - / 12.5; V = 5000, 160 / 80 / 40: 10.1 / 9.3 / 9.3).
static int few_splits(int T) { return std::min(T, std::min(160, std::max(40, T / 6))); }

static size_t few_bytes(const ModelDev &m) { return (size_t)m.Vp * m.Hp * (m.dtype == RNNLM_BF16 ? 2 : 4); }

// Do the words asked for, P = N * K, suit the launch?  Up to 2048 its last workgroup finishes them beside the partials.  Beyond, every further 2048
// are a round of that workgroup, about 1 us, and more than a batch for every wave another batch, 1.5; the query kernel pays 1.4 us for every 32
// words of a query beyond the first 32.  Small weights leave it 1.5 us ahead.  (In units of half a microsecond.)  Replayed steps of N queries of K
// words from 8 rows, us, three launches / this one:
//   V = 1000, Hp = 64, fp32    128 of 32 11.1 / 9.8, 256 of 24 11.2 / 12.5, 100 of 64 12.6 / 13.1, 64 of 128 15.6 / 13.6, 1000 of 8 11.2 / 13.5, 1 of 8192 302 / 13.3
//   V = 4000, Hp = 128, fp32   128 of 32 12.2 / 12.1, 256 of 24 12.2 / 14.7, 100 of 64 13.5 / 15.2, 64 of 128 16.1 / 15.7, 1000 of 8 12.2 / 15.8
//   V = 8000, Hp = 256, bf16 (6 rows)    256 of 8 12.0 / 11.9, 100 of 30 11.9 / 14.2, 64 of 64 13.2 / 14.5, 32 of 128 15.5 / 14.5, 64 of 128 15.6 / 19.1
//   V = 90000, Hp = 128, bf16 (4 rows)   256 of 8 12.1 / 11.7, 100 of 30 12.2 / 12.7, 64 of 64 13.4 / 12.8, 64 of 128 16.5 / 14.4, 1000 of 8 12.1 / 14.2
static bool words_chosen(const ModelDev &m, int N, int K) {
    const long long P = (long long)N * K;
    if (P <= 2048) return P > 0;
    if (P > kMostPairs) return false;
    const int per_batch = few_splits(m.Vp / 32) * kWaves * (m.Hp <= 128 ? 16 : 8);       // (Pairs::per_batch of every wave)
    const int rounds = ((int)P - 1) / 2048, batches = ((int)P - 1) / per_batch, old_rounds = (K - 1) / 32;
    return 2 * rounds + 3 * batches < 3 * old_rounds + (m.Hp <= 128 && few_bytes(m) <= 8u << 20 ? 3 : 0);
}

// Replayed steps of 8 words per query, us, three launches / this one (the host's part, 14 to 16.5 us for three launches, 9 to 10.5 for
// one, is not in it):
//   V = 1200    Hp = 128 rows 1, 16, 32   10.4 / 7.7, 11.0 / 8.7, 11.0 / 10.4;  Hp = 192, 32   11.7 / 13.1;  Hp = 256, 16   11.7 / 11.4
//   V = 5000    Hp = 128 rows 1, 16   10.5 / 8.1, 11.0 / 9.3;  Hp = 192, 16   11.6 / 11.0
//   V = 20000   Hp = 128 rows 1, 16   10.5 / 9.2, 11.3 / 10.2;  Hp = 192, 1, 16   11.2 / 10.4, 11.8 / 12.0
//   V = 80000   Hp = 128 rows 1, 16   11.2 / 11.2, 11.9 / 12.3;  Hp = 256, 1   16.2 / 17.1
// and with the ids to group in front: V = 20000, Hp = 128, 16, 32 rows 12.7 / 10.8, 13.0 / 12.7, V = 80000 1, 16 rows 12.8 / 12.1, 13.6 / 13.0,
// Hp = 192 1 row 14.1 / 13.4.  What this launch pays more for is rows x units, computed in every workgroup (Hp = 192 beyond 16 rows in a third
// piece a thread: 21 rows, V = 5000 11.4 / 11.8, grouped V = 20000 13.1 / 13.4), and the weights it cannot request meanwhile; what it saves is launches.
// fp32 models pay twice the latter.  Rows the caller has told apart, weights that the L2s still hold from the step before:
//   V = 4000    Hp = 128 rows 24, 32   12.1 / 11.8, 12.2 / 12.6;  V = 22000   Hp = 64, 24, 32   11.4 / 10.9, 11.4 / 11.4
//   V = 30000   Hp = 64 rows 16, 24, 32   11.1 / 10.9, 11.4 / 11.5, 11.5 / 12.1;  V = 70000   Hp = 64, 8, 16   11.8 / 11.5, 11.9 / 12.2
//   Hp = 128 rows 1, 8   V = 40000 12.3 / 12.5, 12.6 / 12.8;  V = 46000 12.2 / 13.1, 12.7 / 13.4;  V = 58000 12.7 / 13.5, 13.4 / 13.7
// and beyond them   V = 70000   Hp = 128 rows 1, 8   15.7 / 14.6, 16.2 / 14.9;  V = 130000   Hp = 64, 16   14.8 / 14.0;  grouped   V = 5000   Hp = 64, 32
// 11.5 / 10.6, V = 50000   Hp = 128, 16   15.6 / 14.9.
bool step_few_chosen(const ModelDev &m, int rows, bool grouped, int N, int K) {
    if (rows <= 0 || rows > kHereRows || !m.Wfrag || !words_chosen(m, N, K)) return false;
    const size_t bytes = few_bytes(m);
    const int units = rows * m.Hp;
    if (bytes <= (grouped ? 8u : 2u) << 20) return m.Hp == 192 ? rows <= 16 : units <= (m.dtype != RNNLM_BF16 && !grouped ? 3072 : 4096);
    if (m.dtype != RNNLM_BF16 && !grouped && bytes <= kAllL2s) {
        if (bytes <= 8u << 20) return units <= 2048 && (rows <= 16 || bytes <= 6u << 20);
        return rows <= 8 && (m.Hp <= 64 || bytes <= 22u << 20);
    }
    if (bytes <= 8u << 20) return units <= 2048;
    return bytes <= 48u << 20 && m.Hp <= (grouped ? 192 : 128) && units <= (grouped ? 2048 : 1024);
}

template <auto Kernel>
static hipError_t launch_kernel(const ModelDev &m, const FewStep &a, int S, size_t lds_bytes, hipStream_t stream) {
    static LdsLimit limit;
    if (hipError_t e = limit.ensure(reinterpret_cast<const void *>(Kernel), lds_bytes); e != hipSuccess) return e;
    hipLaunchKernelGGL(Kernel, dim3(S), dim3(kThreads), lds_bytes, stream, m, a);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_type(const ModelDev &m, const FewStep &a, bool fixed_offset, hipStream_t stream) {
    const int S = few_splits(m.Vp / 32);
    const size_t bytes = few_lds_bytes(sizeof(T) == 4 ? 2 : 1, m.Hp);
    return fixed_offset ? launch_kernel<step_few_kernel<T, true>>(m, a, S, bytes, stream) : launch_kernel<step_few_kernel<T, false>>(m, a, S, bytes, stream);
}

hipError_t launch_step_few(const ModelDev &m, const FewStep &a, bool fixed_offset, hipStream_t stream) {
    return m.dtype == RNNLM_BF16 ? launch_type<bf16_t>(m, a, fixed_offset, stream) : launch_type<float>(m, a, fixed_offset, stream);
}

}  // namespace rnnlm
