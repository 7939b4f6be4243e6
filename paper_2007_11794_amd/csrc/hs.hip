// Hierarchical output layer (Section 2.1 of the paper): the words are the leaves of a Huffman
// tree, and the probability of a word is normalised only over the nodes on its path from the
// root: log p(w | h') = sum over the path nodes i of log sigmoid(+-theta_i . h'), + for code bit
// 0, - for code bit 1.  About log2 V dot products per queried word instead of V per row: the
// whole-vocabulary contraction of the full softmax disappears, what is left is a gather of node
// vectors (one contiguous row each), bound by L2 / HBM traffic.
//
// One wave per (query, word) pair, eight path nodes at a time: the eight node rows are requested
// together, the eight dot products are reduced over the wave at once, and the lane that ends up
// with node u turns its dot product into log sigmoid.  The tree comes with the model
// (rnnlm_hs_load); rnnlm_huffman_build below makes one from word frequencies on the host.
#include <algorithm>
#include <numeric>
#include <vector>

#include "device_utils.h"
#include "recur_math.h"
#include "rnnlm_internal.h"

namespace rnnlm {

namespace {

constexpr int kHsBatch = 8;

// log sigmoid(x) = min(x, 0) - log(1 + exp(-|x|))
__device__ __forceinline__ float log_sigmoid_f32(float x) {
    const float t = fast_exp2(-fabsf(x) * kLog2e);
    return fminf(x, 0.f) - fast_log2(1.0f + t) * kLn2;
}

__device__ __forceinline__ float weight_f32(bf16_t w) { return bf16_to_f32(w); }
__device__ __forceinline__ float weight_f32(float w) { return w; }

template <typename T>
__global__ __launch_bounds__(256) void hs_query_kernel(
    ModelDev m, int rows, const int *__restrict__ B_dev, int N, int K,
    const int32_t *__restrict__ query_word, const int32_t *__restrict__ row_of_query,
    const float *__restrict__ h_out, const float *__restrict__ base_score, float *__restrict__ logprob) {
    const int B = B_dev ? *B_dev : rows;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long pair = (long long)blockIdx.x * 4 + wave;
    if (pair >= (long long)N * K) return;                // wave-uniform; no barrier in this kernel
    const int n = (int)(pair / K);
    const int H = m.H, Hp = m.Hp;
    const int r_raw = row_of_query ? row_of_query[n] : n;
    const bool r_ok = r_raw >= 0 && r_raw < B;
    const int r = r_ok ? r_raw : 0;
    const int q_raw = query_word[pair];
    const bool q_ok = q_raw >= 0 && q_raw < m.V;
    const int q = q_ok ? q_raw : 0;
    const int off0 = m.path_off[q], len = m.path_off[q + 1] - off0;      // wave-uniform
    const T *Theta = static_cast<const T *>(m.Theta);
    const float *hrow = h_out + (size_t)r * H;
    const bool vec_ok = (H % 4) == 0;
    const int umine = batch_slot_of_lane(lane);
    float total = 0.f;
    for (int i0 = 0; i0 < len; i0 += kHsBatch) {
        const bool valid = i0 + umine < len;
        const uint32_t entry = valid ? (uint32_t)m.path_entry[off0 + i0 + umine] : 0u;
        const int node_mine = (int)(entry & 0x7FFFFFFFu);
        int node[kHsBatch];
#pragma unroll
        for (int u = 0; u < kHsBatch; ++u) node[u] = __builtin_amdgcn_readlane(node_mine, lane_of_batch_slot(u));
        float acc[kHsBatch];
#pragma unroll
        for (int u = 0; u < kHsBatch; ++u) acc[u] = 0.f;
        for (int j0 = lane * 8; j0 < Hp; j0 += 512) {
            float h8[8];
            load8_row(hrow, j0, H, vec_ok, 0.f, h8);
            float w8[kHsBatch][8];
#pragma unroll
            for (int u = 0; u < kHsBatch; ++u) load8_weights(Theta, (size_t)node[u] * Hp + j0, w8[u]);
#pragma unroll
            for (int u = 0; u < kHsBatch; ++u)
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[u] = fmaf(w8[u][i], h8[i], acc[u]);
        }
        const float x = wave_sum8(acc, lane);
        float term = valid ? log_sigmoid_f32((entry >> 31) ? -x : x) : 0.f;
        float a, b;
        half_pair(term, term, a, b); term = a + b;       // the eight slots differ in lane bits 5, 4, 3
        row_pair(term, term, a, b); term = a + b;
        term += lane_xor<8>(term);
        total += term;
    }
    if (lane == 0) {
        if (r_ok && q_ok) {
            logprob[pair] = base_score ? total - base_score[pair] : total;
        } else {
            atomicOr(m.flag, r_ok ? RNNLM_FLAG_BAD_QUERY_WORD : RNNLM_FLAG_BAD_ROW);
            logprob[pair] = quiet_nan();
        }
    }
}

// ---- the same for a raw query with several words: the paths of its K words share their upper
// nodes (every path starts at the root), so the workgroup of a raw query first collects the
// DISTINCT nodes of all K paths (a small LDS hash table, 23 KB in all: six workgroups per compute
// unit -- the kernel is a chain of dependent loads and lives on occupancy), computes one dot product per distinct
// node, and only then adds up log sigmoid along each path.  At the headline shape (K = 32, Zipf
// words) that is 163 instead of 304 node vectors per query.
// Two sizes of the workgroup of a raw query: up to 1024 path entries (all K words together) with 256
// threads, and up to 256 entries with 128 threads -- few words per query (a search step that extends
// every hypothesis by a handful of words): a third of the LDS, twice the queries in flight per
// compute unit, and the kernel lives on how many chains of dependent loads are in flight.
template <int THREADS, int LOG2_TABLE, int MAX_ENTRIES, int MAX_K>
struct HsShape {
    static constexpr int kThreads = THREADS;
    static constexpr int kLog2Table = LOG2_TABLE, kTable = 1 << LOG2_TABLE;   // slots of the node table (at most half full)
    static constexpr int kMaxEntries = MAX_ENTRIES;                          // path entries of one raw query
    static constexpr int kMaxK = MAX_K;
    static_assert(kTable >= 2 * MAX_ENTRIES && kTable <= 32768 && MAX_ENTRIES % THREADS == 0, "");
};
typedef HsShape<256, 11, 1024, 256> HsLarge;
typedef HsShape<128, 9, 256, 64> HsSmall;
// The same with twice the threads, while the queries leave compute units idle or half empty: a query's chain of
// dependent loads gets shorter (fewer rounds of node rows), the number of chains does not matter then.  Steps at V =
// 65536, H = 512, bf16, us, half as many threads / these: 40 queries of 25 words 17.6 / 13.9, 512 queries 20.8 / 17.3,
// 640 of 30 words 22.4 / 24.4, 1024 of 32 words 26.1 / 28.9; 512 queries of 6 words 16.6 / 14.2, 640 15.6 / 13.9.  With few words four
// workgroups of the doubled shape fit a compute unit (sixteen waves), so the line lies at 1024 queries there: 1024 of 6 words 15.6 / 14.6, of 12, H =
// 400, 17.5 / 15.9, H = 1024 32.7 / 27.7, fp32, H = 320, 21.0 / 20.2; 700 of 8, H = 640, 21.1 / 17.5; 1300 of 8 20.4 / 20.6, of 4, H = 320, 13.0 /
// 13.9; 2048 of 8 21.2 / 23.1.  Short rows have
// several in a wave's round already: up to 256 queries (V = 300000, H = 128, 40 queries 12.1 / 11.3; H = 250, fp32, 512 queries
// 19.8 / 23.5), and with the large shape only once the words' nodes are more than one round of half as many threads: kernel at V =
// 250000, H = 128, bf16, 100 queries of 17 words 0.3 slower, 24 words 0.3 faster, 32 words 1.3 faster; rows that are not 16-byte
// aligned, which every wave reads for itself, H = 75, 17, 24 and 32 words 1.0, 0.3 and 0.5 slower; V = 60000, H = 256, 17 words 1.0
// faster, H = 250 0.3 slower, 24 words 0.3 faster.  Steps at Hp = 64 and 192, which have several rows in a wave's round as well: V =
// 250000, H = 64, fp32, 512 queries of 15 words 13.2 / 9.8 with the narrow shape, of 30 14.9 / 12.1; V = 60000, H = 192, bf16, 256 queries
// of 30 words 10.5 with the wide one, of 15 words 10.3 wide, 10.9 narrow.
typedef HsShape<512, 11, 1024, 256> HsLargeWide;
typedef HsShape<256, 9, 256, 64> HsSmallWide;
inline bool hs_wide(int N, int K, int H, int Hp, bool small) {
    if (Hp > 256) return N <= (small ? 1024 : 512);
    const bool aligned = H % 4 == 0;
    return N <= 256 && (small || (Hp <= 128 ? aligned && K >= 24 : K >= (aligned ? 16 : 24)));
}

// Dot products of the distinct nodes for a short hidden vector (Hp = 8 * LPR elements at most, LPR = 16 or
// 32; lanes beyond the row drop what they compute): a node row takes only LPR lanes of a wave, so the wave works on 64 / LPR rows side by side,
// eight per lane group in flight: 32 (16) rows per wave and round trip to memory instead of 8 (steps at H = 64, fp32, V = 250000, 4096
// queries of 30 words, a wave per eight rows / this 70.6 / 42.9 us, 32 queries 12.5 / 9.7; H = 192, bf16, V = 60000 58.9 / 40.7, 12.0 / 10.2).  Lane
// group g of wave w takes the nodes d = first + g + G * u, u = 0..7; the eight sums of a group are
// reduced together (a lane passes on the half it will not finish, as in wave_sum8).
// row(d): which row of the weights; asked for d < D.
template <typename T, int LPR, int THREADS, class Row>
__device__ __forceinline__ void hs_dots_short_rows(const T *Theta, const float (&h8)[8], int Hp, Row row, float *dx, int D, int wave, int lane) {
    static_assert(LPR == 16 || LPR == 32, "");
    constexpr int G = 64 / LPR, kPerWave = G * kHsBatch;
    const int g = lane / LPR, sl = lane % LPR;
    const bool in_row = sl * 8 < Hp;
    const int j0 = in_row ? sl * 8 : 0;
    constexpr int top = LPR / 2;                           // 8 or 16
    const bool upa = (lane & top) != 0, upb = (lane & (top / 2)) != 0, upc = (lane & (top / 4)) != 0;
    const int u_mine = (upa ? 4 : 0) + (upb ? 2 : 0) + (upc ? 1 : 0);
    const bool writer = (lane & (top / 4 - 1)) == 0;
    auto fetch = [&](int first, float (&w8)[kHsBatch][8]) {
#pragma unroll
        for (int u = 0; u < kHsBatch; ++u) {
            const int d = first + g + G * u;
            const int node = d < D ? row(d) : 0;
            load8_weights(Theta, (size_t)node * Hp + j0, w8[u]);
        }
    };
    auto finish = [&](int first, const float (&w8)[kHsBatch][8]) {
        float acc[kHsBatch];
#pragma unroll
        for (int u = 0; u < kHsBatch; ++u) {
            acc[u] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[u] = fmaf(w8[u][i], h8[i], acc[u]);
            acc[u] = in_row ? acc[u] : 0.f;
        }
        // three levels that halve the number of values a lane carries, then the rest of the butterfly
        float v4[4], v2[2], x, y;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (LPR == 32) { row_pair(acc[i], acc[4 + i], x, y); v4[i] = x + y; }
            else v4[i] = (upa ? acc[4 + i] : acc[i]) + lane_xor<8>(upa ? acc[i] : acc[4 + i]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) v2[i] = (upb ? v4[2 + i] : v4[i]) + lane_xor<top / 2>(upb ? v4[i] : v4[2 + i]);
        float v = (upc ? v2[1] : v2[0]) + lane_xor<top / 4>(upc ? v2[0] : v2[1]);
        if constexpr (LPR == 32) v += lane_xor<2>(v);
        v += lane_xor<1>(v);
        const int d = first + g + G * u_mine;
        if (writer && d < D) dx[d] = v;
    };
    // two batches on their way at a time (the second may lie past the end: its loads fetch node 0)
    constexpr int stride = (THREADS / 64) * kPerWave;
    for (int first = wave * kPerWave; first < D; first += 2 * stride) {
        float wa[kHsBatch][8], wb[kHsBatch][8];
        fetch(first, wa);
        fetch(first + stride, wb);
        finish(first, wa);
        finish(first + stride, wb);
    }
}

// The same for bf16 rows that a wave reads in one piece (256 < Hp <= 512, lane l has elements 8 l .. + 7), its eight floats of the hidden
// vector read once.  Bound by the rows' way from the L2s; with more than three rounds of nodes, eight rows are on their way while the eight
// before them are multiplied and reduced.  The rounds past the end, which fetch the first node again, are there so that a wait has the same
// loads in front of it on every way to it (left out, the compiler waited for everything: 4096 queries of 32 words 81 us), and cost more
// than they give in two or three rounds (2000 queries of 5 words 14.8 -> 15.5 us).  Steps, us, general form / this one: V = 65536, H = 512, 4096 queries
// of 32 words from 1229 rows 63.3 / 57.5, of 8 words 34.4 / 32.8, 1024 of 32 words 22.5 / 22.2; V = 100000, H = 300, 1500 of 10 words 21.4 / 18.7;
// V = 20000, H = 320, 2000 of 5 words 15.8 / 15.5; V = 50000, H = 333, 100 of 12 words 13.9 / 12.1.  fp32 rows take twice the registers: not tried.
template <typename T, int THREADS>
__device__ __forceinline__ void hs_dots_one_piece(const T *Theta, const float (&h8)[8], int Hp, const int *dnode, float *dx, int D, int wave, int lane) {
    const int umine = batch_slot_of_lane(lane);
    const bool in_row = lane * 8 < Hp;                     // lanes beyond the row drop what they compute
    const int j0 = in_row ? lane * 8 : 0;
    auto fetch = [&](int first, float (&w8)[kHsBatch][8]) {
        const int node_mine = dnode[first + umine < D ? first + umine : 0];
#pragma unroll
        for (int u = 0; u < kHsBatch; ++u)
            load8_weights(Theta, (size_t)__builtin_amdgcn_readlane(node_mine, lane_of_batch_slot(u)) * Hp + j0, w8[u]);
    };
    auto finish = [&](int first, const float (&w8)[kHsBatch][8]) {
        float acc[kHsBatch];
#pragma unroll
        for (int u = 0; u < kHsBatch; ++u) {
            acc[u] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[u] = fmaf(w8[u][i], h8[i], acc[u]);
            acc[u] = in_row ? acc[u] : 0.f;
        }
        const float x = wave_sum8(acc, lane);
        if ((lane & 7) == 0 && first + umine < D) dx[first + umine] = x;
    };
    constexpr int stride = (THREADS / 64) * kHsBatch;
    int first = wave * kHsBatch;
    float wa[kHsBatch][8], wb[kHsBatch][8];
    if (D <= 3 * stride) {
        for (; first < D; first += stride) {
            fetch(first, wa);
            finish(first, wa);
        }
        return;
    }
    fetch(first, wa);
    for (; first < D; first += 2 * stride) {
        fetch(first + stride, wb);
        finish(first, wa);
        fetch(first + 2 * stride, wa);
        finish(first + stride, wb);
    }
}

// LPR: lanes per node row of the short-row form (16: Hp <= 128, 32: Hp <= 256), 64: bf16 rows in one piece, 0: any hidden size.
// Kernels of their own, so that the registers of the short-row form do not cost the general one occupancy.
// HERE (short rows only): the hidden update is part of the launch.  A workgroup computes the hidden vector of its query's row for
// itself, in plain fp32, while its words' paths are on their way: W (Hp x Hp) comes through the same row dot products.  Without
// row_of_query it also writes the row out; with it, `rows` further workgroups do.
struct HsHidden {
    const int32_t *prev_word;
    const float *h_in;
    float *h_out;
};
template <typename T, int LPR, class S, bool HERE>
__global__ __launch_bounds__(S::kThreads) void hs_query_shared_kernel(
    ModelDev m, int rows, const int *__restrict__ B_dev, int N, int K,
    const int32_t *__restrict__ query_word, const int32_t *__restrict__ row_of_query,
    const float *__restrict__ h_out, const float *__restrict__ base_score, float *__restrict__ logprob, HsHidden hidden) {
    __shared__ int wbase[S::kMaxK + 1];               // start of word k's entries
    __shared__ int woff[S::kMaxK];                    // where word k's path starts in the model's entries
    __shared__ uint16_t eslot[S::kMaxEntries];        // entry -> table slot of its node | code bit << 15
    __shared__ int tnode[S::kTable];                  // hash table: node (-1 free)
    __shared__ uint16_t tidx[S::kTable];              // slot -> index of its node among the distinct ones
    __shared__ int dnode[S::kMaxEntries];             // the distinct nodes
    __shared__ float dx[S::kMaxEntries];              // their dot products
    __shared__ int dcount;
    __shared__ int wsum[S::kThreads / 64 + 1];
    __shared__ __attribute__((aligned(16))) float hvec[HERE ? 8 * LPR : 4];        // W (h - 1/2), then the hidden vector, zeros beyond H
    static_assert(S::kTable <= 32768, "slot index and code bit share sixteen bits");
    static_assert(S::kMaxK <= S::kThreads, "one word per thread in step 1");
    const int B = B_dev ? *B_dev : rows;
    const bool query = !HERE || (int)blockIdx.x < N;        // (HERE) or a row that only has to be written
    const int n = query ? blockIdx.x : 0;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int H = m.H, Hp = m.Hp;
    const int r_raw = !query ? blockIdx.x - N : row_of_query ? row_of_query[n] : n;
    const bool r_ok = r_raw >= 0 && r_raw < B;
    const int r = r_ok ? r_raw : 0;
    int word_before = 0;
    float h8[8];
    if constexpr (HERE) {
        word_before = hidden.prev_word[r];
        load8_row(hidden.h_in + (size_t)r * H, 8 * (lane % LPR), H, (H % 4) == 0 && (reinterpret_cast<uintptr_t>(hidden.h_in) & 15) == 0, 0.5f, h8);
    }
    // 1. lengths of the K paths -> offsets (K <= 256: one word per thread)
    int len = 0;
    if (query && tid < K) {
        const int q_raw = query_word[(size_t)n * K + tid];
        const int q = (q_raw >= 0 && q_raw < m.V) ? q_raw : 0;
        const int o = m.path_off[q];
        len = m.path_off[q + 1] - o;
        woff[tid] = o;
    }
    for (int i = tid; i < S::kTable; i += S::kThreads) tnode[i] = -1;
    if (tid == 0) dcount = 0;
    float embedding = 0.f, half_rowsum = 0.f;
    const bool word_ok = word_before >= 0 && word_before < m.V;
    if constexpr (HERE) {
        if (tid < Hp) {                                    // (further units below)
            embedding = weight_f32(static_cast<const T *>(m.U)[(size_t)(word_ok ? word_before : 0) * Hp + tid]);
            half_rowsum = m.half_rowsum_W[tid];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) h8[i] -= 0.5f;
        hs_dots_short_rows<T, LPR, S::kThreads>(static_cast<const T *>(m.W), h8, Hp, [](int d) { return d; }, hvec, Hp, wave, lane);
    }
    int total;
    const int mybase = block_exclusive_scan(len, wsum, total);      // barriers inside
    if (tid < K) wbase[tid] = mybase;
    if (tid == 0) wbase[K] = total;
    if constexpr (HERE) {                                  // (the sums were there with the scan's barriers)
        const bool writes = query ? !row_of_query : true;
        for (int j = tid; j < Hp; j += S::kThreads) {
            if (j != tid) {
                embedding = weight_f32(static_cast<const T *>(m.U)[(size_t)(word_ok ? word_before : 0) * Hp + j]);
                half_rowsum = m.half_rowsum_W[j];
            }
            const float h = word_ok ? sigmoid_f32(hvec[j] + half_rowsum + embedding) : quiet_nan();
            hvec[j] = j < H ? h : 0.f;
            if (writes && j < H) hidden.h_out[(size_t)r * H + j] = h;
        }
        if (writes && !word_ok && tid == 0) atomicOr(m.flag, RNNLM_FLAG_BAD_PREV_WORD);
        if (!query) return;                                // uniform
    }
    __syncthreads();
    // 2. distinct nodes (a thread per path entry, all entries of a thread requested before the first
    //    is used: one round trip to memory for the whole query): the thread whose insertion claims
    //    a slot numbers the node; every entry remembers its slot and its code bit
    constexpr int kPerThread = S::kMaxEntries / S::kThreads;
    uint32_t entry[kPerThread];
#pragma unroll
    for (int c = 0; c < kPerThread; ++c) {
        const int e = tid + c * S::kThreads;
        entry[c] = 0u;
        if (e < total) {
            int lo = 0, hi = K;                                      // the word k with wbase[k] <= e < wbase[k + 1]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (wbase[mid] <= e) lo = mid; else hi = mid;
            }
            entry[c] = (uint32_t)m.path_entry[woff[lo] + (e - wbase[lo])];
        }
    }
#pragma unroll
    for (int c = 0; c < kPerThread; ++c) {
        const int e = tid + c * S::kThreads;
        if (e < total) {
            const int node = (int)(entry[c] & 0x7FFFFFFFu);
            uint32_t h = (uint32_t)(node * 0x9E3779B1u) >> (32 - S::kLog2Table);
            for (int probe = 0; probe < S::kTable; ++probe) {
                const int old = atomicCAS(&tnode[h], -1, node);
                if (old == -1) {
                    const int d = atomicAdd(&dcount, 1);
                    dnode[d] = node;
                    tidx[h] = (uint16_t)d;
                    break;
                }
                if (old == node) break;
                h = (h + 1) & (S::kTable - 1);
            }
            eslot[e] = (uint16_t)(h | ((entry[c] >> 31) << 15));
        }
    }
    __syncthreads();
    const int D = dcount;
    // 3. one dot product per distinct node, eight nodes of a wave at a time
    const T *Theta = static_cast<const T *>(m.Theta);
    const float *hrow = h_out + (size_t)r * H;
    const bool vec_ok = (H % 4) == 0;
    const int umine = batch_slot_of_lane(lane);
    if constexpr (LPR == 64) {
        load8_row(hrow, lane * 8 < Hp ? lane * 8 : 0, H, vec_ok, 0.f, h8);
        hs_dots_one_piece<T, S::kThreads>(Theta, h8, Hp, dnode, dx, D, wave, lane);
    } else if constexpr (LPR != 0) {
        if constexpr (HERE) {
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(hvec + 8 * (lane % LPR)), hi = *reinterpret_cast<const f32x4 *>(hvec + 8 * (lane % LPR) + 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) { h8[i] = lo[i]; h8[4 + i] = hi[i]; }      // (lanes beyond the row drop what they compute)
        } else {
            load8_row(hrow, 8 * (lane % LPR), H, vec_ok, 0.f, h8);
        }
        hs_dots_short_rows<T, LPR, S::kThreads>(Theta, h8, Hp, [&](int d) { return dnode[d]; }, dx, D, wave, lane);
    } else
    for (int d0 = wave * kHsBatch; d0 < D; d0 += (S::kThreads / 64) * kHsBatch) {
        const int node_mine = (d0 + umine < D) ? dnode[d0 + umine] : 0;
        int node[kHsBatch];
#pragma unroll
        for (int u = 0; u < kHsBatch; ++u) node[u] = __builtin_amdgcn_readlane(node_mine, lane_of_batch_slot(u));
        float acc[kHsBatch];
#pragma unroll
        for (int u = 0; u < kHsBatch; ++u) acc[u] = 0.f;
        for (int j0 = lane * 8; j0 < Hp; j0 += 512) {
            float h8[8];
            load8_row(hrow, j0, H, vec_ok, 0.f, h8);
            float w8[kHsBatch][8];
#pragma unroll
            for (int u = 0; u < kHsBatch; ++u) load8_weights(Theta, (size_t)node[u] * Hp + j0, w8[u]);
#pragma unroll
            for (int u = 0; u < kHsBatch; ++u)
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[u] = fmaf(w8[u][i], h8[i], acc[u]);
        }
        const float x = wave_sum8(acc, lane);
        if ((lane & 7) == 0 && d0 + umine < D) dx[d0 + umine] = x;
    }
    __syncthreads();
    // 4. log sigmoid of every path entry (a thread per entry; the terms go where the node table was,
    //    which nobody has probed since step 2), then eight lanes add up the terms of one word
    float *const eterm = reinterpret_cast<float *>(tnode);
    static_assert(S::kMaxEntries <= S::kTable, "the terms fit the node table");
#pragma unroll
    for (int c = 0; c < kPerThread; ++c) {
        const int e = tid + c * S::kThreads;
        if (e < total) {
            const uint32_t es = eslot[e];
            const float x = dx[tidx[es & 0x7FFFu]];
            eterm[e] = log_sigmoid_f32((es >> 15) ? -x : x);
        }
    }
    __syncthreads();
    for (int k = tid >> 3; k < K; k += S::kThreads / 8) {
        const int b0 = wbase[k], b1 = wbase[k + 1];
        float t = 0.f;
        for (int e = b0 + (tid & 7); e < b1; e += 8) t += eterm[e];
        t += lane_xor<4>(t);
        t += lane_xor<2>(t);
        t += lane_xor<1>(t);
        if ((tid & 7) == 0) {
            const int qk = query_word[(size_t)n * K + k];
            const bool ok = qk >= 0 && qk < m.V;
            const size_t at = (size_t)n * K + k;
            if (r_ok && ok) {
                logprob[at] = base_score ? t - base_score[at] : t;
            } else {
                atomicOr(m.flag, r_ok ? RNNLM_FLAG_BAD_QUERY_WORD : RNNLM_FLAG_BAD_ROW);
                logprob[at] = quiet_nan();
            }
        }
    }
}

}  // namespace

// Several words per query, few enough path entries: one workgroup per raw query, shared path nodes computed once.
static bool hs_shared(const ModelDev &m, int K) { return K >= 4 && K <= HsLarge::kMaxK && (long long)K * m.hs_max_len <= HsLarge::kMaxEntries; }

template <bool HERE>
static hipError_t launch_shared(const ModelDev &m, int rows, const int *B_dev, int N, int K, const int32_t *query_word, const int32_t *row_of_query,
                                const float *h_out, const float *base_score, float *logprob, const HsHidden &hidden, hipStream_t stream) {
    const bool small = K <= HsSmall::kMaxK && (long long)K * m.hs_max_len <= HsSmall::kMaxEntries;
    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(HERE && row_of_query ? N + rows : N), dim3(threads), 0, stream, m, rows, B_dev, N, K, query_word,
                           row_of_query, h_out, base_score, logprob, hidden);
    };
    auto pick_rows = [&](auto tag, auto shape) {
        using T = decltype(tag);
        using S = decltype(shape);
        if (m.Hp <= 128) launch(hs_query_shared_kernel<T, 16, S, HERE>, S::kThreads);
        else if (HERE || m.Hp <= 256) launch(hs_query_shared_kernel<T, 32, S, HERE>, S::kThreads);
        else if constexpr (!HERE) {
            if (sizeof(T) == 2 && m.Hp <= 512) launch(hs_query_shared_kernel<T, sizeof(T) == 2 ? 64 : 0, S, HERE>, S::kThreads);
            else launch(hs_query_shared_kernel<T, 0, S, HERE>, S::kThreads);
        }
    };
    const bool wide = hs_wide(N, K, m.H, m.Hp, small);
    auto pick = [&](auto tag) {
        if (small && wide) pick_rows(tag, HsSmallWide{});
        else if (small) pick_rows(tag, HsSmall{});
        else if (wide) pick_rows(tag, HsLargeWide{});
        else pick_rows(tag, HsLarge{});
    };
    if (m.dtype == RNNLM_BF16) pick(bf16_t{});
    else pick(float{});
    return hipGetLastError();
}

// Every workgroup reads W: while that is little beside its nodes' rows, and the workgroups are few.  Replayed steps, us, two launches
// / this one (the host's part, 9.3 us for two launches, 6 to 7 for one, is not in it): bf16, V = 250000, H = 128, 64 queries of 30 words
// 9.7 / 7.8, 1024 of 6, 30 9.8 / 8.3, 13.1 / 11.7, 2048 of 30 19.5 / 20.3; fp32, V = 60000, H = 128, 512 of 30 11.4 / 9.8, 1024 17.7 /
// 18.3; V = 60000, H = 256, bf16, 200 of 6, 30 9.5 / 7.9, 10.4 / 8.1, 512 11.2 / 13.2, 12.9 / 12.1, fp32 200 of 30 11.8 / 9.1, 512 of
// 6 from 153 rows 11.9 / 13.1.
bool hs_step_chosen(const ModelDev &m, int B, int N, int K, bool mapped) {
    if (m.Hp > 256 || B <= 0 || N <= 0 || !hs_shared(m, K)) return false;
    const int limit = m.Hp > 128 ? 256 : m.dtype == RNNLM_BF16 ? 1024 : 512;
    return N <= limit && (!mapped || N + B <= limit + limit / 2);
}

hipError_t launch_hs_step(const ModelDev &m, int B, int N, int K, const int32_t *prev_word, const float *h_in, const int32_t *query_word,
                          const int32_t *row_of_query, float *h_out, const float *base_score, float *logprob, hipStream_t stream) {
    return launch_shared<true>(m, B, nullptr, N, K, query_word, row_of_query, h_out, base_score, logprob, HsHidden{prev_word, h_in, h_out}, stream);
}

hipError_t launch_hs_query(const ModelDev &m, int rows, const int *B_dev, int N, int K,
                           const int32_t *query_word, const int32_t *row_of_query, const float *h_out,
                           const float *base_score, float *logprob, hipStream_t stream) {
    if (N <= 0 || K <= 0) return hipSuccess;
    if (hs_shared(m, K)) return launch_shared<false>(m, rows, B_dev, N, K, query_word, row_of_query, h_out, base_score, logprob, HsHidden{}, stream);
    const long long pairs = (long long)N * K;
    const dim3 grid((unsigned)((pairs + 3) / 4));
    if (m.dtype == RNNLM_BF16)
        hipLaunchKernelGGL(hs_query_kernel<bf16_t>, grid, dim3(256), 0, stream, m, rows, B_dev, N, K, query_word,
                           row_of_query, h_out, base_score, logprob);
    else
        hipLaunchKernelGGL(hs_query_kernel<float>, grid, dim3(256), 0, stream, m, rows, B_dev, N, K, query_word,
                           row_of_query, h_out, base_score, logprob);
    return hipGetLastError();
}

}  // namespace rnnlm

// Huffman's method with two queues (host code): the words sorted by (frequency, id) ascending,
// and the inner nodes in order of creation, whose weights never decrease.  Every merge takes
// the two lightest queue heads, a word before an inner node of equal weight; the first taken is
// the child with code bit 0.  Inner nodes are numbered in order of creation, the root is V - 2.
extern "C" int rnnlm_huffman_build(int V, const double *frequency, int32_t *path_offset, int32_t *path_entry,
                                   size_t capacity, size_t *needed) {
    if (V < 2 || !frequency || !path_offset) return RNNLM_EINVAL;
    if (V > (1 << 30)) return RNNLM_ERANGE;
    for (int v = 0; v < V; ++v)
        if (!(frequency[v] >= 0.0)) return RNNLM_EINVAL;
    std::vector<int32_t> order, up;          // words by weight; parent of word v / of inner node V + i
    std::vector<double> weight;              // of the inner nodes
    std::vector<uint8_t> code;
    try {
        order.resize(V);
        up.assign(2 * (size_t)V - 1, -1);
        code.assign(2 * (size_t)V - 1, 0);
        weight.resize(V - 1);
    } catch (...) {
        return RNNLM_ENOMEM;
    }
    std::iota(order.begin(), order.end(), 0);
    std::sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        return frequency[a] < frequency[b] || (frequency[a] == frequency[b] && a < b);
    });
    size_t next_word = 0, next_inner = 0;
    for (int created = 0; created < V - 1; ++created) {
        double sum = 0.0;
        for (int side = 0; side < 2; ++side) {
            const bool words_left = next_word < (size_t)V, inner_left = next_inner < (size_t)created;
            const bool take_word = words_left && (!inner_left || frequency[order[next_word]] <= weight[next_inner]);
            size_t child;
            if (take_word) {
                child = (size_t)order[next_word];
                sum += frequency[order[next_word++]];
            } else {
                child = (size_t)V + next_inner;
                sum += weight[next_inner++];
            }
            up[child] = V + created;
            code[child] = (uint8_t)side;
        }
        weight[created] = sum;
    }
    size_t total = 0;
    for (int v = 0; v < V; ++v) {
        size_t depth = 0;
        for (int32_t x = v; up[x] >= 0; x = up[x]) ++depth;
        path_offset[v] = (int32_t)total;
        if (path_entry && total + depth <= capacity) {
            size_t at = total + depth;
            for (int32_t x = v; up[x] >= 0; x = up[x])
                path_entry[--at] = (int32_t)((uint32_t)(up[x] - V) | ((uint32_t)code[x] << 31));
        }
        total += depth;
        if (total > 0x7FFFFFFFull) return RNNLM_ERANGE;
    }
    path_offset[V] = (int32_t)total;
    if (needed) *needed = total;
    return (path_entry && total <= capacity) ? RNNLM_OK : RNNLM_ERANGE;
}
