// Load-time kernels: re-lay the output weights out as [V][H] (one contiguous row per word:
// the K-major operand of the matrix cores and a single contiguous read per queried word),
// and the per-word constants of the centred logit  z = (bias + colsum(O)/2) + O^T (h' - 1/2).
#include "device_utils.h"
#include "recur_math.h"
#include "rnnlm_internal.h"

namespace rnnlm {

namespace {

template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T *__restrict__ O, T *__restrict__ Ot,
                                                        int H, int V, int Hp, int Vp) {
    __shared__ T tile[32][33];
    const int v0 = blockIdx.x * 32, j0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;     // 32 x 8
    for (int r = ty; r < 32; r += 8) {
        int j = j0 + r, v = v0 + tx;
        tile[r][tx] = (j < H && v < V) ? O[(size_t)j * V + v] : T(0);
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        int v = v0 + r, j = j0 + tx;
        if (v < Vp && j < Hp) Ot[(size_t)v * Hp + j] = tile[tx][r];
    }
}

// A workgroup per row at a time; bound by the host copy in front of it.
template <typename T>
__global__ __launch_bounds__(256) void pad_rows_kernel(const T *__restrict__ src, T *__restrict__ dst, size_t rows, int H,
                                                       int Hp) {
    for (size_t r = blockIdx.x; r < rows; r += gridDim.x)
        for (int j = threadIdx.x; j < Hp; j += 256) dst[r * Hp + j] = j < H ? src[r * H + j] : T(0);
}

__device__ __forceinline__ double widen(float x) { return (double)x; }
__device__ __forceinline__ double widen(bf16_t x) { return (double)bf16_to_f32(x); }

// Per word v: half the column sum of O, and bounds on the logit that hold for every hidden
// vector with components in [0,1]:  upper = bias + sum_j max(O[j][v],0),
// lower = bias + sum_j min(O[j][v],0).  fp64 accumulation; upper is rounded up and lower
// down by one float ulp-ish margin on the host.
template <typename T>
__global__ __launch_bounds__(256) void col_stats_kernel(const T *__restrict__ O,
                                                        const float *__restrict__ bias, int H, int V,
                                                        float *__restrict__ half_colsum,
                                                        float *__restrict__ upper,
                                                        float *__restrict__ lower) {
    int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= V) return;
    double pos = 0.0, neg = 0.0;
    for (int j = 0; j < H; ++j) {
        double x = widen(O[(size_t)j * V + v]);
        if (x > 0) pos += x; else neg += x;
    }
    double b = bias ? (double)bias[v] : 0.0;
    half_colsum[v] = (float)(0.5 * (pos + neg));
    upper[v] = (float)(b + pos);
    lower[v] = (float)(b + neg);
}

__global__ __launch_bounds__(256) void fill_cvec_kernel(const float *__restrict__ bias,
                                                        const float *__restrict__ half_colsum, int V,
                                                        int Vp, float m2_fixed, float *__restrict__ bias_out,
                                                        float *__restrict__ cvec,
                                                        float *__restrict__ cvec2_fixed, float *__restrict__ cvec_fixed) {
    int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= Vp) return;
    if (v < V) {
        float b = bias ? bias[v] : 0.f;
        bias_out[v] = b;
        float c = (b + half_colsum[v]) * kLog2e;
        cvec[v] = c;
        cvec2_fixed[v] = c - m2_fixed;
        cvec_fixed[v] = (float)((double)(c - m2_fixed) * 0.6931471805599453);
    } else {
        cvec[v] = -INFINITY;
        cvec2_fixed[v] = -INFINITY;
        cvec_fixed[v] = -INFINITY;
    }
}

// bf16 [Vp][Hp] weights re-laid in MFMA-operand order: 16 bytes per thread.
__global__ __launch_bounds__(256) void frag_weights_kernel(const u32x4 *__restrict__ Ot, size_t n, int KS,
                                                           u32x4 *__restrict__ Ofrag) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;       // (blk, ks, lane)
    if (i >= n) return;
    const int lane = (int)(i & 63);
    const size_t frag = i >> 6, blk = frag / KS;
    const int ks = (int)(frag % KS);
    const size_t word = blk * 32 + (lane & 31);
    Ofrag[i] = Ot[word * (2 * KS) + 2 * ks + (lane >> 5)];           // 2 KS chunks of 8 units per word
}

// fp32 [Hp][Hp] recurrent weights: [blk][ks][half][64 lanes][4]
__global__ __launch_bounds__(256) void frag_recurrent_f32_kernel(const f32x4 *__restrict__ W, int n, int KS, f32x4 *__restrict__ Wfrag) {
    const int i = blockIdx.x * 256 + threadIdx.x;                  // (blk, ks, half, lane)
    if (i >= n) return;
    const int lane = i & 63, half = (i >> 6) & 1, frag = i >> 7, blk = frag / KS, ks = frag % KS;
    Wfrag[i] = W[(blk * 32 + (lane & 31)) * (4 * KS) + 4 * ks + 2 * (lane >> 5) + half];
}

// fp32 W [Hp][Hp] as three bf16 terms in operand order, a thread per eight weights (Wops).
__global__ __launch_bounds__(256) void recurrent_terms_kernel(const float *__restrict__ W, int n, int KS, u32x4 *__restrict__ Wops) {
    const int i = blockIdx.x * 256 + threadIdx.x;                  // (blk, ks, lane)
    if (i >= n) return;
    const int lane = i & 63, ks = (i >> 6) % KS, blk = (i >> 6) / KS;
    float x[8];
    load8_weights(W, (size_t)(blk * 32 + (lane & 31)) * (16 * KS) + 16 * ks + 8 * (lane >> 5), x);
    u32x4 t[3];
    bf16_terms(x, t);
#pragma unroll
    for (int k = 0; k < 3; ++k) Wops[((i >> 6) * 3 + k) * 64 + lane] = t[k];
}

// fp32 [Vp][Hp] weights as two fp16 terms in the same operand order, [blk][ks][term][64 lanes][8 halves].
// One workgroup per block of 32 words: eight threads find the largest weight of a word, then lane
// 32 g + c of fragment ks takes word 32 blk + c, units 16 ks + 8 g .. + 7.  Words scaled to [2^13, 2^14):
// second terms stay normal numbers down to 2^-17 of the largest weight, products stay far below the
// fp32 range.  A word that holds an infinity or a NaN keeps it (its terms are infinities and NaN).
__global__ __launch_bounds__(256) void split2_weights_kernel(const float *__restrict__ Ot, int Hp, uint16_t *__restrict__ Ofrag,
                                                             float *__restrict__ ofac) {
    __shared__ int shift[32];
    const int tid = threadIdx.x, KS = Hp >> 4;
    const size_t blk = blockIdx.x;
    float big = 0.f;
    const float *row = Ot + (blk * 32 + (tid >> 3)) * Hp;
    for (int j = tid & 7; j < Hp; j += 8) big = fmaxf(big, fabsf(row[j]));
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) big = fmaxf(big, __shfl_xor(big, off, 64));
    if ((tid & 7) == 0) {
        int e = 0;
        if (big > 0.f && big < INFINITY) {
            (void)frexpf(big, &e);                                 // big in [2^(e-1), 2^e)
            e = 14 - e;
            if (e > 100) e = 100;                                  // words of denormal size: factors stay normal
        }
        shift[tid >> 3] = e;
        ofac[blk * 32 + (tid >> 3)] = ldexpf(kLog2e, -(e + kSplit2DExp));
    }
    __syncthreads();
    for (int i = tid; i < KS * 64; i += 256) {                     // (ks, lane)
        const int lane = i & 63, ks = i >> 6, w = lane & 31;
        float x[8];
        load8_weights(Ot, (blk * 32 + w) * Hp + 16 * ks + 8 * (lane >> 5), x);
        uint32_t p1[4], p2[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint16_t a1, a2, b1, b2;
            split2_f16(ldexpf(x[2 * q], shift[w]), a1, a2);
            split2_f16(ldexpf(x[2 * q + 1], shift[w]), b1, b2);
            p1[q] = a1 | ((uint32_t)b1 << 16);
            p2[q] = a2 | ((uint32_t)b2 << 16);
        }
        uint16_t *dst = Ofrag + ((blk * KS + ks) * 2 * 64 + lane) * 8;
        *reinterpret_cast<u32x4 *>(dst) = u32x4{p1[0], p1[1], p1[2], p1[3]};
        *reinterpret_cast<u32x4 *>(dst + 512) = u32x4{p2[0], p2[1], p2[2], p2[3]};
    }
}

}  // namespace

hipError_t launch_pad_rows(const void *src, void *dst, int dtype, size_t rows, int H, int Hp, hipStream_t stream) {
    const dim3 grid((unsigned)(rows < 16384 ? rows : 16384));
    if (dtype == RNNLM_BF16)
        hipLaunchKernelGGL(pad_rows_kernel<bf16_t>, grid, dim3(256), 0, stream, static_cast<const bf16_t *>(src),
                           static_cast<bf16_t *>(dst), rows, H, Hp);
    else
        hipLaunchKernelGGL(pad_rows_kernel<float>, grid, dim3(256), 0, stream, static_cast<const float *>(src),
                           static_cast<float *>(dst), rows, H, Hp);
    return hipGetLastError();
}

hipError_t launch_frag_weights(const void *Ot, int Vp, int Hp, void *Ofrag, hipStream_t stream) {
    const size_t n = (size_t)Vp * Hp / 8;
    hipLaunchKernelGGL(frag_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const u32x4 *>(Ot), n, Hp / 16, static_cast<u32x4 *>(Ofrag));
    return hipGetLastError();
}

hipError_t launch_frag_recurrent(const void *W, int dtype, int Hp, void *Wfrag, hipStream_t stream) {
    if (dtype == RNNLM_BF16) return launch_frag_weights(W, Hp, Hp, Wfrag, stream);
    const int n = Hp * Hp / 4;
    hipLaunchKernelGGL(frag_recurrent_f32_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, static_cast<const f32x4 *>(W), n, Hp / 16,
                       static_cast<f32x4 *>(Wfrag));
    return hipGetLastError();
}

hipError_t launch_recurrent_terms(const float *W, int Hp, void *Wops, hipStream_t stream) {
    const int n = Hp * Hp / 8;
    hipLaunchKernelGGL(recurrent_terms_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, W, n, Hp / 16, static_cast<u32x4 *>(Wops));
    return hipGetLastError();
}

hipError_t launch_split2_weights(const float *Ot, int Vp, int Hp, void *Ofrag, float *ofac, hipStream_t stream) {
    hipLaunchKernelGGL(split2_weights_kernel, dim3((unsigned)(Vp / 32)), dim3(256), 0, stream, Ot, Hp,
                       static_cast<uint16_t *>(Ofrag), ofac);
    return hipGetLastError();
}

hipError_t launch_transpose_O(const void *O_dev, void *Ot, int dtype, int H, int V, int Hp, int Vp,
                              hipStream_t stream) {
    dim3 grid((Vp + 31) / 32, (Hp + 31) / 32);
    if (dtype == RNNLM_BF16)
        hipLaunchKernelGGL(transpose_kernel<bf16_t>, grid, dim3(256), 0, stream,
                           static_cast<const bf16_t *>(O_dev), static_cast<bf16_t *>(Ot), H, V, Hp, Vp);
    else
        hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(256), 0, stream,
                           static_cast<const float *>(O_dev), static_cast<float *>(Ot), H, V, Hp, Vp);
    return hipGetLastError();
}

hipError_t launch_col_stats(const void *O_dev, const float *bias, int dtype, int H, int V,
                            float *half_colsum, float *upper, float *lower, hipStream_t stream) {
    dim3 grid((V + 255) / 256);
    if (dtype == RNNLM_BF16)
        hipLaunchKernelGGL(col_stats_kernel<bf16_t>, grid, dim3(256), 0, stream,
                           static_cast<const bf16_t *>(O_dev), bias, H, V, half_colsum, upper, lower);
    else
        hipLaunchKernelGGL(col_stats_kernel<float>, grid, dim3(256), 0, stream,
                           static_cast<const float *>(O_dev), bias, H, V, half_colsum, upper, lower);
    return hipGetLastError();
}

hipError_t launch_fill_cvec(const float *bias, const float *half_colsum, int V, int Vp, float m2_fixed,
                            float *bias_out, float *cvec2, float *cvec2_fixed, float *cvec_fixed,
                            hipStream_t stream) {
    hipLaunchKernelGGL(fill_cvec_kernel, dim3((Vp + 255) / 256), dim3(256), 0, stream, bias, half_colsum,
                       V, Vp, m2_fixed, bias_out, cvec2, cvec2_fixed, cvec_fixed);
    return hipGetLastError();
}

}  // namespace rnnlm
