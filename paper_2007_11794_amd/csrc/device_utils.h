// Small device helpers: bf16 <-> fp32, 8-element loads, wave reductions, MFMA types.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rnnlm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(((uint32_t)b) << 16);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two floats to two bfloat16 (round to nearest even, one v_cvt_pk_bf16_f32), `lo` in the
// low half.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// x = x1 + x2 with fp16 terms, each rounded to nearest even (|x| below 2^15): off by 2^-23 |x| at most, in a quarter of
// all fp32 numbers, as long as the second term is a normal fp16 number (and by 2^-25 at most beyond):
// the split that puts a scaled fp32 operand on the fp16 matrix cores.  Bit patterns.
__device__ __forceinline__ void split2_f16(float x, uint16_t &x1, uint16_t &x2) {
    const _Float16 h = (_Float16)x, l = (_Float16)(x - (float)h);
    x1 = __builtin_bit_cast(uint16_t, h);
    x2 = __builtin_bit_cast(uint16_t, l);
}

// Eight consecutive weights starting at element index `at` (a multiple of 8) as floats.
__device__ __forceinline__ void load8_weights(const uint16_t *p, size_t at, float (&out)[8]) {
    u32x4 v = *reinterpret_cast<const u32x4 *>(p + at);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        out[2 * i] = __uint_as_float(v[i] << 16);
        out[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
    }
}
__device__ __forceinline__ void load8_weights(const float *p, size_t at, float (&out)[8]) {
    f32x4 a = *reinterpret_cast<const f32x4 *>(p + at);
    f32x4 b = *reinterpret_cast<const f32x4 *>(p + at + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) { out[i] = a[i]; out[4 + i] = b[i]; }
}

// Eight consecutive floats row[k0 .. k0+7] of a caller-owned row of length H (not padded);
// elements at or beyond H read as `fill`.  Vector loads when the row allows them.
__device__ __forceinline__ void load8_row(const float *row, int k0, int H, bool vec_ok, float fill,
                                          float (&out)[8]) {
    if (vec_ok && k0 + 8 <= H) {
        f32x4 a = *reinterpret_cast<const f32x4 *>(row + k0);
        f32x4 b = *reinterpret_cast<const f32x4 *>(row + k0 + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) { out[i] = a[i]; out[4 + i] = b[i]; }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = (k0 + i < H) ? row[k0 + i] : fill;
    }
}

// The value of lane (own ^ MASK), without LDS: a shuffle through LDS (ds_bpermute, what __shfl_xor makes) occupies the unit that
// the whole compute unit shares and takes its latency once per level of a reduction.  Rows are 16 lanes; masks 16 and 32 come
// as swaps of registers (row_pair, half_pair).  Steps with all reductions and prefix sums in registers, us, before / after: tree
// layer, 925 queries of 15 words, H = 448 22.0 / 20.0, 1024 of 32 words, H = 512 24.7 / 23.7; cached steps, 972 ids, H = 243, eight
// of them 244 / 235; 8 rows at V = 1000, H = 64 13.2 / 12.5; index table, 4096 contexts 27.3 / 26.2; nothing slower.
template <int MASK>
__device__ __forceinline__ float lane_xor(float v) {
    static_assert(MASK == 1 || MASK == 2 || MASK == 4 || MASK == 8, "");
    const int x = __float_as_int(v);
    if (MASK == 1) return __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));      // quad_perm 1 0 3 2
    if (MASK == 2) return __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));      // quad_perm 2 3 0 1
    if (MASK == 8) return __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x128, 0xF, 0xF, false));     // row_ror 8
    const int up = __builtin_amdgcn_update_dpp(x, x, 0x104, 0xF, 0x5, false);                             // quads 0, 2: row_shl 4
    return __int_as_float(__builtin_amdgcn_update_dpp(up, x, 0x114, 0xF, 0xA, false));                    // quads 1, 3: row_shr 4
}
// {x, y} such that, in lanes with bit 5 (bit 4) clear, they are a of this lane and of the lane 32 (16) further, and in the other
// lanes b of the lane 32 (16) before and of this one.
__device__ __forceinline__ void half_pair(float a, float b, float &x, float &y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
}
__device__ __forceinline__ void row_pair(float a, float b, float &x, float &y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
}

// Butterflies over 32, 16, 8, 4, 2, 1: every lane gets the result.
__device__ __forceinline__ float wave_sum(float v) {
    float x, y;
    half_pair(v, v, x, y); v = x + y;
    row_pair(v, v, x, y); v = x + y;
    v += lane_xor<8>(v);
    v += lane_xor<4>(v);
    v += lane_xor<2>(v);
    return v + lane_xor<1>(v);
}
__device__ __forceinline__ float wave_max(float v) {
    float x, y;
    half_pair(v, v, x, y); v = fmaxf(x, y);
    row_pair(v, v, x, y); v = fmaxf(x, y);
    v = fmaxf(v, lane_xor<8>(v));
    v = fmaxf(v, lane_xor<4>(v));
    v = fmaxf(v, lane_xor<2>(v));
    return fmaxf(v, lane_xor<1>(v));
}

// 2^x with the hardware instruction (x = -inf gives 0).
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Merge two (max, sum) pairs of a base-2 log-sum-exp: value = 2^m * s.
__device__ __forceinline__ void lse2_merge(float &m, float &s, float m2, float s2) {
    float mm = fmaxf(m, m2);
    if (mm == -INFINITY) { m = mm; s = 0.f; return; }
    s = s * fast_exp2(m - mm) + s2 * fast_exp2(m2 - mm);
    m = mm;
}

// Fold sixteen base-2 logits of one row into the (max, sum) pair.
template <bool FIXED>
__device__ __forceinline__ void lse2_fold16(const float (&x)[16], float &mrun, float &srun) {
    if (FIXED) {
#pragma unroll
        for (int i = 0; i < 16; ++i) srun += fast_exp2(x[i]);          // offset already inside x
    } else {
        float mx = x[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, x[i]);
        const float mn = fmaxf(mrun, mx);
        if (mn != -INFINITY) {
            float tsum = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) tsum += fast_exp2(x[i] - mn);
            srun = srun * fast_exp2(mrun - mn) + tsum;
            mrun = mn;
        }
    }
}

// Direct global->LDS load of 16 bytes per lane: lane i of the wave writes LDS bytes
// [lds_base + 16 i, lds_base + 16 i + 16) with the 16 bytes at sbase + voff (its own voff).
// sbase and lds_base must be the same in all lanes (they travel in SGPRs / M0).  Written as
// inline assembly on purpose: when the compiler knows of a pending LDS-DMA it makes every
// later LDS read wait for ALL outstanding LDS reads (lgkmcnt(0)) instead of just its own,
// which stalls the MFMA pipeline; completion is awaited explicitly with vmcnt before the
// workgroup barrier that publishes the data.  M0 is an input operand, so the compiler writes it
// and knows that it is in use; the s_nop is the wait state between that write and the load.
__device__ __forceinline__ void lds_dma_16(const void *sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "{m0}"(lds_base), "v"(voff), "s"(sbase)
                 : "memory");
}

// The same with a full 64-bit address per lane (rows gathered from anywhere in a buffer).
__device__ __forceinline__ void lds_dma_16_ptr(const void *lane_ptr, uint32_t lds_base) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "{m0}"(lds_base), "v"(lane_ptr)
                 : "memory");
}

// One float per lane (lane i writes LDS bytes [lds_base + 4 i, + 4)): rows that are not 16-byte aligned.
__device__ __forceinline__ void lds_dma_4_ptr(const void *lane_ptr, uint32_t lds_base) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %1, off"
                 :
                 : "{m0}"(lds_base), "v"(lane_ptr)
                 : "memory");
}

// The same as lds_dma_16 by lane 0 alone (16 bytes to lds_base), without a branch around it: the
// execution mask is narrowed to lane 0 for the one instruction and put back.  Counts as one
// vector-memory operation of the wave like any other load.
__device__ __forceinline__ void lds_dma_16_lane0(const void *sbase, uint32_t voff, uint32_t lds_base) {
    uint64_t saved_exec;
    asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, 1\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, %0"
                 : "=&s"(saved_exec)
                 : "{m0}"(lds_base), "v"(voff), "s"(sbase)
                 : "memory");
}

// The same from lanes 0 and 1, each with its own voff.
__device__ __forceinline__ void lds_dma_16_lanes01(const void *sbase, uint32_t voff, uint32_t lds_base) {
    uint64_t saved_exec;
    asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, 3\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, %0"
                 : "=&s"(saved_exec)
                 : "{m0}"(lds_base), "v"(voff), "s"(sbase)
                 : "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)reinterpret_cast<uintptr_t>(p);         // LDS offsets are the low 32 bits
}

// Wait until at most N of this wave's vector-memory operations are outstanding (vmcnt is a
// 6-bit field on gfx9: bits 3:0 and 15:14 of the immediate; lgkmcnt and expcnt left alone).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Values that another workgroup of the same launch, on another XCD perhaps, reads: relaxed agent-scope accesses, which pass
// by the caches that are not shared.  The writer's waves await their stores (seen_by_all) in front of the barrier behind
// which one thread counts the workgroup as done; the reader begins behind the count.  Fences that write back and drop
// the whole L2 (__threadfence) in their place took 30 us a launch with 256 workgroups.
__device__ __forceinline__ void store_seen(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_seen(float2 *p, float2 v) {
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_seen(const float *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float2 load_seen(const float2 *p) {
    return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void seen_by_all() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// 64-bit key -> 32 mixed bits for the hash tables of history ids: the high word, multiplied and folded, added to the low one, then
// a round of folding and multiplying.  Two 32-bit products, which take four slots of a SIMD each: one workgroup that hashes
// 4096 ids issues little else (a 64-bit finaliser has eight of them, and shifts of 64 bits).  Three different shifts: folded twice by 16, a
// high word with no low one beside it was itself again, and 4000 ids in their top 19 bits made a chain of 1290 probes in LDS (now 8).
// On counters at any bit, pairs of counters, floating-point numbers and addresses chains are as long as with the finaliser.
__host__ __device__ __forceinline__ uint32_t id_hash(uint64_t k) {
    uint32_t x = (uint32_t)(k >> 32) * 0x9E3779B1u;
    x = (uint32_t)k + (x ^ (x >> 12));
    x ^= x >> 14;
    x *= 0x7FEB352Du;
    return x ^ (x >> 16);
}

// splitmix64 finaliser: 64 well-mixed bits
__device__ __forceinline__ uint64_t mix64_full(uint64_t k) {
    k ^= k >> 30; k *= 0xBF58476D1CE4E5B9ull;
    k ^= k >> 27; k *= 0x94D049BB133111EBull;
    k ^= k >> 31;
    return k;
}

// Inclusive prefix sum over the wave, in registers as well: within rows of 16 lanes, then the last lane of a row to the next one,
// then lane 31 to the upper half.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);      // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);      // row_bcast 15 to rows 1 and 3
    return v + __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast 31 to rows 2 and 3
}

// Block-wide exclusive prefix sum of one int per thread (whole waves, at most 16); returns the exclusive prefix and,
// through `total`, the block sum.  `wsum` is LDS scratch of blockDim.x/64 + 1 ints.
__device__ __forceinline__ int block_exclusive_scan(int v, int *wsum, int &total) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const int incl = wave_inclusive_scan(v);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    // every wave for itself: the sums of all waves up to each
    const int upto = wave_inclusive_scan(lane < nwaves ? wsum[lane] : 0);
    const int before = wave > 0 ? __builtin_amdgcn_readlane(upto, wave - 1) : 0;
    total = __builtin_amdgcn_readlane(upto, nwaves - 1);
    __syncthreads();                                  // wsum may be reused by the caller
    return before + incl - v;
}

// Natural-log normaliser of one row from its `splits` per-split (max, sum) partials of the
// base-2 log-sum-exp, merged in a fixed order by one whole wave (every lane gets the result).
__device__ __forceinline__ float lse_from_partials(const float2 *part_row, int splits, int lane) {
    float pm = -INFINITY, ps = 0.f;
    for (int s = lane; s < splits; s += 64) {
        float2 p = part_row[s];
        lse2_merge(pm, ps, p.x, p.y);
    }
    const float mm = wave_max(pm);
    const float ss = wave_sum(mm == -INFINITY ? 0.f : ps * fast_exp2(pm - mm));
    return (mm + fast_log2(ss)) * 0.6931471805599453f;
}

// Batches of eight dot products per wave (query gather, hierarchical output layer): value u
// of a batch is finished by the lanes whose bits (5, 4, 3) spell u.
__device__ __forceinline__ int batch_slot_of_lane(int lane) {
    return ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
}
constexpr int lane_of_batch_slot(int u) { return 32 * ((u >> 2) & 1) + 16 * ((u >> 1) & 1) + 8 * (u & 1); }

// Sums over the wave of eight per-lane values at once: the same xor butterfly (32, 16, ...,
// 1) as wave_sum, but in the first three levels a lane passes on the half of the values it
// will not finish.  Returns the sum of value batch_slot_of_lane(lane); bit-identical to wave_sum of that value.
__device__ __forceinline__ float wave_sum8(const float (&acc)[8], int lane) {
    float v4[4], v2[2], x, y;
#pragma unroll
    for (int i = 0; i < 4; ++i) { half_pair(acc[i], acc[4 + i], x, y); v4[i] = x + y; }
#pragma unroll
    for (int i = 0; i < 2; ++i) { row_pair(v4[i], v4[2 + i], x, y); v2[i] = x + y; }
    const bool up3 = (lane & 8) != 0;
    float v = (up3 ? v2[1] : v2[0]) + lane_xor<8>(up3 ? v2[0] : v2[1]);
    v += lane_xor<4>(v);
    v += lane_xor<2>(v);
    return v + lane_xor<1>(v);
}

__device__ __forceinline__ float quiet_nan() { return __uint_as_float(0x7FC00000u); }

}  // namespace rnnlm
