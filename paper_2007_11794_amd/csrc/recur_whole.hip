// Hidden update, launches in the whole form: see recur_whole.h.
#include <algorithm>
#include <type_traits>

#include "recur_whole.h"

namespace rnnlm {

namespace {

// GROUP: the launch groups the `rows` raw queries' ids first, the weights on their way meanwhile.  (The rows as well, as if no id came
// twice, and again where one did: nothing gained where none does, 0.3 to 0.5 us lost where some do.)
template <typename WT, int UNITS, int UB, bool VEC, bool GROUP>
__global__ __launch_bounds__(kRecurThreads) void recur_whole_kernel(
    ModelDev m, int rows, const int *__restrict__ B_dev, const int32_t *__restrict__ row_src, const int32_t *__restrict__ row_dst,
    const int32_t *__restrict__ prev_word, const float *__restrict__ h_in, float *__restrict__ h_out, IdGroups ids) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    __shared__ int wsum[kRecurThreads / 64 + 1];
    // the arguments fetched together, not one by one where they are used
    asm volatile("" ::"s"(m.Wops), "s"(m.U), "s"(m.half_rowsum_W), "s"(m.d), "s"(m.dfrag), "s"(m.Hp), "s"(m.H), "s"(m.V), "s"(prev_word), "s"(h_in), "s"(h_out), "s"(row_dst));
    // Workgroup id modulo 8 is the XCD (L2 domain): a row block runs on one of them with all its blocks of units.
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds, J = m.Hp / (32 * UB);
    RecurWhole<WT, UNITS, UB, VEC> t((xcd + kXcds * (local / J)) * 32, local % J * (32 * UB));
    int B, source = min(t.b0 + t.col, rows - 1);
    if constexpr (GROUP) {
        const int *rep;
        B = __builtin_amdgcn_readfirstlane(group_ids(ids, rows, lds, wsum, rep, [&]() { t.request_weights(m); }));
        if (t.b0 >= B) return;
        source = rep[min(t.b0 + t.col, B - 1)];
        __syncthreads();                                                 // the tables are read
    } else {
        if (row_src) source = row_src[source];
        B = B_dev ? *B_dev : rows;
        if (t.b0 >= B) return;
        __builtin_amdgcn_sched_barrier(0);                               // (loads are awaited in order)
        t.request_weights(m);
        if (row_src && B - t.b0 < 32) source = __shfl(source, min(t.lane & 31, B - 1 - t.b0), 64);   // entries from B on are stale
    }
    t.request_rows(m, prev_word, h_in, source, B);
    t.run(m, B, row_dst, h_in, h_out, lds);
}

template <typename WT, int UNITS, int UB, bool VEC, bool GROUP>
hipError_t launch(const ModelDev &m, int rows, const int *B_dev, const int32_t *row_src, const int32_t *row_dst, const int32_t *prev_word,
                  const float *h_in, float *h_out, const IdGroups &ids, hipStream_t stream) {
    static LdsLimit limit;
    const auto kernel = recur_whole_kernel<WT, UNITS, UB, VEC, GROUP>;
    const int bytes = std::max(RecurWhole<WT, UNITS, UB, VEC>::lds_bytes(m.Hp), GROUP ? kGroupLdsBytes : 0);
    if (hipError_t e = limit.ensure(reinterpret_cast<const void *>(kernel), bytes); e != hipSuccess) return e;
    const int blocks = (rows + 31) / 32;
    hipLaunchKernelGGL(kernel, dim3(kXcds * ((blocks + kXcds - 1) / kXcds) * (m.Hp / (32 * UB))), dim3(kRecurThreads), bytes, stream, m, rows, B_dev, row_src,
                       row_dst, prev_word, h_in, h_out, ids);
    return hipGetLastError();
}

template <typename WT, int UNITS>
hipError_t launch_units(const ModelDev &m, bool wide, bool vec, int rows, const int *B_dev, const int32_t *row_src, const int32_t *row_dst,
                        const int32_t *prev_word, const float *h_in, float *h_out, const IdGroups &ids, hipStream_t stream) {
    auto go = [&](auto ub, auto aligned, auto group) -> hipError_t {
        constexpr int UB = decltype(ub)::value;
        constexpr bool VEC = decltype(aligned)::value, GROUP = decltype(group)::value;
        if constexpr (recur_whole_exists(sizeof(WT) == 2, UNITS, 32 * UB, VEC, GROUP))
            return launch<WT, UNITS, UB, VEC, GROUP>(m, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out, ids, stream);
        else return hipErrorInvalidValue;
    };
    auto with_group = [&](auto ub, auto aligned) { return ids.key ? go(ub, aligned, std::true_type{}) : go(ub, aligned, std::false_type{}); };
    auto with_rows = [&](auto ub) { return vec ? with_group(ub, std::true_type{}) : with_group(ub, std::false_type{}); };
    return wide ? with_rows(std::integral_constant<int, 2>{}) : with_rows(std::integral_constant<int, 1>{});
}

}  // namespace

bool recur_whole_supported(int dtype, int Hp) { return Hp <= (dtype == RNNLM_BF16 ? 1024 : 512); }

// 32 units a workgroup while those fit the compute units in one round (more of them at work, a shorter chain), then 64, bf16 models of up to 512
// units two of those side by side: replayed steps, hierarchical layer, us, ring / this: H = 256, 3000, 4096 rows 14.0 / 13.2, 15.4 / 14.6; H = 400, 1100,
// 2048 14.2 / 13.5, 15.4 / 14.8; H = 320, 1600 12.9 / 12.9.  The ring stays for more rows; for few units behind a grouping, which is the longer
// part then (bf16, Hp = 128, 40 ids 10.5 / 10.7, 300 11.1 / 11.1; fp32, Hp = 64, 40 of 12 distinct 10.1 / 10.3); and for unaligned
// rows with 64 units a workgroup (H = 333, 1024 rows 13.2 / 13.4) unless the ring's chunks are many (H = 650 above).
int recur_whole_units(const ModelDev &m, int rows, bool vec, bool grouped) {
    if (!m.Wops || (!vec && m.H < 4)) return 0;
    if (grouped && m.Hp <= (m.dtype == RNNLM_BF16 ? 128 : 64)) return 0;
    const int blocks = kXcds * ((rows + 32 * kXcds - 1) / (32 * kXcds));
    if (blocks * (m.Hp / 32) <= kChipGroups) return 32;
    if (!vec && m.Hp <= 512) return 0;
    return blocks * (m.Hp / 64) <= (m.dtype == RNNLM_BF16 && m.Hp <= 512 ? 2 : 1) * kChipGroups ? 64 : 0;
}

hipError_t launch_recur_whole(const ModelDev &m, int units, bool vec, int rows, const int *B_dev, const int32_t *row_src, const int32_t *row_dst,
                              const int32_t *prev_word, const float *h_in, float *h_out, const IdGroups &ids, hipStream_t stream) {
    auto go = [&](auto fn) { return fn(m, units == 64, vec, rows, B_dev, row_src, row_dst, prev_word, h_in, h_out, ids, stream); };
    if (m.dtype == RNNLM_BF16) {
        switch (recur_whole_top(m.Hp)) {
            case 128: return go(launch_units<bf16_t, 128>);
            case 256: return go(launch_units<bf16_t, 256>);
            case 384: return go(launch_units<bf16_t, 384>);
            case 512: return go(launch_units<bf16_t, 512>);
            case 640: return go(launch_units<bf16_t, 640>);
            case 768: return go(launch_units<bf16_t, 768>);
            case 896: return go(launch_units<bf16_t, 896>);
            case 1024: return go(launch_units<bf16_t, 1024>);
            default: return hipErrorInvalidValue;
        }
    }
    switch (recur_whole_top(m.Hp)) {
        case 128: return go(launch_units<float, 128>);
        case 256: return go(launch_units<float, 256>);
        case 384: return go(launch_units<float, 384>);
        case 512: return go(launch_units<float, 512>);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rnnlm
