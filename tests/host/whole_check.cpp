// Host-side check of the hidden update's whole form, run by tests/test_host_plan.py with the built library: every launch that
// recur_whole_units (linked from there) hands it has a kernel, and every kernel has a launch.  Prints "ok" or what is wrong.
#include <stdio.h>
#include <string.h>

#include <set>
#include <tuple>

#include "rnnlm_internal.h"

using namespace rnnlm;

int main() {
    std::set<std::tuple<bool, int, int, bool, bool>> met, made;
    for (bool bf16 : {true, false}) {
        const int dtype = bf16 ? RNNLM_BF16 : RNNLM_F32;
        for (int Hp = 64; Hp <= 2048; Hp += 64) {
            ModelDev m;
            memset(&m, 0, sizeof m);
            m.H = m.Hp = Hp;
            m.dtype = dtype;
            if (recur_whole_supported(dtype, Hp)) m.Wops = reinterpret_cast<const void *>(0x1000);
            for (bool vec : {true, false})
                for (bool grouped : {true, false})
                    for (int rows = 1; rows <= 9000; ++rows) {
                        if (grouped && !recur_groups_ids(m, rows)) break;
                        const int units = recur_whole_units(m, rows, vec, grouped);
                        if (units == 0) continue;
                        if (units != 32 && units != 64) return printf("FAILED %d units\n", units), 1;
                        // the form for few units comes first: in one round, models it takes for any number of rows
                        const bool one_round = (Hp / 32) * ((rows + 31) / 32) <= kChipGroups;
                        if (!grouped && one_round && (bf16 ? Hp == 128 && !vec : Hp <= 256 || vec || rows <= 16)) continue;
                        const int top = recur_whole_top(Hp);
                        // (a kernel requests the weights of all k-steps up to its largest size)
                        if (top < Hp || top >= Hp + 128) return printf("FAILED Hp %d: kernels up to %d\n", Hp, top), 1;
                        if (!recur_whole_exists(bf16, top, units, vec, grouped))
                            return printf("FAILED %s Hp %d rows %d vec %d grouped %d: no kernel with %d units\n", bf16 ? "bf16" : "fp32", Hp, rows, vec, grouped, units), 1;
                        met.insert({bf16, top, units, vec, grouped});
                    }
        }
        for (int Hp = 64; recur_whole_supported(dtype, Hp); Hp += 64)
            for (int units : {32, 64})
                for (bool vec : {true, false})
                    for (bool grouped : {true, false})
                        if (recur_whole_exists(bf16, recur_whole_top(Hp), units, vec, grouped)) made.insert({bf16, recur_whole_top(Hp), units, vec, grouped});
    }
    for (const auto &k : made)
        if (!met.count(k))
            return printf("FAILED %s up to %d, %d units, vec %d, grouped %d: nothing reaches it\n", std::get<0>(k) ? "bf16" : "fp32", std::get<1>(k), std::get<2>(k), std::get<3>(k),
                          std::get<4>(k)), 1;
    printf("ok\n");
    return 0;
}
