// Host-side check of what a cached step's lookup reads ahead (outproj_weights_ahead, linked from the built library), run by
// tests/test_host_plan.py: rounds of as many blocks of words as the workgroups of the launch behind it have waves, in every form
// that streams its weights for few rows.  Prints "ok" or the first model that is wrong.
#include <stdio.h>
#include <string.h>

#include "rnnlm_internal.h"

using namespace rnnlm;

int main() {
    const int rows_of[] = {1, 64, 65, 127, 128, 300, 1024, 4096}, choices[] = {0, 3, 4, 5};
    for (int dtype : {RNNLM_BF16, RNNLM_F32})
        for (int Hp = 64; Hp <= 2048; Hp += 64)
            for (int rows : rows_of)
                for (int fixed = 0; fixed < 2; ++fixed)
                    for (int choice : choices) {
                        if (choice == 4 && dtype == RNNLM_BF16) continue;
                        ModelDev m;
                        memset(&m, 0, sizeof m);
                        m.V = m.Vp = 65536;
                        m.H = m.Hp = Hp;
                        m.dtype = dtype;
                        m.Ot = m.Ofrag = reinterpret_cast<const void *>(0x1000);
                        if (dtype != RNNLM_BF16) m.ofac = reinterpret_cast<const float *>(0x1000);
                        const char *kernel = outproj_kernel_name(m, rows, fixed != 0, choice);
                        const WeightsAhead a = outproj_weights_ahead(m, rows, fixed != 0, choice);
                        int want = 0;                          // 0: nothing is read ahead
                        if ((size_t)m.Vp * Hp * (dtype == RNNLM_BF16 ? 2 : 4) > kAllL2s) {
                            if (strcmp(kernel, "outproj_stream_kernel") == 0 || strcmp(kernel, "outproj_rowstream_kernel") == 0) want = 8;
                            if (strcmp(kernel, "outproj_split2_kernel") == 0) want = 4;
                            if (strncmp(kernel, "outproj_staged", 14) == 0) want = staged_waves(dtype != RNNLM_BF16, Hp);
                        }
                        if ((a.splits > 0) != (want > 0) || (want > 0 && (a.waves != want || a.splits != kMaxSplits || a.block_kb * 1024 != 32 * Hp * (dtype == RNNLM_BF16 ? 2 : 4)))) {
                            printf("FAILED dtype %d Hp %d rows %d fixed %d choice %d (%s): %d waves in %d splits, blocks of %d KB; %d waves wanted\n", dtype, Hp, rows, fixed, choice,
                                   kernel, a.waves, a.splits, a.block_kb, want);
                            return 1;
                        }
                    }
    printf("ok\n");
    return 0;
}
