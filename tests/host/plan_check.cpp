// Host-side check of the work-split arithmetic the output-projection kernels and the kernels behind
// them share (plan_rows, splits_of in the library's internal header): compiled for the host only and
// run by tests/test_host_plan.py.  Prints "ok" or the first violated property.
#include <stddef.h>
#include <stdio.h>

#include <vector>

#include "rnnlm_internal.h"

using namespace rnnlm;

#define REQUIRE(cond, ...)                       \
    do {                                         \
        if (!(cond)) {                           \
            printf("FAILED %s: ", #cond);        \
            printf(__VA_ARGS__);                 \
            printf("\n");                        \
            return 1;                            \
        }                                        \
    } while (0)

int main() {
    const int group_rows_of[] = {128, 256}, wg_of[] = {1, 4, 32, 64}, cap_of[] = {1, 2, 5, 10, 32, 40, 1000};
    for (int group_rows : group_rows_of)
        for (int wg : wg_of)
            for (int cap : cap_of)
                for (int B = 0; B <= 6000; B += (B < 700 ? 1 : 37)) {
                    const RowPlan p = plan_rows(B, group_rows, wg, cap);
                    REQUIRE(p.RG >= 1 && (long long)p.RG * group_rows >= B, "B=%d rows=%d: RG=%d", B, group_rows, p.RG);
                    REQUIRE(B <= group_rows || (p.RG - 1) * group_rows < B, "B=%d rows=%d: RG=%d too many", B, group_rows, p.RG);
                    REQUIRE(p.Sx >= 1 && p.Sx <= cap && p.Sx <= kMaxSplits / kXcds, "B=%d wg=%d cap=%d: Sx=%d", B, wg, cap, p.Sx);
                    REQUIRE(p.S == kXcds * p.Sx && p.S <= kMaxSplits, "S=%d Sx=%d", p.S, p.Sx);
                    // the items of an XCD fit its workgroups in one round whenever they can
                    REQUIRE(p.RG * p.Sx <= wg || p.Sx == 1, "B=%d wg=%d: RG=%d Sx=%d", B, wg, p.RG, p.Sx);
                    // what the kernel behind derives is what the output projection used
                    const SplitInfo si = {0, wg, group_rows, cap, 0};
                    REQUIRE(splits_of(si, B) == p.S, "B=%d: splits_of=%d S=%d", B, splits_of(si, B), p.S);
                    // a kernel that streams the weights for few rows leaves one partial per workgroup
                    if (kXcds * wg <= kMaxSplits) {
                        const SplitInfo ss = {0, wg, group_rows, cap, 64};
                        const int s = splits_of(ss, B);
                        REQUIRE(s == ((B > 0 && B <= 64) ? kXcds * wg : p.S), "B=%d wg=%d: streamed splits %d", B, wg, s);
                        REQUIRE(s <= kMaxSplits, "B=%d: %d partials", B, s);
                    }
                }
    for (int S = 1; S <= kMaxSplits; ++S)
        for (int B = 0; B < 3000; B += 97) REQUIRE(splits_of(fixed_split_info(S), B) == S, "fixed S=%d B=%d", S, B);
    // the staged kernel's plan: 256 rows per group, every group gets the same number of splits
    for (int B = 1; B <= 5000; ++B) {
        const StagedPlan p = staged_plan(B, 32);
        REQUIRE(p.RG == (B + kStagedRows - 1) / kStagedRows && p.S == kXcds * p.Sx, "staged B=%d", B);
    }
    // the finer splits of groups of 128 rows: kernel and reader agree, partials fit, and no number of splits is better by the rule's own
    // count (the busy part of the rounds that the items take, in 48ths, less five for every round behind the first) where it may choose
    for (int Vp : {256, 16384 - 256, 16384, 65536, 1000192})
        for (int B = 1; B <= 14000; ++B) {
            const RowPlan p = plan_rounds(B, 128, 32, Vp), one = plan_rows(B, 128, 32, kMaxSplits / kXcds);
            const SplitInfo si = {0, 32, -128, Vp, 0, 0};
            REQUIRE(splits_of(si, B) == p.S && p.S == kXcds * p.Sx && p.Sx >= 1 && p.S <= kMaxSplits, "B=%d Vp=%d: S=%d, reader %d", B, Vp, p.S, splits_of(si, B));
            REQUIRE(p.RG == one.RG, "B=%d Vp=%d: RG=%d", B, Vp, p.RG);
            if (p.RG < 5 || Vp < 16384) {
                REQUIRE(p.Sx == one.Sx, "B=%d Vp=%d: Sx=%d", B, Vp, p.Sx);
                continue;
            }
            auto rounds = [&](int Sx) { return (p.RG * Sx + 31) / 32; };
            auto busy = [&](int Sx) { return 48 * p.RG * Sx / (32 * rounds(Sx)) - 5 * (rounds(Sx) - 1); };
            for (int Sx = 1; Sx <= kMaxSplits / kXcds && rounds(Sx) <= 3; ++Sx)
                REQUIRE(busy(p.Sx) >= busy(Sx), "B=%d Vp=%d: Sx=%d keeps %d of 48 busy, Sx=%d %d", B, Vp, p.Sx, busy(p.Sx), Sx, busy(Sx));
        }
    // cutting `units` blocks into `parts` splits: the 32-bit form equals floor(index * units / parts)
    const int units_of[] = {1, 7, 63, 64, 255, 256, 257, 2048, 6250, 31251, 1 << 20, (1 << 25) + 3, 0x7FFFFFFF};
    for (int units : units_of)
        for (int parts = 1; parts <= kMaxSplits; ++parts)
            for (int index = 0; index <= parts; ++index) {
                const long long want = ((long long)index * units) / parts;
                REQUIRE(part_begin(index, units, parts) == (int)want, "part_begin(%d, %d, %d) = %d, want %lld", index, units,
                        parts, part_begin(index, units, parts), want);
            }
    // what a launch reads ahead of a streaming one: inside the workgroup's own share, every piece once, all of them in the end
    const int blocks_of[] = {256, 257, 2047, 2048, 6250, 31250}, hp_of[] = {64, 128, 192, 512, 704, 1024};
    for (int blocks : blocks_of)
        for (int hp : hp_of)
            for (int form = 0; form < 3; ++form) {               // bf16, fp32 with eight waves and with four
                const WeightsAhead a = {nullptr, blocks, hp / 16 * (form ? 2 : 1), kMaxSplits, form == 2 ? 4 : 8};
                for (int split : {0, 1, 100, 255}) {
                    const int b0 = part_begin(split, blocks, kMaxSplits), b1 = part_begin(split + 1, blocks, kMaxSplits);
                    const int rounds = (b1 - b0 + a.waves - 1) / a.waves, pieces = rounds * a.waves * (a.block_kb / 4);
                    std::vector<int> seen((size_t)(b1 - b0) * (a.block_kb / 4));
                    for (int piece = 0; piece < pieces + 40; ++piece) {
                        const long long at = ahead_piece(a, split, piece);
                        if (at < 0) continue;
                        REQUIRE(at % 4 == 0 && at >= (long long)b0 * a.block_kb && at + 4 <= (long long)b1 * a.block_kb, "blocks=%d hp=%d split=%d: %lld",
                                blocks, hp, split, at);
                        REQUIRE(++seen[(size_t)(at / 4 - (long long)b0 * (a.block_kb / 4))] == 1, "blocks=%d hp=%d split=%d: %lld twice", blocks, hp, split, at);
                    }
                    for (int n : seen) REQUIRE(n == 1, "blocks=%d hp=%d split=%d: a piece is left out", blocks, hp, split);
                }
            }
    // the model as an argument of the kernels: what the hidden update asks for first in the first line, nothing in lines further on than it has to be
    REQUIRE(offsetof(ModelDev, half_rowsum_W) + sizeof(void *) <= 64, "half_rowsum_W at %d", (int)offsetof(ModelDev, half_rowsum_W));
    REQUIRE(sizeof(ModelDev) == 8 * sizeof(int) + 2 * 2 * sizeof(float) + 21 * sizeof(void *), "ModelDev has %d bytes", (int)sizeof(ModelDev));
    printf("ok\n");
    return 0;
}
