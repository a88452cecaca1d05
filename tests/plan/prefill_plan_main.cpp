// CPU check of the column sweep's decomposition (csrc/prefill_plan.hpp): for every number of tiles that the valid vision
// rows and the text lengths can leave of a plan, no block of the run is empty, every unit lies in the block that
// unit_block names, and no tile is cut into more pieces than the workspace holds.
#include <stdio.h>
#include <initializer_list>

#include "../../paper_2411_10803_amd/csrc/prefill_plan.hpp"

using namespace md;

int main() {
    long plans = 0, runs = 0, bad = 0;
    const int more_heads[] = {20, 24, 32, 40, 64, 96, 127, 128};
    for (int N : {1, 32, 33, 64, 65, 128, 129, 300, 1024})
        for (int Mv : {1, 64, 65, 144, 576, 900, 2047})
            for (int B : {1, 2, 3, 13})
                for (int hi = 1; hi <= 16 + 8; ++hi) {
                    const int H = hi <= 16 ? hi : more_heads[hi - 17];
                    const ScorePlan s = plan_scores(B, Mv, N, H, 128);
                    const ColPlan& c = s.col;
                    const long all = c.U / H;
                    ++plans;
                    for (long tiles = 1; tiles <= all; tiles += all <= 300 ? 1 : 1 + all / 300) {
                        const ColRun r = effective_run((int)tiles, H, c);
                        ++runs;
                        const char* why = nullptr;
                        if (r.U != tiles * H || r.P < 1 || r.P > c.P) why = "blocks";
                        for (long p = 0; p < r.P && !why; ++p) {
                            const long u0 = index_div(p * r.U, r.P), u1 = index_div((p + 1) * r.U, r.P);
                            if (u0 >= u1) why = "an empty run";
                            else if (unit_block(u0, r.P, r.U) != p || unit_block(u1 - 1, r.P, r.U) != p) why = "a unit's block";
                        }
                        for (long t = 0; t < tiles && !why; ++t)
                            if (unit_block(t * H + H - 1, r.P, r.U) - unit_block(t * H, r.P, r.U) + 1 > c.Gmax) why = "pieces";
                        if (why && ++bad <= 10)
                            printf("B=%d Mv=%d N=%d H=%d: %ld of %ld tiles, P=%d of %d, Gmax=%d: %s\n", B, Mv, N, H, tiles, all, r.P, c.P, c.Gmax, why);
                    }
                }
    printf("%ld plans, %ld runs, %ld wrong\n", plans, runs, bad);
    return bad != 0;
}
