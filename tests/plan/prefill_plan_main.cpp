// CPU check of the column sweep's decomposition (csrc/prefill_plan.hpp): for every number of tiles that the valid vision
// rows and the text lengths can leave of a plan, no block of the run is empty, every unit lies in the block that
// unit_block names, and no tile is cut into more pieces than the workspace holds.  And of the sweep by single tiles: what it keeps
// in the memory of the pieces (V and I per text block, the statistics of more chunks than the workspace has room for)
// fits there, whichever head size the workspace was measured with and whatever a mask or the caller's normalisers change of the
// form, and it is taken where its kernels can.  And of the rules for the form that takes all text rows of a tile, for
// the loads of K in the first sweep and for the stores of the kept K rows.
#include <stdio.h>
#include <stdlib.h>
#include <initializer_list>
#include <random>

#include "../../paper_2411_10803_amd/csrc/prefill_plan.hpp"

using namespace md;

static const char* column_form(const ScorePlan& s) { return s.rows ? "rows" : s.own ? "tiles" : "persistent"; }

// With arguments B Mv N H d masked: the form of that one call.
int main(int argc, char** argv) {
    if (argc == 7) {
        int a[6];
        for (int i = 0; i < 6; ++i) a[i] = atoi(argv[1 + i]);
        const ScorePlan s = plan_scores(a[0], a[1], a[2], a[3], a[4], a[5] != 0);
        printf("%s", column_form(s));
        if (s.rs_wide) printf(" wide %d chunk%s", s.nch, s.nch == 1 ? "" : "s");
        printf(", with normalisers %s\n", column_form(with_normalisers(s)));
        return 0;
    }
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
    std::mt19937 rng(1);
    long own = 0, behind = 0, rows = 0, by_mask = 0;
    auto log_uniform = [&](int lo, int hi) {
        const double r = (double)rng() / 4294967296.0, lg = r * __builtin_log((double)(hi + 1) / lo);
        const int v = (int)(lo * __builtin_exp(lg));
        return v < lo ? lo : (v > hi ? hi : v);
    };
    for (int i = 0; i < 300000; ++i) {
        const int B = log_uniform(1, 200), Mv = log_uniform(1, 10000), N = log_uniform(1, 300), H = log_uniform(1, 128);
        const ScorePlan both[2] = {plan_scores(B, Mv, N, H, 64), plan_scores(B, Mv, N, H, 128)};
        const ScorePlan with_mask[2] = {plan_scores(B, Mv, N, H, 64, true), plan_scores(B, Mv, N, H, 128, true)};
        const long room = both[0].nch_ws > both[1].nch_ws ? both[0].nch_ws : both[1].nch_ws;          // as the workspace has it
        const char* why = nullptr;
        if (both[0].col.Gmax != both[1].col.Gmax || both[0].col.P != both[1].col.P || both[0].nbt != both[1].nbt) why = "sizes by head size";
        for (int m = 0; m < 8 && !why; ++m) {         // head size x mask x normalisers
            const ScorePlan& plain = both[m & 1];
            const ScorePlan s = m & 4 ? with_normalisers(m & 2 ? with_mask[m & 1] : plain) : m & 2 ? with_mask[m & 1] : plain;
            if (s.col.Gmax != plain.col.Gmax || s.col.P != plain.col.P || s.col.U != plain.col.U || s.col.kb != plain.col.kb || s.nbt != plain.nbt ||
                s.nch_ws != plain.nch_ws) why = "sizes by mask";
            if (s.rs_stream && (s.ng != 1 || s.rs_waves != 4 || s.rs_deep)) why = "streamed row statistics";
            if (m & 4 && s.nch != 1) why = "chunks with normalisers";
            if (s.rows && (!s.own || s.nbt > 2)) why = "all text rows of a tile";
            if (s.own && !s.rows && s.nbt == 1) why = "one text block in single tiles";
            by_mask += m < 4 && (m & 2) && s.rows != plain.rows;
            rows += s.rows;
            if (!s.own) {
                if (!(m & 4) && (s.partial_in_pieces || s.nch != s.nch_ws)) why = "chunks of the persistent form";
                continue;
            }
            ++own;
            const long Npad = 32l * s.nbt, pieces = (long)s.col.Gmax * B * Mv * Npad;                // floats
            const long scores = (s.nbt > 1 && !s.rows) || s.partial_in_pieces ? 2l * s.nbt * B * Mv : 0, stats = 2l * B * H * s.nch * Npad;
            if (s.ng != 1 || s.nbt > kOwnParts || Mv > 8192 || s.nch < 1 || s.nch > kOwnChunks || s.own_blocks != (long)B * ((Mv + 31) / 32) * s.nbt) why = "form";
            else if (scores > pieces) why = "scores";
            else if (m & 4) continue;                 // (one statistic per row, in memory of its own)
            else if (s.partial_in_pieces ? scores + stats > pieces : s.nch > room) why = "chunk statistics";
            behind += s.partial_in_pieces;
        }
        if (why && ++bad <= 10) printf("B=%d Mv=%d N=%d H=%d: %s\n", B, Mv, N, H, why);
    }
    // Blocks that take all text rows of a key tile: few heads as well as many, whole rounds of blocks and those that leave
    // little of the last one idle.  plan: without and with the caller's normalisers.
    struct { int B, Mv, N, H, d; bool masked, rows, rows_lse; } const forms[] = {
        {60, 576, 32, 12, 64, true, true, true}, {60, 576, 32, 8, 128, true, true, true}, {24, 1600, 60, 4, 128, true, true, true},
        {32, 576, 60, 12, 128, false, true, true}, {24, 576, 20, 4, 128, false, true, true},
        {16, 576, 60, 32, 128, true, true, true}, {8, 1085, 20, 32, 128, false, true, false}, {8, 2109, 20, 32, 128, false, true, false},
        {8, 2662, 20, 32, 128, false, true, true}, {8, 1843, 60, 32, 128, false, true, true}, {8, 2355, 60, 32, 128, false, false, false},
        {8, 3235, 60, 32, 128, false, false, false}, {24, 1600, 60, 32, 128, true, true, true}, {16, 2600, 60, 16, 128, true, false, true},
        {8, 2355, 60, 16, 128, false, true, true}, {16, 576, 60, 32, 64, false, false, true}, {4, 7000, 60, 32, 64, true, true, true},
        {4, 1000, 60, 32, 128, true, false, false}, {5, 8193, 20, 12, 64, true, false, false}, {1, 576, 20, 96, 64, false, false, false},
        {40, 1600, 20, 1, 128, true, true, true}, {200, 576, 20, 4, 128, true, false, false}, {64, 8000, 20, 4, 64, true, true, true},
        {2048, 128, 20, 4, 64, true, false, false}, {96, 576, 60, 2, 128, true, false, false}, {40, 1600, 60, 4, 128, true, true, true}};
    for (const auto& f : forms) {
        const ScorePlan s = plan_scores(f.B, f.Mv, f.N, f.H, f.d, f.masked);
        if ((s.rows != f.rows || with_normalisers(s).rows != f.rows_lse) && ++bad)
            printf("B=%d Mv=%d N=%d H=%d d=%d masked=%d: all text rows of a tile %d %d\n", f.B, f.Mv, f.N, f.H, f.d, f.masked, s.rows, with_normalisers(s).rows);
    }
    // which calls read K for the row statistics past the Infinity Cache: heads of 128, one text group and K well beyond the cache
    struct { int B, Mv, N, H, d; bool want; } const reads[] = {
        {24, 2880, 100, 32, 128, true}, {10, 3000, 100, 32, 128, true}, {8, 2880, 128, 32, 128, false}, {7, 9172, 113, 28, 64, false},
        {20, 2800, 40, 32, 128, true}, {12, 2880, 60, 32, 128, false}, {2, 18500, 32, 32, 128, false}, {3, 18500, 32, 32, 128, true}, {18, 1883, 10, 40, 128, false}, {2, 18700, 64, 32, 128, true},
        {8, 9161, 30, 33, 64, false}, {8, 9200, 48, 32, 64, false}, {6, 6000, 384, 32, 128, false}, {1, 1, 1, 1, 64, false}};
    for (const auto& r : reads)
        if (plan_scores(r.B, r.Mv, r.N, r.H, r.d).rs_stream != r.want && ++bad)
            printf("B=%d Mv=%d N=%d H=%d d=%d: K of the row statistics\n", r.B, r.Mv, r.N, r.H, r.d);
    // and for the column sweep: where sweep 1 leaves K in the cache and the copies read much of it again, and where several
    // text groups share it with few fragments
    struct { int B, Mv, N, H, d, Rcap; bool threshold, want, want_lse; } const again[] = {
        {16, 576, 128, 32, 128, 115, false, false, true}, {4, 2880, 120, 32, 128, 180, false, true, true}, {8, 2880, 128, 32, 128, 320, false, true, true},
        {8, 2880, 128, 32, 128, 576, false, false, true}, {8, 2880, 128, 32, 128, 2880, true, false, true}, {10, 2880, 100, 32, 128, 576, false, true, true},
        {8, 2000, 100, 40, 64, 200, false, false, true}, {8, 3000, 100, 40, 64, 300, false, true, true}, {1, 9000, 40, 32, 128, 3000, false, true, true}, {1, 9000, 20, 32, 128, 3000, false, true, true},
        {3, 4608, 300, 32, 128, 4608, true, false, false}, {6, 1152, 384, 32, 128, 10, false, false, false}, {20, 576, 200, 32, 128, 192, false, true, true}};
    for (const auto& r : again) {
        const ScorePlan s = plan_scores(r.B, r.Mv, r.N, r.H, r.d);
        auto streams = [&](const ScorePlan& p, bool lse) { return streams_col_k(p, r.B, r.Mv, r.H, r.d, r.Rcap, r.threshold, lse); };
        if ((streams(s, false) != r.want || streams(with_normalisers(s), true) != r.want_lse) && ++bad)
            printf("B=%d Mv=%d N=%d H=%d d=%d Rcap=%d: K of the column sweep\n", r.B, r.Mv, r.N, r.H, r.d, r.Rcap);
    }
    // which calls write the kept K rows past the Infinity Cache: not those whose next reader finds them there
    struct { int B, Mv, N, H, d, Rcap; bool threshold, k_streams, want; } const moves[] = {
        {16, 576, 64, 32, 128, 192, false, false, true}, {16, 192, 64, 32, 128, 128, false, false, false},       // successive layers
        {16, 128, 64, 32, 128, 64, false, false, false}, {4, 4608, 64, 32, 128, 512, false, false, true},
        {8, 2880, 128, 32, 128, 320, false, false, true}, {8, 2880, 128, 32, 128, 320, false, true, false},      // 29 MB
        {24, 1600, 30, 32, 128, 400, false, true, true}, {8, 576, 64, 32, 128, 192, false, false, false},
        {4, 576, 64, 32, 128, 576, true, false, false}, {12, 516, 12, 32, 128, 516, true, false, false}, {24, 576, 20, 32, 128, 576, true, true, false},
        {4, 6907, 110, 32, 128, 6907, true, true, true}, {14, 576, 64, 32, 128, 128, false, false, true}, {16, 576, 64, 32, 128, 128, false, true, false},
        {24, 516, 12, 32, 128, 516, true, false, true}, {4, 2880, 12, 32, 128, 360, false, false, true},         // few rows of large calls
        {16, 576, 64, 32, 128, 576, true, false, true}, {8, 2880, 64, 32, 128, 2880, true, false, true},
        {1, 1, 1, 1, 64, 1, true, true, false}, {1, 64, 1, 1, 64, 0, false, false, false}};
    for (const auto& m : moves)
        if (streams_k_out(m.B, m.Mv, m.N, m.H, m.d, m.H * m.d, m.Rcap, m.threshold, m.k_streams) != m.want && ++bad)
            printf("B=%d Mv=%d N=%d Rcap=%d threshold=%d K streams=%d: K rows out\n", m.B, m.Mv, m.N, m.Rcap, m.threshold, m.k_streams);
    if (!streams_k_out(4, 3000, 20, 34, 128, 8, 1000, false, false) && ++bad) printf("K rows out of the head-major test\n");
    if (own < 10000 || behind < 1000 || rows < 10000 || by_mask < 1000) { ++bad; printf("too few single tiles looked at\n"); }
    printf("%ld plans of single tiles, %ld with statistics behind the scores, %ld with all text rows of a tile, %ld so by the mask\n", own, behind, rows, by_mask);
    printf("%ld plans, %ld runs, %ld wrong\n", plans, runs, bad);
    return bad != 0;
}
