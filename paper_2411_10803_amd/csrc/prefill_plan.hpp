// How the two score sweeps of stage 2 are cut into blocks: host arithmetic for the launch and the workspace, and
// the part of it that the kernels repeat for the rows that matter.  Plain integer arithmetic without any HIP
// header, so that a CPU test can compile it and go through the shapes.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define MD_PLAN_FN __host__ __device__ __forceinline__
#else
#define MD_PLAN_FN inline
#endif

namespace md {
namespace {

constexpr int kMaxChunks = 16;                       // key chunks per (sample, head) in the row-statistics sweep, at most
constexpr int kNumCU = 256;                          // MI355X
constexpr int kOwnChunks = 4, kOwnParts = 4;         // key chunks that the sweep for single tiles merges, text blocks it takes apart

MD_PLAN_FN int text_blocks_of(int tl) { return (tl + 31) >> 5; }
MD_PLAN_FN int text_groups_of(int blocks, int nbw) { return (blocks + nbw - 1) / nbw; }

struct ColPlan { int P; long U; int nkg; int Gmax; int kb; int nbw; };   // kb: vision keys per unit (a power of two); nbw: text blocks

// n / d; the index arithmetic of the sweeps fits 32 bits at all but the largest sizes, and a 64-bit division is four
// times the instructions
MD_PLAN_FN long index_div(long n, long d) {
    return ((n | d) >> 32) == 0 ? (long)((uint32_t)n / (uint32_t)d) : n / d;
}
MD_PLAN_FN int unit_block(long u, int P, long U) { return (int)index_div((u + 1) * P - 1, U); }

// The same decomposition over what matters (SampleRows, one entry per sample; written by the kernel before this
// sweep): a sample has key_groups(vision) x text_groups(text_blocks) tiles, the text groups of a key group next to
// each other, so that the blocks that read the same K rows run side by side on one XCD.
// Fewer units than the host planned for means fewer blocks at work only where a tile would otherwise be cut into more
// pieces than the workspace holds (Gmax), and never more blocks than units: an empty run between two others would count
// as a piece of their tile that nobody writes.
MD_PLAN_FN int key_groups(int rows, int kb) { return (rows + kb - 1) / kb; }
struct ColRun { long U; int P; };
MD_PLAN_FN ColRun effective_run(int tiles, int H, ColPlan cp) {
    ColRun r;
    r.U = (long)tiles * H;
    long P = (long)(cp.Gmax - 1) * tiles;             // pieces per tile <= ceil(H*P/U) + 1 <= Gmax
    if (cp.Gmax >= H || P > cp.P) P = cp.P;           // (non-empty runs cut a tile's H units into H pieces at most)
    if (P > r.U) P = r.U;
    if (P >= 8) P &= ~7L;                             // whole rounds over the 8 XCDs
    if (P < 1) P = 1;
    r.P = (int)P;
    return r;
}

// Launch shapes of the two sweeps; pure host arithmetic shared by the workspace size and the launch.
struct ScorePlan {
    int nbt, nbw, ng;                                 // text blocks of 32 rows; those of one group; groups
    int nch, rs_waves;                                // sweep 1: key chunks per (sample, head, group), waves of a block
    bool rs_stream, rs_deep, rs_wide;                 // streaming loads of K; three LDS slots; the wide form
    bool own, own_lse, partial_in_pieces;             // sweep 2 by single tiles; so with normalisers; chunk statistics behind V and I
    int nch_ws;                                       // chunks that the workspace has room for
    long own_blocks;
    bool rows, rows_lse, rows_stream;                 // single tiles with all text rows; so with normalisers; streaming loads of K there
    ColPlan col;
    int occ;
};

// masked: the call has a validity mask.  (It decides about forms, not about sizes.)
inline ScorePlan plan_scores(int B, int Mv, int N, int H, int d, bool masked = false) {
    ScorePlan s;
    s.nbt = (N + 31) / 32;                            // 32-row text blocks
    s.nbw = s.nbt == 1 ? 1 : (s.nbt == 2 ? 2 : 4);    // text blocks per block, one per wave column
    s.ng = (s.nbt + s.nbw - 1) / s.nbw;               // text groups: each goes over K, side by side
    const double k_mb = (double)B * Mv * H * d * 2 / 1e6;
    // Sweep 1 reads K of heads of 128 with streaming loads where it outgrows the Infinity Cache and there is one text
    // group: from 230 MB on with 65 to 128 text rows, from 300 with 33 to 64, from 450 with fewer.  Plain loads leave part of K
    // to the second sweep, but on inputs that were just written they push the others' dirty lines out under the sweep.
    // us per call, plain / streaming, on three states in turn and on inputs just made: 100 to 128 rows 8 x 2880 keys of 40 heads
    // (236 MB) 176 / 187 and 218 / 192, 10 x 3000 (246) 178 / 185 and 220 / 193, 12 x 2880 (283) 197 / 207 and 224 / 211,
    // 16 x 2880 (377) 246 / 255 and 275 / 258, 24 x 2880 (566) 360 / 372 and 393 / 379; 40 to 60 rows 8 x 2880 (189) 120 / 125 and 143 /
    // 139, 12 x 2880 (283) 172 / 179 and 225 / 210, 14 x 2880 (330) 191 / 194 and 246 / 228, 16 x 2880 (377) 218 / 228 and 249 / 233,
    // 20 x 2800 (459) 287 / 285 and 314 / 305; 30 rows 24 x 1700 (334) 208 / 211 and 232 / 233, 24 x 2880 (566) 298 / 297 and 338 / 328,
    // 10 rows 18 x 1883 at 3/5, 40 heads (347) 221 / 230 and 237 / 247.  Several text groups go over K one after the other and
    // find it in the cache: 6 x 6000 (295), 384 rows 477 / 480 and 483 / 514, 10 x 3600 (295), 200 rows 325 / 345 and 357 / 382.
    // (Not of heads of 64: K of that size is rare there, and more code in the object costs the other calls: 8 x 2880 keys at 3/4,
    // 128 rows, 123.6 us, 125.0 with three more forms of the kernel, its own code being the same.)
    const bool big_k = s.ng == 1 && d == 128 && k_mb > (s.nbw == 1 ? 450.0 : s.nbw == 2 ? 300.0 : 230.0);
    // sweep 2: a persistent grid; units of (kb keys, one head), at least four per block
    ColPlan& c = s.col;
    c.kb = s.nbw == 1 ? 128 : 64;
    c.nkg = (Mv + c.kb - 1) / c.kb;
    c.nbw = s.nbw;
    c.U = (long)B * c.nkg * H * s.ng;
    // Blocks per CU: two where a block holds four text blocks (the second one covers the first one's waits), and with two
    // text blocks when the runs stay long enough (20 units per CU); otherwise one (fewer, longer runs: fewer pieces,
    // fewer prologues; measured faster there).
    s.occ = s.nbw == 4 || (s.nbw == 2 && c.U >= 20L * kNumCU) ? 2 : 1;
    // Units per block, at least: four; two where a single text block would leave most CUs idle.
    // us per call, four / two: 1 x 9000 keys, 28 text rows, 3 heads of 128 62.2 / 59.6, 2 x 9000, 1 head 66.3 / 62.8.  Of small images the
    // persistent form only takes those of very many heads, which lose by the sum of the pieces (1 x 512 keys, 64 heads 36.9 / 36.7,
    // 1 x 256, 127 heads 47.5 / 49.5); for all others this sizes the memory in which single tiles keep the statistics of their chunks.
    const long least = s.nbw == 1 && c.U < kNumCU ? 2 : 4;
    long P = (c.U + least - 1) / least;
    if (P > kNumCU * s.occ) P = kNumCU * s.occ;
    if (P < 1) P = 1;
    c.P = (int)P;
    // Pieces a key group can be cut into: sized for half the planned units (samples whose valid vision rows are a prefix of
    // their slots bring fewer key groups), beyond that fewer blocks work.
    c.Gmax = (int)((2L * H * c.P + c.U - 1) / c.U) + 1;
    if (c.Gmax > H) c.Gmax = H;
    // Sweep 2 by blocks of one tile (32 keys, 32 text rows, all heads): where they are no more than two rounds, of one block
    // per CU or, with heads of 64, of two; with the caller's normalisers one round, as K has not been read before.  The blocks of the
    // persistent form hand over their sums through memory and another launch, and leave most of the chip idle on small
    // calls; behind two rounds the query fragments, read for every 32 keys, come to more.
    // (Up to 64 text rows the form further down has taken these calls over where it may; it keeps the line of one text block.)
    // us per call, persistent / single tiles: 1 x 576 keys, 32 text rows 33 / 28, 128 rows 39 / 28; 14 x 576, 32 rows 64 / 57 (252
    // blocks), 28 x 576 118 / 111 (504), 2 x 1246, 114 rows, 16 heads 41 / 35 (312); heads of 64, 12 x 300, 20 rows 28 / 20,
    // 20 x 1000, 28 rows 84 / 72 (640).  Beyond: 4 x 4248, 25 rows 112 / 119 (532), 8 x 1955, 118 rows 144 / 183 (1984); heads of 64,
    // 3 x 7055, 92 rows 125 / 134 (1989).  With normalisers 23 x 181, 45 rows 50 / 54 (276).  (Of 26 calls of 257 to 512 blocks
    // 20 gain 2 to 15 %, none loses more than 1.5.)
    const long own_round = d == 64 ? 2l * kNumCU : kNumCU;
    s.own_blocks = (long)B * ((Mv + 31) / 32) * s.nbt;
    // And not of many heads on few tiles: a block takes in all heads one after the other on one CU, the persistent form
    // spreads them.  Heads of 64 count for 1 / 1.4.
    // us per call, persistent / single tiles, heads of 128: 1 x 576 keys, 32 text rows (18 blocks), 56 heads 37.3 / 36.8, 64 37.2 /
    // 38.0, 96 43.7 / 49.8, 128 49.3 / 58.9; 128 rows (72) 80 heads 50.6 / 47.8, 96 53.4 / 56.4; 6 x 576, 32 rows (108) 96 85.8 /
    // 85.2, 128 105.8 / 108.4; with normalisers 1 x 576, 32 rows 48 heads 31.1 / 31.0, 64 33.9 / 35.6; 4000 keys (125) 72 44.8 /
    // 43.4, 80 47.9 / 49.1.  Heads of 64, 18 blocks: 80 34.7 / 33.7, 96 34.9 / 36.5; 72 blocks 112 44.3 / 43.0.
    const double heads = d == 64 ? H / 1.4 : H;
    s.own = s.nbt <= kOwnParts && Mv <= 8192 && s.own_blocks <= 2 * own_round && heads <= 54 + 0.4 * s.own_blocks;
    s.own_lse = s.own && s.own_blocks <= own_round && heads <= 46 + 0.22 * s.own_blocks;
    // Up to 64 text rows: blocks of 32 keys that take all text rows and heads (prefill_colrows_kernel).  K is read once and
    // there is one (V, I) pair per key, but a block is long, and the CUs that the last round of blocks leaves idle
    // are what the form can lose by.  (With a mask four fifths of the slots are taken to be valid: stage 1 leaves three quarters.)
    // idle: that part of a round, times its length in heads.
    //
    // One text block: always; with the caller's normalisers (no first sweep, whose merge of chunks this form takes over)
    // where idle is at most 20.  Two: beyond one round of single tiles of one text block, where idle is at most 20 with
    // normalisers, else 16 in two rounds, 12 in three, 10 in four.  The bounds are a fit to what follows.  Heads of 64 share a CU
    // between two blocks, which evens the rounds out: they need only be beyond the two rounds of single tiles.
    // With fewer than 16 heads a block's start and end count for more than what it saves in many rounds: 6.5 rounds at most, 4.5 with
    // fewer than four heads and two text blocks; any number with heads of 64 and one text block, up to 1024 samples (every block
    // looks through all of them).
    //
    // us per call, persistent or single tiles / this form, 32 heads of 128 unless said otherwise:
    // one text block, 8 x 1085 keys (1.06 rounds) 60.1 / 60.4, 8 x 2918 (2.85) 126.7 / 120.8, 24 x 1600 at 4/5 192.6 / 181.3; with
    // normalisers 1.06 rounds 51.7 / 53.2, 1.4 61.4 / 58.9, 2.06 78.4 / 80.5, 2.85 99.5 / 94.2;
    // two, 16 x 576 at 4/5 75.6 / 66.0; 1.2 rounds 75.1 / 75.8, 1.6 88.7 / 86.3, 2.3 112.1 / 119.2, 2.85 133.4 / 134.8, 3.16 147.3 / 154.4,
    // 3.75 (24 x 1600 at 4/5) 228.0 / 211.4; 16 heads, 1.2 rounds 52.5 / 49.3, 2.6 79.8 / 75.2, 3.06 88.6 / 90.2, 4.1 at 4/5 115.1 /
    // 122.9; 8 heads, 3.4 rounds 76.4 / 70.6; with normalisers 1.2 rounds 61.7 / 64.7, 1.6 73.1 / 70.9, 2.06 86.1 / 90.8, 3.4 127.7 /
    // 124.5, 16 heads 2.06 57.9 / 58.1, 3.4 76.9 / 74.5; 4 x 1000 at 4/5 (128 tiles) 40.6 / 44.4;
    // heads of 64, two text blocks, 16 x 576 44.3 / 45.6, 24 x 900 89.9 / 84.4, 4 x 7000 at 4/5 97.0 / 88.8, 12 heads 60 x 576 66.1 / 60.9; with
    // normalisers 16 x 576 45.8 / 39.8, 24 x 1600 105.6 / 101.7;
    // few heads, one text block, 4 heads of 128: 80 x 576 (5.6 rounds) 56.3 / 48.3, 40 x 1600 at 4/5 (6.3) 63.5 / 58.5, 200 x 576 at 4/5 (11)
    // 108.5 / 114.4, 24 x 8000 (23) 152 / 159; 12 heads 40 x 1600 119 / 115, 24 x 8000 360 / 365; one head 40 x 1600 50.3 / 47.4, 64 x 8000
    // 185 / 246; two text blocks, 4 heads 40 x 1600 69.8 / 67.6, 64 x 2000 at 4/5 107 / 118, one head 4 x 8000 (3.9) 52.9 / 51.2, 96 x
    // 576 at 4/5 (5.4) 55.2 / 58.4; heads of 64, one text block, 4 heads 64 x 8000 at 4/5 234 / 211, 2048 x 128 439 / 437.
    const long tiles = (long)B * ((Mv + 31) / 32);
    const double rounds = (masked ? 0.8 : 1.0) * tiles / kNumCU;
    const long whole = (long)rounds + (rounds > (long)rounds ? 1 : 0);
    const double idle = (whole - rounds) * H;
    const double most = s.nbt == 1 || H >= 4 ? 6.5 : 4.5;
    const bool enough = H >= 16 || rounds <= most || (d == 64 && s.nbt == 1 && B <= 1024);
    s.rows = s.rows_lse = false;
    if (Mv <= 8192 && (s.nbt == 1 || (s.nbt == 2 && tiles > kNumCU / 2))) {
        s.rows = enough && heads <= 54 + 0.4 * tiles && (s.nbt == 1 || whole <= 1 || (d == 64 ? !s.own : idle <= 4.0 + 24.0 / whole));
        s.rows_lse = enough && heads <= 46 + 0.22 * tiles && (whole <= 1 || d == 64 || idle <= 20.0);
    }
    s.own |= s.rows;
    // There, K by streaming loads where it has not been read before and is more than 70 MB.
    // us per call, streaming / plain: with normalisers heads of 64, 16 x 1024 keys, 67 MB, 20 rows 41.8 / 40.6; 16 x 576 of 128, 75 MB,
    // 45.6 / 46.9, 4 x 2880, 94 MB, 57.3 / 62.4.  Behind a first sweep 24 x 1200, 236 MB, 60 rows 200.7 / 195.0, 16 x 1024 109.1 / 108.3.
    s.rows_stream = k_mb > 70.0;
    // Sweep 1: blocks of four waves (two per CU) or of eight (one per CU; the chunks two small blocks would take meet in
    // LDS), and the number of key chunks per (sample, head, text group), of at least four units of 128 keys.  Whole
    // rounds of blocks are what a shape can lose most by, so both are picked by an estimate of the time in us: a block's
    // start (5), the keys it takes (ns per key, from alone on the chip to every place taken), the merge of several chunks.
    // Measured to within 20 % at 17 shapes; before -> after e.g. 13 x 1039 keys, 32 heads, 10 text rows 36.6 -> 23.1, 6 x 1152,
    // 384 rows 250 -> 49 (in the wide form), 5 x 774, 16 heads, 60 rows 14.5 -> 13.1.
    const int units = (Mv + N + 127) / 128;
    const long n = (long)B * H * s.ng;
    // The wide form takes all calls with several text groups.  With one, K comes from HBM and bounds the sweep: there it only
    // takes the place of the blocks of four waves at d = 128 (13 x 1039 keys, 32 heads, 128 text rows 43 -> 40, 20 x 576, 40
    // heads, 70 rows 53 -> 49), where it is one chunk as well of those of eight; heads of 64 have three smaller blocks
    // per CU (8 x 2000, 128 rows 25 and 28).
    // Three slots (rs_deep) for K of up to 160 MB; beyond, two are as good (us per call, two / three: 8 x 2880 keys, 20 text rows, 189 MB
    // 102.1 / 102.3, 4 x 8000, 30 rows, 262 MB 134.6 / 134.9), and the workspace hangs on the estimate.
    const bool deep_k = k_mb <= 160.0;
    auto pick = [&](double merge_us, int most, int least_units) {
        double best = 0;
        for (int waves = 4; waves <= (s.ng > 1 ? 4 : 8); waves += 4)
            for (int nch = 1; nch <= most && (nch == 1 || nch <= units / least_units); ++nch) {
                const long blocks = n * nch, places = waves == 4 ? (s.nbw == 4 && s.ng == 1 && d == 64 ? 3 : 2) * kNumCU : kNumCU;
                const double fill = blocks < places ? (double)blocks / places : 1.0;
                double alone = s.nbw == 1 ? 7.5 : (s.nbw == 2 ? (waves == 8 ? 8.0 : 9.0) : (waves == 8 ? 11.0 : 14.0));
                double full = waves == 8 ? (s.nbw < 4 ? 11.5 : 16.0) : 21.0;
                // (heads of 64 with four text blocks: three blocks of four waves share a CU, one of eight waves no better than at
                // d = 128; 2 x 8661 keys, 64 heads, 95 text rows 49.8 -> 38.6)
                if (s.nbw == 4 && d == 64) { alone = waves == 8 ? 10.0 : 11.5; full = waves == 8 ? 10.5 : 21.0; }
                if (s.nbw == 1 && d == 128 && waves == 4 && blocks <= kNumCU && deep_k) { alone = 6.0; full = 16.0; }   // (three slots: rs_deep)
                if (s.nbw == 4 && d == 128 && waves == 4) full = 30.0;
                const double per_key = alone + (full - alone) * fill;
                double t = (double)((blocks + places - 1) / places) * (5.0 + 1e-3 * per_key * (Mv + N) / nch) + (nch > 1 ? merge_us : 0.0);
                if (s.ng > 1) {
                    // Several text groups: the last round by itself, at the full rate once a CU has two blocks of it.  Priced by its
                    // share of the places, it looked cheaper than it is: 4 x 5284 keys of 64, 32 heads, 374 text rows in 384 blocks
                    // 80 us, in 768 with the merge 71; 6 x 6000, 256 rows 97 and 86; 3 x 1592 keys of 128, 40 heads, 171 rows 27.6
                    // and 22.8.  At 84 random shapes the sweep and its merge take 2 % less, none more than 3 % more.
                    alone = d == 64 ? 8.0 : 11.0;
                    full = d == 64 ? 13.0 : 18.0;
                    const double keys = 1e-3 * (Mv + N) / nch;
                    const long last = blocks % places;
                    t = (double)(blocks / places) * (4.0 + full * keys) + (last > 0 ? 4.0 + (last > kNumCU ? full : alone) * keys : 0.0) + (nch > 1 ? 4.0 : 0.0);
                }
                if (best == 0 || t < 0.97 * best) { best = t; s.rs_waves = waves; s.nch = nch; }
            }
    };
    pick(5.0, kMaxChunks, 4);
    // Where the estimate is off: one wide block of four waves per (sample, head) for 65 to 128 text rows when
    // - the heads of all samples are more than two rounds of the CUs, or
    // - they nearly fill the CUs, the keys are many, and K is small or the estimate picks several chunks, which cost the merge too.
    // us per call, picked / wide: 17 x 500 keys, 128 rows (544 heads in all) 111.4 / 101.7, 24 x 1700 (768) 255 / 247; 6 x 2600, 100
    // rows (192) 107.2 / 103.5, 6 x 4000, 128 rows 147.3 / 139.3, 7 x 2880 (224) 132.5 / 126.9, 6 x 2880, 40 heads (240) 131.3 / 126.3;
    // not 5 x 2600 (160) 93.8 / 95.2, 8 x 576, 128 rows 62.0 / 63.1, 9 x 1700 (288) 119.7 / 122.1.  Eight waves in one chunk (256 heads)
    // stay where K is large: 8 x 2880, 128 rows 124.6 / 123.3 with K half in the Infinity Cache, but the sweep alone on new
    // inputs, all of K from HBM, 57.2 / 63.7 (1800: 46.0 / 47.5, 1152: 25.6 / 23.7).
    const bool fills = n > 176 && n <= kNumCU && Mv + N >= 1000 && (s.nch > 1 || k_mb <= 105.0);
    if (s.nbw == 4 && s.ng == 1 && d == 128 && !s.own && (n > 2 * kNumCU || fills)) { s.rs_waves = 4; s.nch = 1; }
    s.nch_ws = s.nch;
    s.partial_in_pieces = false;
    if (s.own) {
        // Single tiles: the merge of the chunks is part of sweep 2, and a chunk may be shorter (2 x 576 keys, 128 text rows 36 ->
        // 32 us).  The workspace stays as it is: more chunks than the persistent form would take have their statistics in
        // the memory of the pieces, behind V and I, as many as fit there.
        const long Npad = 32l * s.nbt, fit = ((long)s.col.Gmax * Mv * Npad - 2l * s.nbt * Mv) / (2l * H * Npad);
        const long most = fit > s.nch_ws ? fit : s.nch_ws;
        pick(1.0, most < kOwnChunks ? (int)most : kOwnChunks, s.nbw < 4 ? 1 : 2);
        s.partial_in_pieces = s.nch > s.nch_ws;
    }
    s.rs_stream = big_k && s.rs_waves == 4;           // (what the estimate picks for K of that size)
    s.rs_wide = s.ng > 1 || (s.nbw == 4 && d == 128 && s.rs_waves == 4);
    s.rs_deep = s.nbw == 1 && d == 128 && s.rs_waves == 4 && n * s.nch <= kNumCU && deep_k;
    return s;
}

// The plan of a call whose caller brings the row normalisers: one statistic per row, and K has not been read before.
inline ScorePlan with_normalisers(ScorePlan s) {
    s.nch = 1;
    s.rows = s.rows_lse;
    s.own = s.own_lse || s.rows;
    return s;
}

// Whether the persistent column sweep reads K by streaming loads, which leave the cache to the query fragments.
//
// Rule: unless K is likely to be found in the cache, or to be wanted there.  One text group of 65 to 128 rows: plain where sweep 1 has
// read K with plain loads, except for K of more than 85 MB of which no more than an eighth is kept (the copies read the kept rows
// again; how many a threshold keeps is not known).  Several groups read K one after the other: plain, unless the fragments are
// many (28 MB).
//
// us per call, plain / streaming, on three states in turn and on inputs just made, 128 rows, all valid unless said otherwise: 4 x 2880
// keys, a sixteenth kept 85.8 / 82.3 and 93.5 / 94.7, a ninth 90.1 / 87.0 and 96.9 / 98.4, a fifth 93.8 / 95.6 and 104.8 / 106.8;
// 8 x 2880 at 3/4 117.2 / 115.6 and 124.2 / 124.3, 124.2 / 123.9 and 132.6 / 133.5, 138.1 / 140.5 and 145.8 / 149.6; 16 x 1600, 100 rows
// 146.2 / 145.5 and 169.3 / 168.5, 156.3 / 157.3 and 178.1 / 179.0, 171.1 / 175.6 and 192.4 / 196.7.  Smaller K, a tenth kept: 5 x 2000
// (82 MB) 86.6 / 85.6 and 93.4 / 93.5, 16 x 700, 80 rows, 16 heads (46) 60.3 / 61.4 and 63.8 / 64.2, 2 x 3000, 70 rows (49) 58.3 / 59.9
// and 62.8 / 63.0, 4 x 2880, 100 rows, 40 heads of 64 (59) 73.3 / 75.1 and 77.3 / 78.2.
// Behind streaming loads, a fifth kept, 10 x 2880 (236 MB) 199.8 / 202.9 and 213.0 / 207.1, 16 x 2600 (341) 263.1 / 268.6 and 275.8 /
// 271.5; with normalisers 6 x 2000 81.1 / 77.6 and 85.0 / 80.6, 8 x 2880 at 3/4 110.8 / 113.7 and 120.5 / 119.0, 16 x 2600 199.5 /
// 200.6 and 212.6 / 207.9.  Several groups: 3 x 9000, 300 rows, normalisers 198 / 211, 8 x 2880, 200 rows 135 / 143, without 6 x 1152, 384
// rows, 19 MB of fragments 140 / 142; 20 x 576, 200 rows, 37 MB 184 / 181.
inline bool streams_col_k(const ScorePlan& s, int B, int Mv, int H, int d, int Rcap, bool threshold, bool row_lse) {
    if (s.ng > 1) return (double)B * H * d * 2e-6 * 32 * s.nbt >= 28.0;
    return s.nbw < 4 || row_lse || s.rs_stream || (!threshold && 8L * Rcap <= Mv && (double)B * Mv * H * d * 2e-6 > 85.0);
}

// Whether the kept K rows leave by streaming stores, as the kept rows of V and hidden always do.
//
// Rule: where the call's K, V and hidden, in and out, come to more than 200 MB, so that the Infinity Cache (256 MB) would have to
// write them back before anything that is sure to come reads them; where the call reads K by streaming loads alone (with the caller's
// row normalisers), only from 34 MB of K rows out on: such loads leave the lines in the cache.
// In threshold mode Rcap is no more than room: a quarter of the slots is taken to be kept (the printed rule keeps 64 of 576 tokens
// on average; long inputs that keep a third have 4 x 6907 keys, 110 rows, normalisers 166.8 / 157.1).
//
// us per call, plain / streaming stores, on three states in turn and on inputs just made: 16 x 576 keys, 64 text rows, 192 kept (34 MB
// out, 352 in all) 95.7 / 88.8; 24 x 516, 12 rows, 64 kept (15, 356) 75.6 / 70.9 and 80.5 / 80.9; 4 x 2880, 12 rows, 360 kept (12,
// 321) 66.4 / 63.3 and 74.2 / 73.9, 128 rows, 320 kept (15, 340) 88.3 / 88.1 and 98.7 / 99.5; 16 x 1000, 20 rows, 64 kept (11, 434) 79.7 /
// 74.4 and 86.1 / 86.7; 8 x 2880, 8 rows, 32 kept (3, 576) 90.6 / 87.8 and 104.7 / 105.1; 12 x 576, 64 rows, 72 kept (13, 229) 52.9 /
// 52.7 and 59.3 / 59.0; 8 x 576 (17, 176) 49.7 / 49.4; heads of 64, 24 x 1000 (12, 281) 63.6 / 60.4 and 70.4 / 70.8.
// By threshold 24 x 516, 12 rows 81.2 / 74.7 and 86.1 / 84.8, 14 x 576, 64 rows 63.3 / 59.1 and 68.9 / 68.5, 12 x 516 (178) 42.5 /
// 42.8 and 46.0 / 46.2, 4 x 2880, 128 rows 97.2 / 92.7 and 102.0 / 104.6, 4 x 576 29.6 / 30.1.
// With normalisers and streaming loads of K 16 x 576, 128 kept (25 MB) 56.3 / 56.7, 192 kept (34) 77.3 / 77.1, 16 x 1152, 100 rows (38)
// 108.4 / 103.5, 24 x 576 (50) 104.9 / 98.8; by threshold 24 x 576, 20 rows (32) 62.4 / 67.3 and 64.3 / 69.9; with plain ones, by
// threshold, 14 x 576, 64 rows 54.0 / 49.3 and 56.8 / 58.0, 4 x 2044, 216 rows 81.2 / 74.9, 8 x 1576, 340 rows, 16 heads 96.0 / 90.0.
// With 600 MB of other data read before each call, that time included, 16 x 576 255.0 / 252.8 and 8 x 2880 287.0 / 281.7.
// Call after call on the same buffers the rows never leave the cache, and streaming them costs: 16 x 576 above 86.6 /
// 88.8, with normalisers 8 x 2880, 128 rows (29 MB) 103.1 / 106.3 and 24 x 576 95.2 / 102.3.  So it does where the next
// layer's filter reads them at once: 16 x 576 -> 192 -> 128 -> 64 takes 183.5 us all plain, 188.5 with the first call's
// streamed (as here), 190.2 with all calls' streamed (24 x 576 -> 192 -> 64: 177.9, 176, 175.4).  Nothing in a call tells the
// one use from the other.
inline bool streams_k_out(int B, int Mv, int N, int H, int d, int C, int Rcap, bool threshold, bool k_streams) {
    const int kept = threshold && Rcap > Mv / 4 ? Mv / 4 : Rcap;
    const double out_mb = (double)B * (kept + N) * H * d * 2e-6;
    const double all_mb = (double)B * (Mv + kept + 2.0 * N) * (2.0 * H * d + C) * 2e-6;
    return all_mb > 200.0 && (!k_streams || out_mb > 34.0);
}

}  // namespace
}  // namespace md
