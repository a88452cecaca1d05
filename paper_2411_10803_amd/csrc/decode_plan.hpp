// How the row moves of a cache cut are shaped into pieces and how the blocks of the move launch come by them, and which logits
// the selection asks for ahead: the arithmetic of the host and of the kernels.  Without any HIP header, so that a CPU test can
// compile it, claim its way through and follow every request.
#pragma once
#include <stdint.h>

#ifndef MD_PLAN_FN
#ifdef __HIPCC__
#define MD_PLAN_FN __host__ __device__ __forceinline__
#else
#define MD_PLAN_FN inline
#endif
#endif

namespace md {
namespace {

// Counters from which blocks claim their pieces, 128 bytes apart (one counter for all takes 12 ns a claim: 683 us instead of 320
// for the moves of 64 caches of 4096 entries cut to 1024).
constexpr int kClaims = 16, kClaimStride = 32;
// Just under two blocks per CU.  us with 320 / 448 / 512 / 640 blocks, heads of 128: 64 caches of 4096 entries cut to 1024 284 /
// 273 / 281 / 282, 32 layers x 16 x 640 to 128 296 / 296 / 309 / 309, 64 x 1000 to a half 91.5 / 90.5 / 92.7 / 94.3, 14 x 882 of 40
// heads to a quarter 19.1 / 19.3 / 19.4 / 19.2, 4 x 2000 to a half 14.8 / 14.3 / 14.5 / 15.2; 300 x 500 of 8 heads to 2/5 61 / 54 / 52 / 54
constexpr int kMoveBlocks = 448;

struct MovePieces {
    int per_piece, per_move;                         // moves per piece, pieces per move: one of them is 1
    int vectors, threads;                            // of a thread; of a block that have any
    int pair;                                        // vectors of a K row and a V row together
};
// Pairs of 1025 to 2048 vectors as one piece of two vectors per thread, not as two with a third of the threads idle: 14 caches of
// 882 entries cut to 208, 40 heads of 128, 26.6 us in two, 22.5 in one.
inline MovePieces move_pieces(int H, int d) {
    MovePieces mp;
    mp.pair = 2 * H * (d / 8);
    mp.vectors = mp.pair <= 1024 ? 1 : 2;
    mp.per_piece = mp.pair < 1024 ? 1024 / mp.pair : 1;
    mp.per_move = (mp.pair + 1024 * mp.vectors - 1) / (1024 * mp.vectors);
    mp.threads = (mp.per_piece * mp.pair + mp.per_move * mp.vectors - 1) / (mp.per_move * mp.vectors);
    return mp;
}
MD_PLAN_FN int pieces_of(int moves, const MovePieces& mp) { return (moves + mp.per_piece - 1) / mp.per_piece * mp.per_move; }

// Rows of one sample that can move when a cache of Lcap slots is cut to `budget` entries or more (protected entries stay beyond
// the budget): a hole below the new length for each of them, and the new length is at least the budget.
inline int most_moves(int Lcap, int budget) {
    return Lcap <= budget ? 0 : (Lcap - budget < Lcap / 2 ? Lcap - budget : Lcap / 2);
}
// Blocks of the move launch: no more than pieces there can be.
inline int move_blocks(const MovePieces& mp, int n_layers, int B, int moves) {
    const long most = (long)n_layers * B * pieces_of(moves, mp);
    return (int)(most < kMoveBlocks ? (most > 1 ? most : 1) : kMoveBlocks);
}

// The pieces of a call go layer by layer, `total` in each.  A layer's fit 31 bits (a call has at most 2^28 slots, and a piece that is
// but part of a move stands for 16 KiB and more of each tensor); those of all layers need not: 65536 rows moved in each of
// 65535 layers come close to 2^32, and a sum that wrapped would leave rows behind.
MD_PLAN_FN uint64_t piece_count(uint32_t total, int n_layers) { return (uint64_t)total * (uint32_t)n_layers; }
struct PieceAt { int layer, r; };                    // r: piece of the layer
MD_PLAN_FN PieceAt piece_at(uint64_t piece, uint32_t total, int n_layers) {
    PieceAt at;
    if (n_layers == 1) at.layer = 0;
    else if ((piece >> 32) == 0) at.layer = (int)((uint32_t)piece / total);       // (a quarter of the instructions)
    else at.layer = (int)(piece / total);
    at.r = (int)(piece - (uint64_t)total * (uint32_t)at.layer);
    return at;
}

// A block's first piece is the one of its number.  Block i draws from counter i % claim_counters(blocks) -- a counter without
// blocks would hand out its share to nobody -- and the n-th claim from counter c is piece claimed_piece(blocks, c, n).
MD_PLAN_FN int claim_counters(int blocks) { return blocks < kClaims ? blocks : kClaims; }
MD_PLAN_FN uint64_t claimed_piece(int blocks, int c, uint32_t n) {
    return (uint64_t)n * (uint32_t)claim_counters(blocks) + (uint32_t)(blocks + c);
}

// What a wave of the selection asks for of a sample's logits [.., H] in one go: the vectors of the entries from `entry` on, up to
// entry `ahead`, as the base and the range of a buffer of its own.  The wave's place is in the base and not in the scalar offset of
// the loads: that one is not part of what is compared with the range, or wraps round where it is larger.
struct LogitRange { long first; int bytes; };        // first float; bytes that may be read from it on
MD_PLAN_FN LogitRange logit_range(int entry, int ahead, int H) {
    const int e = entry < ahead ? entry : ahead;
    return LogitRange{(long)e * H, (ahead - e) * H * 4};
}
// byte of a lane's u-th vector, `entry` entries further on
MD_PLAN_FN int logit_vector(int lane, int u, int entry, int H) { return lane * 16 + u * 1024 + entry * H * 4; }

}  // namespace
}  // namespace md
