// CPU check of the move launch's claims (csrc/decode_plan.hpp): whatever entries a cache cut keeps, no more rows move than the
// host reckons with, and blocks that claim in any order take every piece exactly once, also where blocks are few or layers many.
// And of the selection's requests: a wave's range ends with the last entry that may be asked for, wherever it begins, and what lies
// before that is all there.
#include <stdio.h>
#include <initializer_list>
#include <random>
#include <vector>

#include "../../paper_2411_10803_amd/csrc/decode_plan.hpp"

using namespace md;

// Lets `blocks` blocks take `items` pieces in a random order; false: a piece was left out or taken twice.
static bool drains(int blocks, long items, std::mt19937& rng) {
    std::vector<uint32_t> claims(kClaims, 0u);
    std::vector<char> taken(items, 0);
    std::vector<long> at(blocks);
    std::vector<int> active;
    for (int i = 0; i < blocks; ++i)
        if ((at[i] = i) < items) active.push_back(i);
    long done = 0;
    while (!active.empty()) {
        const size_t a = rng() % active.size();
        const int i = active[a], c = i % claim_counters(blocks);
        if (taken[at[i]]++) return false;
        ++done;
        at[i] = (long)claimed_piece(blocks, c, claims[c]++);
        if (at[i] >= items) { active[a] = active.back(); active.pop_back(); }
    }
    return done == items;
}

int main() {
    std::mt19937 rng(1);
    long cuts = 0, bad = 0;
    for (int H : {1, 3, 4, 8, 32, 40, 65, 128, 1024})
        for (int d : {8, 32, 64, 128, 256, 512})
            for (int B : {1, 2, 15, 64})
                for (int Lcap : {1, 2, 9, 200, 1000, 4352, 9000})
                    for (int budget : {0, 1, 5, 16, 499, 1024, 4351, 20000})
                        for (int share = 0; share <= 4; ++share) {
                            const int n = Lcap - (share == 4), np = n * share / 4;       // entries, protected ones
                            const MovePieces mp = move_pieces(H, d);
                            const int extra = budget > np ? budget - np : 0, new_len = np + extra < n ? np + extra : n;
                            const int moves = n <= budget ? 0 : (new_len < n - new_len ? new_len : n - new_len);
                            const long items = (long)B * pieces_of(moves, mp);
                            ++cuts;
                            const char* why = nullptr;
                            if (mp.per_piece != 1 && mp.per_move != 1) why = "piece";
                            else if (mp.per_piece * mp.pair > mp.per_move * mp.vectors * mp.threads || mp.threads > 1024) why = "threads";
                            else if (moves > most_moves(Lcap, budget)) why = "more moves than reckoned with";
                            else if (items < 200000 && !drains(move_blocks(mp, 1, B, most_moves(Lcap, budget)), items, rng)) why = "pieces";
                            if (why && ++bad <= 10) printf("H=%d d=%d B=%d Lcap=%d budget=%d protected=%d: %s\n", H, d, B, Lcap, budget, np, why);
                        }
    for (int blocks = 1; blocks <= 40; ++blocks)
        for (long items : {0l, 1l, 15l, 16l, 17l, 333l, 1000l})
            if (!drains(blocks, items, rng) && ++bad <= 10) printf("%ld pieces, %d blocks\n", items, blocks);
    // as many layers and samples as a call takes: pieces beyond 2^32 keep their layer, and a claim stays behind the last one
    for (uint32_t total : {1u, 3u, 65535u, 65537u, 98765u, 1u << 27})
        for (int layers : {1, 2, 32, 65535}) {
            const uint64_t all = (uint64_t)total * (uint64_t)layers;
            bool ok = piece_count(total, layers) == all;
            for (int i = 0; i < 2000; ++i) {
                const uint64_t item = i == 0 ? all - 1 : (((uint64_t)rng() << 32) | rng()) % all;
                const PieceAt at = piece_at(item, total, layers);
                ok &= at.layer >= 0 && at.layer < layers && at.r >= 0 && (uint32_t)at.r < total && (uint64_t)at.layer * total + (uint64_t)at.r == item;
                // the claim that hands out this piece, and the last ones from its counter
                if (item < kMoveBlocks || all > (1ull << 36)) continue;
                const uint64_t n = (item - kMoveBlocks) / kClaims;
                const int c = (int)((item - kMoveBlocks) % kClaims);
                ok &= claimed_piece(kMoveBlocks, c, (uint32_t)n) == item;
                const uint64_t behind = (all - kMoveBlocks) / kClaims + kMoveBlocks;
                ok &= behind >> 32 != 0 || claimed_piece(kMoveBlocks, c, (uint32_t)behind) >= all;
            }
            if (!ok && ++bad <= 10) printf("%u pieces in each of %d layers\n", total, layers);
        }
    for (int H = 4; H <= 128; H += 4)
        for (int ahead : {1, 2, 31, 32, 63, 64, 65, 66, 130, 1000, 1023, 1024, 1025, 1088, 2047, 2048, 3000, 8192}) {
            const int vpe = H / 4;
            const long end = (long)ahead * H;                                  // floats that may be read
            const bool by_lanes = vpe == 1 || vpe == 2 || vpe == 4 || vpe == 8;
            bool ok = true;
            for (int round = 0; round < (by_lanes ? 2 : 1); ++round)
                for (int wave = 0; wave < 16; ++wave) {
                    const int e0 = round * 1024 + wave * 64;
                    const LogitRange r = logit_range(e0, ahead, H);
                    ok &= r.first >= 0 && r.bytes >= 0 && r.first + r.bytes / 4 <= end && r.bytes % 16 == 0;
                    std::vector<char> got(64 * vpe, 0);
                    for (int step = 0; step < (by_lanes ? 1 : 2); ++step)
                        for (int u = 0; u < (by_lanes ? vpe : 5); ++u)
                            for (int lane = 0; lane < 64; ++lane) {
                                const int byte = logit_vector(lane, u, 32 * step, H);
                                ok &= byte >= 0;
                                if (byte + 16 > r.bytes) continue;             // reads as zero
                                if (byte / 16 < 64 * vpe) got[byte / 16] = 1;
                            }
                    if (!by_lanes && vpe > 10) continue;                       // asked for later
                    for (int x = 0; x < 64 * vpe; ++x)
                        if (e0 + x / vpe < ahead) ok &= got[x] == 1;
                }
            if (!ok && ++bad <= 10) printf("requests of %d heads up to entry %d\n", H, ahead);
        }
    printf("%ld cuts, %ld wrong\n", cuts, bad);
    return bad != 0;
}
