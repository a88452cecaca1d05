// Stage 2 -- prefill (Sec. 3.4): text-to-vision attention scores, the dual filter (Eq. 8-10) and
// token drop (stable compaction of hidden states, K and V).
//
// The column statistics V_j = sum_i a_ij and I_j = max_i a_ij need the row softmax normaliser of
// every text row over the WHOLE key axis, and the head mean has to be taken before the max over
// text rows.  The normalisers are a by-product of the layer's own attention (Sec. 3.4): a caller
// that has them (row_lse) pays one sweep over K; otherwise a first sweep computes them:
//   prefill_rowstats_kernel  per (sample, head, key chunk): S = K Q^T on the MFMA units, online
//                            (max, sum-exp) per text row -> row statistics (prefill_cstat_kernel
//                            merges the chunks); prefill_rowstats_wide_kernel where there are several
//                            text groups, and for one of three or four text blocks at d = 128 where
//                            blocks of four waves are planned; with row_lse only prefill_qpack_kernel runs
//   prefill_colscore_kernel  persistent blocks over units of (64 or 128 vision keys, one head): recompute
//                            S, p = exp(s - m)/Z, accumulate the head mean a[i][j] of such a key tile
//                            in registers; a block's share of a tile is written as one piece
//   prefill_colfix_kernel    sums a tile's pieces in a fixed order, column sum / max -> V_j, I_j
//   prefill_colown_kernel    in place of both on small calls with two to four text blocks: a block takes a tile (32 keys, 32
//                            text rows) with all heads
//   prefill_colrows_kernel   in place of both for up to 64 text rows: a block takes 32 keys with all text rows and heads
// The N x Mv probability matrix of a head is never written to memory.
//   prefill_select_kernel    per sample: G, the filter rule (threshold) or radix top-k (budget),
//                            prefix sum -> kept_index, row map for the copy
//   prefill_compact_kernel   one block per output row: 16-byte vector copies of hidden, K, V rows
//
// MFMA tile: v_mfma_f32_32x32x16_bf16, keys on the M side (A operand), text rows on the N side
// (B operand).  In the result a lane holds one text row (column lane%32) and 16 of the 32 keys,
// so the row-softmax reductions over keys stay inside a lane (+ one exchange with lane^32).
#include "md_device.hpp"
#include "md_host.hpp"
#include "prefill_plan.hpp"

#include <type_traits>

namespace md {
namespace {

constexpr float kLog2e = 1.4426950408889634f;

struct PrefillDims {
    int B, Mv, N, H, d, C, L;
    int nch;          // key chunks per (sample, head) in the row-statistics sweep
    int Npad;         // 32 * (number of 32-row text blocks)
    int ng;           // text groups a sample of N text rows has (see text_group)
    int Rcap;
    KvLayout q, kv;   // element strides of q_txt and of k (v shares them)
};

// key row of accumulator register r in the 32x32 result tile
__device__ __forceinline__ int tile_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

#define MD_VM_WAIT(n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory")
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Rows of an MFMA operand (one head slice of a key or a text query: 16*KS bf16 = CH chunks of 16
// bytes) on their way from global memory to MFMA fragments, through LDS.
//   global -> LDS  buffer loads that write LDS directly (no staging registers): a wave instruction
//                  moves 1 KiB = RPL whole rows, coalesced; rows outside the buffer resource's range
//                  are never fetched.
//   LDS layout     rows unpadded (pitch ROWB); the chunk a lane fetches for position `pos` of row
//                  `row` is pos ^ swz(row), so that the 128-bit fragment reads below (32 rows, one
//                  chunk index) spread over all banks.
//   LDS -> frags   lane (g = lane/32, r = lane%32) of the 32x32x16 MFMA holds row r, chunks 2*ks+g.
template <int KS>
struct LdsRows {
    static constexpr int CH = 2 * KS;
    static constexpr int ROWB = CH * 16;             // 256 (d = 128) or 128 (d = 64) bytes
    static constexpr int RPL = kWave / CH;           // rows per load instruction
    static_assert(KS == 4 || KS == 8, "rows of 128 or 256 bytes");
    __device__ static __forceinline__ int swz(int row) { return KS == 8 ? (row & 15) : ((row >> 1) & 7); }

    // One wave instruction: rows slot_row .. slot_row+RPL-1 of the LDS block at `lds_base` (wave-uniform)
    // receive the global rows grow0+slot_row.. of the matrix behind `rs` (rows row_bytes apart).
    // `live` (wave-uniform) false: nothing is fetched.
    template <bool STREAM = false>
    __device__ static __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, uint32_t row_bytes, int grow0, int slot_row,
                                                 char* lds_base, int lane, bool live) {
        const int row = slot_row + (int)((uint32_t)lane / CH), pos = (int)((uint32_t)lane % CH);
        const uint32_t off = live ? (uint32_t)(grow0 + row) * row_bytes + (uint32_t)((pos ^ swz(row)) << 4) : 0xFFFFFF00u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(lds_base + slot_row * ROWB), 16, off, 0, 0, STREAM ? 2 : 0);
    }
    // LDS byte address of this lane's fragment row in the 32-row tile at `tile` (aligned to 32*ROWB),
    // with the swizzle and the lane half folded in; chunk index ks is applied with XOR.
    __device__ static __forceinline__ uint32_t frag_base(const char* tile, int lane) {
        const int r = lane & 31, g = lane >> 5;
        const uint32_t a = (uint32_t)(uintptr_t)(lds_ptr_t)const_cast<char*>(tile);
        return (a + r * ROWB) ^ (uint32_t)((g << 4) ^ (swz(r) << 4));
    }
    // the KS fragments of a tile, requested and waited for in one statement
    __device__ static __forceinline__ void frags_wait(uint32_t fb, bf16x8 (&f)[KS]) {
        uint32_t a;
        if constexpr (KS == 8)
            asm volatile("ds_read_b128 %0, %9\n\t"
                         "v_xor_b32 %8, 32, %9\n\tds_read_b128 %1, %8\n\tv_xor_b32 %8, 64, %9\n\tds_read_b128 %2, %8\n\t"
                         "v_xor_b32 %8, 0x60, %9\n\tds_read_b128 %3, %8\n\tv_xor_b32 %8, 0x80, %9\n\tds_read_b128 %4, %8\n\t"
                         "v_xor_b32 %8, 0xa0, %9\n\tds_read_b128 %5, %8\n\tv_xor_b32 %8, 0xc0, %9\n\tds_read_b128 %6, %8\n\t"
                         "v_xor_b32 %8, 0xe0, %9\n\tds_read_b128 %7, %8\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7]),
                           "=&v"(a) : "v"(fb) : "memory");
        else
            asm volatile("ds_read_b128 %0, %5\n\t"
                         "v_xor_b32 %4, 32, %5\n\tds_read_b128 %1, %4\n\tv_xor_b32 %4, 64, %5\n\tds_read_b128 %2, %4\n\t"
                         "v_xor_b32 %4, 0x60, %5\n\tds_read_b128 %3, %4\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(a) : "v"(fb) : "memory");
    }
    // the KS fragments of a tile; returns once they are in registers
    __device__ static __forceinline__ void frags(uint32_t fb, bf16x8 (&f)[KS]) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            uint32_t a;
            asm volatile("v_xor_b32 %1, %2, %3\n\tds_read_b128 %0, %1" : "=v"(f[ks]), "=&v"(a) : "v"(ks << 5), "v"(fb) : "memory");
        }
        if constexpr (KS == 8)
            asm volatile("s_waitcnt lgkmcnt(0)"
                         : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]), "+v"(f[6]), "+v"(f[7]) :: "memory");
        else
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]) :: "memory");
    }
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(const uint16_t* base, long rows, long row_stride, int d) {
    // rows [0, rows) of `d` elements each, row_stride elements apart; anything beyond reads as "not there"
    const long bytes = rows > 0 ? ((rows - 1) * row_stride + d) * 2 : 0;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, (int)bytes, 0x00020000);
}

// Vision rows that matter.  Vision tokens arrive with a validity mask; after the vision-encoder stage
// merged tokens away the valid ones of a sample are a prefix and the rest of its Mv slots is padding.
// Both sweeps skip the slots behind the last valid one: eff = min(Mv, round_up32(last valid + 1))
// (0 when no slot is valid).  Any other pattern of invalid slots is still handled key by key.
// Per-thread part: the largest index this thread saw set among [0, n), or -1.
__device__ __forceinline__ int last_set_partial(const uint8_t* v, int n, int tid, int nthreads) {
    int last = -1;
    const int head = min(n, (int)((16 - ((uintptr_t)v & 15)) & 15));     // bytes before 16-byte alignment
    if (tid < head && v[tid]) last = tid;
    const int nvec = (n - head) / 16;
    const uint4* pv = reinterpret_cast<const uint4*>(v + head);
    for (int q = tid; q < nvec; q += nthreads) {
        const uint4 w = pv[q];
        const int base = head + q * 16;
        if (w.x) last = base + ((31 - __clz((int)w.x)) >> 3);
        if (w.y) last = base + 4 + ((31 - __clz((int)w.y)) >> 3);
        if (w.z) last = base + 8 + ((31 - __clz((int)w.z)) >> 3);
        if (w.w) last = base + 12 + ((31 - __clz((int)w.w)) >> 3);
    }
    for (int j = head + nvec * 16 + tid; j < n; j += nthreads)
        if (v[j]) last = j;
    return last;
}
__device__ __forceinline__ int wave_max_int(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, kWave));
    return v;
}
__device__ __forceinline__ int effective_rows(int last, int Mv) { return last < 0 ? 0 : min(Mv, (last + 32) & ~31); }

// Validity of the 32 keys e0 .. e0+31 of the mask row `vb` of Mv bytes (bit r = key e0 + r is a valid vision token; bytes
// beyond the row count as invalid); e0 is a multiple of 32.
__device__ __forceinline__ uint32_t key_valid_mask(const uint8_t* __restrict__ vb, long e0, int Mv) {
    uint32_t mask = 0;
    if ((reinterpret_cast<uintptr_t>(vb) & 3) == 0) {             // block-uniform: the mask row is word-aligned
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(vb), 0, (Mv + 3) & ~3, 0x00020000);
        uint32_t w[8];
        const int off = (int)min(e0, (long)((Mv + 3) & ~3));    // beyond the row: out of the buffer's range, reads 0
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = __builtin_amdgcn_raw_buffer_load_b32(rv, off + 4 * q, 0, 0);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            mask |= (((w[q] & 0xFFu) ? 1u : 0u) | ((w[q] & 0xFF00u) ? 2u : 0u) | ((w[q] & 0xFF0000u) ? 4u : 0u) |
                     ((w[q] & 0xFF000000u) ? 8u : 0u)) << (4 * q);
    } else {
        for (int r = 0; r < 32; ++r) mask |= (vb[min(e0 + r, (long)Mv - 1)] != 0 ? 1u : 0u) << r;
    }
    const long left = (long)Mv - e0;                            // slots of the row from this tile on
    if (left < 32) mask &= left <= 0 ? 0u : (1u << left) - 1u;
    return mask;
}

// The mask row of a sample for one wave, requested in one go: word w of a lane covers the 32 keys of tile 64 * w + lane, so
// that the last valid key and the tiles' masks come out of the same loads (one round trip; a loop over the row and a
// second look at the wave's own tiles were four to five: 3 x 4608 keys, 100 to 300 text rows, 3/4 of the slots valid 40.2 -> 38.0
// us, 3 x 9000 keys, 200 text rows, 9/10 valid 69.4 -> 64.1).
struct MaskRow {
    static constexpr int W = 5;                       // rows of up to 64 * 32 * W slots
    u32x4 raw[W][2];
    __device__ static __forceinline__ bool fits(const uint8_t* vb, int Mv) {
        return vb && (reinterpret_cast<uintptr_t>(vb) & 3) == 0 && Mv <= W * kWave * 32;
    }
    __device__ __forceinline__ void request(const uint8_t* vb, int Mv, int lane) {
        // (slots beyond the row read as invalid; the up to three bytes that fill its last word are cut off in `word`)
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(vb), 0, (Mv + 3) & ~3, 0x00020000);
#pragma unroll
        for (int w = 0; w < W; ++w)
            if (w * kWave * 32 < Mv) {
                raw[w][0] = __builtin_amdgcn_raw_buffer_load_b128(rv, (w * kWave + lane) * 32, 0, 0);
                raw[w][1] = __builtin_amdgcn_raw_buffer_load_b128(rv, (w * kWave + lane) * 32 + 16, 0, 0);
            } else {
                raw[w][0] = raw[w][1] = u32x4{0, 0, 0, 0};
            }
    }
    __device__ __forceinline__ uint32_t word(int w, int Mv, int lane) const {
        uint32_t mask = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            // byte != 0 -> its top bit (no carry leaves a byte), then the four top bits gathered
            const uint32_t x = raw[w][q >> 2][q & 3], t = ((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x;
            mask |= ((((t >> 7) & 0x01010101u) * 0x01020408u) >> 24 & 15u) << (4 * q);
        }
        const int left = Mv - (w * kWave + lane) * 32;
        return left >= 32 ? mask : left <= 0 ? 0u : mask & ((1u << left) - 1u);
    }
    // the last valid key of the row (-1: none), and this lane's choice of a tile's mask (`tile`: any per lane)
    __device__ __forceinline__ uint32_t digest(int Mv, int lane, int tile, int& last) const {
        uint32_t mine = 0;
        last = -1;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            if (w * kWave * 32 >= Mv) break;
            const uint32_t v = word(w, Mv, lane);
            const unsigned long long any = __ballot(v != 0);
            if (any) {
                const int l = 63 - __builtin_clzll(any);
                last = (w * kWave + l) * 32 + 31 - __builtin_clz((uint32_t)__builtin_amdgcn_readlane((int)v, l));
            }
            const uint32_t got = (uint32_t)__builtin_amdgcn_ds_bpermute((tile & 63) * 4, (int)v);
            if (tile >> 6 == w) mine = got;
        }
        return mine;
    }
};

// What the kernels that follow need to know of a sample, written by the first one of a call.
struct SampleRows { int vision; int text_blocks; };   // effective vision rows; 32-row blocks with text rows below txt_len
// A block of a sweep holds up to `nbw` 32-row text blocks, one per wave column.  More of them (longer prompts) are
// cut into groups that share them out evenly, counted over the blocks that hold rows of the sample at hand: a sample
// with a short prompt has fewer groups than the longest one, or none, and columns without a block only help to move K.
struct TextGroup { int first, count; };
__device__ __forceinline__ TextGroup text_group(int g, int blocks, int groups) {
    if (groups <= 1) return TextGroup{0, blocks};
    // blocks / groups for at most 32 blocks: (blocks + 1/2) / groups stays 1/16 away from the next whole number
    const int base = (int)(((float)blocks + 0.5f) * __builtin_amdgcn_rcpf((float)groups)), extra = blocks - base * groups;
    return TextGroup{g * base + min(g, extra), base + (g < extra ? 1 : 0)};
}

// Row statistics folded into one constant: a probability of the head mean is
// exp2(s*scale*log2e + c) with c = -m - log2(Z) - log2(H); text rows beyond txt_len get -inf (-> 0).
__device__ __forceinline__ float fold_stats(float m, float z, bool row_ok, int H) {
    return (row_ok && z > 0.f) ? -m - fast_log2(z) - fast_log2((float)H) : -INFINITY;
}

// The 32 text-query rows i0.. of head slice `qb` as MFMA fragments: global -> this wave's LDS tile ->
// registers.  Rows at or beyond `tl` come out as zero rows.
template <int KS>
__device__ __forceinline__ void issue_query_rows(const uint16_t* qb, long tok_stride, int d, int i0, int tl, char* tile, int lane) {
    using T = LdsRows<KS>;
    const __amdgpu_buffer_rsrc_t rq = row_buffer(qb, tl, tok_stride, d);
#pragma unroll
    for (int t = 0; t < 32 / T::RPL; ++t) T::issue(rq, (uint32_t)(tok_stride * 2), i0, t * T::RPL, tile, lane, true);
}
template <int KS>
__device__ __forceinline__ void read_query_frags(int i0, int tl, const char* tile, int lane, bf16x8 (&qf)[KS]) {
    using T = LdsRows<KS>;
    MD_VM_WAIT(0);
    T::frags(T::frag_base(tile, lane), qf);
    const bool row_ok = i0 + (lane & 31) < tl;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        if (!row_ok) qf[ks] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
}
template <int KS>
__device__ __forceinline__ void load_query_frags(const uint16_t* qb, long tok_stride, int d, int i0, int tl, char* tile,
                                                 int lane, bf16x8 (&qf)[KS]) {
    issue_query_rows<KS>(qb, tok_stride, d, i0, tl, tile, lane);
    read_query_frags<KS>(i0, tl, tile, lane, qf);
}

// ---------------------------------------------------------------------------------------------
// Sweep 1: row statistics.  Block = (key chunk, head, sample), 4 or 8 waves, one text group (see the wide form below).  The waves of a
// block share every K tile through LDS: wave w works on text block w % NBW of the group and on key
// tile w / NBW of the TW tiles in flight per step, so a wave keeps the fragments of ONE
// 32-row text block in registers and K is read once per block.  K tiles stream through S LDS slots
// (filled S-1 steps ahead, no staging registers); one block barrier per step.  Inside a step the
// MFMA chain of the current tile is issued before the softmax arithmetic of the previous one (two
// accumulators), so the matrix unit and the vector ALUs overlap within a wave.
// Chunk 0 also stores the text-query fragments in fragment-major order (qfrag), rows beyond txt_len
// zeroed, for the second sweep.
template <int KS>
__device__ __forceinline__ f32x16 score_tile(const bf16x8 (&kf)[KS], const bf16x8 (&qf)[KS]) {
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], acc, 0, 0, 0);
    return acc;
}

// Online (max, sum of exp2) update of one lane's text row with the 16 keys it holds of a tile.
// Fast form: every key of the tile is visible -- straight-line code (so that the compiler can
// interleave it with the MFMA chain of the next tile), maximum and sum as trees.
__device__ __forceinline__ void online_update_all(const f32x16& acc, float scale_log2e, float& m, float& z) {
    const float b0 = fmaxf(fmaxf(acc[0], acc[1]), acc[2]), b1 = fmaxf(fmaxf(acc[3], acc[4]), acc[5]);
    const float b2 = fmaxf(fmaxf(acc[6], acc[7]), acc[8]), b3 = fmaxf(fmaxf(acc[9], acc[10]), acc[11]);
    const float b4 = fmaxf(fmaxf(acc[12], acc[13]), acc[14]);
    const float bm = fmaxf(fmaxf(fmaxf(b0, b1), b2), fmaxf(fmaxf(b3, b4), acc[15]));
    const float mn = fmaxf(m, bm * scale_log2e);     // the scale is positive: applied after the maximum
    const float nmn = -mn;
    float e[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) e[r] = fast_exp2(fmaf(acc[r], scale_log2e, nmn));
    const float s = ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7])) +
                    (((e[8] + e[9]) + (e[10] + e[11])) + ((e[12] + e[13]) + (e[14] + e[15])));
    z = fmaf(z, fast_exp2(m - mn), s);               // m = -inf at the first tile: exp2(-inf) = 0
    m = mn;
}
// General form: `vis` bit r set = accumulator r is a visible key.
__device__ __forceinline__ void online_update_masked(f32x16 acc, uint32_t vis, float scale_log2e, float& m, float& z) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (!((vis >> r) & 1u)) acc[r] = -INFINITY;
    float bm = acc[0];
#pragma unroll
    for (int r = 1; r < 16; r += 2) bm = fmaxf(fmaxf(bm, acc[r]), acc[r + 1 < 16 ? r + 1 : r]);
    const float mn = fmaxf(m, bm * scale_log2e);
    if (mn > -INFINITY) {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            s0 += fast_exp2(fmaf(acc[r], scale_log2e, -mn));
            s1 += fast_exp2(fmaf(acc[r + 1], scale_log2e, -mn));
        }
        z = fmaf(z, fast_exp2(m - mn), s0 + s1);
        m = mn;
    }
}

// The same where keys may be invisible (their scores -inf), up to all that were seen so far.
__device__ __forceinline__ void online_update_any(const f32x16& acc, float scale_log2e, float& m, float& z) {
    const float b0 = fmaxf(fmaxf(acc[0], acc[1]), acc[2]), b1 = fmaxf(fmaxf(acc[3], acc[4]), acc[5]);
    const float b2 = fmaxf(fmaxf(acc[6], acc[7]), acc[8]), b3 = fmaxf(fmaxf(acc[9], acc[10]), acc[11]);
    const float b4 = fmaxf(fmaxf(acc[12], acc[13]), acc[14]);
    const float bm = fmaxf(fmaxf(fmaxf(b0, b1), b2), fmaxf(fmaxf(b3, b4), acc[15]));
    const float mn = fmaxf(m, bm * scale_log2e);
    const float nmn = mn > -INFINITY ? -mn : 0.f;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r += 4) {
        s0 += fast_exp2(fmaf(acc[r], scale_log2e, nmn));
        s1 += fast_exp2(fmaf(acc[r + 1], scale_log2e, nmn));
        s2 += fast_exp2(fmaf(acc[r + 2], scale_log2e, nmn));
        s3 += fast_exp2(fmaf(acc[r + 3], scale_log2e, nmn));
    }
    z = fmaf(z, fast_exp2(m + nmn), (s0 + s1) + (s2 + s3));
    m = mn;
}

// The compiler's scheduler is asked to issue one MFMA, then a few vector and transcendental
// instructions, and so on: a wave issues in order, and a chain of dependent MFMAs issued back to back
// would hold up the independent vector work behind it.
template <int KS>
__device__ __forceinline__ void interleave_mfma_valu() {
#pragma unroll
    for (int q = 0; q < KS; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 48 / KS, 0);
        __builtin_amdgcn_sched_group_barrier(0x400, 16 / KS, 0);
    }
}

template <int NBW, int TW, int KS, bool STREAM, bool DEEP>
__global__ __launch_bounds__(64 * NBW * TW) void prefill_rowstats_kernel(
    const uint16_t* __restrict__ q_txt, const uint16_t* __restrict__ k,
    const uint8_t* __restrict__ vis_valid, const int32_t* __restrict__ txt_len, PrefillDims p, float scale_log2e,
    float2* __restrict__ partial, float* __restrict__ cstat, bf16x8* __restrict__ qfrag, SampleRows* __restrict__ rows)
{
    using T = LdsRows<KS>;
    // NBW wave columns (one 32-row text block each) x TW tile lanes (one 32-key tile of a step each): four waves,
    // or eight (NBW = 4, TW = 2) where one block then covers what two chunk blocks would and their statistics meet
    // in LDS instead of in a separate kernel
    constexpr int NW = NBW * TW;
    // LDS slots.  The eight-wave form runs with two (one step in flight while one is worked on): with more
    // requests outstanding per CU the sweep gets slower, not faster, when K comes from HBM (46.3 against 47.9 us);
    // four tile lanes too: three slots of 128 rows would leave room for one block per CU instead of two, which is
    // all that there is where the grid has no more (DEEP: 4 x 861 keys, 32 heads, 2 text rows 11.1 -> 10.1 us; not for
    // heads of 64, whose rows are half as long: 4 x 1510, 8 heads, 10 text rows 5.1 with two, 5.9 with three)
    constexpr int S = TW == 1 ? 4 : (NBW == 4 || (NBW == 1 && !DEEP) ? 2 : 3);
    constexpr int SLOT_ROWS = 32 * TW, SLOT_BYTES = SLOT_ROWS * T::ROWB;
    constexpr int NLW = SLOT_ROWS / T::RPL / NW;      // load instructions per wave and step
    constexpr int QBYTES = NBW * 32 * T::ROWB;        // the block's query tiles during the prologue (one per wave column)
    __shared__ __attribute__((aligned(1024))) char s_k[S * SLOT_BYTES];
    __shared__ __attribute__((aligned(1024))) char s_q[QBYTES];
    __shared__ float s_m[NW][32], s_z[NW][32];
    __shared__ int s_last[NW];
    const int lane = lane_id(), wv = wave_id();
    const int nbw = wv % NBW, tw = wv / NBW;
    const int ch = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int tl = txt_len ? min(max(txt_len[b], 0), p.N) : p.N;
    const int nbl = text_blocks_of(tl);               // (at most NBW)
    const int nbg = nbw;                              // 32-row text block of this wave
    const bool live = nbg < nbl;
    const int i0 = 32 * nbg;
    const uint16_t* kb = k + (long)b * p.kv.batch + (long)h * p.kv.head;
    const uint16_t* qb = q_txt + (long)b * p.q.batch + (long)h * p.q.head;
    const uint8_t* vb = vis_valid ? vis_valid + (long)b * p.Mv : nullptr;
    const __amdgpu_buffer_rsrc_t rk = row_buffer(kb, p.L, p.kv.token, p.d);
    const uint32_t krow = (uint32_t)(p.kv.token * 2);

    // The sweep runs over "effective" key positions e: the Me vision rows that matter (see
    // effective_rows), then the sample's txt_len text rows (those behind them are seen by no row that counts: 2 x 2000 keys,
    // prompts of up to 600 34.0 -> 30.4 us, 3 x 4608 with up to 300 39.0 -> 37.8); e >= Me is row e + jump of K.  Me is a multiple of 32 (or
    // Mv itself), so a 32-key tile never straddles the jump.  The nch blocks of a (sample, head) take the
    // SLOT_ROWS-key steps in turn (block ch: steps ch, ch + nch, ...): their shares are even whatever Me is,
    // and a block knows where its first steps lie before Me has been found.
    int Me = p.Mv, jump = 0, c1 = 0, nit = 0;
    auto plan = [&]() {
        jump = p.Mv - Me;
        c1 = Me + tl;
        const int steps = (c1 + SLOT_ROWS - 1) / SLOT_ROWS;
        nit = steps > ch ? (steps - ch + p.nch - 1) / p.nch : 0;          // steps of this block
    };
    auto step_row0 = [&](int g) { return (ch + g * p.nch) * SLOT_ROWS; };  // effective position of step g's first key
    // step g's tiles go to slot g % S
    auto issue_step = [&](int g) {
        char* slot = s_k + (g % S) * SLOT_BYTES;
        const int row0 = step_row0(g);
#pragma unroll
        for (int t = 0; t < NLW; ++t) {
            const int sr = (t * NW + wv) * T::RPL;
            T::template issue<STREAM>(rk, krow, row0 + (row0 + sr >= Me ? jump : 0), sr, slot, lane, true);
        }
    };
    // Validity of the 32 keys of this wave's tile in the steps g0 .. g0+63: lane l fetches the 32 mask bytes of
    // step g0 + l and turns them into one word (bit r = key r of the tile is a valid vision token; bytes beyond
    // the sample's Mv slots count as invalid), so a step gets its mask with one lane read and the whole batch
    // costs one round trip.  (A load inside the steady loop would have the compiler wait for everything in
    // flight, the K tiles included, once per step.)
    auto key_valid_masks = [&](int g0) -> uint32_t {
        if (!vb) return 0xFFFFFFFFu;
        return key_valid_mask(vb, (long)step_row0(g0 + lane) + tw * 32, p.Mv);      // first key of the tile
    };

    // Prologue, one round trip: the query tiles (each wave column's tile, its rows split among the column's
    // waves), the scan of the validity mask, and the first S-1 steps of K all go out together.  With a mask the
    // rows that matter (Me) are not known yet: the steps are requested as if they lay below Me, which holds
    // unless the sample has fewer than (S-1) * nch * SLOT_ROWS rows that matter; then they are requested again.
    plan();
#pragma unroll
    for (int g = 0; g < S - 1; ++g)
        if (g < nit) issue_step(g);
    {
        const __amdgpu_buffer_rsrc_t rq = row_buffer(qb, tl, p.q.token, p.d);
#pragma unroll
        for (int t = tw; t < 32 / T::RPL; t += TW)    // this wave's share of its column's 32 query rows
            T::issue(rq, (uint32_t)(p.q.token * 2), i0, t * T::RPL, s_q + nbw * 32 * T::ROWB, lane, true);
    }
    if (vb) {
        const int last = wave_max_int(last_set_partial(vb, p.Mv, threadIdx.x, 64 * NW));
        if (lane == 0) s_last[wv] = last;
    }
    uint32_t vismasks = key_valid_masks(0);           // (its loads belong to the same round trip)
    MD_VM_WAIT(0);
    block_sync_lds();                                 // query tiles complete, mask scanned, first steps landed
    bf16x8 qf[KS];
    read_query_frags<KS>(i0, tl, s_q + nbw * 32 * T::ROWB, lane, qf);
    if (vb) {
        const int nit_guess = nit;
        int last = s_last[0];
#pragma unroll
        for (int w2 = 1; w2 < NW; ++w2) last = max(last, s_last[w2]);
        Me = effective_rows(last, p.Mv);
        plan();
        if (ch == 0 && h == 0 && threadIdx.x == 0) rows[b] = SampleRows{Me, nbl};   // for the second sweep
        const int ahead = min(S - 1, max(nit, nit_guess));
        if (ahead > 0 && step_row0(ahead - 1) + SLOT_ROWS > Me) {            // a requested step reaches beyond Me: again, with the jump
#pragma unroll
            for (int g = 0; g < S - 1; ++g)
                if (g < nit) issue_step(g);
        }
    } else if (ch == 0 && h == 0 && threadIdx.x == 0) {
        rows[b] = SampleRows{p.Mv, nbl};
    }

    float m = -INFINITY, z = 0.f;
    const int i = i0 + (lane & 31);
    // what the arithmetic of a finished tile needs besides its accumulator
    struct Pending { bool all; uint32_t vis; };
    auto visibility = [&](int g) -> Pending {
        const int j0 = step_row0(g) + tw * 32;        // effective position of the tile's first key
        // the tile's 32 keys (vision keys only): valid, and below the rows that matter
        uint32_t vmask = (uint32_t)__builtin_amdgcn_readlane((int)vismasks, g & 63);
        if (j0 + 32 > Me) vmask &= j0 >= Me ? 0u : (1u << (Me - j0)) - 1u;
        Pending pd;
        pd.all = j0 + 32 <= Me && vmask == 0xFFFFFFFFu;
        pd.vis = 0xFFFFu;
        if (!pd.all) {
            uint32_t bits = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = tile_row(r, lane), j = j0 + row;
                const bool vis = j < Me ? ((vmask >> row) & 1u) : (j < c1 && (j - Me) <= i);
                bits |= (vis ? 1u : 0u) << r;
            }
            pd.vis = bits;
        }
        return pd;
    };
    // Step g: wait for its tiles, refill the slot of step g-1, fragments of this wave's tile.
    auto advance = [&](int g) {
        if (g + S - 2 < nit) { MD_VM_WAIT((S - 2) * NLW); } else { MD_VM_WAIT(0); }   // this wave's part of step g has landed
        block_sync_lds();                             // ... and everyone else's; step g-1's slot is free
        if (g + S - 1 < nit) issue_step(g + S - 1);
    };
    auto fetch = [&](int g, bf16x8 (&kf)[KS]) {
        advance(g);
        T::frags(T::frag_base(s_k + (g % S) * SLOT_BYTES + tw * 32 * T::ROWB, lane), kf);
    };
    // The MFMA chain of step g is issued together with the arithmetic on the tile of step g-1.
    auto step = [&](int g, f32x16& acc_new, const f32x16& acc_old, Pending& pend) {
        bf16x8 kf[KS];
        fetch(g, kf);
        if (pend.all) {
            acc_new = score_tile<KS>(kf, qf);
            online_update_all(acc_old, scale_log2e, m, z);
            interleave_mfma_valu<KS>();
        } else {
            acc_new = score_tile<KS>(kf, qf);
            online_update_masked(acc_old, pend.vis, scale_log2e, m, z);
        }
        pend = visibility(g);
        if ((g & 63) == 63 && g + 1 < nit) vismasks = key_valid_masks(g + 1);   // (drains the loads in flight: once per 64 steps)
    };
    f32x16 accA, accB;
    Pending pend{true, 0xFFFFu};
    if (!live) {                                      // wave-uniform: no text rows here, K still comes in through every wave
        for (int g = 0; g < nit; ++g) advance(g);
        nit = 0;
    }
    if (nit > 0) {
        bf16x8 kf[KS];
        fetch(0, kf);
        accA = score_tile<KS>(kf, qf);
        pend = visibility(0);
    }
    int g = 1;
    for (; g + 1 < nit; g += 2) {
        step(g, accB, accA, pend);
        step(g + 1, accA, accB, pend);
    }
    if (g < nit) {
        step(g, accB, accA, pend);
        if (pend.all) online_update_all(accB, scale_log2e, m, z); else online_update_masked(accB, pend.vis, scale_log2e, m, z);
    } else if (nit > 0) {
        if (pend.all) online_update_all(accA, scale_log2e, m, z); else online_update_masked(accA, pend.vis, scale_log2e, m, z);
    }
    MD_VM_WAIT(0);
    // the fragment-major copy of the text queries for the second sweep (here, where no load waits behind the stores)
    if (ch == 0 && tw == 0 && live) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qfrag[((((long)b * p.H + h) * (p.Npad / 32) + nbg) * KS + ks) * kWave + lane] = qf[ks];
    }
    // merge the two lane halves (same text row, the other 16 keys), then the tile lanes
    {
        const float mo = __shfl_xor(m, 32, kWave), zo = __shfl_xor(z, 32, kWave);
        const float mn = fmaxf(m, mo);
        float zn = 0.f;
        if (mn > -INFINITY) zn = z * fast_exp2(m - mn) + zo * fast_exp2(mo - mn);
        if (lane < 32) { s_m[wv][lane] = mn; s_z[wv][lane] = zn; }
    }
    __syncthreads();
    if (threadIdx.x < 32 * NBW) {
        const int nb = threadIdx.x >> 5, r = threadIdx.x & 31;
        float mn = -INFINITY;
#pragma unroll
        for (int t = 0; t < TW; ++t) mn = fmaxf(mn, s_m[t * NBW + nb][r]);
        float zn = 0.f;
        if (mn > -INFINITY) {
#pragma unroll
            for (int t = 0; t < TW; ++t) zn += s_z[t * NBW + nb][r] * fast_exp2(s_m[t * NBW + nb][r] - mn);
        }
        const int ii = 32 * nb + r;
        if (nb < nbl) {
            if (p.nch == 1)     // the only chunk: fold the statistics right away (see fold_stats)
                cstat[((long)b * p.H + h) * p.Npad + ii] = fold_stats(mn, zn, ii < tl, p.H);
            else
                partial[(((long)b * p.H + h) * p.nch + ch) * p.Npad + ii] = make_float2(mn, zn);
        }
    }
}

// The same for one (tile, text block) of the wide form, whose arithmetic starts with a tree of maxima.
template <int KS>
__device__ __forceinline__ void interleave_chain() {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 14, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
#pragma unroll
    for (int q = 2; q < KS; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x400, KS == 8 ? 1 : 4, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, KS == 8 ? 2 : 7, 0);
        __builtin_amdgcn_sched_group_barrier(0x400, KS == 8 ? 2 : 5, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, KS == 8 ? 3 : 7, 0);
    }
}

// The same sweep with all text blocks of a group in every wave: block = (key chunk, text group, head, sample), four
// waves, and a wave holds the fragments of up to four text blocks in registers and has key tiles, LDS slots and a place
// in the sum of its own.  A key fragment is read from LDS once for all of the text blocks, not once per text block, and
// the steady loop has no barrier: a wave waits for its own loads only.  Two such blocks fit a CU, so that one's prologue
// runs beside the other's arithmetic (one block of eight waves per CU: 5 to 35 % slower at the sizes below).
// Bound by the exponentials and the matrix product of a wave, which the steady loop interleaves, wherever K comes from L2,
// as it does for all text groups of a sample but one: 6 x 1152 keys, 32 heads, 384 text rows 69 -> 49 us, 20 x 576 with 200
// rows 77 -> 59, 3 x 9000 with 200 rows 88 -> 77; heads of 64 with the merge, 4 x 4000 keys, 300 rows 63 -> 55, 8 x 2000, 160
// rows 45 -> 31.
template <int KS, bool STREAM>
__global__ __launch_bounds__(256, 2) void prefill_rowstats_wide_kernel(
    const uint16_t* __restrict__ q_txt, const uint16_t* __restrict__ k,
    const uint8_t* __restrict__ vis_valid, const int32_t* __restrict__ txt_len, PrefillDims p, float scale_log2e,
    float2* __restrict__ partial, float* __restrict__ cstat, bf16x8* __restrict__ qfrag, SampleRows* __restrict__ rows)
{
    using T = LdsRows<KS>;
    constexpr int NW = 4, NBMAX = 4;
    constexpr int S = KS == 8 ? 2 : 4;                // tiles under way per wave: 64 KB per block, two blocks per CU
    constexpr int TILE_BYTES = 32 * T::ROWB;
    constexpr int NLT = 32 / T::RPL;                  // load instructions per tile
    // slot s of wave w at (s * NW + w) * TILE_BYTES; the query tiles lie in the last slots until they are in registers,
    // a wave's statistics in its first one once the sweep is done
    __shared__ __attribute__((aligned(1024))) char s_k[S * NW * TILE_BYTES];
    static_assert(NBMAX <= NW && NBMAX * 32 * (int)sizeof(float2) <= TILE_BYTES, "query tiles and statistics fit the slots");
    char* const s_q = s_k + (S - 1) * NW * TILE_BYTES;
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    // one text group: grid (chunk, head, sample).  Several: the blocks of one (chunk, head, sample) read the same K at the
    // same time, so they follow each other on one XCD (blocks go round-robin over the 8 XCDs, each with its own L2)
    int ch = blockIdx.x, tg = 0, h = blockIdx.y, b = blockIdx.z;
    if (p.ng > 1) {
        const int q = (int)blockIdx.x >> 3;
        tg = q % p.ng;
        int item = (q / p.ng) * 8 + ((int)blockIdx.x & 7);
        if (item >= p.B * p.H * p.nch) return;
        ch = item % p.nch; item /= p.nch;
        h = item % p.H; b = item / p.H;
    }
    const int tl = txt_len ? min(max(txt_len[b], 0), p.N) : p.N;
    const int nbl = text_blocks_of(tl), ngl = text_groups_of(nbl, NBMAX);
    if (tg > 0 && tg >= ngl) return;                  // (group 0 stays: it says how many rows matter)
    const TextGroup grp = ngl > 0 ? text_group(tg, nbl, ngl) : TextGroup{0, 0};
    const uint16_t* kb = k + (long)b * p.kv.batch + (long)h * p.kv.head;
    const uint16_t* qb = q_txt + (long)b * p.q.batch + (long)h * p.q.head;
    const uint8_t* vb = vis_valid ? vis_valid + (long)b * p.Mv : nullptr;
    const __amdgpu_buffer_rsrc_t rk = row_buffer(kb, p.L, p.kv.token, p.d);
    const uint32_t krow = (uint32_t)(p.kv.token * 2);

    // effective key positions as in prefill_rowstats_kernel; tile g of this wave is tile (g * nch + ch) * NW + wv
    int Me = p.Mv, jump = 0, c1 = 0, nit = 0;
    auto tile_row0 = [&](int g) { return ((g * p.nch + ch) * NW + wv) * 32; };
    auto plan = [&]() {
        jump = p.Mv - Me;
        c1 = Me + tl;
        const int tiles = (c1 + 31) / 32, first = ch * NW + wv, every = p.nch * NW;
        nit = tiles > first ? (tiles - first + every - 1) / every : 0;
    };
    auto slot_of = [&](int g) { return s_k + ((g % S) * NW + wv) * TILE_BYTES; };
    auto issue_tile = [&](int g, bool live = true) {
        const int row0 = tile_row0(g), src0 = row0 + (row0 >= Me ? jump : 0);
        char* slot = slot_of(g);
        int l = lane;
        asm volatile("" : "+v"(l));                   // the lane's offsets are made anew: registers are what this kernel lacks
#pragma unroll
        for (int t = 0; t < NLT; ++t) T::template issue<STREAM>(rk, krow, src0, t * T::RPL, slot, l, live);
    };
    // validity of the 32 keys of the tiles g0 .. g0+63, one per lane (see prefill_rowstats_kernel)
    auto key_valid_masks = [&](int g0) -> uint32_t {
        if (!vb) return 0xFFFFFFFFu;
        return key_valid_mask(vb, (long)tile_row0(g0 + lane), p.Mv);
    };

    // prologue, one round trip: the query tiles, the first S-1 tiles of K as if they lay below Me, the scan of the mask
    // (every wave for itself)
    plan();
    {
        const __amdgpu_buffer_rsrc_t rq = row_buffer(qb, tl, p.q.token, p.d);
        for (int e = wv; e < grp.count * NLT; e += NW)
            T::issue(rq, (uint32_t)(p.q.token * 2), 32 * (grp.first + e / NLT), (e % NLT) * T::RPL, s_q + (e / NLT) * TILE_BYTES, lane, true);
    }
    const bool one_go = MaskRow::fits(vb, p.Mv);      // block-uniform
    MaskRow mrow;
    if (one_go) mrow.request(vb, p.Mv, lane);
#pragma unroll
    for (int g = 0; g < S - 1; ++g) issue_tile(g, g < nit);
    int last = p.Mv - 1;
    uint32_t vismasks = 0xFFFFFFFFu;
    if (one_go) {
        vismasks = mrow.digest(p.Mv, lane, tile_row0(lane) / 32, last);
    } else if (vb) {
        last = __builtin_amdgcn_readfirstlane(wave_max_int(last_set_partial(vb, p.Mv, lane, kWave)));
        vismasks = key_valid_masks(0);
    }
    MD_VM_WAIT((S - 1) * NLT);
    block_sync_lds();                                 // query tiles complete
    const int guess = nit;
    Me = effective_rows(last, p.Mv);
    plan();

    auto sweep = [&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        bf16x8 qf[NB][KS];
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            T::frags_wait(T::frag_base(s_q + t * TILE_BYTES, lane), qf[t]);
            const int rows_here = tl - 32 * (grp.first + t);
            if (rows_here < 32) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    if ((lane & 31) >= rows_here) qf[t][ks] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
            }
        }
        block_sync_lds();                             // the query tiles' place is free
        {
            const int ahead = min(S - 1, max(nit, guess));
            const bool again = Me < p.Mv && ahead > 0 && tile_row0(ahead - 1) + 32 > Me;   // a requested tile reaches beyond Me
#pragma unroll 1
            for (int g = again ? 0 : S - 1; g < S; ++g)
                if (g < nit) issue_tile(g);
        }

        float m[NB], z[NB];
#pragma unroll
        for (int t = 0; t < NB; ++t) { m[t] = -INFINITY; z[t] = 0.f; }
        struct TileVis { bool all; int j0; uint32_t vmask; };         // first key; its valid vision keys
        auto visibility = [&](int g) -> TileVis {
            TileVis v;
            v.j0 = tile_row0(g);
            v.vmask = (uint32_t)__builtin_amdgcn_readlane((int)vismasks, g & 63);
            if (v.j0 + 32 > Me) v.vmask &= v.j0 >= Me ? 0u : (1u << (Me - v.j0)) - 1u;
            v.all = v.j0 + 32 <= Me && v.vmask == 0xFFFFFFFFu;
            return v;
        };
        // scores of invisible keys to -inf: text row i of block t sees the valid vision keys and text keys 0 .. i
        auto hide = [&](f32x16& acc, const TileVis& v, int t) {
            int l = lane;
            asm volatile("" : "+v"(l));
            auto below = [](int n) { return n >= 32 ? 0xFFFFFFFFu : n <= 0 ? 0u : (1u << n) - 1u; };
            const int i = 32 * (grp.first + t) + (l & 31);
            const uint32_t text = below(min(c1, Me + i + 1) - v.j0) & ~below(Me - v.j0);
            const uint32_t vis = (v.vmask | text) >> (4 * (l >> 5));          // bit 8 * (r / 4) + r % 4: key of register r
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = (vis >> tile_row(r, 0)) & 1u ? acc[r] : -INFINITY;
        };
        // The MFMA chain of a (tile, text block) is issued together with the arithmetic on the one before it.
        TileVis prev{false, c1, 0u};                  // before the first tile: nothing visible
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        for (int g = 0; g < nit; ++g) {
            if (g + S - 1 < nit) { MD_VM_WAIT((S - 1) * NLT); } else { MD_VM_WAIT(0); }
            bf16x8 kf[KS];
            T::frags_wait(T::frag_base(slot_of(g), lane), kf);
            if (g + S < nit) issue_tile(g + S);
            const TileVis cur = visibility(g);
            auto chain = [&](int t, int tu) {
                const f32x16 nw = score_tile<KS>(kf, qf[t]);
                online_update_any(acc, scale_log2e, m[tu], z[tu]);
                acc = nw;
            };
            // (the two forms apart, so that the common one is straight-line code)
            if (prev.all) {
                chain(0, NB - 1);
                interleave_chain<KS>();
            } else {
                hide(acc, prev, NB - 1);
                chain(0, NB - 1);
            }
            if (cur.all) {
#pragma unroll
                for (int t = 1; t < NB; ++t) {
                    __builtin_amdgcn_sched_barrier(0);
                    chain(t, t - 1);
                    interleave_chain<KS>();
                }
            } else {
#pragma unroll
                for (int t = 1; t < NB; ++t) {
                    hide(acc, cur, t - 1);
                    chain(t, t - 1);
                }
            }
            prev = cur;
            if ((g & 63) == 63 && g + 1 < nit) vismasks = key_valid_masks(g + 1);
        }
        if (!prev.all) hide(acc, prev, NB - 1);
        online_update_any(acc, scale_log2e, m[NB - 1], z[NB - 1]);
        // a wave that the mask left without tiles has waited for none of those it requested ahead, and its statistics go to one's place
        MD_VM_WAIT(0);
        // the fragment-major copy of the text queries for the second sweep, shared out over the waves
        if (ch == 0) {
#pragma unroll
            for (int t = 0; t < NB; ++t)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    if (wv == ks % NW) qfrag[((((long)b * p.H + h) * (p.Npad / 32) + grp.first + t) * KS + ks) * kWave + lane] = qf[t][ks];
        }
        // merge the two lane halves (same text row, the other 16 keys); the wave's statistics go to its own first slot
        float2* const sv = reinterpret_cast<float2*>(s_k + wv * TILE_BYTES);
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            const float mo = __shfl_xor(m[t], 32, kWave), zo = __shfl_xor(z[t], 32, kWave);
            const float mn = fmaxf(m[t], mo);
            float zn = 0.f;
            if (mn > -INFINITY) zn = z[t] * fast_exp2(m[t] - mn) + zo * fast_exp2(mo - mn);
            if (lane < 32) sv[t * 32 + lane] = make_float2(mn, zn);
        }
    };
    if (ch == 0 && tg == 0 && h == 0 && threadIdx.x == 0) rows[b] = SampleRows{effective_rows(last, p.Mv), nbl};   // for the second sweep
    if (grp.count == 0) return;                       // no text rows in this sample
    if (grp.count == 4) sweep(std::integral_constant<int, 4>());
    else if (grp.count == 3) sweep(std::integral_constant<int, 3>());
    else if (grp.count == 2) sweep(std::integral_constant<int, 2>());
    else sweep(std::integral_constant<int, 1>());
    __syncthreads();
    if ((int)threadIdx.x < 32 * grp.count) {
        const int r = threadIdx.x;
        auto stat = [&](int w) { return reinterpret_cast<const float2*>(s_k + w * TILE_BYTES)[r]; };
        float mn = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) mn = fmaxf(mn, stat(w).x);
        float zn = 0.f;
        if (mn > -INFINITY) {
#pragma unroll
            for (int w = 0; w < NW; ++w) zn += stat(w).y * fast_exp2(stat(w).x - mn);
        }
        const int ii = 32 * grp.first + r;
        if (p.nch == 1) cstat[((long)b * p.H + h) * p.Npad + ii] = fold_stats(mn, zn, ii < tl, p.H);
        else partial[(((long)b * p.H + h) * p.nch + ch) * p.Npad + ii] = make_float2(mn, zn);
    }
}

// Several key chunks per (sample, head): merge their partial statistics.  One thread per text row.
__global__ __launch_bounds__(256) void prefill_cstat_kernel(
    const float2* __restrict__ partial, const int32_t* __restrict__ txt_len, PrefillDims p, float* __restrict__ cstat)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)p.B * p.H * p.Npad) return;
    const int i = (int)(e % p.Npad);
    const long bh = e / p.Npad;
    const int b = (int)(bh / p.H);
    const int tl = txt_len ? min(max(txt_len[b], 0), p.N) : p.N;
    const float2* pp = partial + bh * p.nch * p.Npad + i;
    float mn = -INFINITY, zn = 0.f;
    for (int c = 0; c < (i < tl ? p.nch : 0); ++c) {   // (nothing was written for text blocks beyond txt_len)
        const float2 v = pp[(long)c * p.Npad];
        const float m2 = fmaxf(mn, v.x);
        if (m2 > -INFINITY) zn = zn * fast_exp2(mn - m2) + v.y * fast_exp2(v.x - m2);
        mn = m2;
    }
    cstat[e] = fold_stats(mn, zn, i < tl, p.H);
}

// The text-query fragments alone (the caller brought the row statistics, so sweep 1 does not run):
// one wave per (sample, head, 32-row text block).
template <int KS>
__global__ __launch_bounds__(256) void prefill_qpack_kernel(
    const uint16_t* __restrict__ q_txt, const uint8_t* __restrict__ vis_valid, const int32_t* __restrict__ txt_len,
    const float* __restrict__ row_lse, PrefillDims p, bf16x8* __restrict__ qfrag, float* __restrict__ cstat,
    SampleRows* __restrict__ rows)
{
    using T = LdsRows<KS>;
    __shared__ __attribute__((aligned(1024))) char s_q[4 * 32 * T::ROWB];
    __shared__ int s_last[4];
    const int lane = lane_id(), wv = wave_id();
    const int nbt = p.Npad / 32;
    const long items = (long)p.B * p.H * nbt;
    const long item_blocks = (items + 3) / 4;
    if ((long)blockIdx.x >= item_blocks) {            // the last B blocks: the vision rows that matter, per sample
        const int b = (int)(blockIdx.x - item_blocks);
        int last = p.Mv - 1;
        if (vis_valid) {
            last = wave_max_int(last_set_partial(vis_valid + (long)b * p.Mv, p.Mv, threadIdx.x, 256));
            if (lane == 0) s_last[wv] = last;
            __syncthreads();
            last = max(max(s_last[0], s_last[1]), max(s_last[2], s_last[3]));
        }
        if (threadIdx.x == 0)
            rows[b] = SampleRows{effective_rows(last, p.Mv), text_blocks_of(txt_len ? min(max(txt_len[b], 0), p.N) : p.N)};
        return;
    }
    const long item = (long)blockIdx.x * 4 + wv;
    if (item >= items) return;
    const int nbg = (int)(item % nbt), h = (int)(item / nbt % p.H), b = (int)(item / nbt / p.H);
    const int tl = txt_len ? min(max(txt_len[b], 0), p.N) : p.N;
    bf16x8 qf[KS];
    load_query_frags<KS>(q_txt + (long)b * p.q.batch + (long)h * p.q.head, p.q.token, p.d, 32 * nbg, tl,
                         s_q + wv * 32 * T::ROWB, lane, qf);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qfrag[(item * KS + ks) * kWave + lane] = qf[ks];
    // the caller's log-sum-exp (natural log, over the keys the row sees) as the folded statistic:
    // exp(s*scale - lse) / H = exp2(s*scale*log2e + c), c = -lse*log2e - log2(H)
    if (lane < 32) {
        const int i = 32 * nbg + lane;
        const float lse = row_lse[((long)b * p.H + h) * p.N + min(i, p.N - 1)];
        cstat[((long)b * p.H + h) * p.Npad + i] = i < tl ? -lse * kLog2e - fast_log2((float)p.H) : -INFINITY;
    }
}

// ---------------------------------------------------------------------------------------------
// Sweep 2: head-mean probabilities.  The work is cut into units (kb vision keys of a sample, one head; kb = 64,
// or 128 with a single text block: smaller key groups mean smaller pieces and less to hand over, at the price of
// the query fragments being fetched from L2 more often per K byte; 64 measured best where a block holds two or
// four text blocks, 32 worse);
// a persistent grid of P blocks (one or two per CU) takes equal, contiguous runs of units
// [p*U/P, (p+1)*U/P), ordered (sample, key group, head), whatever the shape: no block count has to
// match the chip.  A block of 4 waves holds a [kb keys x 32*NBW text rows] tile of a[i][j] in
// registers (wave w: text block w % NBW, the KT key tiles of tile lane w / NBW) and adds one head's
// probabilities per unit.  With more than 128 text rows the text groups are units of their own in the same launch, next to
// each other: 3 x 4608 keys, 100 to 300 text rows, 84 us with one launch per group and all of them full, 47 us now;
// key groups of 128 there: 47 and 2 us more for the pieces.  Per unit the kb K rows go global -> registers -> LDS (two slots; the rows
// of unit u+2 are requested while unit u is worked on), the wave's text-query fragments come from
// qfrag (coalesced).  The row statistics are folded into one constant per (head, text row):
// p = exp2(s*scale*log2e + c), c = -m - log2(Z*H) (cstat: from sweep 1, or from the caller's
// log-sum-exp), so a probability costs one FMA and one exp2.  The MFMA chain of a key tile is issued together with the exp2 work of the tile before it.
// Where a run leaves a key group (or ends) the block writes its head-partial sums a[j][i] as one
// "piece" (fp32, key-major); prefill_colfix_kernel adds a key group's pieces in a fixed order and
// reduces over the text rows (Eq. 8 / Eq. 10).  Which block holds which piece is a function of the
// shapes alone, so the result does not depend on timing.
struct SampleTiles { int b, tile0, nk, nbl, nt; };                // a sample: first tile, key groups, text blocks and groups
// The samples b0 .. b0 + 63, one per lane: their tiles and the sum of tiles up to and with each (one vector load and a lane
// scan; a loop over scalar loads is a dependent chain).
struct LaneTiles { int nk, nbl, nt, n, incl; };
__device__ __forceinline__ LaneTiles lane_tiles(const SampleRows* __restrict__ rows, int B, int kb, int nbw, int b0, int before) {
    const int b = b0 + lane_id();
    const SampleRows r = rows[min(b, B - 1)];
    LaneTiles lt;
    lt.nk = key_groups(r.vision, kb); lt.nbl = r.text_blocks; lt.nt = text_groups_of(r.text_blocks, nbw);
    lt.n = b < B ? lt.nk * lt.nt : 0;
    lt.incl = wave_incl_scan_i(lt.n) + before;
    return lt;
}
__device__ __forceinline__ SampleTiles sample_at_lane(const LaneTiles& lt, int b0, int l) {
    return SampleTiles{b0 + l, __builtin_amdgcn_readlane(lt.incl - lt.n, l), __builtin_amdgcn_readlane(lt.nk, l),
                       __builtin_amdgcn_readlane(lt.nbl, l), __builtin_amdgcn_readlane(lt.nt, l)};
}
__device__ __forceinline__ unsigned long long lane_with_tile(const LaneTiles& lt, int t) {
    return __ballot(lt.incl > t && lt.n > 0 && lt.incl - lt.n <= t);
}
// All samples: the number of tiles, and in `s` the sample that holds tile `t` (find_tile) or sample `t` itself.
__device__ __forceinline__ int find_sample(const SampleRows* __restrict__ rows, int B, int kb, int nbw, bool find_tile, int t, SampleTiles& s) {
    if (B == 1) {
        const SampleRows r = rows[0];
        s = SampleTiles{0, 0, key_groups(r.vision, kb), r.text_blocks, text_groups_of(r.text_blocks, nbw)};
        return s.nk * s.nt;
    }
    int tiles = 0;
    s = SampleTiles{0, 0, 0, 0, 0};
    for (int b0 = 0; b0 < B; b0 += kWave) {
        const LaneTiles lt = lane_tiles(rows, B, kb, nbw, b0, tiles);
        const unsigned long long hit = find_tile ? lane_with_tile(lt, t) : __ballot(b0 + lane_id() == t);
        if (hit) s = sample_at_lane(lt, b0, __builtin_ctzll(hit));
        tiles = __builtin_amdgcn_readlane(lt.incl, kWave - 1);
    }
    return tiles;
}

// MULTI: samples may have several text groups.  STREAM: K comes by streaming loads.
template <int NBW, int KT, int KS, bool MULTI, bool STREAM>
__global__ __launch_bounds__(256, 2) void prefill_colscore_kernel(
    const bf16x8* __restrict__ qfrag, const uint16_t* __restrict__ k, const float* __restrict__ cstat,
    const SampleRows* __restrict__ rows, PrefillDims p, ColPlan cp, float scale_log2e, float* __restrict__ apart)
{
    constexpr int TW = 4 / NBW;
    constexpr int KB = 32 * TW * KT;                  // keys per unit (= cp.kb)
    constexpr int CH = 2 * KS;                        // 16-byte chunks per row
    constexpr int PITCH = CH * 16 + 16;               // padded row pitch: conflict-free 128-bit accesses
    constexpr int SLOT_BYTES = KB * PITCH;
    constexpr int RPL = kWave / CH;                   // rows per load instruction
    constexpr int NLW = KB / RPL / 4;                 // load instructions per wave and unit
    __shared__ __attribute__((aligned(16))) char s_k[2 * SLOT_BYTES];
    const int lane = lane_id(), wv = wave_id();
    const int nbw = wv % NBW, tw = wv / NBW;
    // Blocks go round-robin over the 8 XCDs (each with its own L2): the blocks of one XCD take neighbouring
    // runs, so a sample's query fragments are fetched into one or two L2s, not all eight.
    // Up to 64 samples stay at hand, one per lane, for all that the block asks about them.
    const bool few = p.B <= kWave;
    LaneTiles lt{};
    SampleTiles st0;
    int tiles;
    if (few) { lt = lane_tiles(rows, p.B, KB, NBW, 0, 0); tiles = __builtin_amdgcn_readlane(lt.incl, kWave - 1); }
    else tiles = find_sample(rows, p.B, KB, NBW, false, 0, st0);
    const ColRun run = effective_run(tiles, p.H, cp);
    const int P = run.P;
    const long U = run.U;
    if ((int)blockIdx.x >= P) return;
    const int pb = (P % 8 == 0) ? (int)(blockIdx.x % 8) * (P / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
    const long u0 = index_div((long)pb * U, P), u1 = index_div((long)(pb + 1) * U, P);
    if (u0 >= u1) return;
    const int nbt = p.Npad / 32;
    const long tok_stride = p.kv.token;

    // unit u = (tile, head); tile = (sample, key group, text group), counted over the ones that matter.  The
    // block walks its run with three cursors (the unit being worked on, the one whose fragments are
    // requested, the one whose K rows are requested), each advanced without divisions.
    struct Unit { int b, kg, tg, h, nk, nt, nbl, t; };   // nk, nt, nbl: key groups, text groups, text blocks of sample b; t: tile
    auto at_sample = [&](Unit& x) {
        if (few) {
            x.nk = __builtin_amdgcn_readlane(lt.nk, x.b); x.nbl = __builtin_amdgcn_readlane(lt.nbl, x.b);
        } else {
            const SampleRows r = rows[x.b];
            x.nk = key_groups(r.vision, KB); x.nbl = r.text_blocks;
        }
        x.nt = MULTI ? text_groups_of(x.nbl, NBW) : min(x.nbl, 1);
    };
    auto unit_at = [&](long u) -> Unit {
        Unit x;
        x.t = (int)index_div(u, p.H);
        x.h = (int)(u - (long)x.t * p.H);
        SampleTiles st;
        if (few) st = sample_at_lane(lt, 0, __builtin_ctzll(lane_with_tile(lt, x.t)));
        else find_sample(rows, p.B, KB, NBW, true, x.t, st);
        x.b = st.b; x.nk = st.nk; x.nt = st.nt; x.nbl = st.nbl;
        x.kg = MULTI ? (x.t - st.tile0) / st.nt : x.t - st.tile0;
        x.tg = MULTI ? x.t - st.tile0 - x.kg * st.nt : 0;
        return x;
    };
    auto advance = [&](Unit& x) {
        if (++x.h == p.H) {
            x.h = 0;
            ++x.t;
            if (!MULTI || ++x.tg == x.nt) {
                x.tg = 0;
                if (++x.kg == x.nk) {
                    x.kg = 0;
                    do {
                        if (++x.b == p.B) break;      // behind the last unit
                        at_sample(x);
                    } while (x.nk * x.nt == 0);
                }
            }
        }
    };
    // this wave's 32-row text block in a unit's group; -1: the group has none for it
    auto text_block = [&](const Unit& x) {
        const TextGroup g = MULTI ? text_group(x.tg, x.nbl, x.nt) : TextGroup{0, x.nbl};
        return nbw < g.count ? g.first + nbw : -1;
    };
    // This wave's share of a unit's K rows: NLW x 1 KiB; rows beyond the last vision key repeat it.
    // (`live` false, past the end of the run: every lane reads the same 16 bytes -- the loads stay
    // unconditional, so the compiler can count the loads in flight exactly.)
    auto load_k = [&](const Unit& x, bool live, u32x4 (&st)[NLW]) {
        const uint16_t* kb = k + (long)x.b * p.kv.batch + (long)x.h * p.kv.head + (live ? (lane % CH) * 8 : 0);
#pragma unroll
        for (int t = 0; t < NLW; ++t) {
            const int row = live ? min(x.kg * KB + (t * 4 + wv) * RPL + lane / CH, p.Mv - 1) : 0;
            const u32x4* src = reinterpret_cast<const u32x4*>(kb + (long)row * tok_stride);
            st[t] = STREAM ? __builtin_nontemporal_load(src) : *src;
        }
    };
    auto store_k = [&](int slot, const u32x4 (&st)[NLW]) {
        char* base = s_k + slot * SLOT_BYTES + (lane / CH) * PITCH + (lane % CH) * 16;
#pragma unroll
        for (int t = 0; t < NLW; ++t) *reinterpret_cast<u32x4*>(base + (t * 4 + wv) * RPL * PITCH) = st[t];
    };
    auto load_q = [&](const Unit& x, int nb, bool live, bf16x8 (&qf)[KS]) {
        const bf16x8* qh = qfrag + (((long)x.b * p.H + x.h) * nbt + max(nb, 0)) * KS * kWave + (live ? lane : 0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = qh[live ? ks * kWave : 0];
    };
    // folded row statistic of this lane's text row for the unit's head (-inf beyond txt_len)
    auto load_c = [&](const Unit& x, int nb) -> float {
        return cstat[((long)x.b * p.H + x.h) * p.Npad + 32 * max(nb, 0) + (lane & 31)];
    };
    auto frags = [&](int slot, int kt, bf16x8 (&f)[KS]) {
        const char* q = s_k + slot * SLOT_BYTES + ((tw * KT + kt) * 32 + (lane & 31)) * PITCH + (lane >> 5) * 16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) f[ks] = *reinterpret_cast<const bf16x8*>(q + ks * 32);
    };
    auto add_probs = [&](f32x16& a, const f32x16& acc, float c) {
#pragma unroll
        for (int r = 0; r < 16; ++r) a[r] += fast_exp2(fmaf(acc[r], scale_log2e, c));
    };

    f32x16 a_acc[KT];
    auto clear_acc = [&]() {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) a_acc[kt][r] = 0.f;
    };
    // the piece of the unit's tile that this block holds: apart[piece][b][j][i], text rows contiguous
    auto flush = [&](const Unit& x, int nb) {
        const int piece = pb - unit_block((long)x.t * p.H, P, U);
        if (nb >= 0) {
            float* ap = apart + (((long)piece * p.B + x.b) * p.Mv) * p.Npad + 32 * nb + (lane & 31);
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int j = x.kg * KB + (tw * KT + kt) * 32 + tile_row(r, lane);
                    if (j < p.Mv) ap[(long)j * p.Npad] = a_acc[kt][r];
                }
        }
    };

    // prologue: unit u0 into slot 0, unit u0+1 in registers, fragments and statistic of unit u0
    u32x4 st[NLW];
    bf16x8 qf[KS];
    Unit xc = unit_at(u0), xq = xc, xk = xc;         // cursors: current unit, fragments, K rows
    load_k(xk, true, st);
    int nbc = text_block(xc), nbq = nbc;             // text blocks of the current unit and of the one whose fragments are requested
    load_q(xq, nbq, true, qf);
    float c_cur = load_c(xq, nbq), c_nxt = 0.f;
    store_k(0, st);
    if (u0 + 1 < u1) advance(xk);
    load_k(xk, u0 + 1 < u1, st);
    clear_acc();

    // One unit.  On entry: its K rows are in `slot` (written before the barrier below), the next unit's
    // rows are in `st`, its fragments in qf.  The fragments of the next unit replace them as soon as the
    // last MFMA chain of this unit is under way.
    auto unit_step = [&](long u, int slot) {
        __syncthreads();                              // slot is complete; the other slot is no longer read
        store_k(slot ^ 1, st);                        // unit u+1
        if (u + 2 < u1) advance(xk);
        load_k(xk, u + 2 < u1, st);                   // unit u+2
        if (u + 1 < u1) { advance(xq); nbq = text_block(xq); }
        c_nxt = load_c(xq, nbq);
        // (wave-uniform; a branch only where groups leave columns empty as a rule: it keeps the K traffic above from the
        // arithmetic below, 12 x 634 keys, 32 heads, 34 text rows 14.9 -> 13.6 us; an empty column's sums are not flushed)
        if (!MULTI || nbc >= 0) {
        bf16x8 kfA[KS], kfB[KS];
        f32x16 accA, accB;
        frags(slot, 0, kfA);
        if constexpr (KT > 1) frags(slot, 1, kfB);
        accA = score_tile<KS>(kfA, qf);
#pragma unroll
        for (int kt = 1; kt < KT; ++kt) {
            // the MFMA chain of tile kt together with the exp2 work of tile kt-1
            if (kt & 1) {
                accB = score_tile<KS>(kfB, qf);
                if (kt + 1 < KT) frags(slot, kt + 1, kfA);
                add_probs(a_acc[kt - 1], accA, c_cur);
            } else {
                accA = score_tile<KS>(kfA, qf);
                if (kt + 1 < KT) frags(slot, kt + 1, kfB);
                add_probs(a_acc[kt - 1], accB, c_cur);
            }
        }
        load_q(xq, nbq, u + 1 < u1, qf);              // unit u+1
        add_probs(a_acc[KT - 1], ((KT - 1) & 1) ? accB : accA, c_cur);
        } else {
            load_q(xq, nbq, u + 1 < u1, qf);
        }
        c_cur = c_nxt;
        if (xc.h == p.H - 1 || u + 1 == u1) {         // the run leaves this tile
            flush(xc, nbc);
            clear_acc();
        }
        advance(xc);
        nbc = nbq;
    };
    long u = u0;
    for (; u + 1 < u1; u += 2) {
        unit_step(u, 0);
        unit_step(u + 1, 1);
    }
    if (u < u1) unit_step(u, 0);
}

// The same where one block takes a tile of 32 keys and 32 text rows with all of its heads (ScorePlan::own): no piece is handed
// over and no launch follows.  Block = (sample, 32 vision keys, text block), eight waves of every eighth head each.  A wave's K
// rows lie in two LDS slots of its own, so that the loop over the heads has no barrier; the K rows of the next head and the fragments
// of several are under way while a head is worked on.  What the waves have summed up meets in LDS, where V and I
// come out of it, of each text block by itself (the selection adds them up).  The row statistics of several key chunks are merged here.
// Bound by what a CU can take in: half a megabyte of K and query fragments per block at 64 bytes per clock, 3.6 us, asked for as far
// ahead as the registers hold (four heads' fragments; one head's, measured with one text block: 1 x 3810 keys, 18 text rows, 16 heads
// 34.6 -> 33.2 us a call).  For two to four text blocks (one, and two on more than half of the CUs: prefill_colrows_kernel).
// 1 x 576 keys, 128 text rows: 39 us a call in the persistent form with its sum of the pieces, 28 so; the first sweep gains too, as its
// chunks may be shorter.
template <int KS>
__global__ __launch_bounds__(512) void prefill_colown_kernel(
    const bf16x8* __restrict__ qfrag, const uint16_t* __restrict__ k, const float* __restrict__ cstat, const float2* __restrict__ partial,
    const uint8_t* __restrict__ vis_valid, const int32_t* __restrict__ txt_len, const SampleRows* __restrict__ rows, PrefillDims p,
    float scale_log2e, float* __restrict__ Vout, float* __restrict__ Iout)
{
    using T = LdsRows<KS>;
    constexpr int W = 8, TILE_BYTES = 32 * T::ROWB, NLT = 32 / T::RPL;
    constexpr int CH = kOwnChunks;
    __shared__ __attribute__((aligned(1024))) char s_k[W * 2 * TILE_BYTES];
    const int lane = lane_id(), wv = wave_id(), i = lane & 31;
    // neighbouring tiles of a sample on one XCD (blocks go round the 8 of them), whose L2 then holds the sample's query fragments
    const int nbt = p.Npad / 32, nkg = (p.Mv + 31) / 32, items = p.B * nkg * nbt, per_xcd = (items + 7) / 8;
    const int item = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (item >= items) return;
    const int tile = item / nbt, nb = item - tile * nbt, b = tile / nkg, j0 = (tile - b * nkg) * 32;
    const uint16_t* kb = k + (long)b * p.kv.batch;
    const uint32_t krow = (uint32_t)(p.kv.token * 2);
    char* const slots = s_k + wv * 2 * TILE_BYTES;
    // (behind the last head the last one is asked for again: the loads stay unconditional, so that those in flight can be counted)
    auto issue_k = [&](int h, int slot) {
        const __amdgpu_buffer_rsrc_t rk = row_buffer(kb + (long)min(h, p.H - 1) * p.kv.head, p.L, p.kv.token, p.d);
#pragma unroll
        for (int t = 0; t < NLT; ++t) T::issue(rk, krow, j0, t * T::RPL, slots + slot * TILE_BYTES, lane, true);
    };
    struct Query { bf16x8 f[KS]; float c; float2 st[CH]; };
    auto load_q = [&](int h, Query& q) {
        const long bh = (long)b * p.H + min(h, p.H - 1);
        const bf16x8* qh = qfrag + (bh * nbt + nb) * KS * kWave + lane;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) q.f[ks] = qh[ks * kWave];
        if (p.nch == 1) q.c = cstat[bh * p.Npad + 32 * nb + i];
        else {
#pragma unroll
            for (int u = 0; u < CH; ++u) q.st[u] = partial[(bh * p.nch + min(u, p.nch - 1)) * p.Npad + 32 * nb + i];
        }
    };
    const int tl = txt_len ? min(max(txt_len[b], 0), p.N) : p.N;
    // the statistic of this lane's text row: see prefill_cstat_kernel
    auto statistic = [&](const Query& q) -> float {
        if (p.nch == 1) return q.c;
        float mn = -INFINITY, zn = 0.f;
#pragma unroll
        for (int u = 0; u < CH; ++u)
            if (u < p.nch) mn = fmaxf(mn, q.st[u].x);
        if (mn > -INFINITY) {
#pragma unroll
            for (int u = 0; u < CH; ++u)
                if (u < p.nch) zn = fmaf(q.st[u].y, fast_exp2(q.st[u].x - mn), zn);
        }
        return fold_stats(mn, zn, 32 * nb + i < tl, p.H);
    };
    f32x16 sum;
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[r] = 0.f;
    // K rows of two heads and the fragments of QH are asked for before it is known whether the tile has a valid key
    constexpr int QH = KS == 8 ? 4 : 2;               // (heads of 64: two blocks per CU keep their registers; 4 x 2122 keys, 50 rows 52 us, 57 with four)
    Query q[QH];
    issue_k(wv, 0);
    issue_k(wv + W, 1);
#pragma unroll
    for (int u = 0; u < QH; ++u)
        if (wv + u * W < p.H) load_q(wv + u * W, q[u]);
    const bool work = j0 < rows[b].vision && 32 * nb < tl;                 // block-uniform
    if (work) {
        for (int h0 = wv; h0 < p.H; h0 += QH * W) {
#pragma unroll
            for (int u = 0; u < QH; ++u) {
                const int h = h0 + u * W;
                if (h >= p.H) break;
                const int slot = u & 1;
                MD_VM_WAIT(NLT);                      // all but the K rows of the next head
                bf16x8 kf[KS];
                T::frags_wait(T::frag_base(slots + slot * TILE_BYTES, lane), kf);
                issue_k(h + 2 * W, slot);
                const f32x16 acc = score_tile<KS>(kf, q[u].f);
                const float c = statistic(q[u]);
                if (h + QH * W < p.H) load_q(h + QH * W, q[u]);
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[r] += fast_exp2(fmaf(acc[r], scale_log2e, c));
            }
        }
    }
    MD_VM_WAIT(0);                                    // (nothing writes LDS any more)
    float v_sum = 0.f, i_max = 0.f;                   // of the key 4 * wv + lane / 16, whose text rows 16 lanes share
    if (work) {
        // sums of the waves, [wave][key][text row]
        float* mine = reinterpret_cast<float*>(s_k) + wv * 1024;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[tile_row(r, lane) * 32 + i] = sum[r];
        __syncthreads();
        const float2* part = reinterpret_cast<const float2*>(s_k) + (4 * wv + (lane >> 4)) * 16 + (lane & 15);
        float2 a = make_float2(0.f, 0.f);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float2 x = part[w * 512];
            a.x += x.x;
            a.y += x.y;
        }
        v_sum = group_sum<16>(a.x + a.y);
        i_max = fmaxf(0.f, fmaxf(a.x, a.y));         // (of scores that are not numbers, 0: see prefill_colfix_kernel)
        i_max = fmaxf(i_max, dpp_f<0xB1>(i_max));
        i_max = fmaxf(i_max, dpp_f<0x4E>(i_max));
        i_max = fmaxf(i_max, dpp_f<0x141>(i_max));
        i_max = fmaxf(i_max, dpp_f<0x140>(i_max));
    }
    const int j = j0 + 4 * wv + (lane >> 4);
    if ((lane & 15) == 0 && j < p.Mv) {
        const bool ok = !vis_valid || vis_valid[(long)b * p.Mv + j];
        const long o = ((long)nb * p.B + b) * p.Mv + j;
        Vout[o] = ok ? v_sum : 0.f;
        Iout[o] = ok ? i_max : 0.f;
    }
}

// The same with all text rows of a prompt of up to 64 in a block (ScorePlan::rows; NB text blocks): K is read once, and a head's
// query fragments once per 32 keys.  Nothing is asked for before it is known which tiles have a valid key (a block that takes
// loads along for a tile without one holds up those that wait for its CU: 16 x 576 keys at 3/4, 64 rows, 22.0 us that way, 18.3 so),
// one head's fragments at a time (two heads': 18.3 and 18.0), and the K rows of the next head are what is asked for last, so that the wait
// for the fragments leaves them under way.
// Bound by what comes in: with the fragments of the first head kept, 14.8 us, with K from L2 as well 12.3, which is the launch, the
// plan, the first round trip and the sums; the matrix products and exponentials interleaved instead of one after the other changed
// nothing.  16 x 576 keys at 3/4, 64 rows, row normalisers: 21.1 + 4.3 us for the persistent form and the sum of its pieces, 19.1 here (3.6
// TB/s of K and 7 of fragments from L2); 20 rows 18.5 + 4.4 and 14.0.
// STREAM: K comes by streaming loads.  CHUNKS: the row statistics of several key chunks are merged here.
template <int KS, int NB, bool STREAM, bool CHUNKS>
__global__ __launch_bounds__(512) void prefill_colrows_kernel(
    const bf16x8* __restrict__ qfrag, const uint16_t* __restrict__ k, const float* __restrict__ cstat, const float2* __restrict__ partial,
    const uint8_t* __restrict__ vis_valid, const int32_t* __restrict__ txt_len, const SampleRows* __restrict__ rows, PrefillDims p,
    float scale_log2e, float* __restrict__ Vout, float* __restrict__ Iout)
{
    using T = LdsRows<KS>;
    constexpr int W = 8, TILE_BYTES = 32 * T::ROWB, NLT = 32 / T::RPL;
    constexpr int CH = kOwnChunks;
    __shared__ __attribute__((aligned(1024))) char s_k[W * 2 * TILE_BYTES];
    const int lane = lane_id(), wv = wave_id(), i = lane & 31;
    // The tiles that matter, an eighth of them for each XCD (blocks go round the 8 of them), whose L2 then holds the query fragments of
    // few samples and which all have the same to do whatever the samples' lengths are.
    const int xcd = (int)(blockIdx.x & 7), at = (int)(blockIdx.x >> 3);
    const int nkg = (p.Mv + 31) / 32;
    int tiles = p.B * nkg, b, j0, nbl = NB;           // nbl: text blocks of the sample
    const bool masked = vis_valid || txt_len, few = p.B <= kWave;
    LaneTiles lt{};
    SampleTiles sm{};
    if (masked) {
        if (few) { lt = lane_tiles(rows, p.B, 32, NB, 0, 0); tiles = __builtin_amdgcn_readlane(lt.incl, kWave - 1); }
        else tiles = find_sample(rows, p.B, 32, NB, false, 0, sm);
    }
    const int tile = (int)((long)tiles * xcd >> 3) + at;
    const bool work = tile < (int)((long)tiles * (xcd + 1) >> 3);      // block-uniform
    // keys behind the last valid one, or without text rows (in the end: no block waits for this before its tile)
    auto others = [&]() {
        const long e = (long)blockIdx.x * 512 + threadIdx.x;           // (16 threads for each slot are there)
        if (e >= (long)p.B * p.Mv) return;
        const long s = index_div(e, p.Mv);
        const SampleRows r = rows[s];
        if (r.text_blocks == 0 || (int)(e - s * p.Mv) >= 32 * key_groups(r.vision, 32)) { Vout[e] = 0.f; Iout[e] = 0.f; }
    };
    if (masked) {
        if (!work) { others(); return; }
        if (few) sm = sample_at_lane(lt, 0, __builtin_ctzll(lane_with_tile(lt, tile)));
        else find_sample(rows, p.B, 32, NB, true, tile, sm);
        b = sm.b; j0 = (tile - sm.tile0) * 32; nbl = sm.nbl;
    } else {
        if (!work) return;
        b = tile / nkg; j0 = (tile - b * nkg) * 32;
    }
    // this thread's key at the end: 4 * wv + lane / 16
    const int j = j0 + 4 * wv + (lane >> 4);
    const bool ok = j < p.Mv && (!vis_valid || vis_valid[(long)b * p.Mv + min(j, p.Mv - 1)]);
    float v_sum = 0.f, i_max = 0.f;
    {
        const int tl = txt_len ? min(max(txt_len[b], 0), p.N) : p.N;
        const uint16_t* kb = k + (long)b * p.kv.batch;
        const uint32_t krow = (uint32_t)(p.kv.token * 2);
        char* const slots = s_k + wv * 2 * TILE_BYTES;
        auto issue_k = [&](int h, int slot) {
            const __amdgpu_buffer_rsrc_t rk = row_buffer(kb + (long)h * p.kv.head, p.L, p.kv.token, p.d);
#pragma unroll
            for (int t = 0; t < NLT; ++t) T::template issue<STREAM>(rk, krow, j0, t * T::RPL, slots + slot * TILE_BYTES, lane, true);
        };
        bf16x8 qf[NB][KS];
        float c[NB];
        float2 st[CHUNKS ? CH : 1][NB];
        auto load_q = [&](int h) {
            const long bh = (long)b * p.H + h;
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const bf16x8* qh = qfrag + (bh * NB + t) * KS * kWave + lane;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) qf[t][ks] = qh[ks * kWave];
                if constexpr (!CHUNKS) c[t] = cstat[bh * p.Npad + 32 * t + i];
                else {
#pragma unroll
                    for (int u = 0; u < CH; ++u) st[u][t] = partial[(bh * p.nch + min(u, p.nch - 1)) * p.Npad + 32 * t + i];
                }
            }
        };
        // the statistic of this lane's text row: see prefill_cstat_kernel
        auto statistic = [&](int t) -> float {
            if constexpr (!CHUNKS) return c[t];
            else {
                float mn = -INFINITY, zn = 0.f;
#pragma unroll
                for (int u = 0; u < CH; ++u)
                    if (u < p.nch) mn = fmaxf(mn, st[u][t].x);
                if (mn > -INFINITY) {
#pragma unroll
                    for (int u = 0; u < CH; ++u)
                        if (u < p.nch) zn = fmaf(st[u][t].y, fast_exp2(st[u][t].x - mn), zn);
                }
                return fold_stats(mn, zn, 32 * t + i < tl, p.H);
            }
        };
        f32x16 sum[NB];
#pragma unroll
        for (int t = 0; t < NB; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[t][r] = 0.f;
        if (wv < p.H) { issue_k(wv, 0); load_q(wv); }
        if (wv + W < p.H) issue_k(wv + W, 1);
        int slot = 0;
        for (int h = wv; h < p.H; h += W, slot ^= 1) {
            // all but what was asked for last, the K rows of the next head
            if (h + W < p.H) { MD_VM_WAIT(NLT); } else { MD_VM_WAIT(0); }
            bf16x8 kf[KS];
            T::frags_wait(T::frag_base(slots + slot * TILE_BYTES, lane), kf);
            f32x16 acc[NB];
            float cc[NB];
#pragma unroll
            for (int t = 0; t < NB; ++t) { acc[t] = score_tile<KS>(kf, qf[t]); cc[t] = statistic(t); }
            __builtin_amdgcn_sched_barrier(0);
            if (h + W < p.H) load_q(h + W);
            __builtin_amdgcn_sched_barrier(0);
            if (h + 2 * W < p.H) issue_k(h + 2 * W, slot);
#pragma unroll
            for (int t = 0; t < NB; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) sum[t][r] += fast_exp2(fmaf(acc[t][r], scale_log2e, cc[t]));
        }
        // (nothing writes LDS any more)  Sums of the waves, [wave][key][text row], a text block at a time
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            if (t < nbl) {                 // (nobody wrote fragments and statistics of the others)
                float* mine = reinterpret_cast<float*>(s_k) + (t * W + wv) * 1024;
                if (t == 0) __syncthreads();
#pragma unroll
                for (int r = 0; r < 16; ++r) mine[tile_row(r, lane) * 32 + i] = sum[t][r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            if (t >= nbl) break;
            const float2* part = reinterpret_cast<const float2*>(s_k) + t * W * 512 + (4 * wv + (lane >> 4)) * 16 + (lane & 15);
            float2 a = make_float2(0.f, 0.f);
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const float2 x = part[w * 512];
                a.x += x.x;
                a.y += x.y;
            }
            v_sum += a.x + a.y;
            i_max = fmaxf(i_max, fmaxf(a.x, a.y));    // (of scores that are not numbers, 0: see prefill_colfix_kernel)
        }
        v_sum = group_sum<16>(v_sum);
        i_max = fmaxf(i_max, dpp_f<0xB1>(i_max));
        i_max = fmaxf(i_max, dpp_f<0x4E>(i_max));
        i_max = fmaxf(i_max, dpp_f<0x141>(i_max));
        i_max = fmaxf(i_max, dpp_f<0x140>(i_max));
    }
    if ((lane & 15) == 0 && j < p.Mv) {
        Vout[(long)b * p.Mv + j] = ok ? v_sum : 0.f;
        Iout[(long)b * p.Mv + j] = ok ? i_max : 0.f;
    }
    if (masked) others();
}

// Column statistics (Eq. 8 / Eq. 10): a[i][j] = sum over the pieces of j's key group (fixed order);
// V_j = sum_i a[i][j], I_j = max_i a[i][j].  A wave takes four neighbouring vision keys (same key group, same pieces), 16 lanes
// each, with four text rows per lane and load.  How many pieces there are takes a round trip and two divisions; the
// first `early` pieces of the first text group wait only for the sample's rows to reach the keys at all (what a piece that does
// not exist holds is not added; slots behind the last valid one have none, and reading there all the same took 8 x 950 of 2880
// keys 8.8 us).  us per launch, a row of a key per load and every piece behind that chain / now: 16 x 432 of 576 keys, 64 text
// rows 5.8 / 4.3, 3 x 3456 of 4608, 100 to 300 rows 8.8 / 8.0, 8 x 2160 of 2880, 128 rows 8.4 / 7.7, 8 x 950 6.9 / 5.8.
constexpr int kFixKeys = 4;
// NP: pieces whose loads go out together.
template <int NP>
__global__ __launch_bounds__(256) void prefill_colfix_kernel(
    const float* __restrict__ apart, const uint8_t* __restrict__ vis_valid, const SampleRows* __restrict__ rows,
    PrefillDims p, ColPlan cp, int early, int early_rows, float* __restrict__ Vout, float* __restrict__ Iout)
{
    const int lane = lane_id(), wv = wave_id(), b = blockIdx.y;
    const long gstride = (long)p.B * p.Mv * p.Npad;
    const int j0 = (blockIdx.x * 4 + wv) * kFixKeys;
    if (j0 >= p.Mv) return;
    const int j = j0 + (lane >> 4), c = 4 * (lane & 15);                  // this lane's key; its first text row of 64
    const float* own = apart + ((long)b * p.Mv + min(j, p.Mv - 1)) * p.Npad;
    // text rows `first` + c .. and 64 rows further, of `nrows`; lanes behind them read the last four and drop them
    auto load = [&](int piece, int first, int nrows, f32x4& lo, f32x4& hi) {
        const float* q = own + piece * gstride + first;
        lo = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(q + min(c, nrows - 4)));       // a piece is read once
        hi = nrows > 64 ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(q + min(c + 64, nrows - 4))) : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    constexpr int EARLY = 3;
    f32x4 lo[NP > EARLY ? NP : EARLY], hi[NP > EARLY ? NP : EARLY];
#pragma unroll
    for (int u = 0; u < EARLY; ++u)
        if (u < early && j0 < rows[b].vision) load(u, 0, early_rows, lo[u], hi[u]);
    SampleTiles sm;
    const ColRun run = effective_run(find_sample(rows, p.B, cp.kb, cp.nbw, false, b, sm), p.H, cp);
    // keys behind the rows that matter: no pieces were written, their scores are zero
    const int kg = j0 / cp.kb;
    float s = 0.f, mx = 0.f;
    for (int tg = 0; tg < (kg < sm.nk ? sm.nt : 0); ++tg) {
        const long tile = sm.tile0 + (long)kg * sm.nt + tg;
        const int npieces = unit_block(tile * p.H + p.H - 1, run.P, run.U) - unit_block(tile * p.H, run.P, run.U) + 1;
        const TextGroup grp = text_group(tg, sm.nbl, sm.nt);
        const int first = 32 * grp.first, nrows = 32 * grp.count;         // (at most 128)
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, a2 = {0.f, 0.f, 0.f, 0.f};
        int g = 0;
        if (tg == 0 && nrows <= early_rows) {
#pragma unroll
            for (int u = 0; u < EARLY; ++u)
                if (u < min(npieces, early)) { a += lo[u]; a2 += hi[u]; }
            g = early;
        }
        for (; g < npieces; g += NP) {
#pragma unroll
            for (int u = 0; u < NP; ++u) load(min(g + u, npieces - 1), first, nrows, lo[u], hi[u]);
#pragma unroll
            for (int u = 0; u < NP; ++u)
                if (g + u < npieces) { a += lo[u]; a2 += hi[u]; }
        }
        if (c >= nrows) a = f32x4{0.f, 0.f, 0.f, 0.f};
        if (c + 64 >= nrows) a2 = f32x4{0.f, 0.f, 0.f, 0.f};
        s += ((a.x + a.y) + (a.z + a.w)) + ((a2.x + a2.y) + (a2.z + a2.w));
        mx = fmaxf(mx, fmaxf(fmaxf(fmaxf(a.x, a.y), fmaxf(a.z, a.w)), fmaxf(fmaxf(a2.x, a2.y), fmaxf(a2.z, a2.w))));
    }
    s = group_sum<16>(s);
    mx = fmaxf(mx, dpp_f<0xB1>(mx));
    mx = fmaxf(mx, dpp_f<0x4E>(mx));
    mx = fmaxf(mx, dpp_f<0x141>(mx));
    mx = fmaxf(mx, dpp_f<0x140>(mx));
    if (c == 0 && j < p.Mv) {
        const bool ok = !vis_valid || vis_valid[(long)b * p.Mv + j];
        Vout[(long)b * p.Mv + j] = ok ? s : 0.f;
        Iout[(long)b * p.Mv + j] = ok ? mx : 0.f;
    }
}

// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void prefill_select_kernel(
    PrefillDims p, const float* __restrict__ V, const float* __restrict__ I,
    const uint8_t* __restrict__ vis_valid, const int32_t* __restrict__ txt_len, const uint8_t* __restrict__ is_key,
    int mode, int budget, float gamma, float alpha,
    float* __restrict__ score, int32_t* __restrict__ src_row,
    int32_t* __restrict__ kept_index, int32_t* __restrict__ kept_count,
    int32_t* __restrict__ out_len, uint8_t* __restrict__ out_protect,
    float* __restrict__ score_global, float* __restrict__ score_indiv)
{
    __shared__ float s_redf[16];
    __shared__ int s_red[16];
    __shared__ int s_hist[256];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int Mv = p.Mv;
    const float* Vb = V + (long)b * Mv;
    const float* Ib = I + (long)b * Mv;
    const uint8_t* vb = vis_valid ? vis_valid + (long)b * Mv : nullptr;
    const uint8_t* kb = is_key ? is_key + (long)b * Mv : nullptr;
    float* sc = score + (long)b * Mv;
    const int tl = txt_len ? min(max(txt_len[b], 0), p.N) : p.N;
    const int rows_cap = p.Rcap + p.N;

    // G = sum of V_j over valid vision tokens (Eq. 9, right-hand side); fixed summation tree
    float part = 0.f;
    for (int j = tid; j < Mv; j += blockDim.x) {
        const float v = Vb[j];
        part += v;                                   // invalid tokens carry 0
        if (score_global) score_global[(long)b * Mv + j] = v;
        if (score_indiv) score_indiv[(long)b * Mv + j] = Ib[j];
    }
    const float G = block_sum(part, s_redf);

    SelectBound sb{0ull, 63};
    int extra = 0;
    if (mode == MD_FILTER_BUDGET) {
        int nk = 0, no = 0;
        const float gG = gamma * G;
        for (int j = tid; j < Mv; j += blockDim.x) {
            const bool ok = !vb || vb[j];
            const bool key = ok && kb && kb[j];
            nk += key;
            no += ok && !key;
            const float s1 = G > 0.f ? Vb[j] / gG : 0.f;
            const float s2 = Ib[j] / alpha;
            sc[j] = fmaxf(s1, s2);
        }
        nk = block_sum_i(nk, s_red);
        no = block_sum_i(no, s_red);
        extra = min(max(budget - nk, 0), no);
        __syncthreads();
        if (extra > 0) {
            auto keyfn = [&](int i, bool& ok) -> uint64_t {
                ok = (!vb || vb[i]) && !(kb && kb[i]);
                return ok ? rank_key(sc[i], i) : 0ull;
            };
            sb = block_radix_select(keyfn, Mv, extra, s_hist);
        }
    }
    const float thrV = gamma * G;

    int running = 0;
    for (int base = 0; base < Mv; base += blockDim.x) {
        const int j = base + tid;
        bool keep = false, key = false;
        if (j < Mv && (!vb || vb[j])) {
            key = kb && kb[j];
            if (mode == MD_FILTER_THRESHOLD) {
                const bool drop = (Vb[j] <= thrV) && (Ib[j] < alpha) && !key;
                keep = !drop;
            } else {
                keep = key || (extra > 0 && (rank_key(sc[j], j) >> sb.shift) >= sb.bound);
            }
        }
        int total;
        const int r = block_rank(keep, s_red, total);
        const int o = running + r;
        if (keep && o < p.Rcap) {
            kept_index[(long)b * p.Rcap + o] = j;
            src_row[(long)b * rows_cap + o] = j;
            if (out_protect) out_protect[(long)b * rows_cap + o] = key ? 1 : 0;
        }
        running += total;
    }
    const int nkept = min(running, p.Rcap);
    for (int i = tid; i < rows_cap - nkept; i += blockDim.x) {
        const int o = nkept + i;
        src_row[(long)b * rows_cap + o] = i < tl ? Mv + i : -1;
        if (out_protect && i < tl) out_protect[(long)b * rows_cap + o] = 1;
    }
    if (tid == 0) {
        kept_count[b] = running;
        if (out_len) out_len[b] = nkept + tl;
    }
}

// The same selection with a sample's scores held in registers (Mv <= 1024*IPT): tokens are dealt
// round-robin (thread t owns t, t+1024, ...), every global load is issued up front, the radix passes
// and the prefix sums touch no memory.
// The text rows of the outputs need no selection: in budget mode their place follows from counting the
// valid and the key tokens.  While the one block per sample of the selection kernel works through its
// dependent steps on 1 CU in 16, further blocks of the same launch copy those rows (hidden, K, V).
struct TextRows {
    const u32x4* hidden; const u32x4* k; const u32x4* v;
    u32x4* hidden_out; u32x4* k_out; u32x4* v_out;
    int enabled;
    int stream_k;                                    // see prefill_compact_kernel
};
constexpr int kTextRowsPerBlock = 4;                 // 1024 threads = four rows of 256 threads

template <int IPT>
__device__ __forceinline__ void copy_text_rows(
    const PrefillDims& p, const TextRows& tr, const uint8_t* __restrict__ vis_valid, const int32_t* __restrict__ txt_len,
    const uint8_t* __restrict__ is_key, int budget, int* s_red)
{
    const int tid = threadIdx.x, Mv = p.Mv;
    const int bps = (p.N + kTextRowsPerBlock - 1) / kTextRowsPerBlock;        // blocks per sample
    const int e = blockIdx.x - p.B, b = e / bps, i = (e % bps) * kTextRowsPerBlock + tid / 256;
    // the number of vision rows kept, exactly as the selection block of this sample counts it
    uint32_t vv[IPT], kk[IPT];
#pragma unroll
    for (int t = 0; t < IPT; ++t) vv[t] = vis_valid ? vis_valid[(long)b * Mv + min(tid + t * 1024, Mv - 1)] : 1u;
#pragma unroll
    for (int t = 0; t < IPT; ++t) kk[t] = is_key ? is_key[(long)b * Mv + min(tid + t * 1024, Mv - 1)] : 0u;
    const int tl = txt_len ? min(max(txt_len[b], 0), p.N) : p.N;
    int cnt = 0;
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        const bool ok = tid + t * 1024 < Mv && vv[t] != 0;
        cnt += (ok && kk[t] != 0 ? 1 : 0) + ((ok && kk[t] == 0) ? 1 << 16 : 0);
    }
    cnt = block_sum_i(cnt, s_red);
    const int nk = cnt & 0xFFFF, no = cnt >> 16;
    const int nkept = min(nk + min(max(budget - nk, 0), no), p.Rcap);
    if (i >= tl) return;
    const int rows_cap = p.Rcap + p.N;
    const int hv = p.C / 8, kv = p.H * p.d / 8, c0 = tid % 256;
    const long src = (long)b * p.L + Mv + i, dst = (long)b * rows_cap + nkept + i;
    // (a loop each: a branch around the one store would be folded into a plain one)
    auto kv_rows = [&](auto stream_k) {
        for (int c = c0; c < kv; c += 256) {
            const u32x4 a = __builtin_nontemporal_load(tr.k + src * kv + c), a2 = __builtin_nontemporal_load(tr.v + src * kv + c);
            if constexpr (decltype(stream_k)::value) __builtin_nontemporal_store(a, tr.k_out + dst * kv + c);
            else tr.k_out[dst * kv + c] = a;
            __builtin_nontemporal_store(a2, tr.v_out + dst * kv + c);      // streaming stores: see prefill_compact_kernel
        }
    };
    if (tr.stream_k) kv_rows(std::true_type()); else kv_rows(std::false_type());
    for (int c = c0; c < hv; c += 256)
        __builtin_nontemporal_store(__builtin_nontemporal_load(tr.hidden + src * hv + c), tr.hidden_out + dst * hv + c);
}

// PARTS: V and I come as one array per text block.
template <int IPT, bool PARTS>
__global__ __launch_bounds__(1024) void prefill_select_fast_kernel(
    PrefillDims p, const float* __restrict__ V, const float* __restrict__ I, int parts,
    const uint8_t* __restrict__ vis_valid, const int32_t* __restrict__ txt_len, const uint8_t* __restrict__ is_key,
    int mode, int budget, float gamma, float alpha,
    int32_t* __restrict__ src_row,
    int32_t* __restrict__ kept_index, int32_t* __restrict__ kept_count,
    int32_t* __restrict__ out_len, uint8_t* __restrict__ out_protect,
    float* __restrict__ score_global, float* __restrict__ score_indiv, TextRows tr)
{
    __shared__ float s_redf[16];
    __shared__ int s_red[16];
    __shared__ int s_hist[kSelectHistInts];
    __shared__ int s_rounds[16 * IPT];
    if ((int)blockIdx.x >= p.B) {                    // block-uniform: the blocks that copy the text rows
        copy_text_rows<IPT>(p, tr, vis_valid, txt_len, is_key, budget, s_red);
        return;
    }
    const int b = blockIdx.x, tid = threadIdx.x;
    if (tid < 256) s_hist[tid] = 0;                  // for block_select_topk, after later barriers
    const int Mv = p.Mv;
    const int rows_cap = p.Rcap + p.N;
    float v[IPT], iv[IPT];
    bool ok[IPT], key[IPT];
    {
        // every load at a clamped address and none guarded by another's result: one round trip
        uint32_t vv[IPT], kk[IPT];
#pragma unroll
        for (int t = 0; t < IPT; ++t) v[t] = V[(long)b * Mv + min(tid + t * 1024, Mv - 1)];
#pragma unroll
        for (int t = 0; t < IPT; ++t) iv[t] = I[(long)b * Mv + min(tid + t * 1024, Mv - 1)];
#pragma unroll
        for (int t = 0; t < IPT; ++t) vv[t] = vis_valid ? vis_valid[(long)b * Mv + min(tid + t * 1024, Mv - 1)] : 1u;
#pragma unroll
        for (int t = 0; t < IPT; ++t) kk[t] = is_key ? is_key[(long)b * Mv + min(tid + t * 1024, Mv - 1)] : 0u;
        if constexpr (PARTS) {
            float vq[kOwnParts - 1][IPT], iq[kOwnParts - 1][IPT];
#pragma unroll
            for (int q = 1; q < kOwnParts; ++q)
#pragma unroll
                for (int t = 0; t < IPT; ++t) {
                    const long o = ((long)min(q, parts - 1) * p.B + b) * Mv + min(tid + t * 1024, Mv - 1);
                    vq[q - 1][t] = V[o];
                    iq[q - 1][t] = I[o];
                }
#pragma unroll
            for (int q = 1; q < kOwnParts; ++q)
#pragma unroll
                for (int t = 0; t < IPT; ++t)
                    if (q < parts) { v[t] += vq[q - 1][t]; iv[t] = fmaxf(iv[t], iq[q - 1][t]); }
        }
#pragma unroll
        for (int t = 0; t < IPT; ++t) {
            const bool in = tid + t * 1024 < Mv;
            if (!in) { v[t] = 0.f; iv[t] = 0.f; }
            ok[t] = in && vv[t] != 0;
            key[t] = ok[t] && kk[t] != 0;
        }
    }
    const int tl = txt_len ? min(max(txt_len[b], 0), p.N) : p.N;
    // G = sum of V_j over valid vision tokens (Eq. 9, right-hand side); fixed summation tree
    float part = 0.f;
    int cnt = 0;                                     // keys in the low half, other valid tokens in the high half
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        part += v[t];                                // invalid tokens carry 0
        cnt += (key[t] ? 1 : 0) + ((ok[t] && !key[t]) ? 1 << 16 : 0);
        const int j = tid + t * 1024;
        if (j < Mv) {
            if (score_global) score_global[(long)b * Mv + j] = v[t];
            if (score_indiv) score_indiv[(long)b * Mv + j] = iv[t];
        }
    }
    const float G = block_sum(part, s_redf);
    bool keep[IPT];
    if (mode == MD_FILTER_BUDGET) {
        cnt = block_sum_i(cnt, s_red);
        const int nk = cnt & 0xFFFF, no = cnt >> 16;
        const int extra = min(max(budget - nk, 0), no);
        const float gG = gamma * G;
        uint64_t rk[IPT];
#pragma unroll
        for (int t = 0; t < IPT; ++t) {
            const float s1 = G > 0.f ? v[t] / gG : 0.f;
            const float s2 = iv[t] / alpha;
            rk[t] = (ok[t] && !key[t]) ? rank_key(fmaxf(s1, s2), tid + t * 1024) : 0ull;
        }
        const SelectBound sb = block_select_topk<IPT>(rk, extra, s_hist);
#pragma unroll
        for (int t = 0; t < IPT; ++t) keep[t] = key[t] || (rk[t] != 0 && extra > 0 && (rk[t] >> sb.shift) >= sb.bound);
    } else {
        const float thrV = gamma * G;
#pragma unroll
        for (int t = 0; t < IPT; ++t) keep[t] = ok[t] && !((v[t] <= thrV) && (iv[t] < alpha) && !key[t]);
    }
    // ranks of the kept tokens: one barrier for all rounds (two a round before: 5697 tokens 12.8 -> 11.4 us)
    int below[IPT], cnts[IPT], wave_pre[IPT];
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        const unsigned long long kept = __ballot(keep[t]);
        cnts[t] = __popcll(kept);
        below[t] = lanes_below(kept);
    }
    const int running = block_round_prefixes<IPT>(cnts, wave_pre, s_rounds);
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        const int j = tid + t * 1024, o = wave_pre[t] + below[t];
        if (keep[t] && o < p.Rcap) {
            kept_index[(long)b * p.Rcap + o] = j;
            src_row[(long)b * rows_cap + o] = j;
            if (out_protect) out_protect[(long)b * rows_cap + o] = key[t] ? 1 : 0;
        }
    }
    const int nkept = min(running, p.Rcap);
    for (int i = tid; i < rows_cap - nkept; i += blockDim.x) {
        const int o = nkept + i;
        src_row[(long)b * rows_cap + o] = i < tl ? Mv + i : -1;
        if (out_protect && i < tl) out_protect[(long)b * rows_cap + o] = 1;
    }
    if (tid == 0) {
        kept_count[b] = running;
        if (out_len) out_len[b] = nkept + tl;
    }
}

// One block per output row: copies the hidden, K and V rows named by the row map.
// STREAM_K: the K rows too are written with streaming stores.
template <bool STREAM_K>
__global__ __launch_bounds__(256) void prefill_compact_kernel(
    PrefillDims p, const int32_t* __restrict__ src_row,
    const u32x4* __restrict__ hidden, const u32x4* __restrict__ k, const u32x4* __restrict__ v,
    u32x4* __restrict__ hidden_out, u32x4* __restrict__ k_out, u32x4* __restrict__ v_out, int text_done)
{
    const int o = blockIdx.x, b = blockIdx.y;
    const int rows_cap = p.Rcap + p.N;
    const int src = src_row[(long)b * rows_cap + o];
    if (src < 0 || (text_done && src >= p.Mv)) return;     // text rows may have been copied by the selection launch
    const int hv = p.C / 8, kv = p.H * p.d / 8;          // 16-byte vectors per row
    const u32x4* hs = hidden + ((long)b * p.L + src) * hv;
    const u32x4* ks = k + ((long)b * p.L + src) * kv;
    const u32x4* vs = v + ((long)b * p.L + src) * kv;
    u32x4* hd = hidden_out + ((long)b * rows_cap + o) * hv;
    u32x4* kd = k_out + ((long)b * rows_cap + o) * kv;
    u32x4* vd = v_out + ((long)b * rows_cap + o) * kv;
    // every source row is read once (streaming loads; the copies are read again by the next stage),
    // four vectors in flight
    // hidden and V rows are written with streaming stores: nothing on this path reads them again, and left as
    // dirty lines in the Infinity Cache they would be written back in the middle of whatever kernel streams
    // through it next (measured: the sweep that follows 150 MB of plain stores takes 10 us longer); the K
    // rows, which a scoring pass reads next, keep plain stores where streams_k_out says so
    auto put = [](u32x4* q, const u32x4& v, bool nt) { if (nt) __builtin_nontemporal_store(v, q); else *q = v; };
    auto copy2 = [&](const u32x4* __restrict__ s0, u32x4* __restrict__ d0, const u32x4* __restrict__ s1,
                     u32x4* __restrict__ d1, int n, bool nt0, bool nt1) {
        const int step = 2 * blockDim.x;
        for (int c = threadIdx.x; c < n; c += step) {
            const int c2 = c + blockDim.x;
            const bool two = c2 < n;
            const u32x4 a0 = __builtin_nontemporal_load(s0 + c), a1 = __builtin_nontemporal_load(s1 + c);
            u32x4 b0 = a0, b1 = a1;
            if (two) { b0 = __builtin_nontemporal_load(s0 + c2); b1 = __builtin_nontemporal_load(s1 + c2); }
            put(d0 + c, a0, nt0);
            put(d1 + c, a1, nt1);
            if (two) { put(d0 + c2, b0, nt0); put(d1 + c2, b1, nt1); }
        }
    };
    copy2(ks, kd, vs, vd, kv, STREAM_K, true);
    const int half = (hv + 1) / 2;                   // the hidden row as two halves
    copy2(hs, hd, hs + half, hd + half, hv - half, true, true);
    if (hv & 1) {                                    // odd vector count: the first half has one more
        const int c = half - 1;
        if (threadIdx.x == 0) hd[c] = hs[c];
    }
}

// The same for K / V in other layouts: a row is gathered head slice by head slice (d contiguous
// elements each) from the input layout and scattered to the output layout.
template <bool STREAM, bool STREAM_K>
__global__ __launch_bounds__(256) void prefill_compact_strided_kernel(
    PrefillDims p, const int32_t* __restrict__ src_row,
    const u32x4* __restrict__ hidden, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    u32x4* __restrict__ hidden_out, uint16_t* __restrict__ k_out, uint16_t* __restrict__ v_out, KvLayout out)
{
    const int o = blockIdx.x, b = blockIdx.y;
    const int rows_cap = p.Rcap + p.N;
    const int src = src_row[(long)b * rows_cap + o];
    if (src < 0) return;
    const int lph = p.d / 8;                             // 16-byte vectors per head slice
    const int kvn = p.H * lph;
    const long sbase = (long)b * p.kv.batch + (long)src * p.kv.token;
    const long dbase = (long)b * out.batch + (long)o * out.token;
    auto ld = [](const u32x4* q) { return STREAM ? __builtin_nontemporal_load(q) : *q; };
    auto st = [](const u32x4& x, u32x4* q) { if (STREAM) __builtin_nontemporal_store(x, q); else *q = x; };
    for (int c = threadIdx.x; c < kvn; c += blockDim.x) {
        const int h = c / lph, w = c - h * lph;
        const long so = sbase + (long)h * p.kv.head + w * 8, d_o = dbase + (long)h * out.head + w * 8;
        const u32x4 a = ld(reinterpret_cast<const u32x4*>(k + so)), c2 = ld(reinterpret_cast<const u32x4*>(v + so));
        if (STREAM_K) __builtin_nontemporal_store(a, reinterpret_cast<u32x4*>(k_out + d_o));
        else *reinterpret_cast<u32x4*>(k_out + d_o) = a;
        st(c2, reinterpret_cast<u32x4*>(v_out + d_o));
    }
    const int hv = p.C / 8;
    const u32x4* hs = hidden + ((long)b * p.L + src) * hv;
    u32x4* hd = hidden_out + ((long)b * rows_cap + o) * hv;
    for (int c = threadIdx.x; c < hv; c += blockDim.x) st(ld(hs + c), hd + c);
}

struct PrefillWorkspace {
    float2* partial; float* cstat; bf16x8* qfrag; float* apart; float* V; float* I; float* score; int32_t* src_row;
    SampleRows* rows;
    size_t bytes;
    // V and I as the column sweep leaves them: one array each, or one per text block (ScorePlan::own without ::rows, two to
    // four text blocks) in the memory of the pieces, which that form does not write (a piece is at least 32 floats per key and text block)
    struct ScoreParts { float* V; float* I; int parts; };
    ScoreParts score_parts(const PrefillDims& p, const ScorePlan& s) const {
        if (!s.own || s.rows) return ScoreParts{V, I, 1};
        return ScoreParts{apart, apart + (size_t)s.nbt * p.B * p.Mv, s.nbt};
    }
    float2* chunk_stats(const PrefillDims& p, const ScorePlan& s) const {
        return s.partial_in_pieces ? reinterpret_cast<float2*>(apart + 2 * (size_t)s.nbt * p.B * p.Mv) : partial;
    }
};

PrefillWorkspace carve_prefill(void* base, int B, int Mv, int N, int H, int Rcap) {
    Carver c(base);
    PrefillWorkspace w;
    const ScorePlan s = plan_scores(B, Mv, N, H, 128);     // (of the sizes only the number of chunks depends on d)
    const int s64 = plan_scores(B, Mv, N, H, 64).nch_ws, nch = s.nch_ws > s64 ? s.nch_ws : s64;
    const int Npad = s.nbt * 32;
    w.partial = c.take<float2>((size_t)B * H * nch * Npad);
    w.cstat = c.take<float>((size_t)B * H * Npad);
    w.qfrag = c.take<bf16x8>((size_t)B * H * Npad * 16);      // [B][H][NB][KS][64] fragments, d <= 128
    w.apart = c.take<float>((size_t)s.col.Gmax * B * Mv * Npad);
    w.V = c.take<float>((size_t)B * Mv);
    w.I = c.take<float>((size_t)B * Mv);
    w.score = c.take<float>((size_t)B * Mv);
    w.src_row = c.take<int32_t>((size_t)B * (Rcap + N));
    w.rows = c.take<SampleRows>((size_t)B);
    w.bytes = c.off;
    return w;
}

template <int KS>
int launch_scores(const PrefillDims& p, const ScorePlan& s, const PrefillWorkspace& w, hipStream_t st, const void* q_txt,
                  const void* k, const uint8_t* vis_valid, const int32_t* txt_len, const float* row_lse, float scale_log2e, bool col_stream) {
    const uint16_t* qp = static_cast<const uint16_t*>(q_txt);
    const uint16_t* kp = static_cast<const uint16_t*>(k);
    float2* const partial = w.chunk_stats(p, s);
    if (!row_lse) {
        const dim3 g1 = s.ng == 1 ? dim3(p.nch, p.H, p.B) : dim3((unsigned)(((long)p.nch * p.H * p.B + 7) / 8 * 8 * s.ng));
#define MD_ROWSTATS2(NBW_, TW_, ST_, DEEP_)                                                                    \
    MD_LAUNCH("prefill_rowstats", st, (prefill_rowstats_kernel<NBW_, TW_, KS, ST_, DEEP_>), g1, 64 * NBW_ * TW_, 0, \
        qp, kp, vis_valid, txt_len, p, scale_log2e, partial, w.cstat, w.qfrag, w.rows)
#define MD_ROWSTATS(NBW_, TW_)                                                                                 \
        do {                                                                                                   \
            if (KS == 8 && NBW_ * TW_ == 4 && s.rs_stream) MD_ROWSTATS2(NBW_, TW_, (KS == 8 && NBW_ * TW_ == 4), false); \
            else if (KS == 8 && NBW_ == 1 && TW_ == 4 && s.rs_deep) MD_ROWSTATS2(NBW_, TW_, false, (KS == 8 && NBW_ == 1 && TW_ == 4)); \
            else MD_ROWSTATS2(NBW_, TW_, false, false);                                                        \
        } while (0)
#define MD_ROWSTATS_WIDE(ST_)                                                                                  \
    MD_LAUNCH("prefill_rowstats", st, (prefill_rowstats_wide_kernel<KS, ST_>), g1, 256, 0,                     \
        qp, kp, vis_valid, txt_len, p, scale_log2e, partial, w.cstat, w.qfrag, w.rows)
        const bool big = s.rs_waves == 8;
        if (s.rs_wide) { if (KS == 8 && s.rs_stream) MD_ROWSTATS_WIDE((KS == 8)); else MD_ROWSTATS_WIDE(false); }
        else if (s.nbw == 1) { if (big) MD_ROWSTATS(1, 8); else MD_ROWSTATS(1, 4); }
        else if (s.nbw == 2) { if (big) MD_ROWSTATS(2, 4); else MD_ROWSTATS(2, 2); }
        else if (big) MD_ROWSTATS(4, 2);
        else if constexpr (KS == 4) MD_ROWSTATS(4, 1);    // (d = 128: the wide form)
#undef MD_ROWSTATS_WIDE
#undef MD_ROWSTATS
#undef MD_ROWSTATS2
        if (p.nch > 1 && !s.own) {
            const long n = (long)p.B * p.H * p.Npad;
            MD_LAUNCH("prefill_cstat", st, (prefill_cstat_kernel), (unsigned)((n + 255) / 256), 256, 0, partial, txt_len, p, w.cstat);
        }
    } else {
        const long items = (long)p.B * p.H * s.nbt;
        MD_LAUNCH("prefill_qpack", st, (prefill_qpack_kernel<KS>), (unsigned)((items + 3) / 4 + p.B), 256, 0, qp, vis_valid, txt_len,
                  row_lse, p, w.qfrag, w.cstat, w.rows);
    }
    if (s.rows) {
        const long tiles = (long)p.B * ((p.Mv + 31) / 32);
#define MD_COLROWS2(NB_, ST_, CH_)                                                                             \
    MD_LAUNCH("prefill_colscore", st, (prefill_colrows_kernel<KS, NB_, ST_, CH_>), (unsigned)((tiles + 7) / 8 * 8), 512, 0, \
        w.qfrag, kp, w.cstat, partial, vis_valid, txt_len, w.rows, p, scale_log2e, w.V, w.I)
#define MD_COLROWS(NB_)                                                                                        \
    do {                                                                                                       \
        if (row_lse && s.rows_stream) MD_COLROWS2(NB_, true, false);                                           \
        else if (p.nch == 1) MD_COLROWS2(NB_, false, false);                                                   \
        else MD_COLROWS2(NB_, false, true);                                                                    \
    } while (0)
        if (s.nbt == 1) MD_COLROWS(1); else MD_COLROWS(2);
#undef MD_COLROWS
#undef MD_COLROWS2
        return MD_OK;
    }
    if (s.own) {
        MD_LAUNCH("prefill_colscore", st, (prefill_colown_kernel<KS>), (unsigned)((s.own_blocks + 7) / 8 * 8), 512, 0, w.qfrag, kp, w.cstat, partial, vis_valid, txt_len, w.rows,
                  p, scale_log2e, w.score_parts(p, s).V, w.score_parts(p, s).I);
        return MD_OK;
    }
#define MD_COLSCORE(NBW_, KT_, M_, ST_)                                                                        \
    MD_LAUNCH("prefill_colscore", st, (prefill_colscore_kernel<NBW_, KT_, KS, M_, ST_>), s.col.P, 256, 0,          \
        w.qfrag, kp, w.cstat, w.rows, p, s.col, scale_log2e, w.apart)
    // 32 * (4 / NBW) * KT keys per unit = s.col.kb
    if (s.nbw == 1) MD_COLSCORE(1, 1, false, true);
    else if (s.nbw == 2) MD_COLSCORE(2, 1, false, true);
    else if (s.ng == 1) { if (!col_stream) MD_COLSCORE(4, 2, false, false); else MD_COLSCORE(4, 2, false, true); }
    else { if (!col_stream) MD_COLSCORE(4, 2, true, false); else MD_COLSCORE(4, 2, true, true); }
#undef MD_COLSCORE
    const int fx = (p.Mv + 4 * kFixKeys - 1) / (4 * kFixKeys);          // four waves of kFixKeys keys per block
    // pieces that a tile has as a rule, by the length of the blocks' runs (one that has fewer reads in vain), and the rows of the
    // first text group of a full prompt
    int early = s.col.U >= 2l * p.H * s.col.P ? 1 : s.col.U >= (long)p.H * s.col.P ? 2 : 3;
    if (early > s.col.Gmax) early = s.col.Gmax;
    const int early_rows = 32 * ((s.nbt + s.ng - 1) / s.ng);
    // small calls cut a tile into many pieces, a chain of round trips unless four are requested at a time (14 pieces
    // 8.2 -> 6.7 us); the two or three of a large one are bound by their bytes, and by occupancy (8.1 -> 11.3)
    if ((long)p.H * s.col.P >= 4 * s.col.U)
        MD_LAUNCH("prefill_colfix", st, (prefill_colfix_kernel<4>), dim3(fx, p.B), 256, 0, w.apart, vis_valid, w.rows, p, s.col, early, early_rows, w.V, w.I);
    else
        MD_LAUNCH("prefill_colfix", st, (prefill_colfix_kernel<2>), dim3(fx, p.B), 256, 0, w.apart, vis_valid, w.rows, p, s.col, early, early_rows, w.V, w.I);
    return MD_OK;
}

}  // namespace
}  // namespace md

using namespace md;

extern "C" size_t mustdrop_prefill_filter_workspace_bytes(int B, int Mv, int N, int H, int Rcap) {
    if (B <= 0 || Mv <= 0 || N <= 0 || H <= 0 || Rcap <= 0) return 0;
    return carve_prefill(nullptr, B, Mv, N, H, Rcap).bytes;
}

namespace md {
namespace {

int prefill_filter_impl(
    const void* q_txt, const void* k, const void* v, const void* hidden,
    const uint8_t* vis_valid, const int32_t* txt_len, const uint8_t* is_key, const float* row_lse,
    int B, int Mv, int N, int H, int d, int C,
    float softmax_scale, md_filter_mode mode, int budget, float gamma, float alpha,
    int Rcap,
    void* hidden_out, void* k_out, void* v_out,
    int32_t* kept_index, int32_t* kept_count, int32_t* out_len, uint8_t* out_protect, int32_t* out_ids,
    float* score_global, float* score_indiv,
    const md_kv_layout* q_layout, const md_kv_layout* kv_layout, const md_kv_layout* kv_out_layout,
    void* workspace, size_t workspace_bytes, void* stream)
{
    clear_error();
    if (mode != MD_FILTER_BUDGET && mode != MD_FILTER_THRESHOLD) return fail(MD_EDTYPE, "prefill_filter: unknown mode %d", (int)mode);
    if (B <= 0 || Mv <= 0 || N <= 0 || H <= 0 || d <= 0 || C <= 0 || Rcap <= 0)
        return fail(MD_EINVAL, "prefill_filter: B, Mv, N, H, d, C, Rcap must be positive");
    if (!q_txt || !k || !v || !hidden || !hidden_out || !k_out || !v_out || !kept_index || !kept_count)
        return fail(MD_EINVAL, "prefill_filter: q_txt, k, v, hidden, the *_out tensors, kept_index and kept_count are required");
    if (d != 64 && d != 128) return fail(MD_ESHAPE, "prefill_filter: head dim %d not supported (64 or 128)", d);
    if (N > 1024) return fail(MD_ESHAPE, "prefill_filter: N=%d text tokens exceeds the limit of 1024", N);
    if (H > 128) return fail(MD_ESHAPE, "prefill_filter: H=%d heads exceeds the limit of 128", H);
    if ((long)B * (Mv + N) > (1l << 28)) return fail(MD_ESHAPE, "prefill_filter: too many tokens");
    if (C % 8) return fail(MD_EALIGN, "prefill_filter: a hidden row of C=%d bf16 is not a multiple of 16 bytes", C);
    if (std::isnan(softmax_scale) || std::isnan(gamma) || std::isnan(alpha)) return fail(MD_EINVAL, "prefill_filter: NaN parameter");
    if (!(softmax_scale > 0.f) || std::isinf(softmax_scale)) return fail(MD_EINVAL, "prefill_filter: softmax_scale must be positive and finite");
    if (mode == MD_FILTER_BUDGET) {
        if (budget < 0) return fail(MD_EINVAL, "prefill_filter: negative budget");
        if (!(gamma > 0.f) || !(alpha > 0.f)) return fail(MD_EINVAL, "prefill_filter: budget mode needs gamma > 0 and alpha > 0");
        if (Rcap < (budget < Mv ? budget : Mv))
            return fail(MD_EINVAL, "prefill_filter: Rcap=%d is smaller than min(budget, Mv)=%d", Rcap, budget < Mv ? budget : Mv);
    }
    const void* big[] = {q_txt, k, v, hidden, hidden_out, k_out, v_out};
    for (const void* ptr : big)
        if (!aligned16(ptr)) return fail(MD_EALIGN, "prefill_filter: tensor pointers must be 16-byte aligned");
    const size_t L = (size_t)Mv + N;
    KvLayout lq, lkv, lout;
    int lrc = read_layout("prefill_filter", "q_txt", q_layout, B, N, H, d, &lq);
    if (lrc == MD_OK) lrc = read_layout("prefill_filter", "k / v", kv_layout, B, (long)L, H, d, &lkv);
    if (lrc == MD_OK) lrc = read_layout("prefill_filter", "k_out / v_out", kv_out_layout, B, (long)Rcap + N, H, d, &lout);
    if (lrc != MD_OK) return lrc;
    if (lq.token > (1l << 26) || lkv.token > (1l << 26))
        return fail(MD_ESHAPE, "prefill_filter: token stride above 2^26 elements");
    // the score sweeps address a sample's head slice with 32-bit byte offsets
    if (((long)L * lkv.token + d) * 2 >= (1l << 31) || ((long)N * lq.token + d) * 2 >= (1l << 31))
        return fail(MD_ESHAPE, "prefill_filter: one head slice of a sample spans more than 2 GiB");
    const size_t kv_in = layout_extent_bytes(lkv, B, (long)L, H, d), h_in = (size_t)B * L * C * 2;
    const size_t kv_out = layout_extent_bytes(lout, B, (long)Rcap + N, H, d), h_out = (size_t)B * (Rcap + N) * C * 2;
    const void* ins[] = {k, v, hidden, q_txt};
    const size_t in_sz[] = {kv_in, kv_in, h_in, layout_extent_bytes(lq, B, N, H, d)};
    const void* outs[] = {k_out, v_out, hidden_out};
    const size_t out_sz[] = {kv_out, kv_out, h_out};
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 4; ++c)
            if (overlaps(outs[a], out_sz[a], ins[c], in_sz[c])) return fail(MD_EALIAS, "prefill_filter: an output tensor overlaps an input");
    const PrefillWorkspace w = carve_prefill(workspace, B, Mv, N, H, Rcap);
    if (!workspace || workspace_bytes < w.bytes)
        return fail(MD_EWORKSPACE, "prefill_filter: workspace of %zu bytes needed, %zu given", w.bytes, workspace ? workspace_bytes : (size_t)0);
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(MD_EALIGN, "prefill_filter: workspace must be 256-byte aligned");

    PrefillDims p;
    p.B = B; p.Mv = Mv; p.N = N; p.H = H; p.d = d; p.C = C; p.L = Mv + N; p.Rcap = Rcap;
    p.q = lq; p.kv = lkv;
    ScorePlan sp = plan_scores(B, Mv, N, H, d, vis_valid != nullptr);
    if (row_lse) sp = with_normalisers(sp);
    p.Npad = sp.nbt * 32;
    p.nch = sp.nch; p.ng = sp.ng;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const float sl2 = softmax_scale * kLog2e;

    const bool col_stream = streams_col_k(sp, B, Mv, H, d, Rcap, mode == MD_FILTER_THRESHOLD, row_lse != nullptr);
    int rc = d == 128 ? launch_scores<8>(p, sp, w, st, q_txt, k, vis_valid, txt_len, row_lse, sl2, col_stream)
                      : launch_scores<4>(p, sp, w, st, q_txt, k, vis_valid, txt_len, row_lse, sl2, col_stream);
    if (rc != MD_OK) return rc;
    int32_t* src_row = out_ids ? out_ids : w.src_row;     // the row map doubles as the optional out_ids
    const bool dense_io = is_dense(lkv, (long)L, H, d) && is_dense(lout, (long)Rcap + N, H, d);
    TextRows tr{static_cast<const u32x4*>(hidden), static_cast<const u32x4*>(k), static_cast<const u32x4*>(v),
                static_cast<u32x4*>(hidden_out), static_cast<u32x4*>(k_out), static_cast<u32x4*>(v_out), 0, 0};
    const bool k_streams = row_lse && (sp.rows ? sp.rows_stream : !sp.own && col_stream);
    const bool stream_k = streams_k_out(B, Mv, N, H, d, C, Rcap, mode == MD_FILTER_THRESHOLD, k_streams);
    tr.stream_k = stream_k ? 1 : 0;
    tr.enabled = (mode == MD_FILTER_BUDGET && dense_io && Mv <= 8192) ? 1 : 0;
    const int sel_blocks = B + (tr.enabled ? B * ((N + kTextRowsPerBlock - 1) / kTextRowsPerBlock) : 0);
    const PrefillWorkspace::ScoreParts parts = w.score_parts(p, sp);
#define MD_PSELECT_FAST2(IPT_, P_)                                                                               \
    MD_LAUNCH("prefill_select", st, (prefill_select_fast_kernel<IPT_, P_>), sel_blocks, 1024, 0,        \
        p, parts.V, parts.I, parts.parts, vis_valid, txt_len, is_key, (int)mode, budget, gamma, alpha,     \
        src_row, kept_index, kept_count, out_len, out_protect, score_global, score_indiv, tr)
#define MD_PSELECT_FAST(IPT_) do { if (parts.parts > 1) MD_PSELECT_FAST2(IPT_, true); else MD_PSELECT_FAST2(IPT_, false); } while (0)
    if (Mv <= 1024) MD_PSELECT_FAST(1);
    else if (Mv <= 2048) MD_PSELECT_FAST(2);
    else if (Mv <= 3072) MD_PSELECT_FAST(3);
    else if (Mv <= 4096) MD_PSELECT_FAST(4);
    else if (Mv <= 5120) MD_PSELECT_FAST(5);
    else if (Mv <= 6144) MD_PSELECT_FAST(6);
    else if (Mv <= 8192) MD_PSELECT_FAST(8);
    else
        MD_LAUNCH("prefill_select", st, (prefill_select_kernel), B, 1024, 0,
            p, w.V, w.I, vis_valid, txt_len, is_key, (int)mode, budget, gamma, alpha,
            w.score, src_row, kept_index, kept_count, out_len, out_protect, score_global, score_indiv);
#undef MD_PSELECT_FAST
#undef MD_PSELECT_FAST2
    dim3 gc(tr.enabled ? Rcap : Rcap + N, B);         // the text rows beyond the kept vision rows are already in place
    if (dense_io) {
#define MD_COMPACT(SK_)                                                                                        \
        MD_LAUNCH("prefill_compact", st, (prefill_compact_kernel<SK_>), gc, 256, 0, p, src_row,                    \
            static_cast<const u32x4*>(hidden), static_cast<const u32x4*>(k), static_cast<const u32x4*>(v),         \
            static_cast<u32x4*>(hidden_out), static_cast<u32x4*>(k_out), static_cast<u32x4*>(v_out), tr.enabled)
        if (stream_k) MD_COMPACT(true); else MD_COMPACT(false);
#undef MD_COMPACT
    } else {
        // Streaming where K, V and hidden together outgrow the Infinity Cache, so that the rows left in it are not written
        // back under the next sweep (21 x 1163 keys, 40 heads of 64, 125 MB: compact + next row statistics 56.9 -> 53.8 us);
        // smaller calls find their rows in L2, which streaming loads pass by (12 x 634, 32 heads of 64, 31 MB: 8.2 -> 6.0).  K out as
        // streams_k_out says, but not with row normalisers (head-major, 24 x 1200, 60 rows 184 -> 181, with them 140 -> 143)
#define MD_COMPACT_STRIDED(ST_, SK_)                                                                           \
        MD_LAUNCH("prefill_compact", st, (prefill_compact_strided_kernel<ST_, SK_>), gc, 256, 0, p, src_row,       \
            static_cast<const u32x4*>(hidden), static_cast<const uint16_t*>(k), static_cast<const uint16_t*>(v),   \
            static_cast<u32x4*>(hidden_out), static_cast<uint16_t*>(k_out), static_cast<uint16_t*>(v_out), lout)
        if ((double)B * p.L * H * d * 2 <= 100e6) MD_COMPACT_STRIDED(false, false);
        else if (stream_k && !row_lse) MD_COMPACT_STRIDED(true, true);
        else MD_COMPACT_STRIDED(true, false);
#undef MD_COMPACT_STRIDED
    }
    return check_launch("prefill_filter");
}

}  // namespace
}  // namespace md

extern "C" int mustdrop_prefill_filter(
    const void* q_txt, const void* k, const void* v, const void* hidden,
    const uint8_t* vis_valid, const int32_t* txt_len, const uint8_t* is_key, const float* row_lse,
    int B, int Mv, int N, int H, int d, int C,
    float softmax_scale, md_filter_mode mode, int budget, float gamma, float alpha,
    int Rcap,
    void* hidden_out, void* k_out, void* v_out,
    int32_t* kept_index, int32_t* kept_count, int32_t* out_len, uint8_t* out_protect, int32_t* out_ids,
    float* score_global, float* score_indiv,
    void* workspace, size_t workspace_bytes, void* stream)
{
    return prefill_filter_impl(q_txt, k, v, hidden, vis_valid, txt_len, is_key, row_lse, B, Mv, N, H, d, C, softmax_scale, mode,
                               budget, gamma, alpha, Rcap, hidden_out, k_out, v_out, kept_index, kept_count, out_len,
                               out_protect, out_ids, score_global, score_indiv, nullptr, nullptr, nullptr,
                               workspace, workspace_bytes, stream);
}

extern "C" int mustdrop_prefill_filter_strided(
    const void* q_txt, const void* k, const void* v, const void* hidden,
    const uint8_t* vis_valid, const int32_t* txt_len, const uint8_t* is_key, const float* row_lse,
    int B, int Mv, int N, int H, int d, int C,
    float softmax_scale, md_filter_mode mode, int budget, float gamma, float alpha,
    int Rcap,
    void* hidden_out, void* k_out, void* v_out,
    int32_t* kept_index, int32_t* kept_count, int32_t* out_len, uint8_t* out_protect, int32_t* out_ids,
    float* score_global, float* score_indiv,
    const md_kv_layout* q_layout, const md_kv_layout* kv_layout, const md_kv_layout* kv_out_layout,
    void* workspace, size_t workspace_bytes, void* stream)
{
    return prefill_filter_impl(q_txt, k, v, hidden, vis_valid, txt_len, is_key, row_lse, B, Mv, N, H, d, C, softmax_scale, mode,
                               budget, gamma, alpha, Rcap, hidden_out, k_out, v_out, kept_index, kept_count, out_len,
                               out_protect, out_ids, score_global, score_indiv, q_layout, kv_layout, kv_out_layout,
                               workspace, workspace_bytes, stream);
}
