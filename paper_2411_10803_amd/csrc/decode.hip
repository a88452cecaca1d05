// Stage 3 -- decode (Sec. 3.5): score the KV cache against the query of the token being generated
// (attention of Eq. 4), keep a running score per entry, evict down to a budget and compact the
// cache by hole filling.
//
//   decode_logits_stream_kernel / decode_logits_kernel
//                         one wave per cache entry at a time: an entry's K row (H heads x d, all
//                         contiguous) is read once with 16-byte loads, 16 lanes per head slice;
//                         segmented butterflies give the H logits.  Pure streaming: a GEMV at about
//                         1 flop per byte, so plain ALUs, not MFMA.
//   decode_select_fast_kernel / decode_select_kernel
//                         softmax statistics per head, head mean, running score update, radix top-k among
//                         unprotected entries, hole/mover lists, moves of the small per-entry arrays; for
//                         short or few caches also the row moves (several blocks per sample, the same selection in each)
//   decode_move_kernel    copies the K and V rows of the movers into the holes, where many may move, in every layer
#include "md_device.hpp"
#include "md_host.hpp"
#include "decode_plan.hpp"

#include <type_traits>

namespace md {
namespace {

constexpr float kLog2eD = 1.4426950408889634f;

struct DecodeDims { int B, Lcap, H, d; };
// The counters from which the blocks of decode_move_kernel claim their pieces, cleared by the kernel before it.
__device__ __forceinline__ void clear_claims(int32_t* claims, int tid) {
    if (tid < kClaims) claims[tid * kClaimStride] = 0;
}
constexpr int kMaxStatParts = 256;               // blocks per sample of the streaming logits kernel

// The small per-entry state of a cache, [B, Lcap] each and len [B].
struct StateArrays { float* acc; int32_t* ids; uint8_t* protect; int32_t* len; };

// logits[b][j][h] = scale * q[b][h] . k[b][j][h]      (token-major so an entry's H logits are contiguous)
// LPH = lanes per head slice = d / 8.  Generic shape: walks an entry's row in 1 KiB pieces.
template <int LPH>
__global__ __launch_bounds__(256) void decode_logits_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache, const int32_t* __restrict__ len,
    DecodeDims p, KvLayout lay, float scale, int tokens_per_block, float* __restrict__ logits)
{
    const int lane = lane_id(), wv = wave_id();
    const int b = blockIdx.y;
    const int n = min(len[b], p.Lcap);
    const int t0 = blockIdx.x * tokens_per_block;
    if (t0 >= n) return;
    const int t1 = min(t0 + tokens_per_block, n);
    const int row = p.H * p.d;                      // elements per entry
    const int nvec = row / 8;                       // 16-byte vectors per entry
    const int iters = (nvec + kWave - 1) / kWave;
    const uint16_t* qb = q + (long)b * row;
    const uint16_t* kb = k_cache + (long)b * lay.batch;
    float* lb = logits + (long)b * p.Lcap * p.H;

    for (int it = 0; it < iters; ++it) {
        const int idx = it * kWave + lane;
        float qv[8];
        if (idx < nvec) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(qb + idx * 8);
            qv[0] = bf16_lo(w.x); qv[1] = bf16_hi(w.x); qv[2] = bf16_lo(w.y); qv[3] = bf16_hi(w.y);
            qv[4] = bf16_lo(w.z); qv[5] = bf16_hi(w.z); qv[6] = bf16_lo(w.w); qv[7] = bf16_hi(w.w);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) qv[e] = 0.f;
        }
        const int head = idx / LPH;
        const long in_row = (long)head * lay.head + (idx % LPH) * 8;      // dense: idx * 8
        for (int j = t0 + wv; j < t1; j += 4) {
            float part = 0.f;
            if (idx < nvec) {
                const u32x4 w = *reinterpret_cast<const u32x4*>(kb + (long)j * lay.token + in_row);
                part = qv[0] * bf16_lo(w.x);
                part = fmaf(qv[1], bf16_hi(w.x), part);
                part = fmaf(qv[2], bf16_lo(w.y), part);
                part = fmaf(qv[3], bf16_hi(w.y), part);
                part = fmaf(qv[4], bf16_lo(w.z), part);
                part = fmaf(qv[5], bf16_hi(w.z), part);
                part = fmaf(qv[6], bf16_lo(w.w), part);
                part = fmaf(qv[7], bf16_hi(w.w), part);
            }
            part = group_sum<LPH>(part);
            if (idx < nvec && (lane & (LPH - 1)) == 0) lb[(long)j * p.H + head] = part * scale;
        }
    }
}

__device__ __forceinline__ float dot8(const u32x4& a, const float (&qv)[8]) {
    float s = qv[0] * bf16_lo(a.x);
    s = fmaf(qv[1], bf16_hi(a.x), s);
    s = fmaf(qv[2], bf16_lo(a.y), s);
    s = fmaf(qv[3], bf16_hi(a.y), s);
    s = fmaf(qv[4], bf16_lo(a.z), s);
    s = fmaf(qv[5], bf16_hi(a.z), s);
    s = fmaf(qv[6], bf16_lo(a.w), s);
    s = fmaf(qv[7], bf16_hi(a.w), s);
    return s;
}

// Streaming shape: an entry's row is at most NIT KiB (H*d*2 bytes, d = 64 or 128).  A wave keeps the whole query
// in registers and reads each entry's row in one go: NIT independent 16-byte loads per lane, every
// load instruction covering 1 KiB of consecutive addresses.  Waves stride over the sample's entries.
// Where the row ends inside a piece the lanes behind it read its last vector again against a zero query.
// Each wave also keeps online softmax statistics (max, sum of exp2) of every head over the entries
// it has seen; the block's four waves are merged and written as one partial per (sample, block, head),
// so the selection kernel does not have to sweep the logits for them.
// Bound by the read of K: 64 caches of 1025 entries, 32 heads of 128, 90 us = 6.0 TB/s; 60 of 748 entries, 40 heads,
// head-major, 81 us = 5.7 TB/s (93 through the generic form).  A second register set with the next row in flight did
// not help (89 us at half the waves), nor did one store per entry with the statistics spread over the lanes of a
// group (91 and 89 us).
// LAYOUT 0: dense rows of exactly NIT KiB (a load's offset is then a constant of the instruction: 0.6 us of 90 on 64
// caches of 1025 entries).  1: dense rows that end inside a piece.  2: any other layout; a load instruction then
// covers kWave/LPH head slices of d*2 contiguous bytes each instead of 1 KiB of one row.
// Rows of more than NIT pieces are shared by gridDim.z blocks, each with heads of its own (layouts 1 and 2 only).
// STREAM_ONCE: the cache is larger than what the L2 / Infinity Cache can hold until the row moves, so
// the K rows are read with streaming loads (they would only evict each other and everything else).
template <int LPH, int NIT, int LAYOUT, bool STREAM_ONCE>
__global__ __launch_bounds__(256) void decode_logits_stream_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache, const int32_t* __restrict__ len,
    DecodeDims p, KvLayout lay, float scale, float* __restrict__ logits, float2* __restrict__ stat_partial,
    StateArrays state, StateArrays copy)
{
    constexpr int HPI = kWave / LPH;                 // heads per load instruction
    __shared__ float s_m[4][NIT * HPI], s_z[4][NIT * HPI];
    const int lane = lane_id(), wv = wave_id();
    const int b = blockIdx.y;
    const int wave_global = blockIdx.x * 4 + wv;
    const int nwaves = gridDim.x * 4;
    const int row = p.H * p.d, nvec = row / 8;
    const int v0 = LAYOUT == 0 ? 0 : (int)blockIdx.z * (NIT * kWave), h0 = v0 / LPH;      // this block's first vector and head
    const u32x4* qb = reinterpret_cast<const u32x4*>(q + (long)b * row);
    const u32x4* kb = reinterpret_cast<const u32x4*>(k_cache + (long)b * p.Lcap * row);
    const uint16_t* ks = k_cache + (long)b * lay.batch;
    int vec[NIT];                                    // this lane's vectors within a row
    long off[NIT];                                   // LAYOUT 2: their element offsets within an entry
    float qv[NIT][8];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int idx = v0 + it * kWave + lane;
        vec[it] = LAYOUT == 0 ? idx : min(idx, nvec - 1);
        off[it] = (long)(vec[it] / LPH) * lay.head + (vec[it] % LPH) * 8;
        u32x4 w = qb[vec[it]];
        if (LAYOUT != 0 && idx >= nvec) w = u32x4{0, 0, 0, 0};
        qv[it][0] = bf16_lo(w.x); qv[it][1] = bf16_hi(w.x); qv[it][2] = bf16_lo(w.y); qv[it][3] = bf16_hi(w.y);
        qv[it][4] = bf16_lo(w.z); qv[it][5] = bf16_hi(w.z); qv[it][6] = bf16_lo(w.w); qv[it][7] = bf16_hi(w.w);
    }
    float* lb = logits + (long)b * p.Lcap * p.H;
    const float scale_l2 = scale * kLog2eD;
    // The maxima start at the lowest finite number, not at -inf: the first entry of a wave may be one that the caller masks
    // (logit -inf), and -inf - -inf would make the head's sum a NaN.
    float m[NIT], z[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) { m[it] = -3.402823466e38f; z[it] = 0.f; }

    const int n = min(max(len[b], 0), p.Lcap);
    // the state as it is before the selection changes it, for the other selection blocks of the sample
    if (copy.acc && blockIdx.z == 0) {
        for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256) {
            const long i = (long)b * p.Lcap + j;
            copy.acc[i] = state.acc[i]; copy.ids[i] = state.ids[i]; copy.protect[i] = state.protect[i];
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) copy.len[b] = n;
    }
    for (int j = wave_global; j < n; j += nwaves) {
        u32x4 kv[NIT];
        if constexpr (LAYOUT == 2) {
            const uint16_t* kr = ks + (long)j * lay.token;
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const u32x4* src = reinterpret_cast<const u32x4*>(kr + off[it]);
                kv[it] = STREAM_ONCE ? __builtin_nontemporal_load(src) : *src;
            }
        } else {
            const u32x4* kr = kb + (long)j * (LAYOUT == 0 ? NIT * kWave : nvec);
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                kv[it] = STREAM_ONCE ? __builtin_nontemporal_load(kr + vec[it]) : kr[vec[it]];
        }
        float part[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) part[it] = dot8(kv[it], qv[it]);
#pragma unroll
        for (int it = 0; it < NIT; ++it) part[it] = group_sum<LPH>(part[it]);
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const float t2 = part[it] * scale_l2;
            const float dlt = t2 - m[it];            // huge on the first entry
            const float e = fast_exp2(-fabsf(dlt));
            z[it] = dlt > 0.f ? fmaf(z[it], e, 1.0f) : z[it] + e;
            m[it] = fmaxf(m[it], t2);
        }
        if ((lane & (LPH - 1)) == 0) {
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                if (LAYOUT == 0 || h0 + it * HPI + lane / LPH < p.H) lb[(long)j * p.H + h0 + it * HPI + lane / LPH] = part[it] * scale;
        }
    }
    if ((lane & (LPH - 1)) == 0) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) { s_m[wv][it * HPI + lane / LPH] = m[it]; s_z[wv][it * HPI + lane / LPH] = z[it]; }
    }
    __syncthreads();
    for (int h = threadIdx.x; h < min(NIT * HPI, p.H - h0); h += blockDim.x) {
        float mn = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) mn = fmaxf(mn, s_m[w][h]);
        float zn = 0.f;
        if (mn > -INFINITY) {
#pragma unroll
            for (int w = 0; w < 4; ++w) zn += s_z[w][h] * fast_exp2(s_m[w][h] - mn);
        }
        stat_partial[((long)b * gridDim.x + blockIdx.x) * p.H + h0 + h] = make_float2(mn, zn);
    }
}

// Rows movers[t] -> holes[t] for t = first, first + step, ... < m of one sample's caches, by a team of 256 threads.
// Source rows (beyond the new length) and destination rows (holes below it) never coincide, but
// the compiler cannot know: the vectors of a round are read into registers before any is written.
// The V rows are not read on this path at all (only moved): always streamed; the K rows where the caches are too large
// to stay in the Infinity Cache until the next step reads them.
template <bool STREAM_ONCE>
__device__ __forceinline__ void move_rows(const DecodeDims& p, const KvLayout& lay, const int* holes, const int* movers, int m,
                                          int first, int step, int tid, uint16_t* k, uint16_t* v) {
    const int lph = p.d / 8, sh = __builtin_ctz(lph), rv = p.H << sh;        // 16-byte vectors per head slice (a power of two), per row
    for (int t = first; t < m; t += step) {
        const long src = (long)movers[t] * lay.token, dst = (long)holes[t] * lay.token;
        for (int c = tid; c < rv; c += 512) {
            const int c2 = c + 256;
            const bool two = c2 < rv;
            const long o = (long)(c >> sh) * lay.head + (c & (lph - 1)) * 8, o2 = (long)(c2 >> sh) * lay.head + (c2 & (lph - 1)) * 8;
            auto at = [](uint16_t* q, long e) { return reinterpret_cast<u32x4*>(q + e); };
            auto ld = [](const u32x4* q) { return STREAM_ONCE ? __builtin_nontemporal_load(q) : *q; };
            auto st = [](u32x4* q, const u32x4& x) { if (STREAM_ONCE) __builtin_nontemporal_store(x, q); else *q = x; };
            const u32x4 k0 = ld(at(k, src + o)), v0 = __builtin_nontemporal_load(at(v, src + o));
            u32x4 k1 = k0, v1 = v0;
            if (two) { k1 = ld(at(k, src + o2)); v1 = __builtin_nontemporal_load(at(v, src + o2)); }
            st(at(k, dst + o), k0);
            __builtin_nontemporal_store(v0, at(v, dst + o));
            if (two) { st(at(k, dst + o2), k1); __builtin_nontemporal_store(v1, at(v, dst + o2)); }
        }
    }
}

// Selection with everything in registers.  Two forms:
//   moves in the same launch (n_move null): gridDim.x blocks per sample work out the same selection, each from the
//     logits and an unchanged copy of the state (`in`; with one block per sample the state itself), the first one writes
//     the new state, and they share the rows to move.  The selection is a chain of latencies on a chip that is idle
//     beside it, and a launch of its own for the moves costs 4 us more.
//   lists (one block per sample): holes, movers and their number go to decode_move_kernel.
// Entries are dealt round-robin: thread t owns the entries
// t, t+1024, ... (coalesced loads; the first one does not depend on the live length, so it is
// requested before the length arrives).  IPT >= ceil(Lcap / 1024).  One round of global loads for
// the common case, then block-level phases only.
// Bound by that chain and by the instructions of sixteen waves on one CU.  In a steady loop one entry leaves: the writer alone works
// (62 blocks per sample that all read the same logits were in each other's way), the row that will move is under way from
// the start and the statistics are read as they lie in memory.  us per launch, before / after: 4 x 778 entries of 40
// heads, head-major 13.2 / 9.4, 64 x 1025 of 32 12.2 / 11.0, 16 x 8001 of 32, whose form spills four registers, 38.2 / 36.5; none
// leaves: 16 x 1000 of 32 heads 9.0 / 8.2, 64 x 1000 6.9 / 7.6; per step 16 x 1025 of 32 heads 42.9 / 39.5, 1 x 1025 20.1 / 16.4.
// LPE = lanes per entry = H / 4 where that is a power of two up to 8; 0: any other H that is a multiple of four.
template <int IPT, int LPE>
__global__ __launch_bounds__(1024) void decode_select_fast_kernel(
    DecodeDims p, const float* __restrict__ logits, const float2* __restrict__ stat_partial, int n_part,
    float decay, int budget, StateArrays in, StateArrays out, KvLayout lay, uint16_t* k_cache, uint16_t* v_cache, int stream_once,
    int32_t* __restrict__ holes, int32_t* __restrict__ movers, int32_t* __restrict__ n_move, int32_t* __restrict__ claims,
    int32_t* __restrict__ evicted_ids, int32_t* __restrict__ evicted_count)
{
    // [Lcap] a_t (and behind it, for LPE = 0, the waves' shares); once every thread has taken its a_t the same
    // memory holds the list of evicted slots below the new length and, in its second half, that of the kept ones behind it
    extern __shared__ __attribute__((aligned(16))) int s_holes[];
    float* s_at = reinterpret_cast<float*>(s_holes);
    __shared__ __attribute__((aligned(16))) float s_cm[128], s_cz[128];      // per head: max (log2 domain), 1 / (Z * H)
    __shared__ float2 s_st[1024];
    __shared__ int s_red[16];
    __shared__ int s_hist[kSelectHistInts];
    __shared__ uint64_t s_red64[16];
    __shared__ int s_rounds[16 * IPT];
    const int b = blockIdx.y, tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const bool writer = blockIdx.x == 0;
    if (tid < 256) s_hist[tid] = 0;                  // for block_select_topk, after later barriers
    if (n_move && b == 0) clear_claims(claims, tid);
    const int H = p.H;
    const float* lb = logits + (long)b * p.Lcap * H;
    const float* ai = in.acc + (long)b * p.Lcap;
    const int32_t* ii = in.ids + (long)b * p.Lcap;
    const uint8_t* pi = in.protect + (long)b * p.Lcap;
    float* ab = out.acc + (long)b * p.Lcap;
    int32_t* ib = out.ids + (long)b * p.Lcap;
    uint8_t* pb = out.protect + (long)b * p.Lcap;
    k_cache += (long)b * lay.batch;
    v_cache += (long)b * lay.batch;
    auto move = [&](const int* from, const int* to, int m) {             // `from`, `to` in LDS
        if (n_move) {                                // up to four rows, one for each team, are moved here all the same
            if (tid == 0) n_move[b] = m > 4 ? m : 0;
            if (m > 4) {
                for (int t = tid; t < m; t += 1024) { movers[(long)b * p.Lcap + t] = from[t]; holes[(long)b * p.Lcap + t] = to[t]; }
                return;
            }
        }
        const int first = blockIdx.x * 4 + (tid >> 8), step = gridDim.x * 4;
        if (stream_once) move_rows<true>(p, lay, to, from, m, first, step, tid & 255, k_cache, v_cache);
        else move_rows<false>(p, lay, to, from, m, first, step, tid & 255, k_cache, v_cache);
    };

    // ---- requests that do not depend on the live length
    float a_old[IPT];
    int id[IPT];
    bool prot[IPT], live[IPT];
    // Logits are read the way they lie in memory: a wave takes 64 consecutive entries (64*H floats)
    // with LPE = H/4 fully coalesced 16-byte loads per lane; lane l then holds heads 4*(l%LPE)..+3 of
    // the entries u*(64/LPE) + l/LPE, u = 0..LPE-1.
    constexpr int PFR = IPT < 2 ? IPT : 2;           // rounds requested before the length is known
    constexpr int LPE1 = LPE ? LPE : 1;
    constexpr int EPI = kWave / LPE1;                // entries per load instruction
    f32x4 lpf[PFR][LPE1], hpf[2][5];
    // Logits are requested ahead only up to where a steady decode loop has entries: behind them a cache with room to
    // spare holds nothing but old logits, which come from far away (33 x 168 of 949 slots, 8 blocks each: 35.6 -> 32.7 us).
    // One block per sample takes all at once: a cut to a quarter would wait twice (6 x 1838 entries: 15 us, 18.6 so)
    // (Buffer loads: what lies behind the last entry that is asked for reads as zero.  A predicate and an address for each of
    // the loads is what four waves per SIMD spend their time on here.)
    const int ahead = gridDim.x > 1 && budget < p.Lcap - 64 ? budget + 64 : p.Lcap;
    // Up to budget + 1 entries one leaves at most, and the writer sees to that alone.  The other blocks wait for the length before
    // they ask for anything: they would all go for the lines that the writer waits for.  (The writer itself does not, and reads the
    // length once its requests are out.)
    if (!writer && in.len[b] <= budget + 1) return;
    uint32_t pbyte[PFR];
#pragma unroll
    for (int t = 0; t < PFR; ++t) {
        const int j = min(tid + t * 1024, p.Lcap - 1);                   // readable whatever the live length is
        a_old[t] = ai[j];
        id[t] = ii[j];
        pbyte[t] = pi[j];
    }
    auto range_from = [&](int entry) -> __amdgpu_buffer_rsrc_t {         // (uniform over the wave)
        const LogitRange r = logit_range(entry, ahead, H);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(lb + r.first), 0, r.bytes, 0x00020000);
    };
    auto request = [&](__amdgpu_buffer_rsrc_t from, int byte) -> f32x4 {
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(from, byte, 0, 0));
    };
#pragma unroll
    for (int t = 0; t < PFR; ++t) {
        const __amdgpu_buffer_rsrc_t from = range_from(t * 1024 + wv * kWave);
#pragma unroll
        for (int u = 0; u < LPE; ++u) lpf[t][u] = request(from, logit_vector(lane, u, 0, H));
    }
    // LPE = 0: the wave's first 64 entries, 32 at a time, where they are no more than five vectors per lane (with six, eight registers
    // more: 4 x 778 entries of 44 heads 10.5 -> 10.0 us a launch, but of 36 and 40 heads 9.4 -> 9.7 and 9.8)
    const int vpe = H >> 2;
    if (LPE == 0 && vpe <= 10) {
        const __amdgpu_buffer_rsrc_t from = range_from(wv * kWave);
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int u = 0; u < 5; ++u) hpf[r][u] = request(from, logit_vector(lane, u, 32 * r, H));
    }
    // the logits kernel's partial statistics, as they lie in memory: thread = (slice of its blocks, head), heads contiguous
    const uint32_t hmul = (1u << 20) / (uint32_t)H + 1u;                 // x / H = x * hmul >> 20 for x <= 1024
    const int nsl = (int)((1024u * hmul) >> 20), sl = (int)(((uint32_t)tid * hmul) >> 20), hh = tid - sl * H;
    float mn = -INFINITY, zn = 0.f;
    if (sl < nsl) {
        const float2* sp = stat_partial + (long)b * n_part * H + hh;
        auto merge = [&](int c0, auto count) {       // count partials, in flight together
            constexpr int N = decltype(count)::value;
            double v[N];                             // (pairs of floats; as such, the halves would be loaded one after the other)
            float m2 = mn;
#pragma unroll
            for (int u = 0; u < N; ++u) v[u] = *reinterpret_cast<const double*>(sp + min(c0 + u * nsl, n_part - 1) * H);
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (c0 + u * nsl < n_part) m2 = fmaxf(m2, __builtin_bit_cast(float2, v[u]).x);
            if (m2 > -INFINITY) {
                zn *= fast_exp2(mn - m2);
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const float2 w = __builtin_bit_cast(float2, v[u]);
                    if (c0 + u * nsl < n_part) zn = fmaf(w.y, fast_exp2(w.x - m2), zn);
                }
            }
            mn = m2;
        };
        if (n_part <= 2 * nsl) merge(sl, std::integral_constant<int, 2>());
        else
            for (int c0 = sl; c0 < n_part; c0 += 8 * nsl) merge(c0, std::integral_constant<int, 8>());
        s_st[tid] = make_float2(mn, zn);
    }
    const int n = min(max(in.len[b], 0), p.Lcap);
    if (n == 0) {
        if (writer && tid == 0 && evicted_count) evicted_count[b] = 0;
        if (n_move && tid == 0) n_move[b] = 0;
        return;
    }
#pragma unroll
    for (int t = 0; t < PFR; ++t) {
        live[t] = tid + t * 1024 < n;
        prot[t] = live[t] && pbyte[t] != 0;
        if (!live[t]) a_old[t] = 0.f;
    }
#pragma unroll
    for (int t = PFR; t < IPT; ++t) {                // further rounds only for long caches
        const int j = tid + t * 1024;
        live[t] = prot[t] = false;
        a_old[t] = 0.f;
        id[t] = 0;
        if (t * 1024 >= n) continue;                 // block-uniform
        live[t] = j < n;
        a_old[t] = live[t] ? ai[j] : 0.f;
        id[t] = live[t] ? ii[j] : 0;
        prot[t] = live[t] ? pi[j] != 0 : false;
    }
    if (LPE > 0 && n > ahead) {                      // block-uniform
#pragma unroll
        for (int t = 0; t < PFR; ++t)
#pragma unroll
            for (int u = 0; u < LPE; ++u) {
                const int base = t * 1024 + wv * kWave, e = base + u * EPI + lane / LPE1;
                if (e >= ahead && e < n) lpf[t][u] = reinterpret_cast<const f32x4*>(lb + (long)base * H)[u * kWave + lane];
            }
    }
    // Where one entry leaves as a rule (a steady decode loop), the last one's rows will fill its place: on their way already
    const int sh_v = __builtin_ctz(p.d / 8), rv = H << sh_v;             // 16-byte vectors of a head slice (log2), of a row
    const bool row_ahead = writer && n == budget + 1 && rv <= 1024;
    u32x4 mrow[2];
    auto row_vector = [&](int i, int slot, bool& of_v) -> u32x4* {       // this thread's i-th vector of the K row and the V row behind it
        const int x = min(tid + i * 1024, 2 * rv - 1);
        of_v = x >= rv;
        const int y = of_v ? x - rv : x;
        return reinterpret_cast<u32x4*>((of_v ? v_cache : k_cache) + (long)slot * lay.token + (long)(y >> sh_v) * lay.head + (y & ((1 << sh_v) - 1)) * 8);
    };
    // (requested whatever the case: behind a branch, a wait for anything older would be one for these rows too.  Where no row will
    // move, the logits at hand take its place: 64 x 1000 entries of which none leaves 8.3 us with the row from far away, 7.6 so)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        bool of_v;
        const u32x4* src = row_vector(i, n - 1, of_v);
        mrow[i] = __builtin_nontemporal_load(row_ahead ? src : reinterpret_cast<const u32x4*>(lb));
    }
    {
        int np = 0;                                  // the wave's protected entries
#pragma unroll
        for (int t = 0; t < IPT; ++t) np += __popcll(__ballot(prot[t]));
        if (lane == 0) s_red[wv] = np;
    }
    __syncthreads();
    // `parts` consecutive lanes (a power of two) finish a head: maximum, then the sum of the rescaled sums
    {
        const int lg = min(31 - __clz(nsl), 6), parts = 1 << lg, sh = tid >> lg, sq = tid & (parts - 1), ns = min(nsl, n_part);
        float gm = -INFINITY, gz = 0.f;
        if (sh < H)
            for (int c = sq; c < ns; c += parts) {
                const float2 v = s_st[c * H + sh];
                const float m2 = fmaxf(gm, v.x);
                if (m2 > -INFINITY) gz = gz * fast_exp2(gm - m2) + v.y * fast_exp2(v.x - m2);
                gm = m2;
            }
        const float own = gm;
        if (parts >= 2) gm = fmaxf(gm, dpp_f<0xB1>(gm));
        if (parts >= 4) gm = fmaxf(gm, dpp_f<0x4E>(gm));
        if (parts >= 8) gm = fmaxf(gm, dpp_f<0x141>(gm));
        if (parts >= 16) gm = fmaxf(gm, dpp_f<0x140>(gm));
        if (parts >= 32) gm = fmaxf(gm, __shfl_xor(gm, 16, kWave));
        if (parts >= 64) gm = fmaxf(gm, __shfl_xor(gm, 32, kWave));
        const float zs = group_sum_rt(gm > -INFINITY ? gz * fast_exp2(own - gm) : 0.f, parts);
        if (sh < H && sq == 0) { s_cm[sh] = gm; s_cz[sh] = __frcp_rn(zs * (float)H); }
    }
    __syncthreads();
    // a_t[j] = mean_h softmax; acc <- decay*acc + a_t.  A lane always works on the same four heads,
    // so their statistics sit in registers; LPE lanes add up an entry's heads and one of them drops
    // the result in LDS, from where the entry's owner picks it up (same wave: LDS keeps program order).
    float a_new[IPT];
    if constexpr (LPE == 0) {
        // H / 4 = `vpe` vectors of 16 bytes per entry, not a power of two: a wave takes 32 entries at a time, 32 * vpe
        // consecutive vectors.  A lane's vectors belong to changing heads, so it takes their statistics from LDS, and
        // a vector's share goes through LDS to the lane that adds up the entry's shares, in head order.
        const uint32_t vmul = 65536u / (uint32_t)vpe + 1u;               // x / vpe = x * vmul >> 16 for x < 32 * vpe <= 1024
        float* s_share = s_at + p.Lcap + wv * (32 * vpe);
        auto shares = [&](int u0, int nv, const f32x4 (&v)[5]) {
#pragma unroll
            for (int u = 0; u < 5; ++u) {
                const int x = u0 + u * kWave + lane;
                if (x < nv) {
                    const int g = x - (int)(((uint32_t)x * vmul) >> 16) * vpe;
                    const f32x4 cm = reinterpret_cast<const f32x4*>(s_cm)[g], cz = reinterpret_cast<const f32x4*>(s_cz)[g];
                    float part = fast_exp2(fmaf(v[u].x, kLog2eD, -cm.x)) * cz.x;
                    part = fmaf(fast_exp2(fmaf(v[u].y, kLog2eD, -cm.y)), cz.y, part);
                    part = fmaf(fast_exp2(fmaf(v[u].z, kLog2eD, -cm.z)), cz.z, part);
                    part = fmaf(fast_exp2(fmaf(v[u].w, kLog2eD, -cm.w)), cz.w, part);
                    s_share[x] = part;
                }
            }
        };
        auto sums = [&](int e0, int ne) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (lane < ne) {
                float sum = 0.f;
                for (int c = 0; c < vpe; ++c) sum += s_share[lane * vpe + c];
                s_at[e0 + lane] = sum;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        int e_first = wv * kWave;
        if (vpe <= 10 && n <= ahead) {               // block-uniform: the first 64 entries are here
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int e0 = wv * kWave + 32 * r, ne = min(n - e0, 32);
                if (ne <= 0) break;
                shares(0, ne * vpe, hpf[r]);
                sums(e0, ne);
            }
            e_first += 1024;
        }
        for (int e0 = e_first; e0 < n; e0 += (e0 & 32) ? 1024 - 32 : 32) {
            const f32x4* lv = reinterpret_cast<const f32x4*>(lb + (long)e0 * H);
            const int ne = min(n - e0, 32), nv = ne * vpe;               // live entries of this round, their vectors
            for (int u0 = 0; u0 < nv; u0 += 5 * kWave) {
                f32x4 v[5];
#pragma unroll
                for (int u = 0; u < 5; ++u) v[u] = lv[min(u0 + u * kWave + lane, nv - 1)];
                shares(u0, nv, v);
            }
            sums(e0, ne);
        }
#pragma unroll
        for (int t = 0; t < IPT; ++t) a_new[t] = live[t] ? fmaf(decay, a_old[t], s_at[tid + t * 1024]) : 0.f;
    } else {
        float cm[4], cz[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) { cm[c] = s_cm[4 * (lane % LPE) + c]; cz[c] = s_cz[4 * (lane % LPE) + c]; }
#pragma unroll
        for (int t = 0; t < IPT; ++t) {
            a_new[t] = 0.f;
            if (t * 1024 >= n) continue;             // block-uniform: no entries in this round
            const int base = t * 1024 + wv * kWave;
#pragma unroll
            for (int u = 0; u < LPE; ++u) {
                if (base + u * EPI >= n) break;
                const int e = base + u * EPI + lane / LPE;
                f32x4 v;
                if (t < PFR) v = lpf[t < PFR ? t : 0][u];
                else v = e < n ? reinterpret_cast<const f32x4*>(lb + (long)base * H)[u * kWave + lane] : f32x4{0.f, 0.f, 0.f, 0.f};
                float part = fast_exp2(fmaf(v.x, kLog2eD, -cm[0])) * cz[0];
                part = fmaf(fast_exp2(fmaf(v.y, kLog2eD, -cm[1])), cz[1], part);
                part = fmaf(fast_exp2(fmaf(v.z, kLog2eD, -cm[2])), cz[2], part);
                part = fmaf(fast_exp2(fmaf(v.w, kLog2eD, -cm[3])), cz[3], part);
                part = group_sum<LPE>(part);
                if (lane % LPE == 0 && e < p.Lcap) s_at[e] = part;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int j = tid + t * 1024;
            a_new[t] = live[t] ? fmaf(decay, a_old[t], s_at[j]) : 0.f;
        }
    }
    const int np = wave_sum_i(lane < 16 ? s_red[lane] : 0);

    if (n <= budget) {                               // nothing leaves: only the scores change
        if (!writer) return;
#pragma unroll
        for (int t = 0; t < IPT; ++t) if (live[t]) ab[tid + t * 1024] = a_new[t];
        if (tid == 0 && evicted_count) evicted_count[b] = 0;
        if (n_move && tid == 0) n_move[b] = 0;
        return;
    }
    const int nu = n - np;
    const int extra = min(max(budget - np, 0), nu);
    const int new_len = np + extra;
    uint64_t key[IPT];
#pragma unroll
    for (int t = 0; t < IPT; ++t) key[t] = (live[t] && !prot[t]) ? rank_key(a_new[t], id[t]) : 0ull;

    if (nu - extra == 1) {
        // Steady state of a decode loop: exactly one entry leaves -- the smallest key.  If it is not
        // the last live slot, the last entry (a survivor) moves into its place.
        if (!writer) return;
        uint64_t mine = ~0ull;
        int mine_slot = 0;
#pragma unroll
        for (int t = 0; t < IPT; ++t)
            if (t * 1024 < n && key[t] != 0 && key[t] < mine) { mine = key[t]; mine_slot = tid + t * 1024; }
        const uint64_t least = wave_min_u64(mine);
        const int least_slot = __builtin_amdgcn_readlane(mine_slot, __builtin_ctzll(__ballot(mine == least)));
        __shared__ int s_slot[16], s_pair[2];
        if (lane == 0) { s_red64[wv] = least; s_slot[wv] = least_slot; }
        __syncthreads();
        const uint64_t other = s_red64[lane & 15];
        const uint64_t victim = wave_min_u64(other);                     // (keys are unique, and there is one)
        const int vslot = s_slot[__builtin_ctzll(__ballot(other == victim))], last = n - 1;
        if (row_ahead) {
            if (n_move && tid == 0) n_move[b] = 0;
            if (vslot != last) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (tid + i * 1024 < 2 * rv) {
                        bool of_v;
                        u32x4* dst = row_vector(i, vslot, of_v);
                        if (stream_once || of_v) __builtin_nontemporal_store(mrow[i], dst);
                        else *dst = mrow[i];
                    }
            }
        } else {
            if (tid == 0) { s_pair[0] = vslot; s_pair[1] = last; }
            __syncthreads();
            move(s_pair + 1, s_pair, vslot != last ? 1 : 0);
        }
#pragma unroll
        for (int t = 0; t < IPT; ++t) {
            const int j = tid + t * 1024;
            if (!live[t]) continue;
            if (j == vslot) {
                if (evicted_ids) evicted_ids[(long)b * p.Lcap] = id[t];
                if (j == last) ab[j] = a_new[t];     // stays behind the new end, as the oracle leaves it
            } else {
                if (j == last) { ab[vslot] = a_new[t]; ib[vslot] = id[t]; pb[vslot] = prot[t] ? 1 : 0; }
                ab[j] = a_new[t];
            }
        }
        if (tid == 0) {
            out.len[b] = new_len;
            if (evicted_count) evicted_count[b] = 1;
        }
        return;
    }

    const SelectBound sb = block_select_topk<IPT>(key, extra, s_hist);
    bool keep[IPT];
#pragma unroll
    for (int t = 0; t < IPT; ++t)
        keep[t] = live[t] && (prot[t] || (extra > 0 && (key[t] >> sb.shift) >= sb.bound));
    // hole / mover / evicted lists in ascending slot order.  Holes are counted in the low half of a word, movers in the
    // high half; an evicted slot's rank is its hole rank below the new length, and behind it what the kept ones leave.
    int cnt[IPT], pre[IPT];
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        const int j = tid + t * 1024;
        const unsigned long long h = __ballot(live[t] && !keep[t] && j < new_len), mv = __ballot(live[t] && keep[t] && j >= new_len);
        cnt[t] = __popcll(h) | (__popcll(mv) << 16);
        pre[t] = lanes_below(h) | (lanes_below(mv) << 16);
    }
    int wave_pre[IPT];
    const int m = block_round_prefixes<IPT>(cnt, wave_pre, s_rounds) & 0xFFFF;      // as many movers as holes
    int* s_movers = s_holes + p.Lcap / 2;
    int mrank[IPT];
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        mrank[t] = -1;
        const int j = tid + t * 1024;
        if (!live[t]) continue;
        const int hr = (pre[t] + wave_pre[t]) & 0xFFFF, mr = (pre[t] + wave_pre[t]) >> 16;
        if (keep[t]) {
            if (j >= new_len) { mrank[t] = mr; s_movers[mr] = j; }
        } else {
            if (j < new_len) s_holes[hr] = j;
            if (writer && evicted_ids) evicted_ids[(long)b * p.Lcap + (j < new_len ? hr : j - (new_len - m) - mr)] = id[t];
        }
    }
    __syncthreads();
    if (writer) {
        // write the scores back; a mover's state goes straight to its hole (no overlap: holes < new_len <= movers)
#pragma unroll
        for (int t = 0; t < IPT; ++t) {
            const int j = tid + t * 1024;
            if (!live[t]) continue;
            if (mrank[t] >= 0) {
                const int dst = s_holes[mrank[t]];
                ab[dst] = a_new[t];
                ib[dst] = id[t];
                pb[dst] = prot[t] ? 1 : 0;
                ab[j] = a_new[t];
            } else if (keep[t] || j >= new_len) {
                ab[j] = a_new[t];
            }
        }
        if (tid == 0) {
            out.len[b] = new_len;
            if (evicted_count) evicted_count[b] = n - new_len;
        }
    }
    move(s_movers, s_holes, m);
}

__global__ __launch_bounds__(1024) void decode_select_kernel(
    DecodeDims p, const float* __restrict__ logits, float decay, int budget,
    float* __restrict__ acc, int32_t* __restrict__ ids, uint8_t* __restrict__ protect, int32_t* __restrict__ len,
    uint8_t* __restrict__ keep, int32_t* __restrict__ holes, int32_t* __restrict__ movers, int32_t* __restrict__ n_move, int32_t* __restrict__ claims,
    int32_t* __restrict__ evicted_ids, int32_t* __restrict__ evicted_count)
{
    extern __shared__ float s_dyn[];                 // [2*H] max / inv, then [32][H] scratch
    __shared__ int s_red[16];
    __shared__ int s_hist[256];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int H = p.H;
    const int n = min(max(len[b], 0), p.Lcap);
    float* s_max = s_dyn;
    float* s_inv = s_dyn + H;
    float* s_part = s_dyn + 2 * H;                   // [parts][H]
    const float* lb = logits + (long)b * p.Lcap * H;
    float* ab = acc + (long)b * p.Lcap;
    int32_t* ib = ids + (long)b * p.Lcap;
    uint8_t* pb = protect + (long)b * p.Lcap;
    uint8_t* kb = keep + (long)b * p.Lcap;
    int32_t* hb = holes + (long)b * p.Lcap;
    int32_t* mvb = movers + (long)b * p.Lcap;

    if (b == 0) clear_claims(claims, tid);
    if (n == 0) {
        if (tid == 0) { n_move[b] = 0; if (evicted_count) evicted_count[b] = 0; }
        return;
    }
    // per-head softmax statistics over the live entries: thread = (part, head)
    const int parts = blockDim.x / H;                // host guarantees H <= blockDim.x; threads beyond parts*H idle here
    const int h = tid % H, part = tid / H;
    {
        float mx = -INFINITY;
        if (part < parts)
            for (int j = part; j < n; j += parts) mx = fmaxf(mx, lb[(long)j * H + h]);
        if (part < parts) s_part[part * H + h] = mx;
        __syncthreads();
        if (tid < H) {
            float m2 = -INFINITY;
            for (int q = 0; q < parts; ++q) m2 = fmaxf(m2, s_part[q * H + tid]);
            s_max[tid] = m2;
        }
        __syncthreads();
        const float mh = s_max[h];
        float z = 0.f;
        if (part < parts)
            for (int j = part; j < n; j += parts) z += fast_exp2((lb[(long)j * H + h] - mh) * kLog2eD);
        if (part < parts) s_part[part * H + h] = z;
        __syncthreads();
        if (tid < H) {
            float z2 = 0.f;
            for (int q = 0; q < parts; ++q) z2 += s_part[q * H + tid];
            s_inv[tid] = 1.0f / (z2 * (float)H);
        }
        __syncthreads();
    }
    // a_t[j] = mean_h softmax ; acc <- decay*acc + a_t
    for (int j = tid; j < n; j += blockDim.x) {
        float a = 0.f;
        for (int hh = 0; hh < H; ++hh) a += fast_exp2((lb[(long)j * H + hh] - s_max[hh]) * kLog2eD) * s_inv[hh];
        ab[j] = fmaf(decay, ab[j], a);
    }
    __syncthreads();

    if (n <= budget) {                               // nothing to evict
        if (tid == 0) { n_move[b] = 0; if (evicted_count) evicted_count[b] = 0; }
        return;
    }
    int np = 0;
    for (int j = tid; j < n; j += blockDim.x) np += pb[j] != 0;
    np = block_sum_i(np, s_red);
    const int nu = n - np;
    const int extra = min(max(budget - np, 0), nu);
    const int new_len = np + extra;
    SelectBound sb{0ull, 63};
    if (extra > 0) {
        auto keyfn = [&](int i, bool& ok) -> uint64_t {
            ok = pb[i] == 0;
            return ok ? rank_key(ab[i], ib[i]) : 0ull;
        };
        sb = block_radix_select(keyfn, n, extra, s_hist);
    }
    // keep flags, hole / mover / evicted lists (ascending slot order by construction of the scan)
    int run_h = 0, run_m = 0, run_e = 0;
    for (int base = 0; base < n; base += blockDim.x) {
        const int j = base + tid;
        bool kp = false;
        if (j < n) {
            kp = pb[j] != 0 || (extra > 0 && (rank_key(ab[j], ib[j]) >> sb.shift) >= sb.bound);
            kb[j] = kp;
        }
        const bool is_hole = j < new_len && !kp;
        const bool is_mover = j >= new_len && j < n && kp;
        const bool is_ev = j < n && !kp;
        int th, tm, te;
        const int rh = block_rank(is_hole, s_red, th);
        const int rm = block_rank(is_mover, s_red, tm);
        const int re = block_rank(is_ev, s_red, te);
        if (is_hole) hb[run_h + rh] = j;
        if (is_mover) mvb[run_m + rm] = j;
        if (is_ev && evicted_ids) evicted_ids[(long)b * p.Lcap + run_e + re] = ib[j];
        run_h += th; run_m += tm; run_e += te;
    }
    __syncthreads();
    // move the small per-entry arrays (sources >= new_len, destinations < new_len: no overlap)
    for (int t = tid; t < run_m; t += blockDim.x) {
        const int src = mvb[t], dst = hb[t];
        ab[dst] = ab[src];
        ib[dst] = ib[src];
        pb[dst] = pb[src];
    }
    if (tid == 0) {
        n_move[b] = run_m;
        len[b] = new_len;
        if (evicted_count) evicted_count[b] = run_e;
    }
}

// The static policy (Sec. 3.5): the entries to keep are given, nothing is scored.  One block per
// sample turns the keep flags into the same hole / mover lists as the selection kernels and moves the
// small per-entry arrays; the row moves then run over every layer's cache.
__global__ __launch_bounds__(1024) void decode_keep_plan_kernel(
    DecodeDims p, const uint8_t* __restrict__ keep, float* __restrict__ acc, int32_t* __restrict__ ids,
    uint8_t* __restrict__ protect, int32_t* __restrict__ len,
    int32_t* __restrict__ holes, int32_t* __restrict__ movers, int32_t* __restrict__ n_move, int32_t* __restrict__ claims,
    int32_t* __restrict__ evicted_ids, int32_t* __restrict__ evicted_count)
{
    __shared__ int s_red[16];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int n = min(max(len[b], 0), p.Lcap);
    const uint8_t* kf = keep + (long)b * p.Lcap;
    float* ab = acc ? acc + (long)b * p.Lcap : nullptr;
    int32_t* ib = ids + (long)b * p.Lcap;
    uint8_t* pb = protect + (long)b * p.Lcap;
    int32_t* hb = holes + (long)b * p.Lcap;
    int32_t* mvb = movers + (long)b * p.Lcap;

    if (b == 0) clear_claims(claims, tid);
    int nk = 0;
    for (int j = tid; j < n; j += blockDim.x) nk += kf[j] != 0;
    const int new_len = block_sum_i(nk, s_red);
    // hole / mover / evicted lists (ascending slot order by construction of the scan)
    int run_h = 0, run_m = 0, run_e = 0;
    for (int base = 0; base < n; base += blockDim.x) {
        const int j = base + tid;
        const bool kp = j < n && kf[j] != 0;
        const bool is_hole = j < new_len && !kp;
        const bool is_mover = j >= new_len && j < n && kp;
        const bool is_ev = j < n && !kp;
        int th, tm, te;
        const int rh = block_rank(is_hole, s_red, th);
        const int rm = block_rank(is_mover, s_red, tm);
        const int re = block_rank(is_ev, s_red, te);
        if (is_hole) hb[run_h + rh] = j;
        if (is_mover) mvb[run_m + rm] = j;
        if (is_ev && evicted_ids) evicted_ids[(long)b * p.Lcap + run_e + re] = ib[j];
        run_h += th; run_m += tm; run_e += te;
    }
    __syncthreads();
    // move the small per-entry arrays (sources >= new_len, destinations < new_len: no overlap)
    for (int t = tid; t < run_m; t += blockDim.x) {
        const int src = mvb[t], dst = hb[t];
        if (ab) ab[dst] = ab[src];
        ib[dst] = ib[src];
        pb[dst] = pb[src];
    }
    if (tid == 0) {
        n_move[b] = run_m;
        len[b] = new_len;
        if (evicted_count) evicted_count[b] = run_e;
    }
}

// Row moves: movers[t] -> holes[t], t < n_move[b], of every sample in the caches of every layer (layer_stride elements
// apart; one layer for the per-step policy).  Bound by the memory's rate at mixed reads and writes, and that depends on how
// close together the rows lie that are under way at a time: blocks that take their rows in a fixed stride drift apart.
// So the rows are cut into pieces of up to 1024 threads (as a rule the K and the V row of one move, a vector a thread, or two)
// in the order of layers, samples and moves, and the blocks claim the next piece whenever they are done with one, as the
// hardware would hand out blocks if the host knew the number of moves.  64 caches of 4096 entries, 896 rows of 8 KiB moved in
// each: 357 us in strides, 320 so (5.9 TB/s); a block per move, their number known, takes 303.
// The kernel before this one has cleared the counters (decode_plan.hpp: which block claims which pieces).
// STREAM: both sides bypass the caches, also where K is small enough to stay there until the next step reads it: kept, the moved
// rows push out as much (14 caches of 882 entries cut to 208, 40 heads: next scores and moves 24.2 + 22.5 us, 26.0 + 22.1 with
// K kept).  Not where a head slice is shorter than a cache line.
// NV: vectors per thread; 0: one, and a piece holds several moves.  MANY: more samples than lanes.
template <bool STREAM, int NV, bool MANY>
__global__ __launch_bounds__(1024) void decode_move_kernel(
    DecodeDims p, KvLayout lay, MovePieces mp, FastDiv by_pair, int n_layers, const int32_t* __restrict__ holes, const int32_t* __restrict__ movers,
    const int32_t* __restrict__ n_move, int32_t* __restrict__ claims, uint16_t* __restrict__ k_cache, uint16_t* __restrict__ v_cache,
    long layer_stride)
{
    __shared__ uint32_t s_next[2];
    __shared__ int s_span[MANY ? kWave : 1], s_pieces[MANY ? kWave * kWave : 1];
    const int tid = threadIdx.x, lane = lane_id(), q = blockIdx.x % claim_counters(gridDim.x);
    int32_t* my_claims = claims + q * kClaimStride;
    // pieces of the 64 samples b0 .. b0 + 63, one per lane, and the sum of pieces up to and with each
    int b0 = 0, mine = 0, incl = 0;
    auto pieces_at = [&](int b) { return b < p.B ? pieces_of(n_move[min(b, p.B - 1)], mp) : 0; };
    auto group = [&](int at, int pieces, int before) {
        b0 = at;
        mine = pieces;
        incl = wave_incl_scan_i(pieces) + before;
    };
    // MANY: 64 spans of samples, one per lane, with the sum of pieces up to and with each.  The waves share the spans, so that
    // all counts are requested at once; a piece is found by its span and a look at 64 samples of it, in LDS up to 4096 samples.
    // In rounds over the samples by every wave the kernel took, for 4096 samples of 64 entries, one of 50 with a row to move,
    // 41 us (a block that looks at one sample only 29), in spans 5; half of the entries cut 86 (75) and 31.
    const int span = (p.B + kWave * kWave - 1) / (kWave * kWave) * kWave;
    int in_span = 0, upto_span = 0;
    if constexpr (MANY) {
        constexpr int SP = kWave / 16;               // spans of a wave
        const int first = wave_id() * SP;
        int sum[SP];
#pragma unroll
        for (int i = 0; i < SP; ++i) sum[i] = 0;
        for (int o = lane; o < span; o += kWave)
#pragma unroll
            for (int i = 0; i < SP; ++i) sum[i] += pieces_at((first + i) * span + o);
#pragma unroll
        for (int i = 0; i < SP; ++i) {
            if (span == kWave) s_pieces[(first + i) * kWave + lane] = sum[i];
            const int all = wave_sum_i(sum[i]);
            if (lane == 0) s_span[first + i] = all;
        }
        block_sync_lds();
        in_span = s_span[lane];
        upto_span = wave_incl_scan_i(in_span);
        b0 = -1;                                     // no samples at hand yet
    } else {
        group(0, pieces_at(lane), 0);
        upto_span = incl;
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane(upto_span, kWave - 1);      // of a layer
    if (total == 0) return;
    const uint64_t items = piece_count(total, n_layers);
    int buf = 0;
    for (uint64_t item = blockIdx.x; item < items;) {
        uint32_t claimed = 0;                        // the claim of the next piece is under way with this one's rows
        if (tid == 0) {
            int at = 0;
            asm volatile("" : "+v"(at));             // an address per lane: for a uniform one the compiler waits for the result on the spot
            claimed = (uint32_t)atomicAdd(my_claims + at, 1);
        }
        const auto [layer, r] = piece_at(item, total, n_layers);
        if (MANY && (r < __builtin_amdgcn_readlane(incl - mine, 0) || r >= __builtin_amdgcn_readlane(incl, kWave - 1))) {
            const int s = __builtin_ctzll(__ballot(upto_span > r));
            auto look = [&](int at, int before) { group(at, span == kWave ? s_pieces[at + lane] : pieces_at(at + lane), before); };
            if (b0 < s * span || r < __builtin_amdgcn_readlane(incl - mine, 0)) look(s * span, __builtin_amdgcn_readlane(upto_span - in_span, s));
            while (r >= __builtin_amdgcn_readlane(incl, kWave - 1)) look(b0 + kWave, __builtin_amdgcn_readlane(incl, kWave - 1));
        }
        const int l = __builtin_ctzll(__ballot(incl > r));
        const int b = b0 + l, at = r - __builtin_amdgcn_readlane(incl - mine, l);        // the sample's piece
        // this thread's move and its vectors of the pair; one move per piece: its rows come by scalar loads, which do not wait
        // for the stores under way
        constexpr int N = NV ? NV : 1;
        int src, dst, x[N];
        bool on = tid < mp.threads;
        if constexpr (NV > 0) {
            const int t = mp.per_move == 1 ? at : at / mp.per_move;
            const long li = (long)b * p.Lcap + t;
            src = movers[li]; dst = holes[li];
            asm volatile("" : "+s"(src), "+s"(dst));  // both requested before either is waited for
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = ((at - t * mp.per_move) * N + i) * mp.threads + tid;
        } else {
            const int u = by_pair.div(tid), t = at * mp.per_piece + u;
            const long li = (long)b * p.Lcap + min(t, p.Lcap - 1);
            src = movers[li]; dst = holes[li];
            x[0] = tid - u * mp.pair;
            on = on && t < n_move[b];
        }
        u32x4 val[N], *to[N];
        if (on) {
            const int rv = mp.pair >> 1, sh = __builtin_ctz(p.d) - 3;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int xi = min(x[i], mp.pair - 1);          // (behind the pair: its last vector, dropped)
                const bool is_v = xi >= rv;
                const int c = is_v ? xi - rv : xi;   // head slices of 2^sh vectors
                uint16_t* base = (is_v ? v_cache : k_cache) + layer * layer_stride + (long)b * lay.batch +
                                 (long)(c >> sh) * lay.head + (c & ((1 << sh) - 1)) * 8;
                const u32x4* from = reinterpret_cast<const u32x4*>(base + (long)src * lay.token);
                to[i] = reinterpret_cast<u32x4*>(base + (long)dst * lay.token);
                val[i] = STREAM ? __builtin_nontemporal_load(from) : *from;
            }
        }
        buf ^= 1;
        if (tid == 0) s_next[buf] = claimed;         // (requested before the rows; before the stores, which nothing here waits for)
        if (on) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if (N > 1 && x[i] >= mp.pair) continue;
                if (STREAM) __builtin_nontemporal_store(val[i], to[i]); else *to[i] = val[i];
            }
        }
        block_sync_lds();                            // (the stores need not have arrived)
        item = claimed_piece(gridDim.x, q, (uint32_t)__builtin_amdgcn_readfirstlane((int)s_next[buf]));
    }
}

__global__ __launch_bounds__(256) void decode_append_kernel(
    DecodeDims p, const u32x4* __restrict__ k_new, const u32x4* __restrict__ v_new,
    u32x4* __restrict__ k_cache, u32x4* __restrict__ v_cache,
    float* __restrict__ acc, int32_t* __restrict__ ids, uint8_t* __restrict__ protect, int32_t* __restrict__ len,
    int32_t new_id, int protect_new)
{
    const int b = blockIdx.x;
    const int slot = len[b];
    if (slot < 0 || slot >= p.Lcap) return;
    const int rv = p.H * p.d / 8;
    const long dst = ((long)b * p.Lcap + slot) * rv;
    for (int c = threadIdx.x; c < rv; c += blockDim.x) {
        k_cache[dst + c] = k_new[(long)b * rv + c];
        v_cache[dst + c] = v_new[(long)b * rv + c];
    }
    __syncthreads();                                   // every thread has read len[b] before it changes
    if (threadIdx.x == 0) {
        acc[(long)b * p.Lcap + slot] = 0.f;
        ids[(long)b * p.Lcap + slot] = new_id;
        protect[(long)b * p.Lcap + slot] = protect_new ? 1 : 0;
        len[b] = slot + 1;
    }
}

// The same for caches in other layouts: a row is walked head slice by head slice.
__global__ __launch_bounds__(256) void decode_append_strided_kernel(
    DecodeDims p, KvLayout lay, const u32x4* __restrict__ k_new, const u32x4* __restrict__ v_new,
    uint16_t* __restrict__ k_cache, uint16_t* __restrict__ v_cache,
    float* __restrict__ acc, int32_t* __restrict__ ids, uint8_t* __restrict__ protect, int32_t* __restrict__ len,
    int32_t new_id, int protect_new)
{
    const int b = blockIdx.x;
    const int slot = len[b];
    if (slot < 0 || slot >= p.Lcap) return;
    const int lph = p.d / 8, rv = p.H * lph;
    const long dst = (long)b * lay.batch + (long)slot * lay.token;
    for (int c = threadIdx.x; c < rv; c += blockDim.x) {
        const int h = c / lph, w = c - h * lph;
        const long off = dst + (long)h * lay.head + w * 8;
        *reinterpret_cast<u32x4*>(k_cache + off) = k_new[(long)b * rv + c];
        *reinterpret_cast<u32x4*>(v_cache + off) = v_new[(long)b * rv + c];
    }
    __syncthreads();                                   // every thread has read len[b] before it changes
    if (threadIdx.x == 0) {
        acc[(long)b * p.Lcap + slot] = 0.f;
        ids[(long)b * p.Lcap + slot] = new_id;
        protect[(long)b * p.Lcap + slot] = protect_new ? 1 : 0;
        len[b] = slot + 1;
    }
}

#ifndef MD_DEC_BLOCKS
#define MD_DEC_BLOCKS 4096   // target number of blocks of the streaming logits kernel
#endif

struct DecodeWorkspace {
    float* logits; float2* stat_partial; uint8_t* keep; int32_t* holes; int32_t* movers; int32_t* n_move;
    int32_t* claims;
    StateArrays copy;
    size_t bytes;
};

DecodeWorkspace carve_decode(void* base, int B, int Lcap, int H) {
    Carver c(base);
    DecodeWorkspace w;
    w.logits = c.take<float>((size_t)B * Lcap * H);
    w.stat_partial = c.take<float2>((size_t)B * kMaxStatParts * H);
    w.keep = c.take<uint8_t>((size_t)B * Lcap);
    w.holes = c.take<int32_t>((size_t)B * Lcap);
    w.movers = c.take<int32_t>((size_t)B * Lcap);
    w.n_move = c.take<int32_t>((size_t)B);
    w.claims = c.take<int32_t>((size_t)kClaims * kClaimStride);
    // (the general selection's keep flags and lists and the streaming one's copy of the state are never in use together)
    w.copy = StateArrays{reinterpret_cast<float*>(w.holes), w.movers, w.keep, w.n_move};
    w.bytes = c.off;
    return w;
}

// The row moves of every sample in the caches of n_layers layers; at most `most` of them per sample.
void launch_moves(const DecodeDims& p, const KvLayout& lay, const DecodeWorkspace& w, hipStream_t st, bool dense,
                  int n_layers, long layer_stride, int most, void* k_cache, void* v_cache) {
    const MovePieces mp = move_pieces(p.H, p.d);
    const int blocks = move_blocks(mp, n_layers, p.B, most);
    uint16_t* kc = static_cast<uint16_t*>(k_cache);
    uint16_t* vc = static_cast<uint16_t*>(v_cache);
#define MD_MOVE3(STREAM_, NV_, MANY_)                                                                          \
    MD_LAUNCH("decode_move", st, (decode_move_kernel<STREAM_, NV_, MANY_>), blocks, 1024, 0, p, lay, mp, FastDiv::make(mp.pair), n_layers, w.holes, \
        w.movers, w.n_move, w.claims, kc, vc, layer_stride)
#define MD_MOVE2(STREAM_, NV_) do { if (p.B > kWave) MD_MOVE3(STREAM_, NV_, true); else MD_MOVE3(STREAM_, NV_, false); } while (0)
#define MD_MOVE(NV_) do { if (dense || p.d >= 64) MD_MOVE2(true, NV_); else MD_MOVE2(false, NV_); } while (0)
    if (mp.per_piece > 1) MD_MOVE(0);
    else if (mp.vectors == 1) MD_MOVE(1);
    else MD_MOVE(2);
#undef MD_MOVE3
#undef MD_MOVE2
#undef MD_MOVE
}

int check_decode_dims(const char* who, int B, int Lcap, int H, int d) {
    if (B <= 0 || Lcap <= 0 || H <= 0 || d <= 0) return fail(MD_EINVAL, "%s: B, Lcap, H, d must be positive", who);
    if (d != 8 && d != 16 && d != 32 && d != 64 && d != 128 && d != 256 && d != 512)
        return fail(MD_ESHAPE, "%s: head dim %d must be a power of two in [8, 512]", who, d);
    if (H > 1024) return fail(MD_ESHAPE, "%s: H=%d exceeds the limit of 1024 heads", who, H);
    if ((long)B * Lcap > (1l << 28)) return fail(MD_ESHAPE, "%s: cache too large", who);
    return MD_OK;
}

}  // namespace
}  // namespace md

using namespace md;


extern "C" size_t mustdrop_decode_evict_workspace_bytes(int B, int Lcap, int H) {
    if (B <= 0 || Lcap <= 0 || H <= 0) return 0;
    return carve_decode(nullptr, B, Lcap, H).bytes;
}

namespace md {
namespace {

int decode_evict_impl(
    const void* q, void* k_cache, void* v_cache,
    float* acc, int32_t* ids, uint8_t* protect, int32_t* len,
    int B, int Lcap, int H, int d,
    float softmax_scale, float decay, int budget,
    int32_t* evicted_ids, int32_t* evicted_count,
    const md_kv_layout* cache_layout,
    void* workspace, size_t workspace_bytes, void* stream)
{
    clear_error();
    int rc = check_decode_dims("decode_evict", B, Lcap, H, d);
    if (rc != MD_OK) return rc;
    KvLayout lay;
    rc = read_layout("decode_evict", "cache", cache_layout, B, Lcap, H, d, &lay);
    if (rc != MD_OK) return rc;
    const bool dense = is_dense(lay, Lcap, H, d);
    if (!q || !k_cache || !v_cache || !acc || !ids || !protect || !len)
        return fail(MD_EINVAL, "decode_evict: q, the caches and the state arrays are required");
    if (budget < 0) return fail(MD_EINVAL, "decode_evict: negative budget");
    if (std::isnan(softmax_scale) || std::isnan(decay)) return fail(MD_EINVAL, "decode_evict: NaN parameter");
    // the selection ranks entries by the bit pattern of their running score, which orders non-negative values only
    if (decay < 0.f) return fail(MD_EINVAL, "decode_evict: decay must be >= 0 (running scores stay non-negative)");
    if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache))
        return fail(MD_EALIGN, "decode_evict: q and the caches must be 16-byte aligned");
    const size_t cache_bytes = layout_extent_bytes(lay, B, Lcap, H, d);
    if (overlaps(k_cache, cache_bytes, v_cache, cache_bytes)) return fail(MD_EALIAS, "decode_evict: k_cache overlaps v_cache");
    if (overlaps(q, (size_t)B * H * d * 2, k_cache, cache_bytes) || overlaps(q, (size_t)B * H * d * 2, v_cache, cache_bytes))
        return fail(MD_EALIAS, "decode_evict: q overlaps a cache");
    const DecodeWorkspace w = carve_decode(workspace, B, Lcap, H);
    {
        // the small state arrays, the optional outputs and the workspace against the caches, q and one another
        const size_t n = (size_t)B * Lcap;
        const void* pa[] = {acc, ids, protect, len, evicted_ids, evicted_count, workspace, k_cache, v_cache, q};
        const size_t sa[] = {n * 4, n * 4, n, (size_t)B * 4, n * 4, (size_t)B * 4, workspace ? w.bytes : 0,
                             cache_bytes, cache_bytes, (size_t)B * H * d * 2};
        for (int a = 0; a < 7; ++a)
            for (int c = a + 1; c < 10; ++c)
                if (overlaps(pa[a], sa[a], pa[c], sa[c]))
                    return fail(MD_EALIAS, "decode_evict: the state arrays, outputs, workspace, caches and q must not overlap");
    }
    if (!workspace || workspace_bytes < w.bytes)
        return fail(MD_EWORKSPACE, "decode_evict: workspace of %zu bytes needed, %zu given", w.bytes, workspace ? workspace_bytes : (size_t)0);
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(MD_EALIGN, "decode_evict: workspace must be 256-byte aligned");

    DecodeDims p{B, Lcap, H, d};
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint16_t* qp = static_cast<const uint16_t*>(q);
    const uint16_t* kp = static_cast<const uint16_t*>(k_cache);
    const int row_bytes = H * d * 2;
    // 1 KiB pieces of a row, rounded up to a form that is compiled (a piece behind the row's end costs a cached load)
    const int pieces = (row_bytes + 1023) / 1024;
    // Sixteen pieces take all registers of a wave.  Only dense rows of exactly 16 KiB, whose offsets need none, are read so;
    // other rows of more than ten pieces are shared by two blocks (32 x 1025 entries of 128 per head, 48 heads: 120 us in
    // one, 74 in halves, the general kernel 102; 64 heads, head-major: 140, 96 and 127; 64 heads, dense, in one: 96)
    const bool halves = pieces > 10 && !(dense && row_bytes == 16 * 1024);
    const int nit = pieces <= 2 ? pieces : (pieces <= 4 ? 4 : (pieces <= 5 ? 5 : (pieces <= 8 || halves ? 8 : (pieces <= 10 ? 10 : 16))));
    int n_part = 0;                                   // > 0: the logits kernel left per-block softmax statistics
    // selection in registers: up to 8192 slots, and heads in fours (a power of two up to 32: sums over lanes; any other
    // number, where a wave's shares still fit the 64 KB a launch gets: sums through LDS)
    const bool lane_sums = H == 4 || H == 8 || H == 16 || H == 32;
    const size_t select_lds = sizeof(int) * ((size_t)Lcap + (lane_sums ? 0 : 16 * 32 * ((size_t)H / 4)));
    const bool select_fast = (d == 128 || d == 64) && pieces <= 16 && Lcap <= 8192 && H % 4 == 0 && H <= 128 && select_lds <= 64 * 1024;
    // Moves in the selection's launch: blocks per sample that together cover the CUs but do not share one (33 x 168
    // entries: 264 blocks 16.7 us, 231 10.0, 132 9.4; as two launches 8.3 + 4.3), with no more teams than rows that can leave,
    // and reading no more than 32 MB of logits between them, 64 MB where all logits fit half of an XCD's 4 MB L2.  Where that leaves
    // neither half the chip nor all the teams nor 64 blocks for the one sample, the caches are long or many, and a launch
    // for the moves is the smaller price (us, one launch / two:
    // 4 x 778 entries of 40 heads 13.1 / 15.7, 1 x 1724 of 16 heads 8.7 / 12.8, 60 x 748 of 40 heads 14.4 / 16.7;
    // 64 x 1025 of 4352 slots 18.4 / 16.2, 18 x 4036 40.4 / 25.8, 64 x 4096 cut to 1024 407 / 387).
    // A few caches cut by much need the blocks for their rows, a steady loop does not mind them: 1 x 3500 entries of 32 heads
    // cut to 1000, the call, 54.2 us with 32 blocks and 44.6 with 128 (two launches 50.6), one entry leaving 18.2 and 18.2;
    // 2 x 2449 cut to 523 49.6 with 64 blocks, 46.4 with 212 (two launches 47.2), one leaving 19.2 and 19.3
    int select_x = B <= 256 ? 256 / B : 1;
    const long logit_bytes = (long)B * Lcap * H * 4;
    const long leave_x = Lcap > budget ? (Lcap - budget + 3l) / 4 : 1, read_x = (logit_bytes <= (2l << 20) ? 64l << 20 : 32l << 20) / logit_bytes;
    if (select_x > leave_x) select_x = (int)leave_x;
    if (select_x > 128) select_x = 128;
    if (select_x > read_x) select_x = (int)read_x;
    // (and where 64 MB or more could move, counted read and written: 138 blocks move the rows of 6 x 1838 entries cut to 345
    // more slowly than a launch over the whole chip, 30.3 against 15.1 + 13.1)
    const double move_bytes = (double)B * (Lcap > budget ? (Lcap - budget < budget ? Lcap - budget : budget) : 0) * H * d * 8;
    const bool one_launch = select_fast && select_x >= 1 && move_bytes < 64e6 && (select_x * (long)B >= 128 || select_x == leave_x || select_x >= 64);
    if (!one_launch) select_x = 1;
    const StateArrays state{acc, ids, protect, len};
    const StateArrays copy = one_launch && select_x > 1 ? w.copy : StateArrays{nullptr, nullptr, nullptr, nullptr};
    // a cache beyond half of the 256 MB Infinity Cache is streamed; a smaller one is kept cached for
    // the row moves and the steps that follow
    const bool stream_once = cache_bytes > (size_t)128 << 20;
    if ((d == 128 || d == 64) && pieces <= 16) {
        // streaming shape: about 16 waves per CU in flight, each striding over its sample's entries
        const int parts = halves ? 2 : 1;
        int blocks_x = (MD_DEC_BLOCKS / parts + B - 1) / B;
        const int max_x = (Lcap + 3) / 4;
        if (blocks_x > max_x) blocks_x = max_x;
        if (blocks_x > kMaxStatParts) blocks_x = kMaxStatParts;
        if (blocks_x < 1) blocks_x = 1;
        dim3 g1(blocks_x, B, parts);
#define MD_STREAM2(LPH_, NIT_, Y_, O_)                                                                             \
        MD_LAUNCH("decode_logits", st, (decode_logits_stream_kernel<LPH_, NIT_, Y_, O_>), g1, 256, 0,              \
            qp, kp, len, p, lay, softmax_scale, w.logits, w.stat_partial, state, copy)
#define MD_STREAM1(LPH_, NIT_)                                                                                     \
        do {                                                                                                       \
            if (!dense) { if (stream_once) MD_STREAM2(LPH_, NIT_, 2, true); else MD_STREAM2(LPH_, NIT_, 2, false); }                 \
            else if (row_bytes == NIT_ * 1024) { if (stream_once) MD_STREAM2(LPH_, NIT_, 0, true); else MD_STREAM2(LPH_, NIT_, 0, false); } \
            else { if (stream_once) MD_STREAM2(LPH_, NIT_, 1, true); else MD_STREAM2(LPH_, NIT_, 1, false); }                        \
        } while (0)
#define MD_STREAM(NIT_) do { if (d == 128) MD_STREAM1(16, NIT_); else MD_STREAM1(8, NIT_); } while (0)
        switch (nit) {
            case 1: MD_STREAM(1); break;
            case 2: MD_STREAM(2); break;
            case 4: MD_STREAM(4); break;
            case 5: MD_STREAM(5); break;
            case 8: MD_STREAM(8); break;
            case 10: MD_STREAM(10); break;
            default:                                  // dense rows of exactly 16 KiB
                if (d == 128) { if (stream_once) MD_STREAM2(16, 16, 0, true); else MD_STREAM2(16, 16, 0, false); }
                else { if (stream_once) MD_STREAM2(8, 16, 0, true); else MD_STREAM2(8, 16, 0, false); }
                break;
        }
#undef MD_STREAM2
#undef MD_STREAM1
#undef MD_STREAM
        n_part = blocks_x;
    } else {
        int tpb = (int)(((long)B * Lcap + 4095) / 4096);
        tpb = tpb < 4 ? 4 : (tpb > 32 ? 32 : tpb);
        dim3 g1((Lcap + tpb - 1) / tpb, B);
        switch (d / 8) {
            case 1: MD_LAUNCH("decode_logits", st, (decode_logits_kernel<1>), g1, 256, 0, qp, kp, len, p, lay, softmax_scale, tpb, w.logits); break;
            case 2: MD_LAUNCH("decode_logits", st, (decode_logits_kernel<2>), g1, 256, 0, qp, kp, len, p, lay, softmax_scale, tpb, w.logits); break;
            case 4: MD_LAUNCH("decode_logits", st, (decode_logits_kernel<4>), g1, 256, 0, qp, kp, len, p, lay, softmax_scale, tpb, w.logits); break;
            case 8: MD_LAUNCH("decode_logits", st, (decode_logits_kernel<8>), g1, 256, 0, qp, kp, len, p, lay, softmax_scale, tpb, w.logits); break;
            case 16: MD_LAUNCH("decode_logits", st, (decode_logits_kernel<16>), g1, 256, 0, qp, kp, len, p, lay, softmax_scale, tpb, w.logits); break;
            case 32: MD_LAUNCH("decode_logits", st, (decode_logits_kernel<32>), g1, 256, 0, qp, kp, len, p, lay, softmax_scale, tpb, w.logits); break;
            default: MD_LAUNCH("decode_logits", st, (decode_logits_kernel<64>), g1, 256, 0, qp, kp, len, p, lay, softmax_scale, tpb, w.logits); break;
        }
    }
    if (select_fast) {
        const int ipt = (Lcap + 1023) / 1024;
#define MD_SELECT_FAST(I, E)                                                                                       \
    MD_LAUNCH("decode_select", st, (decode_select_fast_kernel<I, E>), dim3(select_x, B), 1024, select_lds,         \
        p, w.logits, w.stat_partial, n_part, decay, budget, copy.acc ? copy : state, state, lay,                   \
        static_cast<uint16_t*>(k_cache), static_cast<uint16_t*>(v_cache), stream_once ? 1 : 0,               \
        w.holes, w.movers, one_launch ? nullptr : w.n_move, w.claims, evicted_ids, evicted_count)
#define MD_SELECT_FAST_H(I)                                                                                        \
    switch (H) {                                                                                                   \
        case 4: MD_SELECT_FAST(I, 1); break;                                                                       \
        case 8: MD_SELECT_FAST(I, 2); break;                                                                       \
        case 16: MD_SELECT_FAST(I, 4); break;                                                                      \
        case 32: MD_SELECT_FAST(I, 8); break;                                                                      \
        default: MD_SELECT_FAST(I, 0); break;                                                                      \
    }
        if (ipt <= 1) { MD_SELECT_FAST_H(1) }
        else if (ipt <= 2) { MD_SELECT_FAST_H(2) }
        else if (ipt <= 3) { MD_SELECT_FAST_H(3) }
        else if (ipt <= 4) { MD_SELECT_FAST_H(4) }
        else if (ipt <= 5) { MD_SELECT_FAST_H(5) }
        else if (ipt <= 6) { MD_SELECT_FAST_H(6) }
        else { MD_SELECT_FAST_H(8) }
#undef MD_SELECT_FAST_H
#undef MD_SELECT_FAST
        if (one_launch) return check_launch("decode_evict");
    } else {
        const size_t lds = sizeof(float) * ((size_t)2 * H + 1024);
        MD_LAUNCH("decode_select", st, (decode_select_kernel), B, 1024, lds,
            p, w.logits, decay, budget, acc, ids, protect, len, w.keep, w.holes, w.movers, w.n_move, w.claims, evicted_ids, evicted_count);
    }
    launch_moves(p, lay, w, st, dense, 1, 0l, most_moves(Lcap, budget), k_cache, v_cache);
    return check_launch("decode_evict");
}

int decode_keep_impl(
    void* k_cache, void* v_cache, const uint8_t* keep,
    float* acc, int32_t* ids, uint8_t* protect, int32_t* len,
    int n_layers, int B, int Lcap, int H, int d,
    int32_t* evicted_ids, int32_t* evicted_count,
    const md_kv_layout* cache_layout, int64_t layer_stride_in,
    void* workspace, size_t workspace_bytes, void* stream)
{
    clear_error();
    int rc = check_decode_dims("decode_keep", B, Lcap, H, d);
    if (rc != MD_OK) return rc;
    if (n_layers <= 0 || n_layers > 65535) return fail(MD_EINVAL, "decode_keep: n_layers=%d out of range", n_layers);
    KvLayout lay;
    rc = read_layout("decode_keep", "cache", cache_layout, B, Lcap, H, d, &lay);
    if (rc != MD_OK) return rc;
    const size_t layer_bytes = layout_extent_bytes(lay, B, Lcap, H, d);
    long layer_stride = cache_layout ? (long)layer_stride_in : (long)B * Lcap * H * d;
    if (n_layers == 1) layer_stride = (long)(layer_bytes / 2);
    if (layer_stride <= 0 || layer_stride % 8 || (size_t)layer_stride * 2 < layer_bytes)
        return fail(MD_ESHAPE, "decode_keep: layer_stride=%ld must be a multiple of 8 elements covering one layer (%zu elements)",
                    layer_stride, layer_bytes / 2);
    const bool dense = is_dense(lay, Lcap, H, d);
    if (!k_cache || !v_cache || !keep || !ids || !protect || !len)
        return fail(MD_EINVAL, "decode_keep: null pointer among the required arguments");
    if ((H * d * 2) % 16) return fail(MD_EALIGN, "decode_keep: a row of H*d=%d bf16 is not a multiple of 16 bytes", H * d);
    if (!aligned16(k_cache) || !aligned16(v_cache)) return fail(MD_EALIGN, "decode_keep: caches must be 16-byte aligned");
    const size_t cache_bytes = (size_t)(n_layers - 1) * layer_stride * 2 + layer_bytes;
    if (overlaps(k_cache, cache_bytes, v_cache, cache_bytes)) return fail(MD_EALIAS, "decode_keep: k_cache overlaps v_cache");
    const DecodeWorkspace w = carve_decode(workspace, B, Lcap, H);
    if (!workspace || workspace_bytes < w.bytes)
        return fail(MD_EWORKSPACE, "decode_keep: workspace of %zu bytes needed, %zu given", w.bytes, workspace ? workspace_bytes : (size_t)0);
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(MD_EALIGN, "decode_keep: workspace must be 256-byte aligned");

    DecodeDims p{B, Lcap, H, d};
    hipStream_t st = static_cast<hipStream_t>(stream);
    MD_LAUNCH("decode_keep_plan", st, (decode_keep_plan_kernel), B, 1024, 0,
        p, keep, acc, ids, protect, len, w.holes, w.movers, w.n_move, w.claims, evicted_ids, evicted_count);
    launch_moves(p, lay, w, st, dense, n_layers, layer_stride, most_moves(Lcap, 0), k_cache, v_cache);
    return check_launch("decode_keep");
}

int decode_append_impl(
    const void* k_new, const void* v_new, void* k_cache, void* v_cache,
    float* acc, int32_t* ids, uint8_t* protect, int32_t* len,
    int B, int Lcap, int H, int d, int32_t new_id, int protect_new, const md_kv_layout* cache_layout, void* stream)
{
    clear_error();
    int rc = check_decode_dims("decode_append", B, Lcap, H, d);
    if (rc != MD_OK) return rc;
    KvLayout lay;
    rc = read_layout("decode_append", "cache", cache_layout, B, Lcap, H, d, &lay);
    if (rc != MD_OK) return rc;
    if (!k_new || !v_new || !k_cache || !v_cache || !acc || !ids || !protect || !len)
        return fail(MD_EINVAL, "decode_append: all pointers are required");
    if (new_id < 0) return fail(MD_EINVAL, "decode_append: ids must be non-negative");
    if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_cache) || !aligned16(v_cache))
        return fail(MD_EALIGN, "decode_append: tensors must be 16-byte aligned");
    DecodeDims p{B, Lcap, H, d};
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (is_dense(lay, Lcap, H, d))
        MD_LAUNCH("decode_append", st, (decode_append_kernel), B, 256, 0,
            p, static_cast<const u32x4*>(k_new), static_cast<const u32x4*>(v_new),
            static_cast<u32x4*>(k_cache), static_cast<u32x4*>(v_cache), acc, ids, protect, len, new_id, protect_new);
    else
        MD_LAUNCH("decode_append", st, (decode_append_strided_kernel), B, 256, 0,
            p, lay, static_cast<const u32x4*>(k_new), static_cast<const u32x4*>(v_new),
            static_cast<uint16_t*>(k_cache), static_cast<uint16_t*>(v_cache), acc, ids, protect, len, new_id, protect_new);
    return check_launch("decode_append");
}

}  // namespace
}  // namespace md

extern "C" int mustdrop_decode_evict(
    const void* q, void* k_cache, void* v_cache, float* acc, int32_t* ids, uint8_t* protect, int32_t* len,
    int B, int Lcap, int H, int d, float softmax_scale, float decay, int budget,
    int32_t* evicted_ids, int32_t* evicted_count, void* workspace, size_t workspace_bytes, void* stream)
{
    return decode_evict_impl(q, k_cache, v_cache, acc, ids, protect, len, B, Lcap, H, d, softmax_scale, decay, budget,
                             evicted_ids, evicted_count, nullptr, workspace, workspace_bytes, stream);
}

extern "C" int mustdrop_decode_evict_strided(
    const void* q, void* k_cache, void* v_cache, float* acc, int32_t* ids, uint8_t* protect, int32_t* len,
    int B, int Lcap, int H, int d, float softmax_scale, float decay, int budget,
    int32_t* evicted_ids, int32_t* evicted_count, const md_kv_layout* cache_layout,
    void* workspace, size_t workspace_bytes, void* stream)
{
    return decode_evict_impl(q, k_cache, v_cache, acc, ids, protect, len, B, Lcap, H, d, softmax_scale, decay, budget,
                             evicted_ids, evicted_count, cache_layout, workspace, workspace_bytes, stream);
}

extern "C" int mustdrop_decode_keep(
    void* k_cache, void* v_cache, const uint8_t* keep, float* acc, int32_t* ids, uint8_t* protect, int32_t* len,
    int n_layers, int B, int Lcap, int H, int d, int32_t* evicted_ids, int32_t* evicted_count,
    void* workspace, size_t workspace_bytes, void* stream)
{
    return decode_keep_impl(k_cache, v_cache, keep, acc, ids, protect, len, n_layers, B, Lcap, H, d, evicted_ids,
                            evicted_count, nullptr, 0, workspace, workspace_bytes, stream);
}

extern "C" int mustdrop_decode_keep_strided(
    void* k_cache, void* v_cache, const uint8_t* keep, float* acc, int32_t* ids, uint8_t* protect, int32_t* len,
    int n_layers, int B, int Lcap, int H, int d, int32_t* evicted_ids, int32_t* evicted_count,
    const md_kv_layout* cache_layout, int64_t layer_stride, void* workspace, size_t workspace_bytes, void* stream)
{
    return decode_keep_impl(k_cache, v_cache, keep, acc, ids, protect, len, n_layers, B, Lcap, H, d, evicted_ids,
                            evicted_count, cache_layout, layer_stride, workspace, workspace_bytes, stream);
}

extern "C" int mustdrop_decode_append(
    const void* k_new, const void* v_new, void* k_cache, void* v_cache,
    float* acc, int32_t* ids, uint8_t* protect, int32_t* len,
    int B, int Lcap, int H, int d, int32_t new_id, int protect_new, void* stream)
{
    return decode_append_impl(k_new, v_new, k_cache, v_cache, acc, ids, protect, len, B, Lcap, H, d, new_id, protect_new,
                              nullptr, stream);
}

extern "C" int mustdrop_decode_append_strided(
    const void* k_new, const void* v_new, void* k_cache, void* v_cache,
    float* acc, int32_t* ids, uint8_t* protect, int32_t* len,
    int B, int Lcap, int H, int d, int32_t new_id, int protect_new, const md_kv_layout* cache_layout, void* stream)
{
    return decode_append_impl(k_new, v_new, k_cache, v_cache, acc, ids, protect, len, B, Lcap, H, d, new_id, protect_new,
                              cache_layout, stream);
}
