// Stage 1 -- vision encoding (Sec. 3.3): Key Retaining (Eq. 6-7, budget form) and Local Spatial
// Merging (Eq. 5), followed by stable compaction of the survivors.
//
// Launch plan (all on the caller's stream, no host synchronisation):
//   encode_scores_kernel one launch, two kinds of waves (two launches for many tokens, see ScoreBlocks):
//       window waves     one wave per window: Gram matrix in registers -> S    (HBM: reads x once)
//       key-row waves    one wave per eight key rows, or per 64-vector slice of   (HBM: reads k_cls once)
//                        them: q_cls . k_j per head
//   encode_decide_*      one block per sample: softmax + head mean (or ready-made key scores), radix top-k -> O,
//                        merge decisions, prefix sum of survivors, small outputs    (tiny)
//   encode_emit_kernel  one wave per window: row copies / mass-weighted means (re-reads x, writes out_x); not launched
//                        where several blocks per sample make the decisions and write the rows behind them
#include "md_device.hpp"
#include "md_host.hpp"
#include "encode_plan.hpp"

#include <mutex>

namespace md {
namespace {

constexpr float kLog2eE = 1.4426950408889634f;
constexpr int kMaxWindow = 16;                   // = the length of EncodeDims::moff
#ifndef MD_ENC_WAVES
#define MD_ENC_WAVES 4
#endif
constexpr int kEncWaves = MD_ENC_WAVES;          // waves (= work items) per block of the wave-per-item kernels
constexpr int kMaxClsHeads = 256;
constexpr int kNumCU = 256;                      // MI355X

struct EncodeDims {
    int B, T, Hg, Wg, D, Hc, dc;
    int kt, kh, kw;
    int M, W, ws, nwx, nwy, nwt;
    int clipped;      // the window does not divide the grid: windows at the far border hold fewer tokens
    // members m < ws, filled by the host so that kernels get them as scalars: token = window_base + moff[m], and the
    // place inside the window, mpos[m] = dt << 16 | dy << 8 | dx
    int moff[16], mpos[16];
    FastDiv by_W, by_nwx, by_nwy, by_kw, by_kh;
};

// A window on the grid: its first token and how far it reaches (clipped windows hold fewer tokens).
struct WindowAt { int base, rt, ry, rx; };
__device__ __forceinline__ WindowAt window_at(const EncodeDims& p, int w) {
    const int row = p.by_nwx.div(w), wx = w - row * p.nwx, wt = p.by_nwy.div(row), wy = row - wt * p.nwy;
    const int t = wt * p.kt, y = wy * p.kh, x = wx * p.kw;
    return WindowAt{(t * p.Hg + y) * p.Wg + x, p.T - t, p.Hg - y, p.Wg - x};
}
__device__ __forceinline__ bool member_exists(const EncodeDims& p, const WindowAt& a, int m) {
    return !p.clipped || ((p.mpos[m] >> 16) < a.rt && ((p.mpos[m] >> 8) & 0xFF) < a.ry && (p.mpos[m] & 0xFF) < a.rx);
}
// A wave that works on one window: lane m < ws computes member m's token (-1 where a clipped window does not have
// it); read back with wave_member().
__device__ __forceinline__ int lane_member_token(const EncodeDims& p, int w, int lane) {
    const WindowAt a = window_at(p, w);
    const int row = p.by_kw.div(lane), dx = lane - row * p.kw, dt = p.by_kh.div(row), dy = row - dt * p.kh;
    if (lane >= p.ws) return 0;
    return dt < a.rt && dy < a.ry && dx < a.rx ? a.base + (dt * p.Hg + dy) * p.Wg + dx : -1;
}
__device__ __forceinline__ int wave_member(int per_lane, int m) { return __builtin_amdgcn_readlane(per_lane, m); }

__device__ __forceinline__ int window_of_token(const EncodeDims& p, int tok) {
    const int x = tok % p.Wg, y = (tok / p.Wg) % p.Hg, t = tok / (p.Wg * p.Hg);
    return ((t / p.kt) * p.nwy + (y / p.kh)) * p.nwx + (x / p.kw);
}

// One 16-byte vector of a row, widened to fp32.  VEC = 4 (fp32) or 8 (bf16).
template <bool BF> struct Vec;
template <> struct Vec<false> {
    static constexpr int N = 4;
    // a vector as loaded, and the dot product of two of them added to acc (elements in ascending order)
    using Raw = f32x4;
    __device__ static __forceinline__ Raw load_raw(const void* row, int c) { return *reinterpret_cast<const f32x4*>(static_cast<const float*>(row) + c); }
    __device__ static __forceinline__ Raw load_raw_once(const void* row, int c) { return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(static_cast<const float*>(row) + c)); }
    __device__ static __forceinline__ Raw zero() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
    __device__ static __forceinline__ float dot(const Raw& a, const Raw& b, float acc) {
        acc = fmaf(a.x, b.x, acc); acc = fmaf(a.y, b.y, acc); acc = fmaf(a.z, b.z, acc); return fmaf(a.w, b.w, acc);
    }
    __device__ static __forceinline__ void load(const void* row, int c, float (&o)[4]) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(static_cast<const float*>(row) + c);
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    }
    // data that is not read again: streaming load
    __device__ static __forceinline__ void load_once(const void* row, int c, float (&o)[4]) {
        const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(static_cast<const float*>(row) + c));
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    }
    __device__ static __forceinline__ void store(void* row, int c, const float (&o)[4]) {
        f32x4 v; v.x = o[0]; v.y = o[1]; v.z = o[2]; v.w = o[3];
        *reinterpret_cast<f32x4*>(static_cast<float*>(row) + c) = v;
    }
};
template <> struct Vec<true> {
    static constexpr int N = 8;
    // bf16 pairs stay packed: v_dot2c_f32_bf16 multiplies two pairs and adds both products to an fp32
    // accumulator (the products of bf16 values are exact in fp32), one instruction per two elements and
    // no widening
    using Raw = u32x4;
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    __device__ static __forceinline__ Raw load_raw(const void* row, int c) { return *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(row) + c); }
    __device__ static __forceinline__ Raw load_raw_once(const void* row, int c) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(row) + c)); }
    __device__ static __forceinline__ Raw zero() { return u32x4{0u, 0u, 0u, 0u}; }
    __device__ static __forceinline__ float dot2(uint32_t a, uint32_t b, float acc) {
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), acc, false);
    }
    __device__ static __forceinline__ float dot(const Raw& a, const Raw& b, float acc) {
        acc = dot2(a.x, b.x, acc); acc = dot2(a.y, b.y, acc); acc = dot2(a.z, b.z, acc); return dot2(a.w, b.w, acc);
    }
    __device__ static __forceinline__ void widen(const u32x4 v, float (&o)[8]) {
        o[0] = bf16_lo(v.x); o[1] = bf16_hi(v.x); o[2] = bf16_lo(v.y); o[3] = bf16_hi(v.y);
        o[4] = bf16_lo(v.z); o[5] = bf16_hi(v.z); o[6] = bf16_lo(v.w); o[7] = bf16_hi(v.w);
    }
    __device__ static __forceinline__ void load(const void* row, int c, float (&o)[8]) {
        widen(*reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(row) + c), o);
    }
    __device__ static __forceinline__ void load_once(const void* row, int c, float (&o)[8]) {
        widen(__builtin_nontemporal_load(reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(row) + c)), o);
    }
    __device__ static __forceinline__ void store(void* row, int c, const float (&o)[8]) {
        u32x4 v;
        v.x = f32_to_bf16(o[0]) | (f32_to_bf16(o[1]) << 16);
        v.y = f32_to_bf16(o[2]) | (f32_to_bf16(o[3]) << 16);
        v.z = f32_to_bf16(o[4]) | (f32_to_bf16(o[5]) << 16);
        v.w = f32_to_bf16(o[6]) | (f32_to_bf16(o[7]) << 16);
        *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(row) + c) = v;
    }
};

// ---------------------------------------------------------------------------------------------
// Eq. 6, the part that needs no global view.  With x[h][j] = log2(e) * q_cls[b][h] . k_cls[b][j][h] / sqrt(dc),
// j = 0..M, one wave takes kClsRows consecutive key rows of a sample (their loads are in flight
// together) and leaves, per head h and for its group g of rows,
//     part[b][h][g] = (m, z):  m = max of x over the rows that count (the CLS row and the valid tokens),
//                              z = sum of exp2(x - m) over them,
//     num[b][j][h]  = exp2(x[h][j] - m)   for each of those rows (heads contiguous),
// so that the decision kernel gets a probability as num * exp2(m - m_h) / Z_h with one factor per
// (head, group): no exponential per (head, token) on the one CU that decides for a sample.
// A head covers vph = dc/VEC consecutive 16-byte vectors (a power of two), so the per-head sums are
// segmented butterflies over vph lanes (or whole-wave sums if vph >= 64).
constexpr int kClsRows = 8;
__host__ __device__ __forceinline__ int cls_groups(int M) { return (M + 1 + kClsRows - 1) / kClsRows; }

// it_first, it_end: the rows' 64-vector slices to work on (all of them, or with SLICED the one of this wave).
// MERGED: the block's waves merge their groups' statistics through s_stat (see ScoreBlocks); `part` then takes the
// maxima m alone, as floats [b][h][group].
template <bool BF, bool SLICED, bool MERGED>
__device__ __forceinline__ void cls_logits_rows(
    int b, int g, int it_first, int it_end, const void* __restrict__ q_cls, const void* __restrict__ k_cls, const uint8_t* __restrict__ valid,
    const EncodeDims& p, float* __restrict__ logits, float2* __restrict__ part, float2* s_stat)
{
    constexpr int VEC = Vec<BF>::N;
    constexpr int R = kClsRows;
    const int lane = lane_id();
    const int gps = cls_groups(p.M), j0 = g * R;
    // wave-uniform.  Loads are never guarded one by one (a guarded load waits for the one before it):
    // addresses are clamped into the sample instead and what was read for an inactive row is ignored.
    bool act[R];
    uint32_t vbyte[R];
#pragma unroll
    for (int r = 0; r < R; ++r) vbyte[r] = valid ? valid[(size_t)b * p.M + min(max(j0 + r - 1, 0), p.M - 1)] : 1u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = j0 + r;
        act[r] = j <= p.M && (j == 0 || vbyte[r] != 0);
    }

    const size_t esz = BF ? 2 : 4;
    const char* qrow = static_cast<const char*>(q_cls) + (size_t)b * p.D * esz;
    const size_t rowb = (size_t)p.D * esz;
    const char* kb0 = static_cast<const char*>(k_cls) + (size_t)b * (p.M + 1) * rowb;
    const char* krow[R];
#pragma unroll
    for (int r = 0; r < R; ++r) krow[r] = kb0 + (size_t)min(j0 + r, p.M) * rowb;
    const int nvec = p.D / VEC, vph = p.dc / VEC;
    const float scale = 1.0f / sqrtf((float)p.dc);
    float* out = logits + ((size_t)b * (p.M + 1) + j0) * p.Hc;
    float2* pout = part + (size_t)b * p.Hc * gps + g;
    float* pmax = reinterpret_cast<float*>(part) + (size_t)b * p.Hc * gps + g;
    // the R logits of one head -> numerators (in place) and their statistics (every lane that holds
    // them computes the same values)
    auto finish = [&](float (&lg)[R]) -> float2 {
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (act[r]) mx = fmaxf(mx, lg[r] * kLog2eE);
        float z = 0.f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            lg[r] = act[r] ? fast_exp2(fmaf(lg[r], kLog2eE, -mx)) : 0.f;
            z += lg[r];
        }
        return make_float2(mx, z);
    };

    float acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.f;
    // slices of the rows per round: fp32 rows are twice as long, and a lone image waits half as often with two in
    // flight (scores of 1 x 576 tokens 10.6 -> 9.8 us); bf16 with two is slower (8 x 2880 tokens 18.1 -> 20.0 us)
    constexpr int UNR = BF || SLICED ? 1 : 2;
    for (int it0 = it_first; it0 < it_end; it0 += UNR) {
        typename Vec<BF>::Raw kv[UNR][R], qv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int ic = min((it0 + u) * kWave + lane, nvec - 1);  // lanes beyond the row repeat its last vector and drop it
            qv[u] = Vec<BF>::load_raw(qrow, ic * VEC);
            // the key rows are read exactly once: streaming loads, so that they do not push x (read again by
            // the emit kernel) out of the Infinity Cache
#pragma unroll
            for (int r = 0; r < R; ++r) kv[u][r] = Vec<BF>::load_raw_once(krow[r], ic * VEC);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int it = it0 + u, idx = it * kWave + lane;
            if (it >= it_end) break;
            float part_r[R];
#pragma unroll
            for (int r = 0; r < R; ++r) part_r[r] = act[r] && idx < nvec ? Vec<BF>::dot(qv[u], kv[u][r], 0.f) : 0.f;
            if (SLICED || vph < kWave) {
                float lg[R];
#pragma unroll
                for (int r = 0; r < R; ++r) lg[r] = group_sum_rt(part_r[r], vph) * scale;
                if (idx < nvec && (lane & (vph - 1)) == 0) {
                    const int h = idx / vph;
                    const float2 st = finish(lg);
                    if (MERGED) { s_stat[h] = st; pmax[(size_t)h * gps] = st.x; }
                    else pout[(size_t)h * gps] = st;
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (act[r]) out[(size_t)r * p.Hc + h] = lg[r];
                }
            } else {
                const int per_head = vph / kWave;                 // iterations per head
#pragma unroll
                for (int r = 0; r < R; ++r) acc[r] += part_r[r];
                if ((it + 1) % per_head == 0) {
                    float lg[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) { lg[r] = wave_sum(acc[r]) * scale; acc[r] = 0.f; }
                    if (lane == 0) {
                        const int h = it / per_head;
                        const float2 st = finish(lg);
                        if (MERGED) { s_stat[h] = st; pmax[(size_t)h * gps] = st.x; }
                        else pout[(size_t)h * gps] = st;
#pragma unroll
                        for (int r = 0; r < R; ++r)
                            if (act[r]) out[(size_t)r * p.Hc + h] = lg[r];
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Eq. 5: S_w = mean over unordered pairs of valid members of cos(x_m, x_n).  One wave per window;
// each lane owns a strided slice of the feature dimension and keeps the upper triangle of the
// Gram matrix (norms on the diagonal) in registers.  What follows the loads is a chain on one wave, so it is kept
// short: all sums in one butterfly that halves its list as it goes, then a lane per pair for the cosines (against 36
// separate wave sums and 28 divisions on one lane: 4 x 4608 tokens, 2x2x2 windows, 22.4 -> 15.6 us = 4.8 TB/s).
template <int WSM, bool BF>
__device__ __forceinline__ void window_sim_item(
    int item, const void* __restrict__ x, const uint8_t* __restrict__ valid, const EncodeDims& p, float* __restrict__ sim,
    float* s_gram)
{
    constexpr int VEC = Vec<BF>::N;
    const int lane = lane_id();
    if (item >= p.B * p.W) return;
    const int b = p.by_W.div(item), w = item - b * p.W;
    const size_t esz = BF ? 2 : 4;

    const char* rows[WSM];
    bool ok[WSM];
    const int tok_l = lane_member_token(p, w, lane);
    const int ok_l = lane < p.ws && tok_l >= 0 && (!valid || valid[(size_t)b * p.M + max(tok_l, 0)]);
#pragma unroll
    for (int m = 0; m < WSM; ++m) {
        // every slot gets a readable row (members beyond the window repeat member 0, invalid members
        // keep their own row): the loads below are unconditional and what they return is zeroed
        const int mm = m < p.ws ? m : 0;
        ok[m] = m < p.ws && wave_member(ok_l, mm) != 0;
        rows[m] = static_cast<const char*>(x) + ((size_t)b * p.M + max(wave_member(tok_l, mm), 0)) * p.D * esz;
    }
    constexpr int NG = WSM * (WSM + 1) / 2;
    float G[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) G[i] = 0.f;

    // slices of the feature dimension per round: a small window has the whole 1024 elements in flight (fp32: 16
    // loads; 16 x 576 tokens 19.7 -> 17.7 us, 8 x 2880 tokens 41 -> 37 us against two slices)
    constexpr int NS = WSM <= 4 ? (BF ? 2 : 4) : 1;
    for (int c0 = lane * VEC; c0 < p.D; c0 += NS * kWave * VEC) {
        typename Vec<BF>::Raw v[NS][WSM];
        bool in[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int c = c0 + q * kWave * VEC;
            in[q] = c < p.D;
#pragma unroll
            for (int m = 0; m < WSM; ++m) v[q][m] = Vec<BF>::load_raw(rows[m], in[q] ? c : c0);
        }
#pragma unroll
        for (int q = 0; q < NS; ++q)
#pragma unroll
            for (int m = 0; m < WSM; ++m)
                if (!ok[m] || !in[q]) v[q][m] = Vec<BF>::zero();
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            int idx = 0;
#pragma unroll
            for (int m = 0; m < WSM; ++m)
#pragma unroll
                for (int n = m; n < WSM; ++n) {
                    G[idx] = Vec<BF>::dot(v[q][m], v[q][n], G[idx]);
                    ++idx;
                }
        }
    }
    wave_sums(G, lane);
    // the sums change hands through LDS: lane q takes the pairs q, q + 64, ...
    constexpr int NP = WSM * (WSM - 1) / 2;
#pragma unroll
    for (int r = 0; r < WaveSums<NG>::H3; ++r) {
        const int i = wave_sums_index<NG>(lane, r);
        if (lane < 16 && i >= 0) s_gram[i] = G[r];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint64_t okmask = __ballot(ok_l);
    float S = 0.f;
    int npairs = 0;
#pragma unroll
    for (int q0 = 0; q0 < NP; q0 += kWave) {
        int m = 0, left = q0 + lane;                 // pair q -> members m < n: WSM-1 pairs with member 0, then WSM-2, ...
#pragma unroll
        for (int mm = 0; mm < WSM - 1; ++mm)
            if (m == mm && left >= WSM - 1 - mm) { left -= WSM - 1 - mm; ++m; }
        const bool in = q0 + lane < NP;
        const int n = in ? m + 1 + left : 0;
        m = in ? m : 0;
        const int at = m * WSM - m * (m - 1) / 2;    // the triangle's row m: (m, m) first
        const float dm = s_gram[at], dn = s_gram[n * WSM - n * (n - 1) / 2], g = s_gram[at + n - m];
        const bool both = in && ((okmask >> m) & (okmask >> n) & 1ull);
        if (both && dm > 0.f && dn > 0.f) S += g / (sqrtf(dm) * sqrtf(dn));
        npairs += __popcll(__ballot(both));
    }
    S = wave_sum(S);
    if (lane == 0) sim[(size_t)b * p.W + w] = npairs > 0 ? S / (float)npairs : 0.f;
}

// Key scores a_cls of kKeyTokens tokens per block, for samples whose decision takes them ready-made
// (encode_decide_large_kernel).  The block merges the per-block statistics of the whole sample (a pair per head and
// kClsRows * kEncWaves key rows), turns its own groups' maxima into factors and adds up num * factor over the heads.
// All of a round's loads are in flight together.
constexpr int kMaxMergedHeads = 64;
constexpr int kKeyTokens = 256;
constexpr int kKeyGroups = kKeyTokens / kClsRows + 1;
__host__ __device__ __forceinline__ int cls_blocks(int M) { return (cls_groups(M) + kEncWaves - 1) / kEncWaves; }
struct KeyScoreLds {
    float f[kKeyGroups * kMaxMergedHeads];           // [group][head]
    float2 st[256];
    float m[kMaxMergedHeads], inv[kMaxMergedHeads];
};
__device__ __forceinline__ void key_scores(
    int b, int chunk, const EncodeDims& p, const uint8_t* __restrict__ valid, const float* __restrict__ logits,
    const float* __restrict__ group_max, const float2* __restrict__ block_stat, float* __restrict__ acls,
    float* __restrict__ a_cls_out, KeyScoreLds& s)
{
    const int tid = threadIdx.x, M = p.M, Hc = p.Hc;
    const int j = chunk * kKeyTokens + tid, jc = min(j, M - 1);      // this thread's token
    const int gps = cls_groups(M), cb = cls_blocks(M), g0 = (chunk * kKeyTokens + 1) / kClsRows;
    const int ng = min(kKeyGroups, gps - g0);
    // the token's first 16 numerators, its validity and the first group maximum depend on nothing
    const f32x4* x = reinterpret_cast<const f32x4*>(logits + ((size_t)b * (M + 1) + 1 + jc) * Hc);
    f32x4 xv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) xv[q] = x[min(q, Hc / 4 - 1)];
    const bool ok = !valid || valid[(size_t)b * M + jc];
    // statistics: thread = (slice, head), eight pairs per round
    const int nsl = 256 / Hc, h = tid % Hc, sl = tid / Hc;
    {
        const float2* bs = block_stat + (size_t)b * cb * Hc + h;
        float mx = -INFINITY, z = 0.f;
        if (sl < nsl)
            for (int c0 = sl; c0 < cb; c0 += 8 * nsl) {
                float2 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = bs[(size_t)min(c0 + u * nsl, cb - 1) * Hc];
                float m2 = mx;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (c0 + u * nsl >= cb) v[u] = make_float2(-INFINITY, 0.f);
                    m2 = fmaxf(m2, v[u].x);
                }
                if (m2 > -INFINITY) {
                    z *= fast_exp2(mx - m2);
#pragma unroll
                    for (int u = 0; u < 8; ++u) z = fmaf(v[u].y, fast_exp2(v[u].x - m2), z);
                }
                mx = m2;
            }
        s.st[tid] = make_float2(mx, z);
    }
    __syncthreads();
    if (tid < Hc) {
        float mx = -INFINITY, z = 0.f;
        for (int q = 0; q < nsl; ++q) mx = fmaxf(mx, s.st[q * Hc + tid].x);
        for (int q = 0; q < nsl; ++q) z = fmaf(s.st[q * Hc + tid].y, fast_exp2(s.st[q * Hc + tid].x - mx), z);
        s.m[tid] = mx;                               // finite: the CLS row always counts
        s.inv[tid] = 1.0f / (z * (float)Hc);
    }
    __syncthreads();
    for (int e = tid; e < ng * Hc; e += 256) {
        const int hh = e / ng, g = e - hh * ng;      // groups contiguous in group_max
        s.f[g * Hc + hh] = fast_exp2(group_max[((size_t)b * Hc + hh) * gps + g0 + g] - s.m[hh]) * s.inv[hh];
    }
    __syncthreads();
    if (j >= M) return;
    const f32x4* f = reinterpret_cast<const f32x4*>(s.f + ((j + 1) / kClsRows - g0) * Hc);
    float a = 0.f;
    auto add = [&](const f32x4& v, const f32x4& w) {
        a = fmaf(v.x, w.x, a); a = fmaf(v.y, w.y, a); a = fmaf(v.z, w.z, a); a = fmaf(v.w, w.w, a);
    };
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (q < Hc / 4) add(xv[q], f[q]);
    for (int q = 4; q < Hc / 4; ++q) add(x[q], f[q]);
    if (!ok) a = -INFINITY;                          // (its numerators were never written)
    acls[(size_t)b * M + j] = a;
    if (a_cls_out) a_cls_out[(size_t)b * M + j] = a;
}

// Both bandwidth-bound score passes: waves that take a window each (Eq. 5) and waves that take a few key rows each
// (Eq. 6 logits; none when no key set is asked for).  A block does one of the three things below; the launch says
// where in the grid each begins.
//   windows, then key rows      one launch
//   key-score blocks, windows   the second of two launches for samples whose decision wants the scores ready-made;
//                               the key scores hide behind the windows.  The first one takes the key rows alone: its
//                               blocks (each within one sample) leave their groups' statistics
//                               merged: block_stat[b][block of the sample][h], in the half of cls_part that the
//                               groups' sums do not need then (their maxima take the first half, as floats; it fits
//                               from two groups on, and such calls have more).
struct ScoreBlocks { int keyscore, windows, rows, slices; };         // blocks of each kind, in grid order; waves per key-row group

// The key rows of one block, with its groups' statistics merged.
template <bool QKBF>
__device__ __forceinline__ void merged_rows(
    int blk, const void* __restrict__ q_cls, const void* __restrict__ k_cls, const uint8_t* __restrict__ valid, const EncodeDims& p,
    float* __restrict__ logits, float2* __restrict__ cls_part, float2* __restrict__ block_stat, float2 (&s_stat)[kEncWaves][kMaxMergedHeads])
{
    const int gps = cls_groups(p.M), cb = cls_blocks(p.M), b = blk / cb, wb = blk % cb, g = wb * kEncWaves + wave_id();
    const int iters = (p.D / Vec<QKBF>::N + kWave - 1) / kWave;
    if (g < gps) cls_logits_rows<QKBF, false, true>(b, g, 0, iters, q_cls, k_cls, valid, p, logits, cls_part, s_stat[wave_id()]);
    __syncthreads();
    const int nw = min(kEncWaves, gps - wb * kEncWaves);
    for (int h = threadIdx.x; h < p.Hc; h += blockDim.x) {
        float mx = -INFINITY, z = 0.f;
        for (int w = 0; w < nw; ++w) mx = fmaxf(mx, s_stat[w][h].x);
        for (int w = 0; w < nw; ++w)
            if (s_stat[w][h].x > -INFINITY) z = fmaf(s_stat[w][h].y, fast_exp2(s_stat[w][h].x - mx), z);
        block_stat[((size_t)b * cb + wb) * p.Hc + h] = make_float2(mx, z);
    }
}

template <int WSM, bool XBF, bool QKBF>
__global__ __launch_bounds__(256) void encode_scores_kernel(
    const void* __restrict__ x, const void* __restrict__ q_cls, const void* __restrict__ k_cls,
    const uint8_t* __restrict__ valid, EncodeDims p, ScoreBlocks nb, float* __restrict__ sim, float* __restrict__ logits,
    float2* __restrict__ cls_part, float2* __restrict__ block_stat, float* __restrict__ acls, float* __restrict__ a_cls_out)
{
    union Lds { KeyScoreLds k; float2 stat[kEncWaves][kMaxMergedHeads]; float gram[kEncWaves][WSM * (WSM + 1) / 2]; };
    __shared__ Lds s;
    int blk = blockIdx.x;
    if (blk < nb.keyscore) {
        const int chunks = (p.M + kKeyTokens - 1) / kKeyTokens;
        if (blk / chunks < p.B)
            key_scores(blk / chunks, blk % chunks, p, valid, logits, reinterpret_cast<const float*>(cls_part), block_stat, acls, a_cls_out, s.k);
        return;
    }
    blk -= nb.keyscore;
    if (blk < nb.windows) {
        window_sim_item<WSM, XBF>(blk * kEncWaves + wave_id(), x, valid, p, sim, s.gram[wave_id()]);
        return;
    }
    blk -= nb.windows;
    const int gps = cls_groups(p.M);
    if (nb.slices > 1) {                             // a wave per (group of key rows, slice of the feature dimension)
        const int item = blk * kEncWaves + wave_id(), gs = item / nb.slices, sl = item - gs * nb.slices, b = gs / gps;
        if (b < p.B) cls_logits_rows<QKBF, true, false>(b, gs - b * gps, sl, sl + 1, q_cls, k_cls, valid, p, logits, cls_part, nullptr);
        return;
    }
    if constexpr (QKBF)
        if (block_stat) { merged_rows<QKBF>(blk, q_cls, k_cls, valid, p, logits, cls_part, block_stat, s.stat); return; }
    const int cb = cls_blocks(p.M), b = blk / cb, g = blk % cb * kEncWaves + wave_id();
    const int iters = (p.D / Vec<QKBF>::N + kWave - 1) / kWave;
    if (g < gps) cls_logits_rows<QKBF, false, false>(b, g, 0, iters, q_cls, k_cls, valid, p, logits, cls_part, nullptr);
}

// The first of the two launches for fp32 keys.  A kernel of its own: as one more path of encode_scores_kernel it made the calls
// without it slower (88 x 416 tokens of 384 features 49.4 -> 51.8 us, 55 x 290 of 256 23.9 -> 25.0).  With bf16 keys it is
// the other way round (16 x 576 tokens 22.2 with the path, 22.45 without; 8 x 2880 42.3 and 42.5), and it stays there.
__global__ __launch_bounds__(256) void encode_rows_f32_kernel(
    const void* __restrict__ q_cls, const void* __restrict__ k_cls, const uint8_t* __restrict__ valid, EncodeDims p,
    float* __restrict__ logits, float2* __restrict__ cls_part, float2* __restrict__ block_stat)
{
    __shared__ float2 s_stat[kEncWaves][kMaxMergedHeads];
    merged_rows<false>(blockIdx.x, q_cls, k_cls, valid, p, logits, cls_part, block_stat, s_stat);
}

// ---------------------------------------------------------------------------------------------
// Per-sample decisions.  One block per sample.
__global__ __launch_bounds__(1024) void encode_decide_kernel(
    EncodeDims p, const uint8_t* __restrict__ valid, const float* __restrict__ mass_in,
    const float* __restrict__ logits, const float2* __restrict__ cls_part, const float* __restrict__ sim, float tau,
    int key_budget, int key_adaptive, float key_lambda, int32_t* __restrict__ key_count,
    float* __restrict__ acls, uint8_t* __restrict__ iskey, uint8_t* __restrict__ wmerged,
    int32_t* __restrict__ dstpos,
    int32_t* __restrict__ out_index, float* __restrict__ out_mass, uint8_t* __restrict__ out_is_key,
    uint8_t* __restrict__ out_valid, int32_t* __restrict__ out_count, int32_t* __restrict__ key_index,
    float* __restrict__ a_cls_out, float* __restrict__ window_sim_out)
{
    __shared__ float s_max[kMaxClsHeads], s_inv[kMaxClsHeads];
    __shared__ int s_hist[256];
    __shared__ int s_red[16];
    __shared__ float s_redf[16];
    const int b = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wv = wave_id(), nw = blockDim.x >> 6;
    const int M = p.M, W = p.W;
    const uint8_t* vb = valid ? valid + (size_t)b * M : nullptr;
    const float* mb = mass_in ? mass_in + (size_t)b * M : nullptr;
    float* acls_b = acls + (size_t)b * M;
    uint8_t* iskey_b = iskey + (size_t)b * M;
    uint8_t* wm_b = wmerged + (size_t)b * W;
    int32_t* dst_b = dstpos + (size_t)b * M;

    // ---- Key Retaining
    if (key_budget > 0 || key_adaptive) {
        const float* lg = logits + (size_t)b * (M + 1) * p.Hc;       // numerators [row][head], see cls_logits_rows
        const int gps = cls_groups(M);
        const float2* pb = cls_part + (size_t)b * p.Hc * gps;
        for (int h = wv; h < p.Hc; h += nw) {
            const float2* pp = pb + (size_t)h * gps;
            float mx = -INFINITY;
            for (int g = lane; g < gps; g += kWave) mx = fmaxf(mx, pp[g].x);
            mx = wave_max(mx);
            float z = 0.f;
            for (int g = lane; g < gps; g += kWave) {
                const float2 v = pp[g];
                if (v.x > -INFINITY) z = fmaf(v.y, fast_exp2(v.x - mx), z);
            }
            z = wave_sum(z);
            if (lane == 0) { s_max[h] = mx; s_inv[h] = 1.0f / (z * (float)p.Hc); }
        }
        __syncthreads();
        for (int j = tid; j < M; j += blockDim.x) {
            float a = -INFINITY;
            if (!vb || vb[j]) {
                a = 0.f;
                const int g = (j + 1) / kClsRows;
                for (int h = 0; h < p.Hc; ++h)
                    a = fmaf(lg[(size_t)(j + 1) * p.Hc + h], fast_exp2(pb[(size_t)h * gps + g].x - s_max[h]) * s_inv[h], a);
            }
            acls_b[j] = a;
            if (a_cls_out) a_cls_out[(size_t)b * M + j] = a;
        }
        __syncthreads();
        auto keyfn = [&](int i, bool& ok) -> uint64_t {
            ok = !vb || vb[i];
            return ok ? rank_key(acls_b[i], i) : 0ull;
        };
        SelectBound sb{0ull, 63};
        float mu = 0.f;
        if (!key_adaptive) {                         // Eq. 7, budget form
            sb = block_radix_select(keyfn, M, key_budget, s_hist);
        } else {                                     // Eq. 7 as printed: a_cls > mu, mu = mean + lambda * std
            float s1 = 0.f;
            int cnt = 0;
            for (int j = tid; j < M; j += blockDim.x)
                if (!vb || vb[j]) { s1 += acls_b[j]; ++cnt; }
            s1 = block_sum(s1, s_redf);
            cnt = block_sum_i(cnt, s_red);
            const float mean = cnt > 0 ? s1 / (float)cnt : 0.f;
            float s2 = 0.f;
            for (int j = tid; j < M; j += blockDim.x)
                if (!vb || vb[j]) { const float dlt = acls_b[j] - mean; s2 = fmaf(dlt, dlt, s2); }
            s2 = block_sum(s2, s_redf);
            mu = mean + key_lambda * sqrtf(cnt > 0 ? s2 / (float)cnt : 0.f);
        }
        int running = 0;                             // keys so far; key_budget is the capacity of key_index
        for (int base = 0; base < M; base += blockDim.x) {
            const int j = base + tid;
            bool sel = false;
            if (j < M && (!vb || vb[j]))
                sel = key_adaptive ? acls_b[j] > mu : (rank_key(acls_b[j], j) >> sb.shift) >= sb.bound;
            if (j < M) iskey_b[j] = sel;
            int total;
            const int r = block_rank(sel, s_red, total);
            if (sel && running + r < key_budget) key_index[(size_t)b * key_budget + running + r] = j;
            running += total;
        }
        for (int r = running + tid; r < key_budget; r += blockDim.x) key_index[(size_t)b * key_budget + r] = -1;
        if (key_count && tid == 0) key_count[b] = running;
    } else {
        for (int j = tid; j < M; j += blockDim.x) {
            iskey_b[j] = 0;
            if (a_cls_out) a_cls_out[(size_t)b * M + j] = 0.f;
        }
    }
    __syncthreads();

    // ---- merge decision per window: S > tau, >= 2 valid members, no key member
    for (int w = tid; w < W; w += blockDim.x) {
        int n = 0;
        bool has_key = false;
        const WindowAt at = window_at(p, w);
        for (int m = 0; m < p.ws; ++m) {
            const int tok = at.base + p.moff[m];
            if (!member_exists(p, at, m) || (vb && !vb[tok])) continue;
            ++n;
            has_key |= iskey_b[tok] != 0;
        }
        const float S = sim[(size_t)b * W + w];
        wm_b[w] = (n >= 2 && !has_key && S > tau) ? 1 : 0;
        if (window_sim_out) window_sim_out[(size_t)b * W + w] = S;
    }
    __syncthreads();

    // ---- survivors in ascending token index: exclusive prefix sum of the survivor flags
    int running = 0;
    for (int base = 0; base < M; base += blockDim.x) {
        const int j = base + tid;
        bool surv = false, merged = false;
        float mass = 0.f;
        if (j < M && (!vb || vb[j])) {
            const int w = window_of_token(p, j);
            merged = wm_b[w] != 0;
            if (!merged) {
                surv = true;
                mass = mb ? mb[j] : 1.0f;
            } else {
                int first = -1;
                const WindowAt at = window_at(p, w);
                for (int m = 0; m < p.ws; ++m) {
                    const int tok = at.base + p.moff[m];
                    if (!member_exists(p, at, m) || (vb && !vb[tok])) continue;
                    if (first < 0) first = tok;
                    mass += mb ? mb[tok] : 1.0f;
                }
                surv = (first == j);
            }
        }
        int total;
        const int r = block_rank(surv, s_red, total);
        if (j < M) dst_b[j] = surv ? running + r : -1;
        if (surv) {
            const size_t o = (size_t)b * M + running + r;
            out_index[o] = j;
            out_mass[o] = mass;
            out_is_key[o] = merged ? 0 : iskey_b[j];
        }
        running += total;
    }
    if (tid == 0) out_count[b] = running;
    if (out_valid)
        for (int s = tid; s < M; s += blockDim.x) out_valid[(size_t)b * M + s] = s < running;
}

// ---------------------------------------------------------------------------------------------
// The rows of the survivors, written by the blocks that decide (EmitArgs::blocks of them per sample, each of which has worked
// out the whole sample's decisions in its LDS; a launch of its own is 4 us and finds nothing of x requested).  An item is a
// window and a slice of 64 16-byte vectors of its rows.  x does not wait for the decisions: a wave asks for its first item
// before they are made, so that a third of x on 8 x 2880 tokens, and all of it on a few images, comes in behind their chain
// of steps, which is what bounds the launch (17 of its 40 thousand cycles on 8 x 2880 tokens are the rows, the decision with its
// fetch of the numerators the rest).  us per call, a launch for the rows / the deciding blocks: 1 x 576 tokens fp32 15.8 /
// 13.4, 16 x 576 22.3 / 20.5, 8 x 2880 42.3 / 39.7, 16 x 2880 71.7 / 65.4.  Not for windows of more than eight members, whose rows
// do not fit the registers (3 x 1152 tokens in 3x3 windows 22.4 / 23.8), nor beyond 3072 tokens: a call by itself still gains
// up to 5120 (4 x 4608 in 2x2x2 windows 42.8 / 42.0), but the longer decisions on all CUs are in the way of other streams' kernels
// (that workload's whole step, two batches in flight 128 / 135, four 112 / 117; 8 x 2880 165 / 163 and 169 / 169); and with
// ready-made scores it loses by itself too (2 x 9216 46.5 / 47.1).
struct EmitArgs {
    const void* x; void* out_x;
    int blocks, slices, bf16;                        // blocks per sample, slices per row, element type
    FastDiv by_B, by_slices;
};
// a token's fate as the emitting waves read it: its output row (with kRowMerged for the mean of a window), or
enum : int { kRowMerged = 1 << 30, kRowInvalid = -1, kRowGone = -2 };
struct EmitItem { int w, c, tok; };                  // window, this lane's vector of the rows, lane m < ws: member m's token
__device__ __forceinline__ EmitItem emit_item(const EncodeDims& p, const EmitArgs& e, int it, int lane) {
    EmitItem i;
    i.w = e.by_slices.div(it);
    i.c = (it - i.w * e.slices) * kWave + lane;
    i.tok = lane_member_token(p, i.w, lane);
    return i;
}
template <int WS>
__device__ __forceinline__ void emit_load(const EncodeDims& p, const EmitItem& i, const char* xb, int rowb, u32x4 (&v)[WS]) {
    const int off = min(i.c * 16, rowb - 16);        // lanes beyond the row repeat its last vector and drop it
#pragma unroll
    for (int m = 0; m < WS; ++m)                     // (members beyond the window repeat its last one)
        v[m] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(xb + (size_t)max(wave_member(i.tok, min(m, p.ws - 1)), 0) * rowb + off));
}
// What an item's rows become: row_l: lane m's row (s_row), merged: the window is merged, with okmask its valid members.
struct EmitFate { int row_l; uint64_t merged, okmask; float mass_l; };
__device__ __forceinline__ EmitFate emit_fate(const EncodeDims& p, const EmitItem& i, const int* s_row, const float* mb) {
    EmitFate f;
    f.row_l = lane_id() < p.ws && i.tok >= 0 ? s_row[i.tok] : (int)kRowInvalid;
    f.merged = __ballot(f.row_l >= 0 && (f.row_l & kRowMerged));
    f.okmask = __ballot(f.row_l != kRowInvalid);
    f.mass_l = f.merged != 0 && mb && f.row_l != kRowInvalid ? mb[i.tok] : 1.0f;
    return f;
}
template <int WS>
__device__ __forceinline__ void emit_copy(const EmitItem& i, const EmitFate& f, char* ob, int rowb, const u32x4 (&v)[WS]) {
    if (i.c * 16 >= rowb) return;
    char* o = ob + (size_t)i.c * 16;
#pragma unroll
    for (int m = 0; m < WS; ++m) {
        const int row = wave_member(f.row_l, m);     // (lanes beyond the window: kRowInvalid)
        if (row >= 0) __builtin_nontemporal_store(v[m], reinterpret_cast<u32x4*>(o + (size_t)row * rowb));
    }
}
// The mass-weighted mean of the valid members, in ascending order, written at the first one.
template <bool BF, int WS>
__device__ __forceinline__ void emit_mean(const EmitItem& i, const EmitFate& f, char* ob, int rowb, const u32x4 (&v)[WS]) {
    constexpr int VEC = Vec<BF>::N;
    float acc[VEC], msum = 0.f;
#pragma unroll
    for (int q = 0; q < VEC; ++q) acc[q] = 0.f;
#pragma unroll
    for (int m = 0; m < WS; ++m) {
        if (!((f.okmask >> m) & 1ull)) continue;
        const float mm = lane_bcast_f(f.mass_l, m);
        msum += mm;
        float xv[VEC];
        if constexpr (BF) Vec<true>::widen(v[m], xv);
        else { const f32x4 x = __builtin_bit_cast(f32x4, v[m]); xv[0] = x.x; xv[1] = x.y; xv[2] = x.z; xv[3] = x.w; }
#pragma unroll
        for (int q = 0; q < VEC; ++q) acc[q] = fmaf(mm, xv[q], acc[q]);
    }
#pragma unroll
    for (int q = 0; q < VEC; ++q) acc[q] = acc[q] / msum;
    if (i.c * 16 < rowb)
        Vec<BF>::store(ob + (size_t)(wave_member(f.row_l, __builtin_ctzll(f.merged)) & ~kRowMerged) * rowb + (size_t)i.c * 16, 0, acc);
}
// The block's share of the sample's items; the rows of the next one are on their way while one is written.  AHEAD: `cur` and
// `v` are the wave's first item, already asked for.
template <int WS, bool AHEAD>
__device__ __forceinline__ void emit_rows(const EncodeDims& p, const EmitArgs& e, int b, int g, const int* s_row, const float* mb,
                                          EmitItem cur, u32x4 (&v)[WS]) {
    const int lane = lane_id(), rowb = p.D * (e.bf16 ? 2 : 4), items = p.W * e.slices, every = e.blocks * 16;
    const char* xb = static_cast<const char*>(e.x) + (size_t)b * p.M * rowb;
    char* ob = static_cast<char*>(e.out_x) + (size_t)b * p.M * rowb;
    int it = wave_id() * e.blocks + g;
    if (!AHEAD && it < items) {
        cur = emit_item(p, e, it, lane);
        emit_load<WS>(p, cur, xb, rowb, v);
    }
    for (; it < items; it += every) {
        EmitItem nxt = cur;
        u32x4 nv[WS];
        const bool more = it + every < items;
        if (more) {
            nxt = emit_item(p, e, it + every, lane);
            emit_load<WS>(p, nxt, xb, rowb, nv);
        }
        const EmitFate f = emit_fate(p, cur, s_row, mb);
        if (f.merged == 0ull) emit_copy<WS>(cur, f, ob, rowb, v);
        else if (e.bf16) emit_mean<true, WS>(cur, f, ob, rowb, v);
        else emit_mean<false, WS>(cur, f, ob, rowb, v);
        cur = nxt;
        if (more) {
#pragma unroll
            for (int m = 0; m < WS; ++m) v[m] = nv[m];
        }
    }
}

// ---------------------------------------------------------------------------------------------
// The same decisions for M <= 1024*IPT <= 5120 with a sample's tokens in registers (thread t owns the IPT
// consecutive tokens t*IPT ..): the kernel is a chain of dependent steps on one CU per sample, so it
// is built to be short rather than wide.
//   - the softmax denominators come from the per-wave statistics the score kernel left (a few
//     hundred pairs per head), while the own tokens' logits are already on their way;
//   - the top-k radix select starts below the bits that all scores share;
//   - key ranks and survivor ranks come from ONE block scan of a packed pair of counts.
#ifdef MD_DECIDE_TICKS
#define MD_DTICK(k) do { if (threadIdx.x == 0 && blockIdx.x == 0) ticks[k] = __builtin_readcyclecounter(); } while (0)
#else
#define MD_DTICK(k) do { } while (0)
#endif
// EMIT: em.blocks blocks per sample (blocks of a sample em.by_B.d apart: with eight samples and more on one XCD, whose L2 they
// share), each of which makes all of the decisions and then writes its share of the rows and of the small outputs.
template <int IPT, int WS, bool EMIT>
__global__ __launch_bounds__(1024) void encode_decide_fast_kernel(
    EncodeDims p, const uint8_t* __restrict__ valid, const float* __restrict__ mass_in,
    const float* __restrict__ logits, const float2* __restrict__ cls_part, const float* __restrict__ sim,
    float tau, int key_budget, int key_adaptive, float key_lambda, int32_t* __restrict__ key_count,
    uint8_t* __restrict__ wmerged, int32_t* __restrict__ dstpos,
    int32_t* __restrict__ out_index, float* __restrict__ out_mass, uint8_t* __restrict__ out_is_key,
    uint8_t* __restrict__ out_valid, int32_t* __restrict__ out_count, int32_t* __restrict__ key_index,
    float* __restrict__ a_cls_out, float* __restrict__ window_sim_out, EmitArgs em)
{
    // [M] merged-window mass / scores (float), then [M] key flags and [M] token states, which take the place of
    // the [groups][16] factors of Eq. 6 (see decide_fast_lds_bytes)
    extern __shared__ __attribute__((aligned(16))) uint8_t s_dyn[];
    __shared__ int s_hist[kSelectHistInts];
    __shared__ int s_red[16];
    __shared__ float s_redf[16];
#ifdef MD_DECIDE_TICKS
    __shared__ long long ticks[12];
#endif
    MD_DTICK(0);
    const int g = EMIT ? em.by_B.div(blockIdx.x) : 0, b = blockIdx.x - g * p.B, tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const int M = p.M, W = p.W;
    const bool writes = !EMIT || (em.blocks < 16 ? wv % em.blocks : wv) == g;     // the small outputs go by waves
    if (tid < 256) s_hist[tid] = 0;                         // for block_select_topk, after later barriers
    float* s_tmass = reinterpret_cast<float*>(s_dyn);
    uint8_t* s_key = s_dyn + 4 * (size_t)M;
    uint8_t* s_state = s_key + M;                    // 0: not in a merged window, 1: first valid member, 2: merged away
    const uint8_t* vb = valid ? valid + (size_t)b * M : nullptr;
    const float* mb = mass_in ? mass_in + (size_t)b * M : nullptr;
    const int j0 = tid * IPT;                        // first own token (and first own window)
    const bool with_keys = key_budget > 0 || key_adaptive;
    const float* lg = logits + (size_t)b * (M + 1) * p.Hc;           // numerators [row][head], row 0 = CLS

    // ---- everything that depends on nothing is requested first (clamped or range-checked addresses, no
    // guarded loads: a guarded load would wait for the one before it)
    // Eq. 6: wave h owns head h (Hc <= 16 = waves of the block; waves beyond Hc contribute zeros).  Its
    // lanes take the head's per-group statistics (group = kClsRows rows, see cls_logits_rows).
    constexpr int PRE = 16;                          // heads
    constexpr int NPB = 2 * IPT + 1;                 // groups per lane: 64 * NPB >= cls_groups(1024 * IPT)
    constexpr bool EARLY = IPT <= 4;                 // registers allow the first batch to be requested up front
    const int gps = cls_groups(M);
    float2 pv[NPB];
    if (with_keys) {
        const float2* pp = cls_part + ((size_t)b * p.Hc + min(wv, p.Hc - 1)) * gps;
#pragma unroll
        for (int u = 0; u < NPB; ++u) pv[u] = pp[min(lane + u * kWave, gps - 1)];
    }
    // Numerators of the tokens tid + 1024*t: the 16 heads of a token are 64 consecutive bytes, four 16-byte buffer loads (tokens
    // beyond M and heads beyond Hc fall outside the buffer's range and read as zero: see numerator_vector).  The scores change
    // hands through LDS afterwards.
    constexpr int PT = IPT < 4 ? IPT : 4;            // tokens per batch
    const __amdgpu_buffer_rsrc_t rnum = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(lg + p.Hc), 0, numerator_bytes(M, p.Hc), 0x00020000);
    f32x4 xl[PT][4];
    auto request_numerators = [&](int t0) {
#pragma unroll
        for (int t = 0; t < PT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (t0 + t < IPT)
                    xl[t][q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                        rnum, numerator_vector(tid, t0 + t, q, M, p.Hc), 0, 0));
    };
    bool ok[IPT];
    float mass[IPT], simv[IPT];
    {
        uint32_t vbyte[IPT];
#pragma unroll
        for (int t = 0; t < IPT; ++t) vbyte[t] = vb ? vb[min(j0 + t, M - 1)] : 1u;
#pragma unroll
        for (int t = 0; t < IPT; ++t) mass[t] = mb ? mb[min(j0 + t, M - 1)] : 1.0f;
#pragma unroll
        for (int t = 0; t < IPT; ++t) simv[t] = sim[(size_t)b * W + min(tid + 1024 * t, W - 1)];
        if (EARLY && with_keys) request_numerators(0);
#pragma unroll
        for (int t = 0; t < IPT; ++t) {
            const int j = j0 + t;
            ok[t] = j < M && vbyte[t] != 0;
            if (j >= M) mass[t] = 1.0f;
        }
    }
    bool sel[IPT];
#pragma unroll
    for (int t = 0; t < IPT; ++t) sel[t] = false;
    // What a window's decision needs besides the key flags, on its way with the loads above: its first token, which members
    // are valid, and the masses of the first four.  (Nothing here uses what a load of a mass returns: the wave would wait
    // for everything requested so far.)
    struct WinInfo { int base; uint32_t vmask; float mm[4]; };
    auto analyse = [&](int w) -> WinInfo {
        WinInfo wi;
        const WindowAt at = window_at(p, w);
        wi.base = at.base;
        wi.vmask = 0u;
#pragma unroll
        for (int m = 0; m < WS; ++m) wi.vmask |= (m < p.ws && member_exists(p, at, m) ? 1u : 0u) << m;
#pragma unroll
        for (int u = 0; u < 4; ++u) wi.mm[u] = 1.0f;
        if (mb) {
#pragma unroll
            for (int u = 0; u < 4; ++u) wi.mm[u] = mb[(wi.vmask >> u) & 1u ? wi.base + p.moff[u] : wi.base];   // the window's first token is always there
        }
        if (vb) {
            uint32_t vv[WS];
#pragma unroll
            for (int m = 0; m < WS; ++m) vv[m] = vb[(wi.vmask >> m) & 1u ? wi.base + p.moff[m] : wi.base];
#pragma unroll
            for (int m = 0; m < WS; ++m)
                if (vv[m] == 0) wi.vmask &= ~(1u << m);
        }
        return wi;
    };
    WinInfo win0 = analyse(min(tid, W - 1));         // nearly always the thread's only window (W <= 1024)
    constexpr bool AHEAD = EMIT && (WS == 4 || IPT <= 2);      // registers allow the first rows to be requested up front
    EmitItem item{};
    u32x4 rowv[WS];
    if constexpr (AHEAD) {                           // (whatever the case: a wait for anything older could not tell these loads apart)
        const int rowb = p.D * (em.bf16 ? 2 : 4);
        item = emit_item(p, em, min(wv * em.blocks + g, W * em.slices - 1), lane);
        emit_load<WS>(p, item, static_cast<const char*>(em.x) + (size_t)b * M * rowb, rowb, rowv);
    }
    MD_DTICK(8);

    if (with_keys) {
        // head statistics (m_h, Z_h) and the factor of every group: f[g][h] = exp2(m_g - m_h) / (Z_h * Hc)
        float* s_f = reinterpret_cast<float*>(s_dyn + ((4 * (size_t)M + 15) & ~(size_t)15));   // [gps][PRE], gone before the key flags are written
        {
            float mx = -INFINITY;
#pragma unroll
            for (int u = 0; u < NPB; ++u) {
                if (lane + u * kWave >= gps) pv[u] = make_float2(-INFINITY, 0.f);
                mx = fmaxf(mx, pv[u].x);
            }
            const float gm = wave_max(mx);
            MD_DTICK(9);
            float z = 0.f;
#pragma unroll
            for (int u = 0; u < NPB; ++u) {
                pv[u].x = fast_exp2(pv[u].x - gm);   // (gm is finite: the CLS row always counts)
                z = fmaf(pv[u].y, pv[u].x, z);
            }
            const float inv = wv < p.Hc ? 1.0f / (wave_sum(z) * (float)p.Hc) : 0.f;
#pragma unroll
            for (int u = 0; u < NPB; ++u)
                if (lane + u * kWave < gps) s_f[(lane + u * kWave) * PRE + wv] = pv[u].x * inv;
        }
        if (!EARLY) request_numerators(0);
        MD_DTICK(10);
        __syncthreads();
        MD_DTICK(1);
        // a_cls (head mean of the probabilities) of the tokens tid + 1024*t
        float* s_a = s_tmass;                        // free until the merge decisions
#pragma unroll
        for (int t0 = 0; t0 < IPT; t0 += PT) {
            if (t0 > 0) request_numerators(t0);
#pragma unroll
            for (int t = 0; t < PT; ++t) {
                if (t0 + t >= IPT) continue;
                const int j = tid + 1024 * (t0 + t);
                const f32x4* fr = reinterpret_cast<const f32x4*>(s_f + (size_t)(min(j, M - 1) + 1) / kClsRows * PRE);
                float a = 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 f = fr[q];
                    a = fmaf(xl[t][q].x, f.x, a);
                    a = fmaf(xl[t][q].y, f.y, a);
                    a = fmaf(xl[t][q].z, f.z, a);
                    a = fmaf(xl[t][q].w, f.w, a);
                }
                if (j < M) s_a[j] = a;
            }
        }
        __syncthreads();
        MD_DTICK(2);
        uint64_t rk[IPT];
        float av[IPT];
#pragma unroll
        for (int t = 0; t < IPT; ++t) {
            const int j = j0 + t;
            av[t] = s_a[min(j, M - 1)];
            const float a = ok[t] ? av[t] : -INFINITY;
            if (j < M && a_cls_out && writes) a_cls_out[(size_t)b * M + j] = a;
            rk[t] = ok[t] ? rank_key(a, j) : 0ull;
        }
        if (!key_adaptive) {                         // Eq. 7, budget form: the key_budget largest scores
            const SelectBound sb = block_select_topk<IPT>(rk, key_budget, s_hist);
#pragma unroll
            for (int t = 0; t < IPT; ++t) sel[t] = rk[t] != 0 && (rk[t] >> sb.shift) >= sb.bound;
        } else {                                     // Eq. 7 as printed: a_cls > mu, mu = mean + lambda * std
            float s1 = 0.f;
            int cnt = 0;
#pragma unroll
            for (int t = 0; t < IPT; ++t)
                if (ok[t]) { s1 += av[t]; ++cnt; }
            s1 = block_sum(s1, s_redf);
            cnt = block_sum_i(cnt, s_red);
            const float mean = cnt > 0 ? s1 / (float)cnt : 0.f;
            float s2 = 0.f;
#pragma unroll
            for (int t = 0; t < IPT; ++t)
                if (ok[t]) { const float dlt = av[t] - mean; s2 = fmaf(dlt, dlt, s2); }
            s2 = block_sum(s2, s_redf);
            const float mu = mean + key_lambda * sqrtf(cnt > 0 ? s2 / (float)cnt : 0.f);
#pragma unroll
            for (int t = 0; t < IPT; ++t) sel[t] = ok[t] && av[t] > mu;
        }
    } else if (a_cls_out) {
#pragma unroll
        for (int t = 0; t < IPT; ++t)
            if (j0 + t < M && writes) a_cls_out[(size_t)b * M + j0 + t] = 0.f;
    }
    MD_DTICK(3);
#pragma unroll
    for (int t = 0; t < IPT; ++t)
        if (j0 + t < M) { s_key[j0 + t] = sel[t]; s_state[j0 + t] = 0; }
    __syncthreads();
    MD_DTICK(4);

    // ---- merge decision per window: S > tau, >= 2 valid members, no key member.  The window's thread
    // leaves each member's fate (and the merged mass at the first valid member) in LDS, so that the
    // per-token pass below needs no index arithmetic.
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        const int w = tid + 1024 * t;                // windows go round the threads: there are fewer than tokens
        if (w >= W) continue;
        const WinInfo wi = t == 0 ? win0 : analyse(w);
        bool has_key = false;
#pragma unroll
        for (int m = 0; m < WS; ++m)
            if ((wi.vmask >> m) & 1u) has_key |= s_key[wi.base + p.moff[m]] != 0;
        const bool mg = __popc(wi.vmask) >= 2 && !has_key && simv[t] > tau;
        if (mg) {
            int first = -1;
            float total = 0.f, mm[WS];
#pragma unroll
            for (int m = 0; m < WS; ++m) mm[m] = m < 4 ? wi.mm[m & 3] : 1.0f;
            if (WS > 4 && mb) {
#pragma unroll
                for (int m = 4; m < WS; ++m) mm[m] = mb[(wi.vmask >> m) & 1u ? wi.base + p.moff[m] : wi.base];
            }
#pragma unroll
            for (int m = 0; m < WS; ++m) {
                if (!((wi.vmask >> m) & 1u)) continue;
                const int tok = wi.base + p.moff[m];
                s_state[tok] = first < 0 ? 1 : 2;
                if (first < 0) first = tok;
                total += mm[m];
            }
            s_tmass[first] = total;
        }
        if (!EMIT) wmerged[(size_t)b * W + w] = mg;
        if (window_sim_out && writes) window_sim_out[(size_t)b * W + w] = simv[t];
    }
    __syncthreads();
    MD_DTICK(5);

    // ---- keys and survivors in ascending token index: one block scan of (keys << 16 | survivors) per thread
    bool surv[IPT], merged[IPT];
    int packed = 0;
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        surv[t] = false; merged[t] = false;
        if (ok[t]) {
            const int stt = s_state[j0 + t];
            merged[t] = stt != 0;
            surv[t] = stt != 2;
            if (stt == 1) mass[t] = s_tmass[j0 + t];
        }
        packed += (sel[t] ? 0x10000 : 0) + (surv[t] ? 1 : 0);
    }
    const int incl = wave_incl_scan_i(packed);
    if (lane == kWave - 1) s_red[wv] = incl;
    __syncthreads();
    MD_DTICK(6);
    int total;
    int excl = wave_prefix_of_totals(s_red, total) + incl - packed;
    int kpos = excl >> 16, spos = excl & 0xFFFF;
    const int nkeys = total >> 16, nsurv = total & 0xFFFF;
    if constexpr (EMIT) {
        int* s_row = reinterpret_cast<int*>(s_tmass);        // (every mass is in a register)
        int pos = spos;
#pragma unroll
        for (int t = 0; t < IPT; ++t) {
            if (j0 + t < M) s_row[j0 + t] = !ok[t] ? (int)kRowInvalid : !surv[t] ? (int)kRowGone : merged[t] ? pos | kRowMerged : pos;
            pos += surv[t] ? 1 : 0;
        }
        __syncthreads();
        MD_DTICK(7);
        emit_rows<WS, AHEAD>(p, em, b, g, s_row, mb, item, rowv);
        MD_DTICK(11);
    }
    if (!writes) return;
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        const int j = j0 + t;
        if (sel[t]) {
            if (kpos < key_budget) key_index[(size_t)b * key_budget + kpos] = j;
            ++kpos;
        }
        if (j < M && !EMIT) dstpos[(size_t)b * M + j] = surv[t] ? spos : -1;
        if (surv[t]) {
            const size_t o = (size_t)b * M + spos;
            out_index[o] = j;
            out_mass[o] = mass[t];
            out_is_key[o] = merged[t] ? 0 : (sel[t] ? 1 : 0);
            ++spos;
        }
    }
    if (with_keys) {
        for (int r = nkeys + tid; r < key_budget; r += blockDim.x) key_index[(size_t)b * key_budget + r] = -1;
        if (key_count && tid == 0) key_count[b] = nkeys;
    }
    if (tid == 0) out_count[b] = nsurv;
    if (out_valid)
        for (int s2 = tid; s2 < M; s2 += blockDim.x) out_valid[(size_t)b * M + s2] = s2 < nsurv;
#ifdef MD_DECIDE_TICKS
    if (threadIdx.x == 0 && blockIdx.x == 0)
        printf("issue %d gm %d f %d bar %d | acls %d select %d keyflags %d windows %d scan %d rows %d emit %d total %d\n",
               (int)(ticks[8] - ticks[0]), (int)(ticks[9] - ticks[8]), (int)(ticks[10] - ticks[9]), (int)(ticks[1] - ticks[10]),
               (int)(ticks[2] - ticks[1]), (int)(ticks[3] - ticks[2]), (int)(ticks[4] - ticks[3]), (int)(ticks[5] - ticks[4]),
               (int)(ticks[6] - ticks[5]), (int)(ticks[7] - ticks[6]), (int)(ticks[11] - ticks[7]), (int)(__builtin_readcyclecounter() - ticks[0]));
#endif
}

// ---------------------------------------------------------------------------------------------
// The decisions for samples of many tokens.  Bound by the latency of one CU's chain of steps.  In the kernel above that
// CU also fetches 64 bytes of numerators per token, at about 40 GB/s; here the scores a_cls come ready-made (4 bytes
// per token, see key_scores): 2 x 9216 tokens 14.3 us (the memory-resident kernel 95.9), 4 x 8064 12.1 (26.9).  A thread holds the scores of
// the tokens tid + 1024*t in registers for the selection; token flags (and the mass of a merged window at its first
// member) pass through LDS.  The final scan goes by waves: a wave owns a contiguous stretch of tokens and takes 64
// of them at a time, so that the outputs are written coalesced.
constexpr int kLargeTokens = 28672;                  // 5 bytes of LDS each: 140 of the CU's 160 KiB
enum : uint8_t { kTokValid = 1, kTokKey = 2, kTokFirst = 4, kTokGone = 8 };
template <int IPT, int WS>
__global__ __launch_bounds__(1024) void encode_decide_large_kernel(
    EncodeDims p, const uint8_t* __restrict__ valid, const float* __restrict__ mass_in,
    const float* __restrict__ acls, const float* __restrict__ sim, float tau,
    int key_budget, int key_adaptive, float key_lambda, int32_t* __restrict__ key_count,
    uint8_t* __restrict__ wmerged, int32_t* __restrict__ dstpos,
    int32_t* __restrict__ out_index, float* __restrict__ out_mass, uint8_t* __restrict__ out_is_key,
    uint8_t* __restrict__ out_valid, int32_t* __restrict__ out_count, int32_t* __restrict__ key_index,
    float* __restrict__ a_cls_out, float* __restrict__ window_sim_out)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t s_dyn[];
    __shared__ int s_hist[kSelectHistInts];
    __shared__ int s_red[16];
    __shared__ float s_redf[16];
    const int b = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const int M = p.M, W = p.W;
    float* s_tmass = reinterpret_cast<float*>(s_dyn);
    uint8_t* s_flag = s_dyn + 4 * (size_t)M;
    const uint8_t* vb = valid ? valid + (size_t)b * M : nullptr;
    const float* mb = mass_in ? mass_in + (size_t)b * M : nullptr;
    const bool with_keys = key_budget > 0 || key_adaptive;
    if (tid < 256) s_hist[tid] = 0;                  // for block_select_keys, after later barriers
    // the first rounds of windows: where they lie and their similarities, on the way while the keys are selected
    constexpr int PRE = 2;
    WindowAt wat[PRE];
    float wsim[PRE];
#pragma unroll
    for (int r = 0; r < PRE; ++r) {
        const int w = min(tid + 1024 * r, W - 1);
        wsim[r] = sim[(size_t)b * W + w];
        wat[r] = window_at(p, w);
    }
    uint32_t okmask = 0, keymask = 0;                // bit t: the token tid + 1024*t
    {
        float av[IPT];
        uint32_t vv[IPT];
#pragma unroll
        for (int t = 0; t < IPT; ++t) av[t] = with_keys ? acls[(size_t)b * M + min(tid + 1024 * t, M - 1)] : 0.f;
#pragma unroll
        for (int t = 0; t < IPT; ++t) vv[t] = vb ? vb[min(tid + 1024 * t, M - 1)] : 1u;
#pragma unroll
        for (int t = 0; t < IPT; ++t) okmask |= (tid + 1024 * t < M && vv[t] != 0 ? 1u : 0u) << t;
        if (with_keys) {
            __syncthreads();                         // s_hist is clear
            if (!key_adaptive) {                     // Eq. 7, budget form
                const SelectBound sb = block_select_keys([&](auto f) {
#pragma unroll
                    for (int t = 0; t < IPT; ++t) f((okmask >> t) & 1u ? rank_key(av[t], tid + 1024 * t) : 0ull);
                }, key_budget, s_hist);
#pragma unroll
                for (int t = 0; t < IPT; ++t)
                    keymask |= ((rank_key(av[t], tid + 1024 * t) >> sb.shift) >= sb.bound ? 1u : 0u) << t;
            } else {                                 // Eq. 7 as printed: a_cls > mu, mu = mean + lambda * std
                float s1 = 0.f;
#pragma unroll
                for (int t = 0; t < IPT; ++t)
                    if ((okmask >> t) & 1u) s1 += av[t];
                s1 = block_sum(s1, s_redf);
                const int cnt = block_sum_i(__popc(okmask), s_red);
                const float mean = cnt > 0 ? s1 / (float)cnt : 0.f;
                float s2 = 0.f;
#pragma unroll
                for (int t = 0; t < IPT; ++t)
                    if ((okmask >> t) & 1u) { const float dlt = av[t] - mean; s2 = fmaf(dlt, dlt, s2); }
                s2 = block_sum(s2, s_redf);
                const float mu = mean + key_lambda * sqrtf(cnt > 0 ? s2 / (float)cnt : 0.f);
#pragma unroll
                for (int t = 0; t < IPT; ++t) keymask |= (av[t] > mu ? 1u : 0u) << t;
            }
            keymask &= okmask;
        }
    }
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        const int j = tid + 1024 * t;
        if (j >= M) continue;
        s_flag[j] = ((okmask >> t) & 1u ? kTokValid : 0) | ((keymask >> t) & 1u ? kTokKey : 0);
        if (!with_keys && a_cls_out) a_cls_out[(size_t)b * M + j] = 0.f;
    }
    __syncthreads();

    // ---- merge decision per window: S > tau, >= 2 valid members, no key member
    auto decide = [&](int w, const WindowAt& at, float S) {
        uint8_t fl[WS];
#pragma unroll
        for (int m = 0; m < WS; ++m)                 // every flag in flight; members that do not exist read as absent
            fl[m] = s_flag[m < p.ws && member_exists(p, at, m) ? at.base + p.moff[m] : at.base];
        int n = 0, first = -1;
        bool has_key = false;
        float total = 0.f;
#pragma unroll
        for (int m = 0; m < WS; ++m) {
            if (m >= p.ws || !member_exists(p, at, m)) fl[m] = 0;
            if (!fl[m]) continue;
            const int tok = at.base + p.moff[m];
            ++n;
            has_key |= (fl[m] & kTokKey) != 0;
            if (first < 0) first = tok;
            total += mb ? mb[tok] : 1.0f;
        }
        const bool mg = n >= 2 && !has_key && S > tau;
        if (mg) {
#pragma unroll
            for (int m = 0; m < WS; ++m) {
                const int tok = at.base + p.moff[m];
                if (fl[m]) s_flag[tok] = kTokValid | (tok == first ? kTokFirst : kTokGone);
            }
            s_tmass[first] = total;
        }
        wmerged[(size_t)b * W + w] = mg;
        if (window_sim_out) window_sim_out[(size_t)b * W + w] = S;
    };
#pragma unroll
    for (int r = 0; r < PRE; ++r)
        if (tid + 1024 * r < W) decide(tid + 1024 * r, wat[r], wsim[r]);
    for (int w = tid + 1024 * PRE; w < W; w += 1024) decide(w, window_at(p, w), sim[(size_t)b * W + w]);
    __syncthreads();

    // ---- keys and survivors in ascending token index (a stretch is at most 64 * IPT tokens)
    const int stretch = ((M + 1023) / 1024) * kWave;
    const int t0 = wv * stretch, t1 = min(t0 + stretch, M);
    uint8_t fl[IPT];
    int packed = 0;                                  // keys in the high half, survivors in the low half
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        const int j = t0 + t * kWave + lane;
        fl[t] = s_flag[min(j, M - 1)];
        if (j >= t1) fl[t] = 0;
        packed += ((fl[t] & kTokKey) ? 0x10000 : 0) + ((fl[t] && !(fl[t] & kTokGone)) ? 1 : 0);
    }
    packed = wave_sum_i(packed);
    if (lane == 0) s_red[wv] = packed;
    __syncthreads();
    int total;
    const int before = wave_prefix_of_totals(s_red, total);
    int kpos = before >> 16, spos = before & 0xFFFF;
    const int nkeys = total >> 16, nsurv = total & 0xFFFF;
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int t = 0; t < IPT; ++t) {
        const int j = t0 + t * kWave + lane;
        const bool key = (fl[t] & kTokKey) != 0, surv = fl[t] && !(fl[t] & kTokGone);
        const uint64_t kmask = __ballot(key), smask = __ballot(surv);
        if (key) {
            const int r = kpos + __popcll(kmask & below);
            if (r < key_budget) key_index[(size_t)b * key_budget + r] = j;
        }
        const int so = spos + __popcll(smask & below);
        if (j < t1) dstpos[(size_t)b * M + j] = surv ? so : -1;
        if (surv) {
            const size_t o = (size_t)b * M + so;
            out_index[o] = j;
            out_mass[o] = (fl[t] & kTokFirst) ? s_tmass[j] : (mb ? mb[j] : 1.0f);
            s_flag[so] = key ? 1 : 0;                // every flag is in a register: its place holds the output's byte
        }
        kpos += __popcll(kmask);
        spos += __popcll(smask);
    }
    if (with_keys) {
        for (int r = nkeys + tid; r < key_budget; r += 1024) key_index[(size_t)b * key_budget + r] = -1;
        if (key_count && tid == 0) key_count[b] = nkeys;
    }
    if (tid == 0) out_count[b] = nsurv;
    __syncthreads();
    // the byte outputs, four at a time where the rows of the batch allow it
    uint8_t* kb = out_is_key + (size_t)b * M;
    uint8_t* vo = out_valid ? out_valid + (size_t)b * M : nullptr;
    const bool words = (M & 3) == 0 && ((reinterpret_cast<uintptr_t>(kb) | reinterpret_cast<uintptr_t>(vo)) & 3) == 0;
    const int n4 = words ? M / 4 : 0;
    for (int q = tid; q < n4; q += 1024) {
        const int s4 = 4 * q;
        if (s4 + 4 <= nsurv) *reinterpret_cast<uint32_t*>(kb + s4) = *reinterpret_cast<const uint32_t*>(s_flag + s4);
        else
            for (int s2 = s4; s2 < nsurv; ++s2) kb[s2] = s_flag[s2];
        const int live = min(max(nsurv - s4, 0), 4);
        if (vo) *reinterpret_cast<uint32_t*>(vo + s4) = live == 4 ? 0x01010101u : 0x01010101u & ((1u << (8 * live)) - 1u);
    }
    for (int s2 = 4 * n4 + tid; s2 < M; s2 += 1024) {
        if (s2 < nsurv) kb[s2] = s_flag[s2];
        if (vo) vo[s2] = s2 < nsurv;
    }
}

// ---------------------------------------------------------------------------------------------
// Writes the surviving rows.  One wave per window.
template <bool BF>
__global__ __launch_bounds__(256) void encode_emit_kernel(
    const void* __restrict__ x, const uint8_t* __restrict__ valid, const float* __restrict__ mass_in,
    EncodeDims p, const uint8_t* __restrict__ wmerged, const int32_t* __restrict__ dstpos,
    void* __restrict__ out_x)
{
    constexpr int VEC = Vec<BF>::N;
    const int lane = lane_id();
    const int item = blockIdx.x * kEncWaves + wave_id();
    if (item >= p.B * p.W) return;
    const int b = p.by_W.div(item), w = item - b * p.W;
    const size_t esz = BF ? 2 : 4;
    const size_t rowb = (size_t)p.D * esz;
    const char* xb = static_cast<const char*>(x) + (size_t)b * p.M * rowb;
    char* ob = static_cast<char*>(out_x) + (size_t)b * p.M * rowb;
    const uint8_t* vb = valid ? valid + (size_t)b * p.M : nullptr;
    const float* mb = mass_in ? mass_in + (size_t)b * p.M : nullptr;
    const int32_t* dst_b = dstpos + (size_t)b * p.M;

    // lane m < ws: token, validity, destination row and mass of member m, all requested at once
    const int is_merged = wmerged[(size_t)b * p.W + w];
    const int tok_l = lane_member_token(p, w, lane);
    const int ok_l = lane < p.ws && tok_l >= 0 && (!vb || vb[max(tok_l, 0)]);
    const int pos_l = ok_l ? dst_b[tok_l] : -1;
    const float mass_l = ok_l ? (mb ? mb[tok_l] : 1.0f) : 0.f;
    const int nchunk = (int)(rowb / 16);

    if (!is_merged) {
        // plain copies, up to four rows in flight
        for (int m0 = 0; m0 < p.ws; m0 += 4) {
            const u32x4* src[4];
            u32x4* dst[4];
            bool okm[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int m = min(m0 + u, p.ws - 1);
                okm[u] = m0 + u < p.ws && wave_member(ok_l, m) != 0;
                src[u] = reinterpret_cast<const u32x4*>(xb + (size_t)max(wave_member(tok_l, m), 0) * rowb);
                dst[u] = reinterpret_cast<u32x4*>(ob + (size_t)max(wave_member(pos_l, m), 0) * rowb);
            }
            for (int c = lane; c < nchunk; c += kWave) {
                u32x4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(src[u] + c);   // unguarded: all in flight
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (okm[u]) __builtin_nontemporal_store(v[u], dst[u] + c);
            }
        }
        return;
    }
    // mass-weighted mean of the valid members (members in ascending order), written at the first one
    const uint64_t okmask = __ballot(ok_l != 0);
    if (okmask == 0ull) return;                      // cannot happen: a merged window has >= 2 valid members
    const int first_m = __builtin_ctzll(okmask);
    float msum = 0.f;
    for (int m = 0; m < p.ws; ++m)
        if ((okmask >> m) & 1ull) msum += __builtin_bit_cast(float, wave_member(__builtin_bit_cast(int, mass_l), m));
    char* orow = ob + (size_t)wave_member(pos_l, first_m) * rowb;
    for (int c = lane * VEC; c < p.D; c += kWave * VEC) {
        float acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
        for (int m0 = 0; m0 < p.ws; m0 += 4) {
            float v[4][VEC], mm[4];
            bool okm[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int m = min(m0 + u, p.ws - 1);
                okm[u] = m0 + u < p.ws && ((okmask >> m) & 1ull);
                mm[u] = __builtin_bit_cast(float, wave_member(__builtin_bit_cast(int, mass_l), m));
                Vec<BF>::load_once(xb + (size_t)max(wave_member(tok_l, m), 0) * rowb, c, v[u]);   // unguarded, see above
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (!okm[u]) continue;
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[e] = fmaf(mm[u], v[u][e], acc[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = acc[e] / msum;
        Vec<BF>::store(orow, c, acc);
    }
}

struct EncodeWorkspace {
    float* logits; float2* cls_part; float* acls; float* sim; uint8_t* iskey; uint8_t* wmerged;
    int32_t* dstpos;
    size_t bytes;
};

EncodeWorkspace carve_encode(void* base, int B, int M, int W, int Hc) {
    Carver c(base);
    EncodeWorkspace ws;
    ws.logits = c.take<float>((size_t)B * (Hc > 0 ? Hc : 1) * (M + 1));
    ws.cls_part = c.take<float2>((size_t)B * (Hc > 0 ? Hc : 1) * cls_groups(M));
    ws.acls = c.take<float>((size_t)B * M);
    ws.sim = c.take<float>((size_t)B * W);
    ws.iskey = c.take<uint8_t>((size_t)B * M);
    ws.wmerged = c.take<uint8_t>((size_t)B * W);
    ws.dstpos = c.take<int32_t>((size_t)B * M);
    ws.bytes = c.off;
    return ws;
}

// Dynamic LDS of the fast decision kernel: [M] floats, then the larger of ([M] + [M] flag bytes) and the
// [groups][16] factors (16-byte aligned).
size_t decide_fast_lds_bytes(int M) {
    const size_t head = (4 * (size_t)M + 15) & ~(size_t)15;
    const size_t factors = (size_t)cls_groups(M) * 16 * 4, flags = 2 * (size_t)M + 16;
    return head + (factors > flags ? factors : flags);
}
struct ScoreArgs {
    const void* x; const void* q_cls; const void* k_cls; const uint8_t* valid; float* sim; float* logits; float2* cls_part;
    float2* block_stat; float* acls; float* a_cls_out;
};
template <int WSM>
void launch_scores(ScoreBlocks nb, hipStream_t st, bool xbf, bool qkbf, const EncodeDims& p, const ScoreArgs& a) {
    const unsigned grid = (unsigned)(nb.keyscore + nb.windows + nb.rows);
#define MD_ENC_SCORES(X_, K_)                                                                                  \
    MD_LAUNCH("encode_scores", st, (encode_scores_kernel<WSM, X_, K_>), grid, 64 * kEncWaves, 0, a.x, a.q_cls, a.k_cls, a.valid, p, nb, \
        a.sim, a.logits, a.cls_part, a.block_stat, a.acls, a.a_cls_out)
    if (xbf && qkbf) MD_ENC_SCORES(true, true);
    else if (xbf) MD_ENC_SCORES(true, false);
    else if (qkbf) MD_ENC_SCORES(false, true);
    else MD_ENC_SCORES(false, false);
#undef MD_ENC_SCORES
}
void launch_scores(int ws, ScoreBlocks nb, hipStream_t st, bool xbf, bool qkbf, const EncodeDims& p, const ScoreArgs& a) {
    if (ws <= 2) launch_scores<2>(nb, st, xbf, qkbf, p, a);
    else if (ws <= 4) launch_scores<4>(nb, st, xbf, qkbf, p, a);
    else if (ws <= 8) launch_scores<8>(nb, st, xbf, qkbf, p, a);
    else if (ws == 9) launch_scores<9>(nb, st, xbf, qkbf, p, a);     // 3 x 3: a third of the pairs of 16 members
    else launch_scores<16>(nb, st, xbf, qkbf, p, a);
}

}  // namespace
}  // namespace md

using namespace md;

extern "C" size_t mustdrop_encode_merge_workspace_bytes(int B, int T, int Hg, int Wg, int Hc, int kt, int kh, int kw) {
    if (B <= 0 || T <= 0 || Hg <= 0 || Wg <= 0 || kt <= 0 || kh <= 0 || kw <= 0) return 0;
    const long M = (long)T * Hg * Wg;
    const long W = (long)((T + kt - 1) / kt) * ((Hg + kh - 1) / kh) * ((Wg + kw - 1) / kw);
    return carve_encode(nullptr, B, (int)M, (int)W, Hc).bytes;
}

namespace md {
namespace {
// Both forms of the key set (Eq. 7): key_adaptive == 0: the key_budget largest scores; key_adaptive == 1:
// a_cls > mean + key_lambda * std, key_budget = capacity of key_index, key_count = size of the set.
int encode_merge_impl(
    const void* x, md_dtype x_dtype,
    const void* q_cls, const void* k_cls, md_dtype qk_dtype,
    const float* mass_in, const uint8_t* valid,
    int B, int T, int Hg, int Wg, int D, int Hc, int dc,
    int kt, int kh, int kw, float tau, int key_adaptive, int key_budget, float key_lambda,
    void* out_x, int32_t* out_index, float* out_mass, uint8_t* out_is_key, uint8_t* out_valid,
    int32_t* out_count, int32_t* key_index, int32_t* key_count,
    float* a_cls_out, float* window_sim_out,
    void* workspace, size_t workspace_bytes, void* stream)
{
    clear_error();
    if (x_dtype != MD_F32 && x_dtype != MD_BF16) return fail(MD_EDTYPE, "encode_merge: unknown x_dtype %d", (int)x_dtype);
    if (B <= 0 || T <= 0 || Hg <= 0 || Wg <= 0 || D <= 0)
        return fail(MD_EINVAL, "encode_merge: B, T, Hg, Wg, D must be positive (got %d %d %d %d %d)", B, T, Hg, Wg, D);
    if (kt <= 0 || kh <= 0 || kw <= 0) return fail(MD_EINVAL, "encode_merge: window sizes must be positive");
    const long ws_l = (long)kt * kh * kw;
    if (ws_l > kMaxWindow) return fail(MD_ESHAPE, "encode_merge: window of %ld tokens exceeds the limit of %d", ws_l, kMaxWindow);
    const long M_l = (long)T * Hg * Wg;
    if (M_l > (1l << 24) || (long)B * M_l > (1l << 30)) return fail(MD_ESHAPE, "encode_merge: too many tokens");
    const int nwt = (T + kt - 1) / kt, nwy = (Hg + kh - 1) / kh, nwx = (Wg + kw - 1) / kw;   // border windows are clipped
    const int M = (int)M_l, ws = (int)ws_l, W = nwt * nwy * nwx;
    if (key_budget < 0 || (!key_adaptive && key_budget > M))
        return fail(MD_EINVAL, "encode_merge: key_budget %d outside [0, %d]", key_budget, M);
    if (key_adaptive && (std::isnan(key_lambda) || !key_count))
        return fail(MD_EINVAL, "encode_merge: the adaptive key rule needs a key_lambda that is a number and key_count");
    const bool with_keys = key_adaptive || key_budget > 0;
    if (!x || !out_x || !out_index || !out_mass || !out_is_key || !out_count)
        return fail(MD_EINVAL, "encode_merge: x and the out_* arrays are required");
    if (std::isnan(tau)) return fail(MD_EINVAL, "encode_merge: tau is NaN");
    const size_t xe = elt_size(x_dtype);
    if ((D * xe) % 16) return fail(MD_EALIGN, "encode_merge: a row of D=%d elements is not a multiple of 16 bytes", D);
    if (!aligned16(x) || !aligned16(out_x)) return fail(MD_EALIGN, "encode_merge: x / out_x must be 16-byte aligned");
    if (with_keys) {
        if (qk_dtype != MD_F32 && qk_dtype != MD_BF16) return fail(MD_EDTYPE, "encode_merge: unknown qk_dtype %d", (int)qk_dtype);
        if (!q_cls || !k_cls || (key_budget > 0 && !key_index))
            return fail(MD_EINVAL, "encode_merge: q_cls, k_cls (and key_index, if it has room) are required when keys are selected");
        if (Hc <= 0 || dc <= 0) return fail(MD_EINVAL, "encode_merge: Hc and dc must be positive");
        if (Hc > kMaxClsHeads) return fail(MD_ESHAPE, "encode_merge: Hc=%d exceeds the limit of %d", Hc, kMaxClsHeads);
        if ((long)Hc * dc != D) return fail(MD_ESHAPE, "encode_merge: Hc*dc = %ld differs from D = %d", (long)Hc * dc, D);
        const int vec = qk_dtype == MD_BF16 ? 8 : 4;
        if ((dc & (dc - 1)) || dc < vec) return fail(MD_ESHAPE, "encode_merge: dc=%d must be a power of two >= %d", dc, vec);
        if (!aligned16(q_cls) || !aligned16(k_cls)) return fail(MD_EALIGN, "encode_merge: q_cls / k_cls must be 16-byte aligned");
    } else if (q_cls || k_cls) {
        return fail(MD_EINVAL, "encode_merge: q_cls / k_cls given but key_budget == 0");
    }
    const size_t xbytes = (size_t)B * M * D * xe;
    if (overlaps(x, xbytes, out_x, xbytes)) return fail(MD_EALIAS, "encode_merge: out_x overlaps x");
    const EncodeWorkspace wsp = carve_encode(workspace, B, M, W, with_keys ? Hc : 0);
    if (!workspace || workspace_bytes < wsp.bytes)
        return fail(MD_EWORKSPACE, "encode_merge: workspace of %zu bytes needed, %zu given", wsp.bytes, workspace ? workspace_bytes : (size_t)0);
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(MD_EALIGN, "encode_merge: workspace must be 256-byte aligned");

    EncodeDims p;
    p.B = B; p.T = T; p.Hg = Hg; p.Wg = Wg; p.D = D; p.Hc = with_keys ? Hc : 0; p.dc = dc;
    p.kt = kt; p.kh = kh; p.kw = kw; p.M = M; p.W = W; p.ws = ws;
    p.nwx = nwx; p.nwy = nwy; p.nwt = nwt;
    p.clipped = (T % kt || Hg % kh || Wg % kw) ? 1 : 0;
    p.by_W = FastDiv::make(W); p.by_nwx = FastDiv::make(nwx); p.by_nwy = FastDiv::make(nwy);
    p.by_kw = FastDiv::make(kw); p.by_kh = FastDiv::make(kh);
    for (int m = 0; m < kMaxWindow; ++m) {
        const int mm = m < ws ? m : 0, dx = mm % kw, dy = mm / kw % kh, dt = mm / (kw * kh);
        p.moff[m] = (dt * Hg + dy) * Wg + dx;
        p.mpos[m] = dt << 16 | dy << 8 | dx;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);

    const int win_blocks = (int)(((long)B * W + kEncWaves - 1) / kEncWaves);
    const int row_blocks = with_keys ? B * cls_blocks(M) : 0;
    // Up to 5120 tokens the decision kernel fetches the numerators itself; beyond that the scores are made beforehand
    // (two score launches, about 5 us more, against a decision 8 to 15 us shorter).  Measured, us per call, numerators /
    // ready-made: 4 x 4608 tokens 41.1 / 41.7, 4 x 5760 48.5 / 45.8, 4 x 6144 51.3 / 47.9, 16 x 5760 135.5 / 131.5,
    // 4 x 8064 66.8 / 56.5.  (The LDS of the former stays below 64 KiB.)
    // With more heads than the former merges (16) the other choice is the general kernel behind the one score launch,
    // sliced: its decision grows with tokens times heads, the two launches cost 10 to 20 us more in the scores.  General /
    // ready-made: 1 x 351 tokens of 32 heads 22.4 / 32.0, 4 x 756 30.1 / 34.6, 16 x 756 53.3 / 53.9, 16 x 1024 66.8 / 65.1;
    // 1 x 756 of 64 heads 34.6 / 41.4, 4 x 1024 51.7 / 48.3; 1 x 2048 of 20 heads 33.4 / 29.9.
    const size_t dlds = decide_fast_lds_bytes(M), llds = 5 * (size_t)M;
    const bool fast_ok = M <= 5120 && (!with_keys || (Hc <= 16 && Hc % 4 == 0));
    const bool few_ok = M <= 1024 && (long)M * Hc <= (B == 1 ? 49152 : 24576);
    const bool large_ok = !fast_ok && M <= kLargeTokens && (!with_keys || (Hc <= kMaxMergedHeads && Hc % 4 == 0 && !few_ok));
    const bool xbf = x_dtype == MD_BF16, qkbf = qk_dtype == MD_BF16;
    const ScoreArgs sa{x, q_cls, k_cls, valid, wsp.sim, wsp.logits, wsp.cls_part,
                       large_ok && with_keys ? wsp.cls_part + (size_t)B * Hc * cls_groups(M) / 2 : nullptr, wsp.acls, a_cls_out};
    if (large_ok && with_keys) {
        if (qkbf) launch_scores(ws, ScoreBlocks{0, 0, row_blocks, 1}, st, xbf, qkbf, p, sa);
        else
            MD_LAUNCH("encode_scores", st, (encode_rows_f32_kernel), (unsigned)row_blocks, 64 * kEncWaves, 0,
                q_cls, k_cls, valid, p, wsp.logits, wsp.cls_part, sa.block_stat);
        // (a multiple of 8 of them: blocks go round the 8 XCDs in turn, and a window's rows are then still in the L2 of the
        // XCD whose block of the emit kernel reads them again: 2 x 756 tokens, 3072 fp32 features, emit 34.3 -> 18.6 us)
        const int score_blocks = (B * ((M + kKeyTokens - 1) / kKeyTokens) + 7) & ~7;
        launch_scores(ws, ScoreBlocks{score_blocks, win_blocks, 0, 1}, st, xbf, qkbf, p, sa);
    } else {
        const int vec = qkbf ? 8 : 4, iters = (D / vec + kWave - 1) / kWave;
        // A wave per 64-vector slice of its key rows, where a head lies inside a slice: the slices were a chain of round
        // trips (scores of 1 x 576 tokens fp32 10.5 -> 5.2 us, 16 x 576 11.2 -> 10.4, 75 x 400 fp32 46.7 -> 41.0).  Not
        // for many tokens in windows of more than nine members, whose registers leave room for few waves.
        const bool sliced = with_keys && iters > 1 && dc / vec < kWave && (ws <= 9 || (long)B * M <= 8192);
        const int rb = sliced ? (int)(((long)B * cls_groups(M) * iters + kEncWaves - 1) / kEncWaves) : row_blocks;
        launch_scores(ws, ScoreBlocks{0, win_blocks, rb, sliced ? iters : 1}, st, xbf, qkbf, p, sa);
    }
    dim3 wgrid((unsigned)win_blocks);
    // Survivors' rows by the deciding blocks (see EmitArgs): as many blocks per sample as have the chip to themselves in one round
    // (more are a second round behind the decisions: 16 x 576 tokens 21.0 us a call with 256 blocks, 26.8 with 384), no more
    // than there are items for their waves.  Two per sample at least (128 x 576 tokens 101.5 us a call with a launch for
    // the rows, 98.3 without; 200 x 576 159.4 and 166.8).
    const int row_slices = (int)(((long)D * xe / 16 + kWave - 1) / kWave);
    const EmitArgs em{x, out_x, (int)min(((long)W * row_slices + 15) / 16, (long)max(kNumCU / B, 1)), row_slices, xbf ? 1 : 0,
                      FastDiv::make(B), FastDiv::make(row_slices)};
    // And only as long as x stays in the 256 MB Infinity Cache between the scores and the rows: few blocks that wait for their
    // decisions fetch from HBM more slowly than a launch over the whole chip (64 x 2048 tokens, 268 MB, 181 us a call with a launch for the
    // rows, 189 without; 112 x 576 fp32, 264 MB, 179 / 190; 42 x 2880, 247 MB, 171 / 177; 48 x 1152 fp32, 226 MB, 157 / 152; 24 x 576 of
    // 4096 fp32 features, 226 MB, 168 / 160).
    // Nor where two blocks per sample leave a fifth of the CUs idle and have neither little to write nor enough to make up for it
    // (86 x 196 tokens 30.6 / 30.9, 86 x 256 36.4 / 37.2, 95 x 196 32.4 / 32.9; 86 x 120 24.2 / 23.1, 86 x 400 51.3 / 50.7, 110 x 256 44.2 / 43.9).
    // (not where an output lies over an input of theirs: a block may still read what another one writes)
    const EncodeOutputs written{out_x, out_index, out_mass, out_is_key, out_valid, out_count, key_index, key_count, a_cls_out, window_sim_out};
    const bool idle = kNumCU / B == 2 && 5 * B < 2 * kNumCU && M > 128 && M <= 256;
    const bool emits = fast_ok && !idle && M <= 3072 && ws <= 8 && 2 * B <= kNumCU && row_slices <= 4096 && xbytes <= 230000000 &&
                       !outputs_over(written, B, M, W, D * xe, key_budget, mass_in, valid);
#define MD_DECIDE_FAST(IPT_, WS_, E_)                                                                             \
    MD_LAUNCH(E_ ? "encode_decide_emit" : "encode_decide", st, (encode_decide_fast_kernel<IPT_, WS_, E_>), E_ ? B * em.blocks : B, 1024, dlds,                  \
        p, valid, mass_in, wsp.logits, wsp.cls_part, wsp.sim, tau, key_budget, key_adaptive, key_lambda, key_count,  \
        wsp.wmerged, wsp.dstpos,                                                                                   \
        out_index, out_mass, out_is_key, out_valid, out_count, key_index, a_cls_out, window_sim_out, em)
#define MD_DECIDE_FAST_WS(IPT_)                                                                               \
    do { if (ws <= 4) MD_DECIDE_FAST(IPT_, 4, false); else if (ws <= 8) MD_DECIDE_FAST(IPT_, 8, false); else MD_DECIDE_FAST(IPT_, 16, false); } while (0)
#define MD_DECIDE_EMIT_WS(IPT_)                                                                               \
    do { if (ws <= 4) MD_DECIDE_FAST(IPT_, 4, true); else MD_DECIDE_FAST(IPT_, 8, true); } while (0)
    if (emits) {
        if (M <= 1024) MD_DECIDE_EMIT_WS(1);
        else if (M <= 2048) MD_DECIDE_EMIT_WS(2);
        else MD_DECIDE_EMIT_WS(3);                           // e.g. five tiles of 24 x 24 tokens
        return check_launch("encode_merge");
    }
    if (fast_ok && M <= 1024) MD_DECIDE_FAST_WS(1);
    else if (fast_ok && M <= 2048) MD_DECIDE_FAST_WS(2);
    else if (fast_ok && M <= 3072) MD_DECIDE_FAST_WS(3);
    else if (fast_ok && M <= 4096) MD_DECIDE_FAST_WS(4);
    else if (fast_ok) MD_DECIDE_FAST_WS(5);                  // e.g. eight frames of 24 x 24 tokens
    else if (large_ok) {
#define MD_DECIDE_LARGE(IPT_, WS_)                                                                             \
    do {                                                                                                       \
        if (llds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void*>(&encode_decide_large_kernel<IPT_, WS_>), \
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)llds) != hipSuccess) \
            return fail(MD_EHIP, "encode_merge: %zu bytes of LDS refused", llds);                              \
        MD_LAUNCH("encode_decide", st, (encode_decide_large_kernel<IPT_, WS_>), B, 1024, llds,                \
            p, valid, mass_in, wsp.acls, wsp.sim, tau, key_budget, key_adaptive, key_lambda, key_count, wsp.wmerged, wsp.dstpos, \
            out_index, out_mass, out_is_key, out_valid, out_count, key_index, a_cls_out, window_sim_out);      \
    } while (0)
#define MD_DECIDE_LARGE_WS(IPT_)                                                                              \
    do { if (ws <= 4) MD_DECIDE_LARGE(IPT_, 4); else if (ws <= 8) MD_DECIDE_LARGE(IPT_, 8); else MD_DECIDE_LARGE(IPT_, 16); } while (0)
        if (M <= 6144) MD_DECIDE_LARGE_WS(6);
        else if (M <= 8192) MD_DECIDE_LARGE_WS(8);
        else if (M <= 10240) MD_DECIDE_LARGE_WS(10);
        else if (M <= 12288) MD_DECIDE_LARGE_WS(12);
        else if (M <= 16384) MD_DECIDE_LARGE_WS(16);
        else MD_DECIDE_LARGE_WS(28);
#undef MD_DECIDE_LARGE_WS
#undef MD_DECIDE_LARGE
    } else
        MD_LAUNCH("encode_decide", st, (encode_decide_kernel), B, 1024, 0,
            p, valid, mass_in, wsp.logits, wsp.cls_part, wsp.sim, tau, key_budget, key_adaptive, key_lambda, key_count,
            wsp.acls, wsp.iskey, wsp.wmerged, wsp.dstpos,
            out_index, out_mass, out_is_key, out_valid, out_count, key_index, a_cls_out, window_sim_out);
#undef MD_DECIDE_EMIT_WS
#undef MD_DECIDE_FAST_WS
#undef MD_DECIDE_FAST
    if (x_dtype == MD_BF16) MD_LAUNCH("encode_emit", st, (encode_emit_kernel<true>), wgrid, 64 * kEncWaves, 0, x, valid, mass_in, p, wsp.wmerged, wsp.dstpos, out_x);
    else MD_LAUNCH("encode_emit", st, (encode_emit_kernel<false>), wgrid, 64 * kEncWaves, 0, x, valid, mass_in, p, wsp.wmerged, wsp.dstpos, out_x);
    return check_launch("encode_merge");
}
}  // namespace
}  // namespace md

extern "C" int mustdrop_encode_merge(
    const void* x, md_dtype x_dtype,
    const void* q_cls, const void* k_cls, md_dtype qk_dtype,
    const float* mass_in, const uint8_t* valid,
    int B, int T, int Hg, int Wg, int D, int Hc, int dc,
    int kt, int kh, int kw, float tau, int key_budget,
    void* out_x, int32_t* out_index, float* out_mass, uint8_t* out_is_key, uint8_t* out_valid,
    int32_t* out_count, int32_t* key_index,
    float* a_cls_out, float* window_sim_out,
    void* workspace, size_t workspace_bytes, void* stream)
{
    return encode_merge_impl(x, x_dtype, q_cls, k_cls, qk_dtype, mass_in, valid, B, T, Hg, Wg, D, Hc, dc, kt, kh, kw, tau,
                             0, key_budget, 0.f, out_x, out_index, out_mass, out_is_key, out_valid, out_count,
                             key_index, nullptr, a_cls_out, window_sim_out, workspace, workspace_bytes, stream);
}

// ---------------------------------------------------------------------------------------------
// The same stage for callers that cannot hand over (or allocate) a workspace: the scratch memory is a
// file-scope device array.  Every GPU the library runs on holds its own copy at its own address; the
// host-side name of the array is only a handle, the address a kernel can use comes from
// hipGetSymbolAddress (once per device, kept).
static __device__ __align__(256) unsigned char scratch[MUSTDROP_STATIC_SCRATCH_BYTES];

namespace md {
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {nullptr};

// Device address of `scratch` on the current device (resolved at the first call on that device).
int static_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(MD_EHIP, "encode_merge_noalloc: hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(MD_EHIP, "encode_merge_noalloc: device index %d not supported", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(MD_EHIP, "encode_merge_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return MD_OK;
}
}  // namespace
}  // namespace md

extern "C" int mustdrop_encode_merge_noalloc(
    const void* x, md_dtype x_dtype,
    const void* q_cls, const void* k_cls, md_dtype qk_dtype,
    const float* mass_in, const uint8_t* valid,
    int B, int T, int Hg, int Wg, int D, int Hc, int dc,
    int kt, int kh, int kw, float tau, int key_budget,
    void* out_x, int32_t* out_index, float* out_mass, uint8_t* out_is_key, uint8_t* out_valid,
    int32_t* out_count, int32_t* key_index,
    float* a_cls_out, float* window_sim_out, void* stream)
{
    clear_error();
    if (B <= 0 || T <= 0 || Hg <= 0 || Wg <= 0 || kt <= 0 || kh <= 0 || kw <= 0)
        return fail(MD_EINVAL, "encode_merge_noalloc: B, T, Hg, Wg and the window sizes must be positive");
    if ((long)T * Hg * Wg > (1l << 24) || (long)B * T * Hg * Wg > (1l << 30))
        return fail(MD_ESHAPE, "encode_merge_noalloc: too many tokens");
    const size_t need = mustdrop_encode_merge_workspace_bytes(B, T, Hg, Wg, key_budget > 0 ? Hc : 0, kt, kh, kw);
    if (need > (size_t)MUSTDROP_STATIC_SCRATCH_BYTES)
        return fail(MD_EWORKSPACE, "encode_merge_noalloc: this shape needs %zu bytes of scratch memory, the static buffer holds %zu; "
                    "use mustdrop_encode_merge with a workspace", need, (size_t)MUSTDROP_STATIC_SCRATCH_BYTES);
    void* ptr = nullptr;
    const int rc = static_scratch(&ptr);
    if (rc != MD_OK) return rc;
    return encode_merge_impl(x, x_dtype, q_cls, k_cls, qk_dtype, mass_in, valid, B, T, Hg, Wg, D, Hc, dc, kt, kh, kw, tau,
                             0, key_budget, 0.f, out_x, out_index, out_mass, out_is_key, out_valid, out_count,
                             key_index, nullptr, a_cls_out, window_sim_out, ptr, (size_t)MUSTDROP_STATIC_SCRATCH_BYTES, stream);
}

extern "C" int mustdrop_encode_merge_adaptive(
    const void* x, md_dtype x_dtype,
    const void* q_cls, const void* k_cls, md_dtype qk_dtype,
    const float* mass_in, const uint8_t* valid,
    int B, int T, int Hg, int Wg, int D, int Hc, int dc,
    int kt, int kh, int kw, float tau, float key_lambda, int key_cap,
    void* out_x, int32_t* out_index, float* out_mass, uint8_t* out_is_key, uint8_t* out_valid,
    int32_t* out_count, int32_t* key_index, int32_t* key_count,
    float* a_cls_out, float* window_sim_out,
    void* workspace, size_t workspace_bytes, void* stream)
{
    return encode_merge_impl(x, x_dtype, q_cls, k_cls, qk_dtype, mass_in, valid, B, T, Hg, Wg, D, Hc, dc, kt, kh, kw, tau,
                             1, key_cap, key_lambda, out_x, out_index, out_mass, out_is_key, out_valid, out_count,
                             key_index, key_count, a_cls_out, window_sim_out, workspace, workspace_bytes, stream);
}
