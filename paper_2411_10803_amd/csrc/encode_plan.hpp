// Where the encode decisions read, and which outputs may not lie there: the arithmetic of the host and of the kernel.  Without any
// HIP header, so that a CPU test can follow it.
#pragma once
#include "md_overlap.hpp"

#ifndef MD_PLAN_FN
#ifdef __HIPCC__
#define MD_PLAN_FN __host__ __device__ __forceinline__
#else
#define MD_PLAN_FN inline
#endif
#endif

namespace md {
namespace {

// The numerators of a sample's M tokens, [M][Hc] floats, as a buffer's range; and the byte in it of the q-th four heads of the
// token that thread `tid` takes in round t, the range itself (which reads as zero) where there are no such heads.  All of it goes
// into the vector offset of the load: the scalar one is not part of what is compared with the range, or wraps round where it is larger.
MD_PLAN_FN int numerator_bytes(int M, int Hc) { return M * Hc * 4; }
MD_PLAN_FN int numerator_vector(int tid, int t, int q, int M, int Hc) {
    return 4 * q < Hc ? (tid + 1024 * t) * Hc * 4 + 16 * q : numerator_bytes(M, Hc);
}

// Everything that a call writes besides its workspace, and whether any of it lies over the masses or the flags.  Several blocks
// per sample that decide and write rows read both while others already write; one block per sample has them in registers by then.
struct EncodeOutputs {
    const void *x, *index, *mass, *is_key, *valid, *count, *key_index, *key_count, *a_cls, *window_sim;
};
inline bool outputs_over(const EncodeOutputs& o, size_t B, size_t M, size_t W, size_t row_bytes, size_t key_index_len,
                         const void* mass_in, const void* valid) {
    const struct { const void* p; size_t n; } out[] = {
        {o.x, B * M * row_bytes}, {o.index, 4 * B * M}, {o.mass, 4 * B * M}, {o.is_key, B * M}, {o.valid, B * M}, {o.count, 4 * B},
        {o.key_index, 4 * B * key_index_len}, {o.key_count, 4 * B}, {o.a_cls, 4 * B * M}, {o.window_sim, 4 * B * W}};
    for (const auto& a : out)
        if (overlaps(a.p, a.n, mass_in, 4 * B * M) || overlaps(a.p, a.n, valid, B * M)) return true;
    return false;
}

}  // namespace
}  // namespace md
