// Where the encode decisions read: the arithmetic of the kernel.  Without any HIP header, so that a CPU test can follow it.
#pragma once

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

}  // namespace
}  // namespace md
