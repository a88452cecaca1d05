// Do two ranges of bytes share one?  Without any HIP header, for the CPU tests.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace md {

inline bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
    if (!a || !b || na == 0 || nb == 0) return false;
    const uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa < pb + nb && pb < pa + na;
}

}  // namespace md
