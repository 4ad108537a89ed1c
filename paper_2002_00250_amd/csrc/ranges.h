// Address arithmetic of the checks that stand before a kernel's writes to a caller's memory (host
// code without HIP, so that it can be tested by itself).
#pragma once

#include <cstddef>
#include <cstdint>

namespace fgs {

// Whether [p, p + bytes) lies in the `size` bytes from `base` on.
inline bool range_within(uintptr_t base, size_t size, uintptr_t p, size_t bytes) {
    return p >= base && p - base <= size && bytes <= size - (p - base);
}

// The bytes from the first of `rows` >= 1 rows of `row` bytes, `stride` >= row apart, to their end;
// SIZE_MAX, which no allocation has, where that is more than a size_t holds.
inline size_t rows_extent(int64_t rows, int64_t stride, size_t row) {
    size_t bytes = 0;
    if (__builtin_mul_overflow((size_t)(rows - 1), (size_t)stride, &bytes) || __builtin_add_overflow(bytes, row, &bytes))
        return SIZE_MAX;
    return bytes;
}

}  // namespace fgs
