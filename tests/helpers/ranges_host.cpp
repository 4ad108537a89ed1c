// range_within and rows_extent of the library, on the host: reads lines "w base size p bytes" and
// "e rows stride row", prints a number for each.
#include <cstdio>

#include "ranges.h"

int main() {
    char kind;
    while (std::scanf(" %c", &kind) == 1) {
        unsigned long long a, b, c, d;
        if (kind == 'w') {
            if (std::scanf("%llu %llu %llu %llu", &a, &b, &c, &d) != 4) return 1;
            std::printf("%d\n", fgs::range_within((uintptr_t)a, (size_t)b, (uintptr_t)c, (size_t)d) ? 1 : 0);
        } else {
            if (std::scanf("%llu %llu %llu", &a, &b, &c) != 3) return 1;
            std::printf("%zu\n", fgs::rows_extent((int64_t)a, (int64_t)b, (size_t)c));
        }
    }
    return 0;
}
