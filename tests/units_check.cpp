// Checks csrc/nlb_units.h on the CPU: for every width, every unit is read
// inside the row, every column of the row is used exactly once, and the
// weights, after unit_shift, meet their own columns (a product over the units
// equals the plain dot product of integers).  Prints "ok <checks>".
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "nlb_units.h"

static unsigned long long checks = 0;

template <uint32_t U>
static bool width(uint32_t dim) {
    const uint32_t padded = (dim + 31) / 32 * 32;
    std::vector<long> row(dim), w(padded + U, 0), staged;
    for (uint32_t c = 0; c < dim; c++) {
        row[c] = rand() % 1000 + 1;
        w[c] = rand() % 1000 + 1;
    }
    for (uint32_t c = dim; c < padded; c++) w[c] = 77777;   // never to be used
    staged = w;
    if (unit_cut(dim, U)) unit_shift<U>(staged.data(), dim);
    std::vector<int> used(dim, 0);
    long got = 0, want = 0;
    for (uint32_t c = 0; c < dim; c++) want += row[c] * w[c];
    for (uint32_t c = 0; c < padded; c += U) {
        const uint32_t from = unit_start(c, dim, U);
        if (from + U > dim) return false;
        checks++;
        if (c >= dim) continue;
        const uint32_t shared = unit_shared(c, dim, U);
        for (uint32_t i = 0; i < U; i++) {
            if (i < shared) {
                if (staged[c + i] != 0) return false;   // an unused value has no weight either
                continue;
            }
            used[from + i]++;
            got += row[from + i] * staged[c + i];
            checks++;
        }
    }
    for (int u : used)
        if (u != 1) return false;
    return got == want;
}

int main() {
    for (uint32_t dim = 4; dim <= 512; dim++) {
        if (!width<4>(dim)) return printf("unit 4, width %u\n", dim), 1;
        if (dim >= 8 && !width<8>(dim)) return printf("unit 8, width %u\n", dim), 1;
    }
    printf("ok %llu\n", checks);
    return 0;
}
