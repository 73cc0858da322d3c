// CPU check of the 32-bit byte offsets into D (devtypes.h), under UndefinedBehaviorSanitizer.
#include <cstdio>

#include "devtypes.h"

using namespace nao;

static_assert(8 * D_OFFSET_MAX_BASIS * D_OFFSET_MAX_BASIS <= int64_t(1) << 32, "every offset fits 32 bits");
static_assert(8 * (D_OFFSET_MAX_BASIS + 1) * (D_OFFSET_MAX_BASIS + 1) > int64_t(1) << 32, "and no limit above it would do");
static_assert(d_offset(23169, 23170, 23169) == 8u * (23169u * 23170u + 23169u), "a constant expression: no signed overflow");

int main()
{
    for (int64_t n : {int64_t(1), int64_t(45), int64_t(16383), int64_t(16384), int64_t(16385), int64_t(20000), D_OFFSET_MAX_BASIS - 1, D_OFFSET_MAX_BASIS})
        for (int64_t i = 0; i < n; i += n / 1000 + 1)
            for (int64_t j : {int64_t(0), n / 2, n - 1})
                for (int64_t r : {i, n - 1 - i})
                    if ((int64_t)d_offset((int)r, n, (int)j) != 8 * (r * n + j)) return std::printf("row %ld of %ld\n", (long)r, (long)n), 1;
    std::printf("offsets: all ok\n");
    return 0;
}
