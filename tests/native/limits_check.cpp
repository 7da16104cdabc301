// Size decisions of the one-workgroup kernels at the largest tables a call may
// have: 100000 rows of 65536 entries, products past 2^31 and 2^32 among them.
#include <cstdio>

#include "../../paper_2401_02852_amd/csrc/internal.h"

#define CHECK(cond)                                                  \
    do {                                                             \
        if (!(cond)) {                                               \
            std::printf("line %d: %s\n", __LINE__, #cond);           \
            return 1;                                                \
        }                                                            \
    } while (0)

int main() {
    constexpr int32_t room = 2048;
    const int32_t lens[] = {1, 2, 255, 256, 2047, 2048, 2049, 32768, 65535, 65536};
    const int32_t rows[] = {0, 1, 2, 8, 31, 32768, 32769, 65535, 65536, 65537, 98304, 100000};
    for (int32_t r : rows)
        for (int32_t l : lens) CHECK(qnae::rows_fit(r, l, room) == ((double)r * l <= room));
    CHECK(!qnae::rows_fit(32768, 65536, room));  // 2^31: negative in 32 bits
    CHECK(!qnae::rows_fit(65536, 65536, room));  // 2^32: zero in 32 bits
    CHECK(qnae::rows_fit(8, 256, room) && !qnae::rows_fit(8, 257, room));
    std::printf("limits ok\n");
    return 0;
}
