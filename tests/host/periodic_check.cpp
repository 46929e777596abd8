// Host check of kbc::periodic_minus (the neighbours of the gradient stencils)
// against 64-bit arithmetic: axes from one node to the largest a box may
// have, every reach up to 4, coordinates at both ends and a tile past the end.
#include <cstdint>
#include <cstdio>

#include "kbc_device.h"

int main()
{
    const uint32_t axes[] = {1, 2, 3, 4, 5, 7, 33, 4096, 536870912u, 858993459u, 858993460u, 900000000u,
                             1073741823u, 1073741824u, 1500000000u, 2147483607u, 2147483647u};
    long bad = 0;
    for (uint32_t n : axes)
        for (uint32_t m = 0; m <= 4; ++m)
            for (int64_t k = -80; k <= 80; ++k)
                for (int64_t base : {(int64_t)0, (int64_t)n / 2, (int64_t)n}) {
                    const int64_t a = base + k;
                    if (a < 0) continue;
                    const int64_t want = ((a - (int64_t)m) % (int64_t)n + (int64_t)n) % (int64_t)n;
                    if (kbc::periodic_minus((uint32_t)a, m, n) != want) ++bad;
                }
    if (bad) std::printf("%ld wrong\n", bad);
    return bad ? 1 : 0;
}
