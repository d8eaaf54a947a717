// Checks the launch shape of the fp32 kernel (f32_grid in fdd_internal.h): enough workgroups, no dimension of 2^32 work items
// or more, which a launch would refuse, and whole rounds of the 8 XCDs in every row of the grid.  Host code only; built and
// run by tests/test_f32_limits.py.
#include <cstdio>

#include "fdd_internal.h"

int main()
{
    using namespace fdd;
    // workgroups: one, around a round of XCDs, ordinary, around 2^23 (2^32 work items of one dimension), the most a call
    // has (2^28: 2^33 query rows in tiles of 32)
    const long long works[] = {1, 7, 8, 9, 224, 1024, 100003, (1 << 22) - 1, 1 << 22, (1 << 22) + 1, (1 << 23) - 1, 1 << 23, (1 << 23) + 8,
                               19000003, (1 << 28) - 1, 1 << 28};
    long bad = 0;
    for (long long w : works) {
        const dim3 g = f32_grid((int)w);
        const long long n = (long long)g.x * g.y;
        const bool ok = n >= w && (long long)g.x * kF32Waves * 64 < (1ll << 32) && g.x % kNumXCD == 0 && g.y < 65536 && g.z == 1 &&
                        n - w < (long long)kNumXCD * g.y;
        if (!ok && bad++ < 5) std::printf("%lld workgroups: grid %u x %u x %u\n", w, g.x, g.y, g.z);
    }
    if (bad) return 1;
    std::puts("launch grid: ok");
    return 0;
}
