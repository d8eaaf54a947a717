// Checks which unmask calls take one launch (unmask_in_one_launch in fdd_internal.h): never a launch of 2^32 work items or more,
// which would be refused, never more positions than the workgroup has records for, and the side of the line that was measured
// faster.  Host code only; built and run by tests/test_unmask_limits.py.
#include <cstdio>

#include "fdd_internal.h"

int main()
{
    using namespace fdd;
    long bad = 0;
    auto expect = [&](bool ok, long long N, long long B, long long bytes) {
        if (!ok && bad++ < 5) std::printf("N=%lld B=%lld, rows of %lld bytes\n", N, B, bytes);
    };
    for (long long B = 1; B <= 300; ++B)
        for (long long N = 1; N * B <= (1ll << 24); N = N < 64 ? N + 1 : N * 2 - N / 3)
            for (long long bytes : {2ll, 4ll, 250ll, 512ll, 1000ll, 2048ll, 4096ll, 4098ll, 304128ll}) {
                const bool one = unmask_in_one_launch((int)N, (int)B, bytes);
                expect(!one || (N * kOneLaunchWaves * 64 < (1ll << 32) && B <= kOneLaunchB && bytes <= 4096), N, B, bytes);
            }
    expect(!unmask_in_one_launch(1 << 23, 1, 2), 1 << 23, 1, 2);            // the first that would be refused
    expect(!unmask_in_one_launch(1 << 24, 1, 2), 1 << 24, 1, 2);
    // N, B, bytes per row, one launch
    const int sides[][4] = {{1, 8, 2048, 1}, {64, 32, 1024, 1}, {1, 16, 4096, 0}, {8, 64, 2048, 0}, {1, 64, 256, 0}, {16, 64, 64, 0}, {64, 64, 256, 1},
                            {1, 128, 64, 0}, {64, 128, 256, 0}, {256, 128, 256, 1}, {1024, 1, 4096, 1}, {4096, 1, 1024, 0}, {65536, 1, 4096, 0},
                            {16384, 4, 1024, 1}, {16384, 4, 2048, 0}, {16384, 8, 2048, 1}, {16384, 8, 4096, 0}, {16384, 32, 1024, 1}, {4096, 12, 2000, 1}};
    for (const auto& c : sides) expect(unmask_in_one_launch(c[0], c[1], c[2]) == (c[3] != 0), c[0], c[1], c[2]);
    if (bad) return 1;
    std::puts("one launch: ok");
    return 0;
}
