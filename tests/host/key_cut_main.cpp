// Checks the cut of a row tile's key tiles among those that share them (key_tiles and key_cut in fdd_internal.h, which the
// kernels call): fp32, among wavefronts, against 64-bit arithmetic, up to the most tiles a call can have; bf16, an M-tile's
// private tiles among the units booked for them; both for lists of positions in any order.  Host code only; built and run by
// tests/test_f32_limits.py.
#include <cstdio>

#include "fdd_internal.h"

int main()
{
    using namespace fdd;
    // row tiles: none or one tile, fewer tiles than wavefronts, the cases' sizes, a list of two far positions of
    // 2^22 .. 2^24 rollouts (the row tile walks the private tiles of every rollout between them), the type's limit
    const int tiles[] = {0, 1, 7, 8, 9, 63, 64, 258, 1026, 32770, 524288, (1 << 22) + 64, (1 << 23) + 512, (1 << 25) + 3,
                         (1 << 26) + 511, 0x7fffffff};
    long bad = 0;
    for (int n : tiles)
        for (int splits : {1, 2, 3, 9, 17, 64}) {
            const int parts = splits * kF32Waves;
            const FastDiv d = make_fastdiv((uint32_t)parts);
            for (int part = 0; part <= parts; ++part) {
                const long long want = (long long)n * part / parts;
                const int got = key_cut(n, part, parts, d);
                if (got != want && bad++ < 5) std::printf("tiles %d part %d of %d: %d, should be %lld\n", n, part, parts, got, want);
            }
        }
    // lists in any order: the parts of a row tile's keys are its prefix tiles and private tiles of rollouts that exist
    const int N = 50;
    for (int prefix : {0, 1, 5, 40})
        for (int per : {1, 3})
            for (int n_lo : {0, 1, 20, N - 1})
                for (int n_hi : {0, 1, 19, 20, N - 1})
                    for (int parts : {2, 8, 9, 24}) {
                        const int n = key_tiles(prefix, per, n_lo, n_hi);
                        const FastDiv d = make_fastdiv((uint32_t)parts);
                        for (int part = 0; part <= parts; ++part) {
                            const int t = key_cut(n, part, parts, d);
                            if ((t < 0 || t > prefix + (N - n_lo) * per) && bad++ < 5)
                                std::printf("rollouts %d to %d, part %d of %d: tile %d\n", n_lo, n_hi, part, parts, t);
                        }
                        if (n_hi >= n_lo && n != prefix + (n_hi - n_lo + 1) * per && bad++ < 5) std::printf("%d tiles\n", n);
                    }
    // bf16: whatever number of units is booked, the cuts at their borders ascend from none to all, so the segments of an M-tile
    // have disjoint shares that add up, and no tile is of a rollout that there is not
    for (int booked = 1; booked <= 64; ++booked) {
        const FastDiv d = make_fastdiv((uint32_t)booked);
        for (int per : {1, 2, 3, 1 << 18})
            for (int n_lo = 0; n_lo < N; ++n_lo)
                for (int n_hi = 0; n_hi < N; ++n_hi) {
                    const int n = key_tiles(0, per, n_lo, n_hi);
                    int before = 0;
                    bool ok = n > 0 && n <= (N - n_lo) * per && (n_hi < n_lo || n == (n_hi - n_lo + 1) * per) && key_cut(n, 0, booked, d) == 0;
                    for (int unit = 1; unit <= booked; ++unit) {
                        const int t = key_cut(n, unit, booked, d);
                        ok = ok && t >= before && t <= n;
                        before = t;
                    }
                    if ((!ok || before != n) && bad++ < 5) std::printf("%d units booked, rollouts %d to %d, %d tiles each\n", booked, n_lo, n_hi, per);
                }
    }
    if (bad) return 1;
    std::puts("key cut: ok");
    return 0;
}
