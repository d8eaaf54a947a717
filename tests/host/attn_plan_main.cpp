// Prints the plans of bf16 attention calls (make_attn_plan, as the library has it), one line per call of nine numbers on the command
// line: N B L Hq Hkv D E, the length of the list of query positions, and splits.  A line holds the rows of an M-tile, the ring
// slots, the workgroups, the equal pieces of an M-tile (0: ranges), its units, those of the prefix, and the bytes of partial results of this
// plan and of the one for calls that bring less scratch, and the stacked rows that one workgroup finishes in either.  Host code only; built
// and run by tests/test_attn_plan.py.
#include <cstdio>
#include <cstdlib>

#include "fdd_internal.h"

// stacked rows of M-tiles whose units all lie with one workgroup
static long long finished(const fdd_attn_params& p, const fdd::AttnPlan& a)
{
    const int MT = a.MT, last = a.R - (MT - 1) * a.mtile_rows;
    long long rows = 0;
    for (long long M = 0; M < (long long)p.Hkv * MT; ++M) {
        const long long base = a.U / a.W, rem = a.U % a.W, cut = rem * (base + 1);
        auto owner = [&](long long u) { return u < cut ? u / (base + 1) : rem + (u - cut) / base; };
        const bool one = a.uniform > 0 ? a.uniform == 1 : owner(M * a.TPU) == owner((M + 1) * a.TPU - 1);
        if (one) rows += M % MT == MT - 1 ? last : a.mtile_rows;
    }
    return rows;
}

int main(int argc, char** argv)
{
    using namespace fdd;
    for (int i = 1; i + 8 < argc; i += 9) {
        int v[9];
        for (int j = 0; j < 9; ++j) v[j] = std::atoi(argv[i + j]);
        fdd_attn_params p = {};
        p.N = v[0]; p.B = v[1]; p.L = v[2]; p.Hq = v[3]; p.Hkv = v[4]; p.D = v[5];
        p.dtype = FDD_BF16;
        p.E = p.ext_capacity = v[6];
        p.n_q_positions = v[7];
        p.splits = v[8];
        AttnPlan a, s;
        make_attn_plan(p, &a);
        make_attn_plan(p, &s, false);
        std::printf("%d %d %d %d %d %d %zu %zu %lld %lld\n", a.mtile_rows, a.slots, a.W, a.uniform, a.TPU, a.TP, a.ws_o_bytes + a.ws_ml_bytes,
                    s.ws_o_bytes + s.ws_ml_bytes, finished(p, a), finished(p, s));
    }
    return 0;
}
