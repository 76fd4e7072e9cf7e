// The choices of csrc/lss_fwd_plan.h on the host: within the limits of workspace and kernels for all sizes, and on launches that were
// measured in every form and split count one of those within 6 % of the shortest.
#include "lss_fwd_plan.h"

#include <cstdio>
#include <initializer_list>
#include <vector>

using namespace lss;

struct Measured {
    SegShape s;
    bool with_drop;
    int most;                       // splits the workspace is sized for
    std::vector<FwdPlan> good;
};

static const Measured measured[] = {
    {{0, 888, 888, 2, 13, 64, 1, 0}, true, 3, {{FWD_2x2, 1}}},     // 16.4 us, 23.2 as chosen before
    {{369, 607, 1163, 2, 14, 64, 1, 0}, true, 4, {{FWD_2x2, 1}}},     // 18.1 us, 25.1 as chosen before
    {{1032, 1259, 8387, 2, 7, 64, 1, 0}, true, 8, {{FWD_4x1, 5}, {FWD_4x1, 6}, {FWD_2x2, 1}, {FWD_2x2, 2}}},     // 34.4 us, 47.0 as chosen before
    {{991, 2345, 6249, 3, 2, 64, 1, 0}, true, 9, {{FWD_4x1, 6}, {FWD_4x1, 7}, {FWD_2x2, 3}, {FWD_2x2, 4}}},     // 37.3 us, 46.8 as chosen before
    {{96, 92, 525, 3, 8, 128, 1, 0}, false, 2, {{FWD_8x1, 1}}},     // 9.1 us, 11.1 as chosen before
    {{3377, 73, 5711, 2, 6, 128, 1, 0}, false, 16, {{FWD_8x1, 12}, {FWD_8x1, 14}, {FWD_8x1, 16}}},     // 15.3 us, 18.3 as chosen before
    {{12, 2952, 3043, 1, 14, 128, 1, 0}, false, 7, {{FWD_4x2, 1}}},     // 51.1 us, 77.6 as chosen before
    {{0, 1099, 1099, 3, 10, 128, 1, 0}, false, 4, {{FWD_4x2, 1}}},     // 24.2 us, 33.2 as chosen before
    {{1586, 88, 1916, 2, 10, 128, 1, 0}, true, 7, {{FWD_8x1, 7}}},     // 17.6 us, 21.6 as chosen before
    {{1155, 83, 8786, 2, 13, 128, 1, 0}, true, 16, {{FWD_8x1, 7}, {FWD_8x1, 8}}},     // 17.8 us, 21.3 as chosen before
    {{0, 715, 715, 4, 12, 128, 1, 0}, true, 3, {{FWD_4x2, 1}}},     // 28.0 us, 40.6 as chosen before
    {{7, 967, 1171, 4, 10, 128, 1, 0}, true, 4, {{FWD_4x2, 1}}},     // 37.7 us, 50.4 as chosen before
    {{0, 1557, 1557, 2, 10, 128, 1, 0}, true, 6, {{FWD_4x2, 1}}},     // 43.0 us, 70.2 as chosen before
    {{22240, 2339, 35978, 4, 7, 64, 1, 0}, false, 2, {{FWD_4x1, 2}}},     // 506 us, 565 as chosen before
    {{1604, 3456, 17209, 4, 8, 64, 1, 0}, false, 2, {{FWD_4x1, 1}}},     // 127 us, 138 as chosen before
    {{0, 1459, 1459, 4, 10, 64, 1, 0}, false, 3, {{FWD_4x1, 1}}},     // 25.6 us, 33.3 as chosen before
    {{1531, 1622, 4513, 2, 6, 64, 1, 0}, false, 7, {{FWD_2x2, 1}}},     // 30.1 us, 36.0 as chosen before
    {{0, 1537, 1537, 3, 16, 128, 1, 0}, false, 4, {{FWD_8x1, 1}}},     // 54.5 us, 65.1 as chosen before
    {{211, 3110, 3517, 2, 11, 128, 1, 0}, false, 4, {{FWD_8x1, 1}}},     // 95.8 us, 106 as chosen before
    {{0, 1257, 1257, 3, 16, 128, 1, 0}, true, 5, {{FWD_4x2, 1}}},     // 56.5 us, 68.0 as chosen before
    {{10452, 1339, 15568, 3, 5, 128, 0, 0}, true, 12, {{FWD_4x2, 3}}},     // 278.4 us, 352.5 as chosen before
};

static int fail(const char *what, const SegShape &s, bool drop, const FwdPlan &p)
{
    std::printf("%s: B %d H %d d %d l_s %d l_x %d s0 %lld causal %d dropout %d: form %d, %d splits\n", what, s.B, s.H, s.d, s.l_s, s.l_x,
                (long long)s.s0, s.causal, drop, p.form, p.splits);
    return 1;
}

int main()
{
    int bad = 0;
    for (const Measured &m : measured) {
        const FwdPlan p = pick_fwd_plan(m.s, m.with_drop, m.most);
        bool good = false;
        for (const FwdPlan &g : m.good) good = good || (g.form == p.form && g.splits == p.splits);
        if (!good) bad += fail("not among the shortest", m.s, m.with_drop, p);
    }
    if (bad) return 1;
    int fours = 0;
    for (int d : {64, 128})
        for (int l_s : {1, 31, 32, 33, 64, 65, 127, 128, 129, 256, 257, 1044, 4096, 70001})
            for (int l_x : {1, 64, 65, 512, 1000, 8192, 50112, 1 << 20})
                for (int heads : {1, 5, 7, 16, 28, 64, 65535})
                    for (int causal : {0, 1})
                        for (int at : {0, 1})
                            for (int most : {1, 2, 3, 16})
                                for (bool drop : {false, true}) {
                                    if (l_s > l_x) continue;
                                    const SegShape s{at * (int64_t)(l_x - l_s), l_s, l_x, 1, heads, d, causal, 0};
                                    const FwdPlan p = pick_fwd_plan(s, drop, most);
                                    const int64_t seen = causal ? s.s0 + l_s : l_x;
                                    if (p.splits < 1 || p.splits > most || (p.splits > 1 && (seen + 63) / 64 / p.splits < 2)) return fail("outside the limits", s, drop, p);
                                    if (d == 64 ? p.form == FWD_8x1 || (drop && p.form == FWD_4x2) : p.form != FWD_8x1 && p.form != FWD_4x2) return fail("no such form", s, drop, p);
                                    // four groups: only where all workgroups run at once, one per compute unit, and not for launches of a few
                                    const int64_t wgs = ((int64_t)l_s + (p.form == FWD_1x4 ? 31 : 63)) / (p.form == FWD_1x4 ? 32 : 64) * heads * p.splits;
                                    if ((p.form == FWD_1x4 || p.form == FWD_2x4) && (wgs <= 16 || wgs > 256)) return fail("four groups in too few or too many workgroups", s, drop, p);
                                    fours += p.form == FWD_1x4 || p.form == FWD_2x4;
                                }
    if (fours < 100) return 1;
    std::printf("clean\n");
    return 0;
}
