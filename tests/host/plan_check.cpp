// Goes over the choices of csrc/lss_bwd_plan.h on the host: of the forms and split counts that a launch may take, the one chosen
// has the smallest estimate under the launcher's own decision whether there is a preprocess launch, every choice stays within
// the limits that the kernels and the workspace have, and on launches with dropout that were measured in every form and split
// count one of those within 6 % of the shortest is taken.  Wavefronts of 16 rows are taken where every compute unit gets one workgroup, and on
// launches measured with and without them only where they were no slower.
#include "lss_bwd_plan.h"

#include <cstdio>
#include <initializer_list>
#include <vector>

static int fail(const char *what, const lss::SegShape &s, const lss::BwdPlan &p)
{
    std::printf("%s: B %d H %d l_s %d l_x %d s0 %lld causal %d: %d splits, %d groups\n", what, s.B, s.H, s.l_s, s.l_x, (long long)s.s0, s.causal,
                p.splits, p.groups);
    return 1;
}

int main()
{
    for (double a : {1e-3, 0.5, 1.0, 7.25, 900.0, 1e5})
        for (double b : {1e-3, 0.5, 0.999, 1.0, 31.0, 1e5}) {
            const double want = pow(pow(a, 6.0) + pow(b, 6.0), 1.0 / 6.0);
            if (!(fabs(lss::larger_or_both(a, b) - want) <= 1e-13 * want)) return 1;
        }
    struct { lss::SegShape s; int most; std::vector<lss::BwdPlan> good; } measured[] = {
        {{1080, 1034, 2121, 1, 6, 64, 0, 0}, 8, {{2, 2}}},     // 40.6 us, 53.5 as chosen before
        {{1330, 1797, 13899, 1, 2, 64, 1, 0}, 16, {{2, 2}, {3, 2}, {4, 2}, {5, 2}, {6, 2}}},     // 56.1 us, 71.0 as chosen before
        {{353, 124, 2363, 1, 5, 64, 1, 0}, 9, {{2, 1}}},     // 17.4 us, 21.5 as chosen before
        {{571, 561, 1527, 3, 2, 64, 1, 0}, 6, {{2, 2}, {3, 2}, {4, 2}}},     // 29.1 us, 33.8 as chosen before
        {{0, 1178, 1178, 2, 8, 64, 1, 0}, 4, {{1, 2}}},     // 41.7 us, 48.1 as chosen before
        {{782, 214, 1031, 1, 11, 64, 1, 0}, 4, {{3, 1}, {3, 2}, {4, 2}}},     // 20.7 us, 23.8 as chosen before
        {{2949, 759, 5697, 2, 2, 64, 1, 0}, 16, {{4, 2}, {5, 2}, {6, 2}}},     // 35.1 us, 40.3 as chosen before
    };
    for (const auto &m : measured) {
        const lss::BwdPlan p = lss::pick_bwd_plan(m.s, true, m.most, true);
        bool good = false;
        for (const lss::BwdPlan &g : m.good) good = good || (g.splits == p.splits && g.groups == p.groups);
        if (!good) return fail("not among the shortest", m.s, p);
    }
    const struct { lss::SegShape s; int splits; bool narrow, with_drop; } forms[] = {
        {{768, 256, 1024, 1, 4, 64, 1, 0}, 2, true, false},    // 15.6 us without, 14.2
        {{2080, 89, 3523, 1, 6, 64, 0, 0}, 14, true, false},          // 252 workgroups, 32 on each XCD: 18.0, 17.4
        {{2066, 126, 2317, 2, 5, 64, 1, 0}, 7, true, false},          // 20.0, 19.0
        {{876, 71, 1474, 1, 15, 64, 0, 0}, 5, false, false},          // 255, 33 on some XCD: 17.3, 19.8
        {{337, 374, 1351, 1, 15, 64, 0, 0}, 2, false, false},         // 26.4, 30.4
        {{2040, 381, 2458, 1, 9, 64, 1, 0}, 3, false, false},         // 23.9, 26.2
        {{103, 123, 3718, 2, 12, 64, 1, 0}, 1, true, false},          // 648 tiles to clear, 184 idle compute units: 17.1, 15.3
        {{42, 137, 4155, 1, 11, 64, 1, 0}, 1, true, false},           // 14.5, 12.8
        {{3477, 174, 49122, 1, 5, 64, 1, 0}, 9, false, false},        // 1775, 21: 26.1, 31.4
        {{3111, 124, 19970, 1, 6, 64, 1, 0}, 11, false, false},       // 18.4, 21.8
        {{2217, 378, 29126, 1, 8, 64, 1, 0}, 3, false, false},        // 25.2, 33.4
        {{2217, 378, 29126, 1, 8, 64, 1, 1}, 3, true, false},         // (left as they are, they cost nothing)
        {{639, 78, 6356, 3, 8, 64, 1, 0}, 3, false, true},     // with dropout 21.6, 24.4
        {{288, 73, 27279, 1, 7, 64, 1, 0}, 1, true, true},     // 19.6, 17.0
        {{44, 116, 7838, 1, 8, 64, 1, 0}, 1, true, true},      // 14.8, 13.2
    };
    for (const auto &f : forms)
        if (lss::bwd_narrow(f.s, f.splits, 1, f.with_drop) != f.narrow) return fail("wavefronts of 16 rows", f.s, {f.splits, 1});
    long long owns = 0, lets = 0;
    for (int l_s : {65, 66, 97, 128, 129, 192, 193, 256, 257, 300, 384, 512, 513, 1024, 1044, 4096, 12661})
        for (int l_x : {65, 129, 512, 1000, 1024, 4100, 8192, 24576, 50112})
            for (int heads : {1, 2, 4, 7, 16, 40, 64, 513})
                for (int causal : {0, 1})
                    for (int at : {0, 1, 2}) {
                        if (l_s > l_x) continue;
                        const int64_t s0 = (int64_t)(l_x - l_s) * at / 2;
                        const lss::SegShape s{s0, l_s, l_x, heads > 16 ? heads / 8 : 1, heads > 16 ? 8 : heads, 64, causal, 0};
                        const lss::BwdWork w = lss::bwd_work(s);
                        for (int most : {1, 2, 5, 16})
                            for (int form = 0; form < 4; ++form) {
                                const bool may_own = form & 1, with_drop = form & 2;
                                const lss::BwdPlan p = lss::pick_bwd_plan(s, with_drop, most, may_own);
                                const int64_t seen = causal ? s0 + l_s : l_x, tiles = (seen + 63) / 64;
                                if (p.splits < 1 || p.splits > most || p.groups < 1 || p.groups > (l_s > 128 ? 2 : 1) || (p.splits > 1 && tiles / p.splits < 4))
                                    return fail("outside the limits", s, p);
                                auto own = [&](int splits, int groups) { return may_own && lss::bwd_own_values(s, splits, groups); };
                                const int64_t heads64 = (int64_t)s.B * s.H, dq_wgs = (l_s + 127) / 128 * heads64 * p.splits, dkv_wgs = (seen + 127) / 128 * heads64;
                                if (lss::bwd_narrow(s, p.splits, p.groups, with_drop) && (p.groups != 1 || l_s <= lss::kSkinnyRows || (dq_wgs + 7) / 8 + (dkv_wgs + 7) / 8 > 32))
                                    return fail("wavefronts of 16 rows, more than one workgroup per compute unit", s, p);
                                if (l_s > lss::kOwnRows && own(p.splits, p.groups)) return fail("start values that do not fit", s, p);
                                (own(p.splits, p.groups) ? owns : lets) += 1;
                                const double t = lss::bwd_estimate(w, p.splits, p.groups, own(p.splits, p.groups), with_drop);
                                if (!(t > 0.0 && t < 1e9)) return fail("no time", s, p);
                                for (int g = 1; g <= (l_s > 128 ? 2 : 1); ++g)
                                    for (int sp = 1; sp <= most && (sp == 1 || tiles / sp >= 4); ++sp)
                                        if (lss::bwd_estimate(w, sp, g, own(sp, g), with_drop) < t) return fail("a shorter one is there", s, p);
                            }
                    }
    if (owns < 100 || lets < 100) return 1;
    std::printf("clean\n");
    return 0;
}
