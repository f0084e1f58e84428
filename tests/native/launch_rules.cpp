// launch_rules.cpp -- prints what the launch rules of mdf_internal.h and
// nn_rules.h choose, for the questions on standard input, one a line.  Built and driven by
// tests/test_launch_rules_cpu.py; no call reaches the device.
#include <cstdio>
#include <cstring>

#include "mdf_internal.h"
#include "nn_rules.h"

int main()
{
    char what[32];
    while (std::scanf("%31s", what) == 1) {
        int a[8] = {};
        if (!std::strcmp(what, "most")) {               // cover storage mask gen
            if (std::scanf("%d%d%d%d", a, a + 1, a + 2, a + 3) != 4) return 1;
            std::printf("%d\n", mdf::march_max(mdf::Cover(a[0]), a[1], a[2] != 0, a[3] != 0));
        } else if (!std::strcmp(what, "two")) {         // cover storage sets pops nodes mask gen walls fields
            long long n = 0;
            int b = 0;
            if (std::scanf("%d%d%d%d%lld%d%d%d%d", a, a + 1, a + 2, a + 3, &n, a + 5, a + 6, a + 7, &b) != 9) return 1;
            const mdf::MarchWork w{a[2], a[3], n, a[5] != 0, a[6] != 0, a[7] != 0, uint32_t(b)};
            std::printf("%d\n", int(mdf::march_two(mdf::Cover(a[0]), a[1], w)));
        } else if (!std::strcmp(what, "next")) {        // left most
            if (std::scanf("%d%d", a, a + 1) != 2) return 1;
            std::printf("%d\n", mdf::march_next(a[0], a[1]));
        } else if (!std::strcmp(what, "grid")) {        // active all
            if (std::scanf("%d%d", a, a + 1) != 2) return 1;
            std::printf("%d\n", mdf::march_grid(a[0], a[1]));
        } else if (!std::strcmp(what, "cover")) {       // nodes storage beyond_cache
            if (std::scanf("%d%d%d", a, a + 1, a + 2) != 3) return 1;
            std::printf("%d\n", int(mdf::march_cover(a[0], a[1], a[2] != 0)));
        } else if (!std::strcmp(what, "emit")) {        // cover fields
            if (std::scanf("%d%d", a, a + 1) != 2) return 1;
            std::printf("%d\n", int(mdf::march_emit_cover(mdf::Cover(a[0]), uint32_t(a[1]))));
        } else if (!std::strcmp(what, "plan")) {        // storage sets q nx ny nz
            if (std::scanf("%d%d%d%d%d%d", a, a + 1, a + 2, a + 3, a + 4, a + 5) != 6) return 1;
            const mdf::Step2zPlan p = mdf::step2z_plan(a[0], a[1], a[2], a[3], a[4], a[5]);
            std::printf("%d %.4f\n", p.zc, p.fill);
        } else if (!std::strcmp(what, "pays")) {        // storage sets q walls nx ny nz
            if (std::scanf("%d%d%d%d%d%d%d", a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6) != 7) return 1;
            std::printf("%d\n", int(mdf::step2z_pays(a[0], a[1], a[2], a[3] != 0, a[4], a[5], a[6])));
        } else if (!std::strcmp(what, "conv")) {        // B H W cin cout bias mask f32
            if (std::scanf("%d%d%d%d%d%d%d%d", a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6, a + 7) != 8) return 1;
            std::printf("%d\n", int(mdfnn::conv_form(a[0], a[1], a[2], a[3], a[4],
                                                         {a[5] != 0, a[6] != 0, a[7] != 0})));
        } else {
            return 1;
        }
    }
    return 0;
}
