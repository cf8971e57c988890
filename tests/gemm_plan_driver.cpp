// The GEMM planner on the CPU: reads "plan <rows> <feature strips> <padded K> <own reduce>" lines, prints "<slices> <k steps a slice>
// <feature strips a tile> <token strips a tile>" for each.
#include <cstdio>
#include <cstring>

#include "../paper_2507_06608_amd/csrc/gemm_plan.hpp"

int main() {
    char what[16];
    int a, b, c, d;
    while (std::scanf("%15s %d %d %d %d", what, &a, &b, &c, &d) == 5) {
        if (!std::strcmp(what, "plan")) {
            const nexus::GemmPlan p = nexus::plan_gemm(a, b, c, d != 0);
            std::printf("%d %d %d %d\n", p.S, p.ksteps_per_split, p.FS, p.TS);
        } else return 1;
    }
    return 0;
}
