// The GEMM planner on the CPU, a line of input for a line of output:
//   plan <rows> <feature strips> <padded K> <own reduce>      -> <slices> <k steps a slice> <feature strips a tile> <token strips a tile>
//   xcds <tiles> <token blocks> <slices> <CUs of the share>   -> <XCDs of 8 that the tiles are dealt to in ranges> on a chip of 256 CUs
//   order <tiles> <XCDs> 0 0                                  -> the tile of each workgroup in turn
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
        } else if (!std::strcmp(what, "xcds")) {
            std::printf("%d\n", nexus::tile_xcds(a, b, c, d, 256, 8));
        } else if (!std::strcmp(what, "order")) {
            for (int i = 0; i < a; ++i) std::printf("%d ", nexus::tile_of_block(i, a, b));
            std::printf("\n");
        } else return 1;
    }
    return 0;
}
