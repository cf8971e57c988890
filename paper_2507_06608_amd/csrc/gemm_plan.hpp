// Which GEMM kernel, tile shape and number of K slices a projection takes.  Plain C++ on host memory, no GPU work.
#pragma once
#include <algorithm>
#include <cstddef>

#if defined(__HIPCC__)
#define NEXUS_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define NEXUS_HOST_DEVICE inline
#endif

namespace nexus {

constexpr int kGemmBK = 64;  // unit of the split-K bookkeeping: ksteps_per_split counts 64-wide k steps

// Tile shapes are features x tokens.  A batch of at most 128 tokens (a decode batch, a short chunk) streams the weights
// once and wants many small workgroups whose rings together keep about 100 KiB per CU in flight: one CU draws at
// most about 50 GB/s from HBM, so a decode share of the chip is bound by per-CU bytes in flight, not by the HBM
// interface.  Longer batches take the tiled kernel in one of the shapes of kTileShapes.
enum GemmVariant {
    GV_P128 = 0,   // gemm_dl_kernel, 128 x 128, 4 waves, 32-wide stages, 64 KiB ring: two workgroups per CU
    GV_P128D,      // the same with a six-stage ring, 96 KiB: one workgroup per CU
    GV_P192x128,   // 4 waves of 3 x 2 MFMA tiles, 120 KiB ring (all from here on: one workgroup per CU)
    GV_P256x128,   // 4 waves of 4 x 2, 144 KiB
    GV_P320x128,   // 4 waves of 5 x 2, 140 KiB
    GV_P192x256,   // 8 waves of 3 x 2, 140 KiB
    GV_P256,       // 256 x 256, 8 waves of 2 x 4, 128 KiB
    GV_P320,       // 320 x 256, 8 waves of 5 x 2, 144 KiB
    GV_S64,       // gemm_stream_kernel, 128 features x 64 tokens, 4 waves: decode batches of 33..64
    GV_S32,       // gemm_stream_kernel, 128 features x 32 tokens, 4 waves: decode batches of at most 32
    GV_S64W,      // gemm_stream_kernel, 256 features x 64 tokens (two feature strips per wave): on a small CU share
                  //   every workgroup re-reads the activations through the same per-CU load path as the weights, and
                  //   twice the features per activation byte is worth more than twice the workgroups
    GV_S128,      // gemm_stream_kernel, 128 features x 128 tokens, 4 waves: batches of 65..128 tokens (a full decode
                  //   pool, a short prefill chunk), still closer to a sweep over the weights than to a tiled GEMM
    GV_S128W,     // gemm_stream_kernel, 256 features x 128 tokens, 8 waves sharing the activation tiles
    GV_R64,       // gemm_dl_kernel with the extent of GV_S64 / GV_S32: k ranges shorter than the streaming
    GV_R32,       //   kernel's pipeline (hidden sizes below 128)
    GV_COUNT
};
struct GemmPlan {
    int variant, S, ksteps_per_split, FS, TS;
};
constexpr int kChipCUs = 256;  // the plan is sized for the whole chip, whatever share the phase runs on

// The tiled GEMM's time, from which tile shape and split count are chosen.  A CU fills its LDS at 65 GB/s at most, and at
// 40 GB/s the whole chip is at its power limit (1.35 PFLOP/s), so the time of a tile per 64 steps of k depends on the
// shape and on how many CUs are busy: `us` holds it for 64, 128, 192 and 256 of them, measured on MI355X as the slope
// between K = 1024, 4096 and 8192 of grids that fill those CUs once and twice.  `round_us` is what a round of the grid
// pays on top (pipeline fill, epilogue).  Two 128 x 128 workgroups share a CU: `us` is the time of such a pair, and a lone
// one takes kLoneTileUs (the pair wins for K up to 1400 or so; the projections of the 8B, 14B and 70B shapes never take
// it).  Against 340 timings (256 to 1021 tokens, 1 to 4 slices, 192 and 256 CUs) the estimate is off by 7 % in the mean;
// outside that range it was checked by whole prefill steps against the planner before it, which knew four shapes and sliced
// 128 x 128 tiles only: 8B shape, 900 to 2304 tokens, 1.04 to 1.22x as fast, 14B, 1021 to 1792, 1.02 to 1.15x, 70B, 1200 to 3072, 1.03x.
struct TileShape {
    int variant, FS, TS, per_cu;
    double us[4], round_us;
    const char *name;  // test hook: NEXUS_GEMM_TILES
};
constexpr TileShape kTileShapes[] = {
    {GV_P320, 10, 8, 1, {1.22, 1.31, 1.60, 1.90}, 11, "320"},     {GV_P256, 8, 8, 1, {1.08, 1.18, 1.30, 1.58}, 8, "256"},
    {GV_P192x256, 6, 8, 1, {0.95, 1.06, 1.14, 1.25}, 7, "192x256"}, {GV_P320x128, 10, 4, 1, {0.90, 0.97, 1.04, 1.15}, 4, "320x128"},
    {GV_P256x128, 8, 4, 1, {0.76, 0.82, 0.87, 0.93}, 4, "256x128"}, {GV_P192x128, 6, 4, 1, {0.60, 0.65, 0.69, 0.74}, 3, "192x128"},
    {GV_P128D, 4, 4, 1, {0.48, 0.50, 0.52, 0.57}, 3, "128d"},     {GV_P128, 4, 4, 2, {0.93, 0.98, 1.05, 1.15}, 3, "128"},
};
constexpr double kLoneTileUs = 0.73;
constexpr int kMaxTileSlices = 4;

inline double tile_round_us(const TileShape &t, int n) {  // one k step of 64 with n CUs busy
    const double x = std::max(0.0, std::min(3.0, n / 64.0 - 1.0));
    const int i = std::min(2, (int)x);
    return t.us[i] + (t.us[i + 1] - t.us[i]) * (x - i);
}
inline double tile_estimate_us(const TileShape &t, int n_ttiles, int n_ftiles, int ksteps_per_split, int S, int cus) {
    const long tiles = (long)((n_ttiles + t.TS - 1) / t.TS) * ((n_ftiles + t.FS - 1) / t.FS) * S, slots = (long)t.per_cu * cus;
    const long full = tiles / slots, rem = tiles % slots;
    const double round = tile_round_us(t, cus);
    double last = 0.0;
    if (rem && t.per_cu == 1) last = tile_round_us(t, (int)rem);
    else if (rem) last = rem <= cus ? kLoneTileUs : kLoneTileUs + (round - kLoneTileUs) * (double)(rem - cus) / cus;
    return 4.0 + (full * round + last) * ksteps_per_split + t.round_us * (double)(full + (rem > 0));
}
inline bool fits_32bit_offsets(int n_strips, int Kp) { return (size_t)n_strips * Kp * 64 < ((size_t)1 << 32); }
// The fastest shape for a GEMM in S slices on `cus` CUs; ties go to the larger tile.  (The two widest shapes address their
// operands with 32-bit offsets; 256 x 256 has a second form that does not.)
inline const TileShape *choose_tile(int n_ttiles, int n_ftiles, int Kp, int ksteps_per_split, int S, int cus, double *us = nullptr) {
    const TileShape *best = nullptr;
    double best_us = 0.0;
    for (const TileShape &t : kTileShapes) {
        if ((t.variant == GV_P320 || t.variant == GV_P192x256) && !(fits_32bit_offsets(n_ftiles, Kp) && fits_32bit_offsets(n_ttiles, Kp))) continue;
        const double e = tile_estimate_us(t, n_ttiles, n_ftiles, ksteps_per_split, S, cus);
        if (!best || e < best_us) best = &t, best_us = e;
    }
    if (us) *us = best_us;
    return best;
}

// Depends on the problem only (never on the CU share): S fixes the summation order, so results are bit-identical
// across layouts.  Up to 128 tokens the slices are doubled until there are 192 workgroups: it is the bytes that the most loaded CU has
// to load that count, and with the projections of the 8B, 14B and 70B shapes that is at most 1.75 times its part on any share.  (As
// many slices as leave at most one workgroup per CU of the whole chip, six for the 40 feature blocks of the 14B shape's O and down
// projections instead of eight, are faster there and slower on most shares, where S has to be the same; beyond 64 rows they also miss
// the wide workgroups, see run_gemm.  Steps of three layers of the 14B shape, 64 / 128 requests, eight -> six slices: 256 CUs 481 -> 447
// us / 594 -> 583, 224 CUs 475 -> 491 / 601 -> 656, 192 590 -> 611 / 745 -> 800, 160 589 -> 613 / 748 -> 812, 128 637 -> 617 / 845 -> 795,
// 96 827 -> 818 / 1047 -> 1081, 32 1635 -> 1634 / 2218 -> 2347.)
// Beyond 128 tokens S is the one with the least estimated time of GEMM and partial sums.  By itself a phase
// pays 0.29 us per MB of them, written and read back (the kernel that sums them reads S slices of fp32 where it would have
// read one of half); they are charged 0.7, because a step's other phase pays for them too: with two slices of the QKV and
// four of the down projection instead of one and two, a 512-token prefill step of the 8B shape takes 1179 us against 1242,
// and the decode phase next to it on 64 CUs, which bounds a mixed step, 2033 to 2063 against 1915 to 2003 (the only mixed step
// that the charge was set on).  A reduce kernel
// of its own, where no later kernel sums the slices in passing, adds 5 us.
inline GemmPlan plan_gemm(int T, int n_ftiles, int Kp, bool own_reduce) {
    const int ksteps = Kp / kGemmBK;
    const int nt = (T + 31) / 32;
    GemmPlan p{};
    int S = 1;
    if (T <= 128) {
        const int min_ksteps = 8;
        p.FS = 4;
        if (T <= 32) p.variant = GV_S32, p.TS = 1;
        else if (T <= 64) p.variant = GV_S64, p.TS = 2;
        else p.variant = GV_S128, p.TS = 4;
        const int blocks = ((n_ftiles + p.FS - 1) / p.FS) * ((nt + p.TS - 1) / p.TS);
        while (S < 8 && blocks * S < (3 * kChipCUs) / 4) S *= 2;
        while (S > 1 && ksteps / S < min_ksteps) --S;
    } else {
        double best = 0.0;
        for (int s = 1; s <= kMaxTileSlices && ksteps / s >= 8; ++s) {
            double us;
            choose_tile(nt, n_ftiles, Kp, (ksteps + s - 1) / s, s, kChipCUs, &us);
            if (s > 1) us += (4 * s - 2) * 0.7e-6 * 32.0 * nt * 32.0 * n_ftiles + (own_reduce ? 5.0 : 0.0);
            if (s == 1 || us < best) best = us, S = s;
        }
    }
    p.ksteps_per_split = (ksteps + S - 1) / S;
    p.S = (ksteps + p.ksteps_per_split - 1) / p.ksteps_per_split;
    if (T > 128) {
        const TileShape *t = choose_tile(nt, n_ftiles, Kp, p.ksteps_per_split, p.S, kChipCUs);
        p.variant = t->variant, p.FS = t->FS, p.TS = t->TS;
    }
    return p;
}

// Tile of a workgroup.  Workgroups are dealt to the XCDs round-robin: every XCD gets a contiguous range of the n tiles, the first
// n % n_xcd of the ranges one longer; n_xcd = 1: launch order.  (Another K slice starts at another XCD if n is no multiple of them,
// which renames the ranges and no more.)
NEXUS_HOST_DEVICE int tile_of_block(int block, int n, int n_xcd) {
    if (n_xcd <= 1) return block;
    const int x = block % n_xcd, longer = n % n_xcd;
    return x * (n / n_xcd) + (x < longer ? x : longer) + block / n_xcd;
}
// XCDs that a grid of n tiles a K slice is dealt to in ranges (1: launch order).  A multiple of the XCDs always is.  Another one is on
// a share of the chip only, and there only if there are two blocks of tokens and all slices fit the share's CUs, more than half of the
// chip: in launch order the two workgroups of a block of weights then run at one time on different XCDs, both fetch the weights, and
// the phase next to it, bound by its own reads, pays for that too.  Kernel times, ranges against launch order (8B, 14B and 70B shapes,
// 160 to 1500 tokens): such grids on shares of 144 to 240 CUs are 1.04 times as fast next to a decode phase in the median if K is in
// one slice (40 timings, 1.01 to 1.17) and 1.01 in several (125, 0.93 to 1.11), and 1.02 (0.97 to 1.06) and 1.00 (0.96 to 1.06) by
// themselves; four layers of the 8B shape, 512 tokens on 192 CUs next to 64 decode requests on 64, 2029 -> 1983 us, on another card
// 1941 -> 1917.  The other grids, next to a decode phase and by themselves: two blocks of tokens on 96 CUs 0.99 and 0.99, in more than
// one round 0.98 (0.95 to 1.02) and 0.99 (0.96 to 1.01), three and more blocks 1.00 (0.87 to 1.08) and 0.99 (0.93 to 1.06), one 1.00 and
// 1.00.  On the whole chip 54 grids of 22 to 540 tiles: 0.99 (0.94 to 1.06).
inline int tile_xcds(int n, int n_tblk, int S, int cus, int n_cus, int n_xcd) {
    const bool pairs = cus < n_cus && 2 * cus > n_cus && n_tblk == 2 && n * S <= cus;
    return n % n_xcd == 0 || pairs ? n_xcd : 1;
}

}  // namespace nexus
