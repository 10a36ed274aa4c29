// The stencil variants the host may run and their launcher.  All give
// bitwise-identical fields; they differ in tile shape, steps per launch and
// speed (tiled depth-only kernels: stencil.hip; nodal: nodal.hip; tile in LDS
// over several steps, both media: blocked.hip; strips streamed through
// registers over several steps: stream.hip; whole solves in LDS: resident.hip).
#include <map>
#include <utility>

#include "internal.h"

namespace eig {

const StencilVariant kVariants[kNumVariants] = {
    {64, 32, EIG_MEDIUM_LAYERED, 1},   // 0: one node per lane
    {128, 32, EIG_MEDIUM_LAYERED, 1, 1},  // 1: two nodes per lane, prefetch 1
    {128, 32, EIG_MEDIUM_LAYERED, 1, 1},  // 2: two nodes per lane, prefetch 2
    {128, 64, EIG_MEDIUM_LAYERED, 1, 1},  // 3: prefetch 2
    {128, 16, EIG_MEDIUM_LAYERED, 1, 1},  // 4: prefetch 2
    {128, 64, EIG_MEDIUM_LAYERED, 1, 1},  // 5: prefetch 1
    {64, 32, EIG_MEDIUM_NODAL, 1},     // 6: nodal media
    {128, 8, EIG_MEDIUM_LAYERED, 1, 1},   // 7: prefetch 2
    {128, 16, EIG_MEDIUM_LAYERED, 1, 1},  // 8: prefetch 1
    {128, 16, EIG_MEDIUM_LAYERED, 2},  // 9: two steps per launch
    {128, 32, EIG_MEDIUM_LAYERED, 2},  // 10: two steps per launch
    {128, 64, EIG_MEDIUM_LAYERED, 2},  // 11: two steps per launch
    {128, 128, EIG_MEDIUM_LAYERED, 2}, // 12: two steps per launch
    {128, 64, EIG_MEDIUM_LAYERED, 2},  // 13: two steps, halo columns up front
    {128, 32, EIG_MEDIUM_LAYERED, 2},  // 14: two steps, halo columns up front
    {128, 64, EIG_MEDIUM_LAYERED, 3},  // 15: three steps per launch
    {128, 32, EIG_MEDIUM_LAYERED, 3},  // 16: three steps per launch
    {128, 16, EIG_MEDIUM_NODAL, 1, 1},    // 17: nodal media, two nodes per lane
    {128, 32, EIG_MEDIUM_NODAL, 1, 1},    // 18: nodal media, two nodes per lane
    {128, 16, EIG_MEDIUM_NODAL, 2},    // 19: nodal media, two steps per launch
    {128, 32, EIG_MEDIUM_NODAL, 2},    // 20: nodal media, two steps per launch
    {0, 0, EIG_MEDIUM_LAYERED, 1, 1, 1},  // 21: resident in LDS, every step in one launch
    {0, 0, EIG_MEDIUM_NODAL, 1, 1, 1},    // 22: resident in LDS, every step in one launch
    {0, 0, EIG_MEDIUM_LAYERED, kStreamSteps, 0, 0, 0, 1},  // 23: strips streamed through registers
    {0, 0, EIG_MEDIUM_NODAL, kNodalStreamSteps, 0, 0, 0, 1},  // 24: the same, nodal media
    {64, 24, EIG_MEDIUM_NODAL, 4, 0, 0, 1},  // 25: as 27, operands read per node (forced only)
    {58, 58, EIG_MEDIUM_LAYERED, 4, 0, 0, 1},  // 26: four steps, tile in LDS (small launches)
    {58, 34, EIG_MEDIUM_NODAL, 4, 0, 0, 1},  // 27: the same, nodal: tile and medium in LDS
    {0, 0, EIG_MEDIUM_LAYERED, kAbsorbingStreamSteps, 0, 0, 1, 1, 1},  // 28: as 23, absorbing edges
};

void launch_stencil(const SolveDesc* descs, const int2* tiles, int ntiles, int step,
                    int variant, int rows, hipStream_t s) {
    if (ntiles <= 0) return;
    if (kVariants[variant].stream && kVariants[variant].medium_kind == EIG_MEDIUM_NODAL)
        launch_nodal_stream(descs, tiles, ntiles, step, rows, s);
    else if (kVariants[variant].stream)
        launch_layered_stream(descs, tiles, ntiles, step, rows, kVariants[variant].absorbing, s);
    else if (kVariants[variant].steps == 4)
        launch_blocked_stencil(descs, tiles, ntiles, step, variant, s);
    else if (kVariants[variant].medium_kind == EIG_MEDIUM_NODAL)
        launch_nodal_stencil(descs, tiles, ntiles, step, variant, s);
    else
        launch_layered_stencil(descs, tiles, ntiles, step, variant, s);
}

// A launch's time in the units of one wide row (K levels of 128 columns) on a
// SIMD of its own, 1.0 us (nodal media 1.44 us): a wave takes rows + 2 K of them, a
// narrow row 0.65, and two waves of a SIMD slow each other down 1.65 times (measured
// per launch over 15 to 960 solves of 128 to 512 columns).  Up to the chip's 2048 waves
// (two per SIMD) a launch takes as long as one wave; a few more wait for a
// whole further one; from 1.25 rounds on the waves' ends are spread enough for
// the work to count, and half a wave for the end.
StreamCut stream_cut(int v, const std::vector<StreamLoad>& all) {
    const int K = kVariants[v].steps;
    constexpr double kPair = 1.65, kSlots = 2048.0;
    std::map<std::pair<int, int>, int64_t> grids;
    for (const auto& l : all) grids[{l.nx, l.nz}] += l.solves;
    std::vector<StreamLoad> loads;
    for (const auto& g : grids) loads.push_back({g.first.first, g.first.second, g.second});
    int nzmax = 2;
    for (const auto& l : loads) nzmax = std::max(nzmax, l.nz);
    StreamCut best;
    double best_t = 1e300;
    for (int narrow = 0; narrow < 2; ++narrow)
        for (int n = 1; n <= std::max(1, (nzmax - 1) / kStreamRowsMin); n += 1 + n / 16) {
            const int rows = stream_chunks(nzmax, n);  // ceil((nz - 1) / n)
            double waves = 0.0, work = 0.0, longest = 0.0;
            for (const auto& l : loads)
                for (const auto& st : stream_strips(l.nx, narrow, K)) {
                    const int c = stream_chunks(l.nz, rows);
                    const double per = st.narrow ? 0.65 : 1.0;
                    waves += (double)l.solves * c;
                    work += (double)l.solves * per * (l.nz - 1 + c * 2.0 * K);
                    longest = std::max(longest, per * (std::min(rows, l.nz - 1) + 2.0 * K));
                }
            const double rounds = waves / kSlots;
            const double t = rounds <= 0.5    ? longest
                             : rounds <= 1.0  ? kPair * longest
                             : rounds <= 1.25 ? (kPair + 1.0) * longest
                                              : kPair * work / kSlots + 0.5 * longest;
            if (t < best_t) {
                best_t = t;
                const bool nodal = kVariants[v].medium_kind == EIG_MEDIUM_NODAL;
                best = StreamCut{rows, narrow, (t * (nodal ? 1.44 : 1.0) + 19.0) * 8.0 / K};
            }
        }
    return best;
}

// Launches of few tiles take four steps with the tile in LDS instead: its 8 waves
// share the tile's rows (58 x 58 nodes, nodal media 58 x 34), while a streaming wave
// takes its rows one after the other however few waves there are.  Both estimates in
// us per eight steps (the LDS kernels' two launches; the streaming ones' rows, and
// 19 us per launch for their start and their rows on the window and the surface).
// Measured, LDS against streaming, depth-only: 1 solve of 512^2 (81 tiles) 26 / 36,
// 30 of 200 x 150 (360) 36 / 48, 60 of 300 x 90 (720) 60 / 63, 60 of four uneven
// grids (915) 69 / 80, 15 of 512^2 (1215) 84 / 84, 120 of 128^2 (1080) 66 / 63, 60
// of 384^2 (2940) 178 / 134, 105 of 256^2 (2625) 144 / 119; nodal: 1 of 512^2 (144)
// 24 / 41, 30 of 200 x 150 (600) 50 / 58, 30 of 300 x 200 (1080) 76 / 82, 120 of
// 128^2 (1440) 85 / 77, 90 of 300 x 200 (3240) 169 / 147.
int small_launch_variant(int v, const std::vector<StreamLoad>& loads) {
    const int lds = kVariants[v].medium_kind == EIG_MEDIUM_NODAL ? 27 : 26;
    const int tw = kVariants[lds].cols, th = kVariants[lds].rows;
    int64_t tiles = 0;
    for (const auto& l : loads)
        tiles += l.solves * ((l.nx + tw - 1) / tw) * ((l.nz - 1 + th - 1) / th);
    // past 16 rounds of tiles the streaming kernel's rate is twice the other's
    if (tiles >= 16 * 512) return v;
    const double us = 16.0 + 26.0 * std::max(0.4, (double)tiles / 512.0);
    return us < stream_cut(v, loads).us ? lds : v;
}

}  // namespace eig
