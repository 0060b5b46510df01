// How a lattice is run: plain host arithmetic on its sizes, storage type and
// boundaries and on the device's compute units.  No HIP here, so that the rules
// can be checked over all of their range without a GPU.
#pragma once

#include "lbm.h"

#include <algorithm>

namespace lbm_host {

// Schedule bits of a tile (lbm_set_tile).
enum : unsigned { SCHED_ALIGN = 1u, SCHED_BANDS = 2u, SCHED_XCD_SLABS = 4u, SCHED_TWO_STEP = 8u, SCHED_REPULL = 16u };

struct Tile {
    int block, seg_rows;
    unsigned sched;
};

// What the rules look at.  bnd: open or moving boundaries are on; cus: compute
// units of the device.
struct PlanInput {
    int nx, ny, storage;
    double tau;
    bool bnd;
    int cus;
};

// The tile of the marching kernels where the caller has set or tuned none: the
// storage's default `t` with two changes.
//
// Relaxation time 1: the kernels keep 4 values per row and component pair
// instead of 18 (FP32 119 registers against 203, FP64 210 against 256 and 122
// accumulation registers), so more wavefronts share a SIMD and wider strips
// pay.  16384 x 2048 channel, us per step, general kernels in the default tile
// / relaxation time 1 in that tile / in this one: FP32 737 / 702 / 653, FP16
// 604 / 520 / 509, BF16 613 / 520 / 505, FP64 (8192 x 2048) 820 / 774 / 702.
// With open edges (us per step alone / with three lattices at a time, 8192 x
// 1024): FP32 in 128 threads 233 / 174, in 256 226 / 162, FP64 - / 467 and 419;
// 16-bit storage, whose default is one step in 128 threads, 232 / 185, takes one
// step in 256 threads and 12 rows, 201 / 165, or two in 64 threads and 24 rows, 206 /
// 145.  The two-step kernel holds three wavefronts per SIMD, 3072 at once, and two
// steps win three at a time from one such round on (BF16 6000 x 1000, 1.5 rounds, 153
// / 120 one step, 162 / 104 two; 4000 x 1000, 1.03, 108 / 81 and 136 / 72) but lose
// alone, less with every round and with a last one that is full (8192 x 1024 in 26
// rows, 1.98 rounds, 206 / 147; 9000 x 1400 in 24, 3.2, 268 / 213 against 288 / 246):
// the line lies where they win both ways, at three rounds.
//
// Rows: a segment is a serial march, so a lattice whose segments are fewer than
// the wavefronts that hide a march's latency (one per SIMD, two in the light
// 16-bit kernels) gets shorter ones, and one whose segments are just more than
// the wavefronts that the registers hold at once (by up to a quarter) gets taller
// ones, as many as fit: the second round would run nearly empty (a lattice so wide
// that one row of segments is more than that keeps the default's).  us per step
// alone / three at a time, the default's rows / these: too few, FP32 at tau 1 1500
// x 600 74 / 33, 55 / 26; at 0.85 78 / 33, 58 / 31; FP16 at 0.85 2000 x 700 99 /
// 41, 60 / 30; FP64 porous at 0.85 1800 x 800 172 / 93, 109 / 98; just too many,
// channels of 3001 x 1027 at 0.85 FP64 258 / 131, 208 / 128, FP32 113 / 63, 92 /
// 63, porous FP32 3200 x 1000 138 / 86, 95 / 84, FP64 2600 x 1100 305 / 178, 199 /
// 179.  More wavefronts than that shorten a lattice alone further, but the halo
// rows cost three at a time (FP32 at 0.85 2000 x 700 in 16 rows 60 / 46 against
// 79 / 44).
//
// A step that runs alone there (the first on given populations, the last of an
// odd number) takes the one-step tile in any case.
//
// A step that runs alone to record diagnostics (`record`) is a one-step launch in
// any case, which loses the fewest columns in wide strips.  In the strips of the
// fused steps it had become slower than it was, for more wavefronts in flight; us
// per step recording every step, at first / in those strips / in these: FP32 open
// 8192 x 1024 at 0.85 395 / 416 / 330, channel 8192 x 2048 718 / 708 / 629, porous
// 2048 x 1024 123 / 107 / 105; FP16 channel 506 / 513 / 418 (256 threads: 379, but
// porous 143 / 90 / 90 and 96), open at tau 1 281 / 285 / 244.  FP64 gained in its
// strips (open 438 / 426, porous 250 / 197, in 256 threads 351 and 219) and stays.
inline Tile march_tile(const PlanInput &l, Tile t, bool two, bool record = false)
{
    const bool half = l.storage == LBM_F16 || l.storage == LBM_BF16;
    const int simds = 4 * l.cus;
    if (record && l.storage != LBM_F64) {
        t = {half ? 128 : 256, 16, SCHED_BANDS};
    } else if (l.tau == 1.0) {
        if (l.storage == LBM_F64) {
            t = {128, l.bnd ? 32 : 24, t.sched};
        } else if (l.storage == LBM_F32) {
            t = {256, 24, t.sched};
        } else if (!l.bnd) {
            t = {128, 32, t.sched};
        } else {
            // (units of one wavefront)
            const long long units = (long long)((l.nx + 53) / 54) * ((l.ny + 23) / 24);
            t = two && units >= 3 * 3LL * simds ? Tile{64, 24, SCHED_TWO_STEP | SCHED_BANDS} : Tile{256, 12, SCHED_BANDS};
        }
    }
    const int w = t.block - (t.sched & SCHED_TWO_STEP ? 10 : 4);
    const long long waves = (long long)((l.nx + w - 1) / w) * (t.block / 64);  // of one segment over the width
    long long segs = (l.ny + t.seg_rows - 1) / t.seg_rows;
    const long long least = half ? 2LL * simds : simds;
    // wavefronts of the two-step kernels without boundary code that the registers hold at once: per
    // SIMD one in FP64, two in FP32 and three in 16-bit storage, one more at relaxation time 1
    const long long held = (long long)simds * ((l.storage == LBM_F64 ? 1 : half ? 3 : 2) + (l.tau == 1.0));
    if (waves * segs < least) segs = std::max<long long>(segs, std::min<long long>(least / waves, l.ny / 8));
    else if (!l.bnd && (t.sched & SCHED_TWO_STEP) && waves <= held && waves * segs > held && 4 * waves * segs <= 5 * held) segs = held / waves;
    t.seg_rows = (int)((l.ny + segs - 1) / segs);
    return t;
}

// Whether the steps of relaxation time 1 run in the kernels that keep momenta in
// this block.  One step per launch, FP32 and FP64 gain nothing by them (the state of
// a row is held for two rows only) and the wavefronts that the registers then admit
// crowd each other's halo out of the L2: channel of 4096 x 2048, us per step, general
// / momenta: FP64 (64, 16) in bands 648 / 681, (256, 16) 580 / 606, FP32 (256, 16)
// 318 / 329; only the porous 2048 x 1024 in FP64 gains, 214 / 203.  Nor do two FP32
// steps in 64-thread strips: channel in 24 rows 214 / 227, with open edges 136 / 146,
// porous 75 / 75.  16-bit storage gains everywhere (FP16 (256, 16) 202 / 194).
inline bool momenta_pay(int storage, int block, bool two)
{
    if (storage == LBM_F32) return two && block >= 128;
    return two || storage != LBM_F64;
}

// Regions of the brick kernel (lbm_brick.hpp), 32 x 16 and 32 x 32: nodes along x
// and y, one thread each, and what is left of a side after the halo of `steps` steps.
constexpr int brick_rx(int) { return 32; }
constexpr int brick_ry(int region) { return region == 0 ? 16 : 32; }
constexpr int brick_core(int side, int steps) { return side - 2 * (3 * steps - 1); }

// Bricks for the steps of a lattice: the region and the steps per launch, or no
// steps where marching strips is the choice.
//
// The line: a lattice stops being a latency chain when the strips fill the chip.
// One lattice on the GPU gains by bricks far beyond that; several stepped at the
// same time fill it together, and there the strips' smaller halo wins (bricks step
// up where they need another round of workgroups).  The line lies where bricks would
// lose, with three lattices, to the strips as they were before bricks came; wide
// channels with few wall nodes, the quickest in strips, decide it.  us per step alone
// / three at a time (per lattice), those strips / bricks / today's strips: FP32
// channels 1732 x 289 56 / 21.2, 17 / 14.6, 35 / 14.0; 2660 x 221 51 / 19.8, 20 /
// 22.2, -; 2049 x 342 60 / 24.6, 22 / 27.0, 41 / 17.4; open 837 x 836 84 / 33.6, 26 /
// 25.6, 62 / 25.0; FP64 channels 2792 x 232 117 / 44.5, 39 / 40.1, -; 2898 x 241 111
// / 41.9, 41 / 42.4, -; 2569 x 428 146 / 59.5, 71 / 64.5, 81 / 52.7; open 2191 x 365
// 219 / 78.8, 64 / 70.3, 96 / 48.7; 1049 x 1049 227 / 85.8, 98 / 91.8, 116 / 70.2;
// 16-bit closed 3746 x 312 82 / 35.3, 31 / 33.3, -; open 2877 x 239 65 / 28.6, 31 /
// 24.9, -; 2939 x 244 61 / 26.8, 34 / 27.9, -; 1000 x 1000 70 / 31.0, 40 / 34.3, 44 /
// 22.6.
//
// Steps per launch: while the bricks fit the chip's compute units once, a
// deeper halo costs only idle units, so the largest region takes the most
// steps that still fit (FP32 100 x 50: 4 steps 3.6, 2 steps 4.4, 1 step 6.7;
// 200 x 200: 3 steps 5.3, 2 6.5, 4 7.0, where 400 bricks no longer fit).
// Past that FP32 and the 16-bit storages take single steps in 32 x 16
// regions, which finish 66 % of their nodes (400 x 400 FP32: 7.9 against 8.7
// for two steps in 32 x 32; FP16 8.6 against 10.2); FP64, whose pulls are
// twice as long, and the boundary instances take two steps in 32 x 32
// (720 x 700 FP64 28.7 against 29.7, 26.6 against 30.2 with three lattices;
// 700 x 300 with open edges, FP32 13.2 against 15.2).  The FP64 boundary
// instance had no registers for 32 x 32 (204 B per lane spilled, 700 x 300 28.3
// us against 22.0) and stays in 32 x 16.
struct BrickPlan {
    int region, steps;
};

inline BrickPlan brick_plan(const PlanInput &l)
{
    const long long most = l.storage == LBM_F32   ? (l.bnd ? 11LL << 16 : 17LL << 15)
                           : l.storage == LBM_F64 ? (l.bnd ? 13LL << 16 : 10LL << 16)
                                                  : (l.bnd ? 21LL << 15 : 18LL << 16);
    if ((long long)l.nx * l.ny > most) return {0, 0};
    auto fits = [&](int region, int steps) {
        const int w = brick_core(brick_rx(region), steps), h = brick_core(brick_ry(region), steps);
        return (long long)((l.nx + w - 1) / w) * ((l.ny + h - 1) / h) <= l.cus;
    };
    if (l.storage == LBM_F64 && l.bnd) return {0, fits(0, 2) ? 2 : 1};
    for (int k = 4; k > 1; --k)
        if (fits(1, k)) return {1, k};
    return l.storage == LBM_F64 || l.bnd ? BrickPlan{1, 2} : BrickPlan{0, 1};
}

// Units of a batch's work list that each XCD takes in a row, 0 to deal them to the XCDs
// in turn.  Runs differ in their walls, and a wavefront at a wall takes longer:
// in one piece per XCD the XCD with the most walls finishes last, in turn they
// finish together but neighbours lose their common L2.  In turn pays from two
// wavefronts per SIMD on in FP32 and FP64, where 16-bit storage, quicker and so
// more dependent on its loads, wants four, and no more than sixteen, where the
// pieces are long enough to even out.  us per two steps, in a row / in turn: 48
// runs of 128 to 512 nodes a side FP32 (64 threads, 16 rows) 298 / 255, (128, 24)
// 315 / 264, FP16 267 / 257, (128, 24) 316 / 296, (64, 32) 282 / 287; 256 runs
// FP32 (64, 16) 1268 / 1215, BF16 1094 / 1113; 24 runs FP32 (128, 48) 252 / 261.
inline int units_per_xcd(int storage, int n_items, int block, int cus)
{
    const long long per_simd = (long long)n_items * (block / 64) / (4 * cus);
    const bool half = storage == LBM_F16 || storage == LBM_BF16;
    const bool turn = half ? per_simd >= 4 && per_simd < 16 : per_simd >= 2;
    return turn ? 0 : (n_items + 7) / 8;
}

}  // namespace lbm_host
