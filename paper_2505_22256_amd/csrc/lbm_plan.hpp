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
// instead of 18 (FP32 119 registers against 203, FP64 211 against 256 and 119
// accumulation registers), so more wavefronts share a SIMD and wider strips
// pay.  16384 x 2048 channel, us per step, general kernels in the default tile
// / relaxation time 1 in that tile / in this one: FP32 737 / 702 / 653, FP16
// 604 / 520 / 509, BF16 613 / 520 / 505, FP64 (8192 x 2048) 820 / 774 / 702.
// With open edges (us per step alone / with three lattices at a time, 8192 x
// 1024): FP32 in 128 threads 233 / 174, in 256 226 / 162, FP64 - / 467 and 419;
// 16-bit storage, whose default is one step in 128 threads, 232 / 185, two steps
// in 64 threads and 24 rows 234 / 155, one step in 256 threads and 12 rows 210 /
// 167.  Two steps need several rounds of wavefronts to be the better both ways
// (9000 x 1400 305 / 229 against 305 / 253, 4000 x 1000 155 / 77 against 117 / 83,
// 2000 x 600 103 / 41 against 66 / 31): three.
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
            const long long units = (long long)((l.nx + 53) / 54) * ((l.ny + 23) / 24);
            t = two && units >= 9LL * simds ? Tile{64, 24, SCHED_TWO_STEP | SCHED_BANDS} : Tile{256, 12, SCHED_BANDS};
        }
    }
    const int w = t.block - (t.sched & SCHED_TWO_STEP ? 10 : 4);
    const long long waves = (long long)((l.nx + w - 1) / w) * (t.block / 64);  // of one segment over the width
    long long segs = (l.ny + t.seg_rows - 1) / t.seg_rows;
    const long long least = half ? 2LL * simds : simds;
    // wavefronts of the two-step kernels without boundary code that the registers hold at once
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
