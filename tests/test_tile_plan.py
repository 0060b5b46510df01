"""The rules that choose tiles (csrc/lbm_plan.hpp) are plain arithmetic on sizes:
compiled for the host and run over lattices of every shape, down to a few rows
and up to the widest that lbm_create takes, every storage, closed and open, on
whole and partitioned GPUs.  A segment has at least one row and no more than the
lattice, and the widest strips are those the kernels are compiled for."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++") or shutil.which("c++")

SWEEP = r"""
#include "lbm_plan.hpp"
#include <cstdio>
using namespace lbm_host;

// the defaults of lbm_create, by storage, closed and open
static Tile dflt(int storage, bool bnd)
{
    const unsigned two = SCHED_TWO_STEP | SCHED_BANDS;
    if (storage == LBM_F32) return {bnd ? 64 : 128, 24, two};
    if (storage == LBM_F64) return {64, 48, two};
    return bnd ? Tile{128, 16, SCHED_BANDS} : Tile{64, 32, two};
}

int main()
{
    long long n = 0, bad = 0;
    const int elem[4] = {8, 4, 2, 2};
    for (int cus : {256, 128, 64, 32})
        for (int storage = 0; storage < 4; ++storage)
            for (int bnd = 0; bnd < 2; ++bnd)
                for (double tau : {1.0, 0.85})
                    for (int ny : {5, 7, 8, 12, 16, 20, 23, 24, 25, 31, 32, 33, 40, 48, 49, 64, 100, 333, 2048, 60000})
                        for (long long nx = 5; nx * ny * 9 * elem[storage] < (1ll << 32); nx += 1 + nx / 37)
                            for (int two = 0; two < 2; ++two) {
                                const PlanInput l = {(int)nx, ny, storage, tau, bnd != 0, cus};
                                const Tile t = march_tile(l, dflt(storage, bnd), two);
                                const bool ok = t.seg_rows >= 1 && t.seg_rows <= ny &&
                                                (t.block == 64 || t.block == 128 || t.block == 256) &&
                                                !(storage == LBM_F64 && t.block == 256 && (t.sched & SCHED_TWO_STEP));
                                ++n;
                                // a recording step runs alone, and not in narrow strips
                                const Tile r = march_tile(l, dflt(storage, bnd), false, true);
                                const bool rok = r.seg_rows >= 1 && r.seg_rows <= ny &&
                                                 (storage == LBM_F64 || (!(r.sched & SCHED_TWO_STEP) && r.block >= 128));
                                if (!rok && bad++ < 5)
                                    std::printf("%lld x %d storage %d bnd %d tau %g cus %d recording: %d %d %u\n", nx, ny,
                                                storage, bnd, tau, cus, r.block, r.seg_rows, r.sched);
                                if (!ok && bad++ < 5)
                                    std::printf("%lld x %d storage %d bnd %d tau %g cus %d: %d %d %u\n", nx, ny, storage,
                                                bnd, tau, cus, t.block, t.seg_rows, t.sched);
                            }
    // bricks: a core is left of every region, small lattices run in them, and wide ones
    // that strips step faster several at a time do not
    for (int cus : {256, 64})
        for (int storage = 0; storage < 4; ++storage)
            for (int bnd = 0; bnd < 2; ++bnd)
                for (int ny : {5, 28, 100, 341, 1000})
                    for (long long nx = 5; nx < 200000; nx += 1 + nx / 29) {
                        const BrickPlan b = brick_plan({(int)nx, ny, storage, 0.85, bnd != 0, cus});
                        const bool ok = b.steps ? b.steps <= 4 && brick_core(brick_rx(b.region), b.steps) > 0 &&
                                                      brick_core(brick_ry(b.region), b.steps) > 0 && nx * ny < 1200000 &&
                                                      (b.region == 0 || (b.region == 1 && !(storage == LBM_F64 && bnd)))
                                                : nx * ny > 500000;
                        ++n;
                        if (!ok && bad++ < 5)
                            std::printf("bricks: %lld x %d storage %d bnd %d cus %d: %d %d\n", nx, ny, storage, bnd, cus,
                                        b.region, b.steps);
                    }
    const int wide[][4] = {{2660, 221, 1, 0}, {2049, 342, 1, 0}, {2898, 241, 0, 0}, {2569, 428, 0, 0},
                           {1049, 1049, 0, 1}, {2939, 244, 2, 1}, {1000, 1000, 3, 1}};
    for (auto &w : wide) {
        ++n;
        if (brick_plan({w[0], w[1], w[2], 0.85, w[3] != 0, 256}).steps && bad++ < 5)
            std::printf("%d x %d storage %d bnd %d runs in bricks\n", w[0], w[1], w[2], w[3]);
    }
    // batches: in turn at the same wavefronts per SIMD whatever the GPU's size
    for (int cus : {256, 128, 64, 32})
        for (int storage = 0; storage < 4; ++storage)
            for (int per_simd = 0; per_simd < 20; ++per_simd) {
                const bool turn = storage < 2 ? per_simd >= 2 : per_simd >= 4 && per_simd < 16;
                const int items = 4 * cus * per_simd + 3, u = units_per_xcd(storage, items, 64, cus);
                ++n;
                if (u != (turn ? 0 : (items + 7) / 8) && bad++ < 5)
                    std::printf("batch: storage %d cus %d items %d: %d in a row\n", storage, cus, items, u);
            }
    std::printf("%lld lattices, %lld bad\n", n, bad);
    return bad ? 1 : 0;
}
"""


@pytest.mark.skipif(CXX is None, reason="no host compiler")
def test_tiles_of_every_lattice(tmp_path):
    src, exe = tmp_path / "sweep.cpp", tmp_path / "sweep"
    src.write_text(SWEEP)
    subprocess.run([CXX, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2505_22256_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)
