// Contact angle of a droplet from the density fields (FP64), for the
// single lattice and for every run of a batch (arXiv 2505.22256, Sec. 3.2;
// the paper does not say how it measures the angle).  Reads the rho1 / rho2
// fields that the fields pass of the step kernel writes.
#pragma once

#include "lbm_regions.hpp"

namespace lbm {

// ---------------------------------------------------------------------------
// Contact angle (FP64): interface points of rho^e = 0 along links, algebraic
// circle fit, Gauss-Newton refinement, angle with the wall.
// ---------------------------------------------------------------------------
struct WallDesc {
    int kind;
    double w0, w1, w2;
};

// The point of the link from node a in direction dir (0: x, 1: y) where
// rho^e changes sign (linear interpolation), and its distance from the wall.
__device__ __forceinline__ void link_point(int nx, const double *r1, const double *r2, const WallDesc &wd, int a, int dir,
                                           double &px, double &py, double &dist)
{
    const int y = (int)((unsigned)a / (unsigned)nx), x = a - y * nx;
    const int b = a + (dir == 0 ? 1 : nx);
    const double ra = (r1[a] - r2[a]) / (r1[a] + r2[a]);
    const double rb = (r1[b] - r2[b]) / (r1[b] + r2[b]);
    const double t = ra / (ra - rb);
    // (t times 0 rather than a choice: a non-finite t rejects the point)
    px = x + t * (dir == 0);
    py = y + t * (dir == 1);
    if (wd.kind == 0) {
        dist = py - wd.w0;
    } else {
        const double dx = px - wd.w0, dy = py - wd.w1;
        dist = __builtin_sqrt(dx * dx + dy * dy) - wd.w2;
    }
}

// Interface links whose point is at least 3 lattice units from the wall.
struct AwayFromWall2 {
    const double *r1, *r2;
    WallDesc wd;
    __device__ __forceinline__ bool accept(const RunGeom &q, int a, int dir) const
    {
        double px, py, dist;
        link_point(q.nx, r1 + q.off, r2 + q.off, wd, a, dir, px, py, dist);
        return dist >= 3.0;
    }
};

// walls: one per run, or null for one lattice with the wall `one`.
static __global__ void __launch_bounds__(256)
k_cc_links(RunSet rs, RegionMem m, const double *__restrict__ rho1, const double *__restrict__ rho2,
           const WallDesc *__restrict__ walls, WallDesc one)
{
    const AwayFromWall2 pt{rho1, rho2, walls ? walls[blockIdx.y] : one};
    links_of_run<2>(rs, m, pt);
}

// One workgroup per run, over the run's list of interface links.  out[run*6]:
// theta (deg), centre x, centre y, radius, number of points, status (0 ok, 1
// too few points, 2 fit failed).  Every pass sums the points in a fixed order,
// so the result is deterministic and the same alone and in a batch.
static __global__ void __launch_bounds__(256)
k_contact_angle(RunSet rs, RegionMem mem, int nblocks, const double *__restrict__ rho1, const double *__restrict__ rho2,
                const WallDesc *__restrict__ walls, WallDesc one, double *out)
{
    constexpr int NT = 256;
    __shared__ double sh[9][NT / 64];
    __shared__ double params[4];
    __shared__ int flag;
    const int run = blockIdx.x, t = threadIdx.x;
    const RunGeom q = run_geom(rs, run);
    const double *r1 = rho1 + q.off, *r2 = rho2 + q.off;
    const WallDesc wd = walls ? walls[run] : one;
    const unsigned *list = mem.list + 2 * q.off;
    const int M = (int)link_total<NT>(q, mem, nblocks);
    auto point = [&](int i, double (&pt)[2]) {
        const unsigned l = list[i];
        double dist;
        link_point(q.nx, r1, r2, wd, (int)(l >> 1), (int)(l & 1), pt[0], pt[1], dist);
    };
    const FitPoints<2, NT, 4, decltype(point)> points(M, point);

    // pass 1: mean
    double mn[2] = {0, 0};
    points.each([&](const double (&pt)[2]) {
        mn[0] += pt[0];
        mn[1] += pt[1];
    });
    block_sum<2, NT>(mn, sh);
    double *o = out + (long long)run * 6;
    if (M < 3) {
        if (t == 0) {
            o[0] = 0; o[1] = 0; o[2] = 0; o[3] = 0; o[4] = M; o[5] = 1;
        }
        return;
    }
    const double mx = mn[0] / M, my = mn[1] / M;
    // pass 2: algebraic fit on centred points
    double k9[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    points.each([&](const double (&pt)[2]) {
        const double u = pt[0] - mx, v = pt[1] - my, z = u * u + v * v;
        k9[0] += u * u; k9[1] += u * v; k9[2] += u;
        k9[3] += v * v; k9[4] += v;
        k9[5] += 1.0;
        k9[6] -= u * z; k9[7] -= v * z; k9[8] -= z;
    });
    block_sum<9, NT>(k9, sh);
    if (t == 0) {
        double A[3][4] = {{k9[0], k9[1], k9[2], k9[6]}, {k9[1], k9[3], k9[4], k9[7]}, {k9[2], k9[4], k9[5], k9[8]}};
        double DEF[3] = {0, 0, 0};
        flag = 0;
        if (!solve_linear<3>(A, DEF)) flag = 2;
        const double r2v = DEF[0] * DEF[0] / 4.0 + DEF[1] * DEF[1] / 4.0 - DEF[2];
        if (!(r2v > 0.0)) flag = 2;
        params[0] = mx - DEF[0] / 2.0;
        params[1] = my - DEF[1] / 2.0;
        params[2] = flag ? 0.0 : __builtin_sqrt(r2v);
    }
    __syncthreads();
    if (flag) {
        if (t == 0) {
            o[0] = 0; o[1] = 0; o[2] = 0; o[3] = 0; o[4] = M; o[5] = 2;
        }
        return;
    }
    // Gauss-Newton on the geometric distance
    for (int it = 0; it < 100; ++it) {
        const double a0 = params[0], b0 = params[1], rr = params[2];
        double g9[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        points.each([&](const double (&pt)[2]) {
            const double dx = pt[0] - a0, dy = pt[1] - b0;
            const double d = __builtin_sqrt(dx * dx + dy * dy);
            if (d == 0.0) return;
            const double J0 = -dx / d, J1 = -dy / d, J2 = -1.0, res = d - rr;
            g9[0] += J0 * J0; g9[1] += J0 * J1; g9[2] += J0 * J2;
            g9[3] += J1 * J1; g9[4] += J1 * J2; g9[5] += J2 * J2;
            g9[6] -= J0 * res; g9[7] -= J1 * res; g9[8] -= J2 * res;
        });
        block_sum<9, NT>(g9, sh);
        if (t == 0) {
            double A[3][4] = {{g9[0], g9[1], g9[2], g9[6]}, {g9[1], g9[3], g9[4], g9[7]}, {g9[2], g9[4], g9[5], g9[8]}};
            double dl[3];
            flag = 1;  // stop
            if (solve_linear<3>(A, dl)) {
                params[0] += dl[0];
                params[1] += dl[1];
                params[2] += dl[2];
                const double step = __builtin_fabs(dl[0]) + __builtin_fabs(dl[1]) + __builtin_fabs(dl[2]);
                flag = step <= 1e-13 * (1.0 + __builtin_fabs(params[2])) ? 1 : 0;
            }
        }
        __syncthreads();
        if (flag) break;
    }
    if (t == 0) {
        double cth;
        if (wd.kind == 0) {
            cth = -(params[1] - wd.w0) / params[2];
        } else {
            const double dx = params[0] - wd.w0, dy = params[1] - wd.w1;
            cth = (wd.w2 * wd.w2 + params[2] * params[2] - (dx * dx + dy * dy)) / (2.0 * wd.w2 * params[2]);
        }
        cth = cth > 1.0 ? 1.0 : (cth < -1.0 ? -1.0 : cth);
        o[0] = acos(cth) * (180.0 / 3.14159265358979323846);
        o[1] = params[0];
        o[2] = params[1];
        o[3] = params[2];
        o[4] = M;
        o[5] = 0;
    }
}

}  // namespace lbm
