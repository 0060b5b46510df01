// Contact angle of a droplet on a 3-D lattice (FP64, on the device): phase
// regions, interface points of rho^e = 0 along x, y and z links, sphere fit
// (arXiv 2505.22256, Sec. 3.5; the paper does not state how it measures the
// angle).  Reads the rho1 / rho2 fields of the 3-D fields pass.
#pragma once

#include "lbm_contact.hpp"

namespace lbm3 {

struct Wall3 {
    int kind;  // 0: flat wall z = w[0]; 1: sphere of centre w[0..2], surface radius w[3]
    double w[4];
};

// The point of the link from node a in direction dir (x, y, z) where rho^e
// changes sign (linear interpolation), and its distance from the wall.
__device__ __forceinline__ void link_point3(int nx, int ny, const double *r1, const double *r2, const Wall3 &wd, int a,
                                            int dir, double (&pt)[3], double &dist)
{
    const unsigned r = (unsigned)a / (unsigned)nx, z = r / (unsigned)ny;
    const unsigned x = (unsigned)a - r * (unsigned)nx, y = r - z * (unsigned)ny;
    const int b = a + (dir == 0 ? 1 : dir == 1 ? nx : nx * ny);
    const double ra = (r1[a] - r2[a]) / (r1[a] + r2[a]);
    const double rb = (r1[b] - r2[b]) / (r1[b] + r2[b]);
    const double t = ra / (ra - rb);
    // (t times 0 rather than a choice: a non-finite t rejects the point)
    pt[0] = x + t * (dir == 0);
    pt[1] = y + t * (dir == 1);
    pt[2] = z + t * (dir == 2);
    if (wd.kind == 0) {
        dist = pt[2] - wd.w[0];
    } else {
        const double dx = pt[0] - wd.w[0], dy = pt[1] - wd.w[1], dz = pt[2] - wd.w[2];
        dist = __builtin_sqrt(dx * dx + dy * dy + dz * dz) - wd.w[3];
    }
}

// Interface links whose point is at least 3 lattice units from the wall.
struct AwayFromWall3 {
    const double *r1, *r2;
    Wall3 wd;
    __device__ __forceinline__ bool accept(const lbm::RunGeom &q, int a, int dir) const
    {
        double pt[3], dist;
        link_point3(q.nx, q.ny, r1, r2, wd, a, dir, pt, dist);
        return dist >= 3.0;
    }
};

static __global__ void __launch_bounds__(256)
k_cc3_links(lbm::RunSet rs, lbm::RegionMem m, const double *__restrict__ r1, const double *__restrict__ r2, Wall3 wd)
{
    const AwayFromWall3 pt{r1, r2, wd};
    lbm::links_of_run<3>(rs, m, pt);
}

// One workgroup of 1024 threads over the list of interface links: out = theta
// (deg), centre (3), radius, number of points, status (0 ok, 1 too few
// points, 2 fit failed).  Every pass sums the points in a fixed order, so the
// result is deterministic.
static __global__ void __launch_bounds__(1024)
k_contact3(lbm::RunSet rs, lbm::RegionMem mem, int nblocks, const double *__restrict__ r1,
           const double *__restrict__ r2, Wall3 wd, double *out)
{
    constexpr int NT = 1024;
    __shared__ double sh[14][NT / 64];
    __shared__ double prm[4];
    __shared__ int flag;
    const int t = threadIdx.x;
    const lbm::RunGeom q = lbm::run_geom(rs, 0);
    const unsigned *list = mem.list;
    const int M = (int)lbm::link_total<NT>(q, mem, nblocks);
    auto point = [&](int i, double (&pt)[3]) {
        const unsigned l = list[i];
        double dist;
        link_point3(q.nx, q.ny, r1, r2, wd, (int)(l / 3u), (int)(l % 3u), pt, dist);
    };
    const lbm::FitPoints<3, NT, 4, decltype(point)> points(M, point);
    double m[3] = {0, 0, 0};
    points.each([&](const double (&p)[3]) {
        for (int d = 0; d < 3; ++d) m[d] += p[d];
    });
    lbm::block_sum<3, NT>(m, sh);
    if (M < 4) {
        if (t == 0) {
            for (int k = 0; k < 5; ++k) out[k] = 0.0;
            out[5] = M;
            out[6] = 1;
        }
        return;
    }
    const double mx = m[0] / M, my = m[1] / M, mz = m[2] / M;
    // algebraic fit x^2 + y^2 + z^2 + D x + E y + F z + G = 0 on centred points
    double k14[14] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    points.each([&](const double (&p)[3]) {
        const double u = p[0] - mx, v = p[1] - my, w = p[2] - mz, s = u * u + v * v + w * w;
        k14[0] += u * u; k14[1] += u * v; k14[2] += u * w; k14[3] += u;
        k14[4] += v * v; k14[5] += v * w; k14[6] += v;
        k14[7] += w * w; k14[8] += w;
        k14[9] += 1.0;
        k14[10] -= u * s; k14[11] -= v * s; k14[12] -= w * s; k14[13] -= s;
    });
    lbm::block_sum<14, NT>(k14, sh);
    if (t == 0) {
        double A[4][5] = {{k14[0], k14[1], k14[2], k14[3], k14[10]}, {k14[1], k14[4], k14[5], k14[6], k14[11]},
                          {k14[2], k14[5], k14[7], k14[8], k14[12]}, {k14[3], k14[6], k14[8], k14[9], k14[13]}};
        double D[4] = {0, 0, 0, 0};
        flag = lbm::solve_linear<4>(A, D) ? 0 : 2;
        const double r2v = (D[0] * D[0] + D[1] * D[1] + D[2] * D[2]) / 4.0 - D[3];
        if (!(r2v > 0.0)) flag = 2;
        prm[0] = mx - D[0] / 2.0;
        prm[1] = my - D[1] / 2.0;
        prm[2] = mz - D[2] / 2.0;
        prm[3] = flag ? 0.0 : __builtin_sqrt(r2v);
    }
    __syncthreads();
    if (flag) {
        if (t == 0) {
            for (int k = 0; k < 5; ++k) out[k] = 0.0;
            out[5] = M;
            out[6] = 2;
        }
        return;
    }
    // Gauss-Newton on the geometric distances
    for (int it = 0; it < 100; ++it) {
        const double cx = prm[0], cy = prm[1], cz = prm[2], rr = prm[3];
        double g14[14] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        points.each([&](const double (&p)[3]) {
            const double dx = p[0] - cx, dy = p[1] - cy, dz = p[2] - cz;
            const double d = __builtin_sqrt(dx * dx + dy * dy + dz * dz);
            if (d == 0.0) return;
            const double J[4] = {-dx / d, -dy / d, -dz / d, -1.0};
            const double res = d - rr;
            g14[0] += J[0] * J[0]; g14[1] += J[0] * J[1]; g14[2] += J[0] * J[2]; g14[3] += J[0] * J[3];
            g14[4] += J[1] * J[1]; g14[5] += J[1] * J[2]; g14[6] += J[1] * J[3];
            g14[7] += J[2] * J[2]; g14[8] += J[2] * J[3];
            g14[9] += J[3] * J[3];
            g14[10] -= J[0] * res; g14[11] -= J[1] * res; g14[12] -= J[2] * res; g14[13] -= J[3] * res;
        });
        lbm::block_sum<14, NT>(g14, sh);
        if (t == 0) {
            double A[4][5] = {{g14[0], g14[1], g14[2], g14[3], g14[10]}, {g14[1], g14[4], g14[5], g14[6], g14[11]},
                              {g14[2], g14[5], g14[7], g14[8], g14[12]}, {g14[3], g14[6], g14[8], g14[9], g14[13]}};
            double dl[4];
            flag = 1;
            if (lbm::solve_linear<4>(A, dl)) {
                for (int k = 0; k < 4; ++k) prm[k] += dl[k];
                const double step = __builtin_fabs(dl[0]) + __builtin_fabs(dl[1]) + __builtin_fabs(dl[2]) +
                                    __builtin_fabs(dl[3]);
                flag = step <= 1e-13 * (1.0 + __builtin_fabs(prm[3])) ? 1 : 0;
            }
        }
        __syncthreads();
        if (flag) break;
    }
    if (t == 0) {
        double cth;
        if (wd.kind == 0) {
            cth = -(prm[2] - wd.w[0]) / prm[3];
        } else {
            const double dx = prm[0] - wd.w[0], dy = prm[1] - wd.w[1], dz = prm[2] - wd.w[2];
            cth = (wd.w[3] * wd.w[3] + prm[3] * prm[3] - (dx * dx + dy * dy + dz * dz)) / (2.0 * wd.w[3] * prm[3]);
        }
        cth = cth > 1.0 ? 1.0 : (cth < -1.0 ? -1.0 : cth);
        out[0] = acos(cth) * (180.0 / 3.14159265358979323846);
        for (int k = 0; k < 4; ++k) out[1 + k] = prm[k];
        out[5] = M;
        out[6] = 0;
    }
}

}  // namespace lbm3
