// Bricks: several fused time steps per launch for lattices too small to fill
// the chip with marching strips.
//
// A workgroup owns a brick of nodes, one thread per node of the brick and
// its halo, and advances it `steps` steps without leaving LDS: psi of the
// whole region for the stencil sums, and the post-collision values for the
// next step's pull.  Every step costs 3 nodes of halo on each side (1 for
// the pull and 2 for the stencil), the first pull comes from HBM and the last
// step writes HBM.
//
// What bounds it: a small lattice is a latency chain.  Marching strips gives
// 100 x 50 nodes 3 workgroups that pass 36 rows one after the other, 58 us
// per two steps (FP32); in bricks the same two steps are two pulls and two
// finishes of all nodes at once.  The price is the halo, computed again by
// every brick that touches it (a 32 x 32 region finishes 22 x 22 nodes of two
// steps, 10 x 10 of four), which idle compute units pay for; brick_plan (in
// lbm_plan.hpp) draws the line.
#pragma once

#include "lbm_kernels.hpp"

namespace lbm {

// psi around the node at index c of a region RX nodes wide.
template <class C, int RX> struct BrickPsi {
    const PsiPair<C> *psi;
    int c;
    __device__ __forceinline__ PsiPair<C> at(int dx, int dy) const { return psi[c + dy * RX + dx]; }
};

// Post-collision values of the region without its outer two nodes (no step
// finishes those): [component][direction][node].
template <int S, int RX, int RY> struct BrickPost {
    static constexpr int FX = RX - 4, FY = RY - 4, N = FX * FY;
    typename Traits<S>::raw_t v[2][9][N];
};

template <int S, int RX, int RY> struct BrickReload {
    static constexpr bool TOGETHER = false;
    const PopMem<S> &m;
    uint32_t off;  // byte offset of the node in HBM
    const BrickPost<S, RX, RY> *post;
    int c;  // its index in `post`
    bool first;
    __device__ __forceinline__ typename Traits<S>::raw_t operator()(int k, int i) const
    {
        return first ? pop_load<S>(m, k, i, off) : post->v[k][i][c];
    }
};

// The node's results: to LDS for the next step, or after the last one to HBM.
template <int S, int RX, int RY> struct BrickOut {
    const PopMem<S> &mw;
    uint32_t voff;
    BrickPost<S, RX, RY> *post;
    int c;
    bool last;
    __device__ __forceinline__ void solid() const
    {
        if (last) return;
#pragma unroll
        for (int i = 0; i < 9; ++i) post->v[0][i][c] = post->v[1][i][c] = Traits<S>::sentinel();
    }
    __device__ __forceinline__ void put(const typename Traits<S>::raw_t (&out)[2][9]) const
    {
        if (last) {
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                pop_store<S>(mw, 0, i, voff, out[0][i]);
                pop_store<S>(mw, 1, i, voff, out[1][i]);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                post->v[0][i][c] = out[0][i];
                post->v[1][i][c] = out[1][i];
            }
        }
    }
};

// Advance brick `unit` of the run `steps` steps.  The region is RX x RY
// nodes, the brick what is left of it after 2 + 3 (steps - 1) nodes of halo
// on each side.  Step s pulls the region without its outer 3 s nodes and
// finishes it without its outer 3 s + 2; region nodes past a periodic edge
// are images of the wrapped node, past a closed one they count as solid.
template <int S, int RX, int RY, int MODE>
__device__ __forceinline__ void process_brick(const KParams<typename Traits<S>::C> &p, int unit, int steps, int tiles_x,
                                              PsiPair<typename Traits<S>::C> *psi, BrickPost<S, RX, RY> *post)
{
    using T = Traits<S>;
    using C = typename T::C;
    using R = typename T::raw_t;
    constexpr bool BND = (MODE & M_BND) != 0;
    const int tid = threadIdx.x, lx = tid % RX, ly = tid / RX;
    const int halo = 3 * steps - 1, w = RX - 2 * halo, h = RY - 2 * halo;
    const int ty = unit / tiles_x, tx = unit - ty * tiles_x;
    const int gx = tx * w - halo + lx, gy = ty * h - halo + ly;
    const Axis cx0 = make_axis(gx, p.nx, p.flags & FL_PERIODIC_X);
    const Axis cx = BND ? open_axis(cx0, p) : cx0;
    const Axis ry = make_axis(gy, p.ny, p.flags & FL_PERIODIC_Y);
    const bool inside = cx.ok && ry.ok && ly < RY;
    const PopMem<S> mr = make_mem<S>(p.A, p.N);
    const PopMem<S> mw = make_mem<S>(p.B, p.N);
    const uint32_t off = (uint32_t)(ry.c * p.nx + cx.c) * (uint32_t)sizeof(R);
    const int c = (ly - 2) * BrickPost<S, RX, RY>::FX + lx - 2;  // in `post`, for the nodes that are finished
    // nodes between this one and the edge of the region
    const int edge = min(min(lx, RX - 1 - lx), min(ly, RY - 1 - ly));
    RedAcc none;
    StateOf<S, M_STORE | MODE> st;
    for (int s = 0; s < steps; ++s) {
        if (edge >= 3 * s) {
            RawRow<S> q;
            if (s == 0) {
                issue_node<S>(mr, p.nx, cx, ry, inside, q);
            } else {
                const bool outflow_col = BND && cx.okp && cx.p == cx.c;
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const int dx = qx(i) == -1 && outflow_col ? 0 : qx(i);
                    const int src = c - qy(i) * BrickPost<S, RX, RY>::FX - dx;
                    q.v[0][i] = post->v[0][i][src];
                    q.v[1][i] = post->v[1][i][src];
                }
            }
            const BrickReload<S, RX, RY> reload{mr, off, post, c, s == 0};
            C r1 = 0, r2 = 0;
            process_node_src<S, M_STORE | MODE>(p, reload, cx, ry, inside, q, st, r1, r2);
            PsiPair<C> ps;
            ps.a = (st.info & 256) ? lds_sentinel<C>() : r1;
            ps.b = (st.info & 256) ? lds_sentinel<C>() : r2;
            psi[tid] = ps;
        }
        __syncthreads();
        const bool last = s == steps - 1;
        // (after the last step only the brick's own nodes inside the lattice)
        if (edge >= 3 * s + 2 && (!last || (gx < p.nx && gy < p.ny))) {
            const BrickOut<S, RX, RY> sink{mw, off, post, c, last};
            finish_node<S, M_STORE | (MODE & (M_SR | M_BND | M_TAU1))>(p, cx, ry.c, ry.c, st, BrickPsi<C, RX>{psi, tid}, sink, none,
                                                              (unsigned)s);
        }
        if (!last) __syncthreads();
    }
}

// Grid: 8 * per_xcd workgroups of RX * RY threads (rounded up to wavefronts);
// workgroup b takes brick (b % 8) * per_xcd + b / 8, so each XCD works on a
// contiguous part of the lattice.
template <int S, int RX, int RY, int MODE>
__global__ void __launch_bounds__((RX * RY + 63) / 64 * 64)
k_brick(const KParams<typename Traits<S>::C> p, int steps, int tiles_x, int per_xcd)
{
    __shared__ PsiPair<typename Traits<S>::C> psi[(RX * RY + 63) / 64 * 64];
    __shared__ BrickPost<S, RX, RY> post;
    const int b = blockIdx.x, unit = (b & 7) * per_xcd + (b >> 3);
    if (unit < p.n_units) process_brick<S, RX, RY, MODE>(p, unit, steps, tiles_x, psi, &post);
}

}  // namespace lbm
