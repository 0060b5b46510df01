// Phase regions and interface links of density fields, for the contact
// angles in two and three dimensions (arXiv 2505.22256, Sec. 3.2 and 3.5;
// the paper does not say how it measures the angle).
//
// Fluid nodes split into rho^e > 0 and rho^e <= 0.  Regions are connected
// along x, y and z links (4- or 6-connected, not across periodic seams), and
// only links between the largest region of each phase (the droplet and the
// fluid around it) are interface links, so pockets trapped under a droplet
// and satellite droplets do not bend the fit.
//
// What bounds it: a handful of passes over the nodes that are short beside
// one time step, so the work is kept to what needs memory.  The first pass
// turns the FP64 fields into two bits per node (64 nodes to a word, one
// wavefront lane per bit), and every later test of a node and its neighbours
// is a shift and a few logic operations on those words.  Labels start at the
// first node of each run inside a word, so that union-find only joins runs,
// one link per pair of runs that touch.  Sizes are summed per wavefront
// before they reach memory, and the interface links are compacted into a
// list, so that the fit reads a few hundred points and not the lattice.
// Measured, fields pass included: 0.25 ms on 400 x 400 (two thirds of it the
// fields pass and the copy back) and 2.4 ms on 200 x 200 x 280, where the
// joining, the links and the fit take 0.3 to 0.5 ms each.  With every node
// its own label and its own atomic increment of one counter, and each pass
// of the fit walking the whole lattice in one workgroup, these took 6.8 ms
// and 754 ms.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace lbm {

// The runs of one call: a batch (dims: nx, ny per run; offs: node offsets),
// or one lattice (dims null).
struct RunSet {
    const int *dims;
    const long long *offs;
    int nx, ny, nz;
};

struct RunGeom {
    int nx, ny, nz, N, groups;  // groups of 64 nodes
    long long off, g0;          // first node and first group in the concatenated arrays
};

__device__ __forceinline__ RunGeom run_geom(const RunSet &rs, int run)
{
    RunGeom g;
    g.nx = rs.dims ? rs.dims[2 * run] : rs.nx;
    g.ny = rs.dims ? rs.dims[2 * run + 1] : rs.ny;
    g.nz = rs.dims ? 1 : rs.nz;
    g.off = rs.dims ? rs.offs[run] : 0;
    g.N = g.nx * g.ny * g.nz;
    g.groups = (g.N + 63) / 64;
    g.g0 = g.off / 64 + run;
    return g;
}

// Scratch of the labelling, carved from one block of 4-byte words (8-byte
// aligned): keys of the chosen regions, class and link words, link counts,
// labels, and the link list, whose first words hold the region sizes until
// the regions are chosen.
struct RegionMem {
    unsigned long long *best;                         // [2 run + phase], size << 32 | ~root
    unsigned long long *fluid, *pos, *link[3];        // one word per group
    unsigned *count;                                  // interface links per block
    int *par, *cnt;                                   // labels, region sizes
    unsigned *list;                                   // ndir * node + dir; run r from word 2 off_r (one lattice: 0)
};

constexpr int REGION_BLOCKS = 512;  // blocks per run of the link passes, at most

inline RegionMem region_mem(void *base, long long nodes, int nruns, int ndir)
{
    RegionMem m;
    const long long tg = nodes / 64 + nruns;
    unsigned long long *q = (unsigned long long *)base;
    m.best = q;
    q += 2 * nruns;
    m.fluid = q;
    q += tg;
    m.pos = q;
    q += tg;
    for (int d = 0; d < 3; ++d) {
        m.link[d] = q;
        if (d < ndir) q += tg;
    }
    m.count = (unsigned *)q;
    m.par = (int *)(m.count + tg);
    m.list = (unsigned *)(m.par + nodes);
    m.cnt = (int *)m.list;
    return m;
}

// Bytes region_mem needs: (9 / 64 + 3) words per node and 13 per run in two
// dimensions, so the two velocity fields (4 words per node, at least 25
// nodes per run) hold it; in three dimensions (11 / 64 + 4) words per node.
inline size_t region_bytes(long long nodes, int nruns, int ndir)
{
    const long long tg = nodes / 64 + nruns;
    return (size_t)(2 * nruns + (2 + ndir) * tg) * 8 + (size_t)(tg + (1 + ndir) * nodes) * 4;
}

__device__ __forceinline__ bool phase_positive(const double *r1, const double *r2, long long a)
{
    return (r1[a] - r2[a]) / (r1[a] + r2[a]) > 0.0;
}

// Root of x.  Loads are device-coherent because other lanes link roots
// concurrently; parents only ever point to smaller indices, so the walk
// ends.  Every node passed is pointed at its grandparent on the way (it
// stays in its tree, and a node that has a parent never becomes a root
// again), which keeps the chains of runs down a column short.
__device__ __forceinline__ int cc_find(int *par, int x)
{
    int p = __hip_atomic_load(par + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (p != x) {
        const int g = __hip_atomic_load(par + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (g == p) return p;
        __hip_atomic_store(par + x, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = g;
        p = __hip_atomic_load(par + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return x;
}

// Link the larger root under the smaller.  A failed compare-and-swap means
// another lane linked that root first; every retry follows a successful link
// elsewhere, so the loop ends.
__device__ __forceinline__ void cc_unite(int *par, int a, int b)
{
    for (;;) {
        const int ra = cc_find(par, a), rb = cc_find(par, b);
        if (ra == rb) return;
        const int hi = ra > rb ? ra : rb, lo = ra > rb ? rb : ra;
        if (atomicCAS(par + hi, hi, lo) == hi) return;
    }
}

// The 64 class bits of nodes 64 g + d .. 64 g + d + 63 (zero past the run).
__device__ __forceinline__ unsigned long long class_bits(const unsigned long long *w, const RunGeom &q, int g, int d)
{
    const int i = g + (d >> 6), s = d & 63;
    unsigned long long v = i < q.groups ? w[q.g0 + i] >> s : 0ull;
    if (s && i + 1 < q.groups) v |= w[q.g0 + i + 1] << (64 - s);
    return v;
}

// Links of group g in direction d (1: x, 2: y, 3: z) between fluid nodes of
// the same phase (`same`) or of different phases.
__device__ __forceinline__ unsigned long long link_bits(const RunGeom &q, const unsigned long long *fluid,
                                                        const unsigned long long *pos, int g, int step, bool inside,
                                                        bool same)
{
    const unsigned long long in = __ballot(inside);
    const unsigned long long f = fluid[q.g0 + g] & class_bits(fluid, q, g, step) & in;
    const unsigned long long p = pos[q.g0 + g] ^ class_bits(pos, q, g, step);
    return f & (same ? ~p : p);
}

// Whether node a has a neighbour at +x, +y, +z inside the lattice.
__device__ __forceinline__ void has_next(const RunGeom &q, int a, bool &x, bool &y, bool &z)
{
    const unsigned r = (unsigned)a / (unsigned)q.nx, zz = r / (unsigned)q.ny;
    x = (int)((unsigned)a - r * (unsigned)q.nx) + 1 < q.nx;
    y = (int)(r - zz * (unsigned)q.ny) + 1 < q.ny;
    z = (int)zz + 1 < q.nz;
}

// Class words, labels (the first node of the run inside the word) and zero
// sizes.  Grid of all labelling kernels: blockIdx.y = run, the wavefronts of
// blockIdx.x stride over the run's groups.
static __global__ void __launch_bounds__(256)
k_cc_class(RunSet rs, RegionMem m, const double *__restrict__ rho1, const double *__restrict__ rho2,
           const uint8_t *__restrict__ solid)
{
    const int run = blockIdx.y, lane = threadIdx.x & 63;
    const RunGeom q = run_geom(rs, run);
    if (blockIdx.x == 0 && threadIdx.x < 2) m.best[2 * run + threadIdx.x] = 0ull;
    for (int g = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)); g < q.groups; g += (int)gridDim.x * 4) {
        const int a = g * 64 + lane;
        const bool fl = a < q.N && !solid[q.off + a];
        const bool ph = fl && phase_positive(rho1 + q.off, rho2 + q.off, a);
        const unsigned long long f = __ballot(fl), p = __ballot(ph);
        const bool row0 = (unsigned)a % (unsigned)q.nx == 0;
        const bool start = lane == 0 || row0 || !((f >> (lane - 1)) & 1) || (((p >> (lane - 1)) & 1) != (ph ? 1u : 0u));
        const unsigned long long st = __ballot(start);
        if (a < q.N) {
            // the last run start at or before this lane
            const unsigned long long upto = st & (~0ull >> (63 - lane));
            m.par[q.off + a] = fl ? g * 64 + 63 - __clzll((long long)upto) : -1;
            m.cnt[2 * q.off + a] = 0;
        }
        if (lane == 0) {
            m.fluid[q.g0 + g] = f;
            m.pos[q.g0 + g] = p;
        }
    }
}

// Join the runs: along x only across words; along y and z one link per pair
// of runs that touch (a link whose left neighbour is the same pair's is
// implied by it).
static __global__ void __launch_bounds__(256) k_cc_hook(RunSet rs, RegionMem m)
{
    const int lane = threadIdx.x & 63;
    const RunGeom q = run_geom(rs, blockIdx.y);
    int *par = m.par + q.off;
    for (int g = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)); g < q.groups; g += (int)gridDim.x * 4) {
        const int a = g * 64 + lane, plane = q.nx * q.ny;
        bool ix, iy, iz;
        has_next(q, a, ix, iy, iz);
        const unsigned long long lx = link_bits(q, m.fluid, m.pos, g, 1, ix, true);
        const unsigned long long ly = link_bits(q, m.fluid, m.pos, g, q.nx, iy, true);
        const unsigned long long lz = q.nz > 1 ? link_bits(q, m.fluid, m.pos, g, plane, iz, true) : 0ull;
        if (lane == 63 && (lx >> 63)) cc_unite(par, a, a + 1);
        if (((ly & ~((lx & ly) << 1)) >> lane) & 1) cc_unite(par, a, a + q.nx);
        if (((lz & ~((lx & lz) << 1)) >> lane) & 1) cc_unite(par, a, a + plane);
    }
}

// After joining: par[a] <- root(a), and the region sizes.  Each wavefront
// takes a contiguous part of the run and keeps the sizes of the two regions
// it met last in registers.
static __global__ void __launch_bounds__(256) k_cc_count(RunSet rs, RegionMem m)
{
    const int lane = threadIdx.x & 63, wave = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)), nw = (int)gridDim.x * 4;
    const RunGeom q = run_geom(rs, blockIdx.y);
    int *par = m.par + q.off, *cnt = m.cnt + 2 * q.off;
    const int span = (q.groups + nw - 1) / nw, g1 = min(q.groups, (wave + 1) * span);
    int ra = -1, na = 0, rb = -1, nb = 0;  // the region met last and the one before it
    for (int g = wave * span; g < g1; ++g) {
        const int a = g * 64 + lane;
        int r = -1;
        if (a < q.N && (r = par[a]) >= 0) {
            for (int n = par[r]; n != r; n = par[r]) r = n;
            par[a] = r;
        }
        unsigned long long todo = __ballot(r >= 0);
        while (todo) {
            const int r0 = __shfl(r, __ffsll(todo) - 1, 64);
            const unsigned long long same = __ballot(r == r0);
            todo &= ~same;
            int n = __popcll(same);
            if (r0 != ra) {
                if (r0 == rb) {
                    n += nb;
                } else if (rb >= 0 && lane == 0) {
                    atomicAdd(cnt + rb, nb);
                }
                rb = ra;
                nb = na;
                ra = r0;
                na = 0;
            }
            na += n;
        }
    }
    if (lane == 0) {
        if (ra >= 0) atomicAdd(cnt + ra, na);
        if (rb >= 0) atomicAdd(cnt + rb, nb);
    }
}

// best[2 run + phase]: size and root of the largest region of that phase
// (ties: the smaller root), 0 when the phase is absent.
static __global__ void __launch_bounds__(256) k_cc_pick(RunSet rs, RegionMem m)
{
    const int run = blockIdx.y, lane = threadIdx.x & 63;
    const RunGeom q = run_geom(rs, run);
    const int *par = m.par + q.off, *cnt = m.cnt + 2 * q.off;
    for (int g = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)); g < q.groups; g += (int)gridDim.x * 4) {
        const int a = g * 64 + lane;
        if (a >= q.N || par[a] != a) continue;
        const int ph = (int)((m.pos[q.g0 + g] >> lane) & 1);
        const unsigned long long k = ((unsigned long long)(unsigned)cnt[a] << 32) | (0xffffffffull - (unsigned long long)a);
        atomicMax(m.best + 2 * run + ph, k);
    }
}

__device__ __forceinline__ int best_root(unsigned long long key)
{
    return key ? (int)(0xffffffffull - (key & 0xffffffffull)) : -1;
}

// Part of a run's groups that wavefront `w` of block b of nb takes.
__device__ __forceinline__ void link_span(const RunGeom &q, int b, int nb, int w, int &g0, int &g1)
{
    const int span = (q.groups + nb - 1) / nb, part = (span + 3) / 4;
    g0 = min(q.groups, b * span + min(span, w * part));
    g1 = min(q.groups, b * span + min(span, (w + 1) * part));
}

// Blocks per run that the link passes use (every run at most its groups).
__device__ __forceinline__ int link_blocks(const RunGeom &q) { return min((int)gridDim.x, q.groups); }

// Interface links: words of those links between the two chosen regions
// whose interpolated point `pt` accepts, and their number per block.
template <int ND, class Point>
__device__ void links_of_run(const RunSet &rs, const RegionMem &m, const Point &pt)
{
    __shared__ unsigned wsum[4];
    const int run = blockIdx.y, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const RunGeom q = run_geom(rs, run);
    const int nb = link_blocks(q);
    if ((int)blockIdx.x >= nb) return;
    const int *par = m.par + q.off;
    const int best[2] = {best_root(m.best[2 * run]), best_root(m.best[2 * run + 1])};
    int g0, g1;
    link_span(q, blockIdx.x, nb, w, g0, g1);
    unsigned n = 0;
    for (int g = g0; g < g1; ++g) {
        const int a = g * 64 + lane;
        bool in[3];
        has_next(q, a, in[0], in[1], in[2]);
        const int step[3] = {1, q.nx, q.nx * q.ny};
        const unsigned long long pw = m.pos[q.g0 + g];
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            const unsigned long long c = link_bits(q, m.fluid, m.pos, g, step[d], in[d], false);
            bool ok = (c >> lane) & 1;
            if (ok) {
                const int ph = (int)((pw >> lane) & 1);
                ok = par[a] == best[ph] && par[a + step[d]] == best[ph ^ 1] && pt.accept(q, a, d);
            }
            const unsigned long long l = __ballot(ok);
            if (lane == 0) m.link[d][q.g0 + g] = l;
            n += __popcll(l);
        }
    }
    if (lane == 0) wsum[w] = n;
    __syncthreads();
    if (threadIdx.x == 0) m.count[q.g0 + blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// The links as a list (ndir * node + dir) in a fixed order: block by block,
// wavefront by wavefront, word by word.
template <int ND>
static __global__ void __launch_bounds__(256) k_cc_list(RunSet rs, RegionMem m)
{
    __shared__ unsigned wsum[4], before[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const RunGeom q = run_geom(rs, blockIdx.y);
    const int nb = link_blocks(q);
    if ((int)blockIdx.x >= nb) return;
    int g0, g1;
    link_span(q, blockIdx.x, nb, w, g0, g1);
    // links before this block, and those of this block's wavefronts
    unsigned pre = 0, n = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += 256) pre += m.count[q.g0 + b];
    for (int g = g0 + lane; g < g1; g += 64)
#pragma unroll
        for (int d = 0; d < ND; ++d) n += __popcll(m.link[d][q.g0 + g]);
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        pre += __shfl_xor(pre, s, 64);
        n += __shfl_xor(n, s, 64);
    }
    if (lane == 0) {
        before[w] = pre;
        wsum[w] = n;
    }
    __syncthreads();
    unsigned at = before[0] + before[1] + before[2] + before[3];
    for (int k = 0; k < w; ++k) at += wsum[k];
    if (n == 0) return;
    unsigned *list = m.list + 2 * q.off;
    for (int g = g0; g < g1; ++g) {
        const int a = g * 64 + lane;
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            const unsigned long long l = m.link[d][q.g0 + g];
            if ((l >> lane) & 1) list[at + __popcll(l & ((1ull << lane) - 1))] = (unsigned)ND * (unsigned)a + (unsigned)d;
            at += __popcll(l);
        }
    }
}

// Number of links of a run, for the workgroup that fits them (all threads).
template <int NT> __device__ unsigned link_total(const RunGeom &q, const RegionMem &m, int nb)
{
    __shared__ unsigned part[NT / 64];
    unsigned s = 0;
    for (int b = threadIdx.x; b < min(nb, q.groups); b += NT) s += m.count[q.g0 + b];
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) s += __shfl_xor(s, k, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    unsigned tot = 0;
    for (int k = 0; k < NT / 64; ++k) tot += part[k];
    return tot;
}

// Sum of v over the workgroup in a fixed order (a butterfly inside each
// wavefront, then the wavefronts in order); every thread gets the result.
template <int NV, int NT> __device__ void block_sum(double (&v)[NV], double (*sh)[NT / 64])
{
#pragma unroll
    for (int k = 0; k < NV; ++k)
        for (int s = 32; s > 0; s >>= 1) v[k] += __shfl_xor(v[k], s, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < NV; ++k) sh[k][threadIdx.x >> 6] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k] = sh[k][0];
        for (int w = 1; w < NT / 64; ++w) v[k] += sh[k][w];
    }
}

// Blocks of the labelling passes for runs of up to max_nodes nodes.
inline dim3 region_grid(long long max_nodes, int nruns)
{
    long long bx = (max_nodes + 255) / 256;
    const long long cap = nruns > 16 ? 64 : nruns > 1 ? 256 : 2048;
    return dim3((unsigned)(bx > cap ? cap : bx < 1 ? 1 : bx), (unsigned)nruns);
}
inline dim3 link_grid(long long max_nodes, int nruns)
{
    long long bx = (max_nodes + 255) / 256;
    const long long cap = nruns > 16 ? 32 : REGION_BLOCKS;
    return dim3((unsigned)(bx > cap ? cap : bx < 1 ? 1 : bx), (unsigned)nruns);
}

// Label the phase regions and choose the largest of each phase.
static inline hipError_t launch_regions(hipStream_t st, const RunSet &rs, int nruns, long long max_nodes,
                                        const double *rho1, const double *rho2, const uint8_t *solid, const RegionMem &m)
{
    const dim3 grid = region_grid(max_nodes, nruns);
    hipLaunchKernelGGL(k_cc_class, grid, dim3(256), 0, st, rs, m, rho1, rho2, solid);
    hipLaunchKernelGGL(k_cc_hook, grid, dim3(256), 0, st, rs, m);
    hipLaunchKernelGGL(k_cc_count, grid, dim3(256), 0, st, rs, m);
    hipLaunchKernelGGL(k_cc_pick, grid, dim3(256), 0, st, rs, m);
    return hipGetLastError();
}

}  // namespace lbm
