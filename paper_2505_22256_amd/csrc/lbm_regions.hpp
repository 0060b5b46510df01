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
// one link per pair of runs that touch.  It works band by band in LDS (a
// workgroup labels 4096 consecutive nodes and counts its regions' nodes there)
// and only links between bands, and one size per band and region, go through
// memory: joined there, every walk up a chain of labels is a round trip to the
// L2 per step, and a chain as long as the lattice is high.  The interface links
// are compacted into a list, so that the fit reads a few hundred points and
// not the lattice.
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

constexpr int BAND_GROUPS = 64, BAND_NODES = BAND_GROUPS * 64;

// The same inside one band of BAND_GROUPS class words: root of x, and joining.
__device__ __forceinline__ int band_find(int *par, int x)
{
    int p = __hip_atomic_load(par + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (p != x) {
        const int g = __hip_atomic_load(par + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (g == p) return p;
        __hip_atomic_store(par + x, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        x = g;
        p = __hip_atomic_load(par + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    return x;
}

__device__ __forceinline__ void band_unite(int *par, int a, int b)
{
    for (;;) {
        const int ra = band_find(par, a), rb = band_find(par, b);
        if (ra == rb) return;
        const int hi = ra > rb ? ra : rb, lo = ra > rb ? rb : ra;
        int want = hi;
        if (__hip_atomic_compare_exchange_strong(par + hi, &want, lo, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
            return;
    }
}

// Links in a band from the nodes of word g to those `step` further on, fluid
// and of one phase (zero past the band).
__device__ __forceinline__ unsigned long long band_links(const unsigned long long *fluid, const unsigned long long *pos,
                                                         int g, int step, bool inside)
{
    auto bits = [&](const unsigned long long *w) {
        const int i = g + (step >> 6), s = step & 63;
        unsigned long long v = i < BAND_GROUPS ? w[i] >> s : 0ull;
        if (s && i + 1 < BAND_GROUPS) v |= w[i + 1] << (64 - s);
        return v;
    };
    return fluid[g] & bits(fluid) & ~(pos[g] ^ bits(pos)) & __ballot(inside);
}

// Class words of one band per workgroup (blockIdx.x; blockIdx.y = run), its
// labels joined inside the band (par[a]: the first node of a's region in the
// band, -1 for solid nodes) and the sizes of those regions at their roots
// (zero at every other node).
static __global__ void __launch_bounds__(1024)
k_cc_band(RunSet rs, RegionMem m, const double *__restrict__ rho1, const double *__restrict__ rho2,
          const uint8_t *__restrict__ solid)
{
    __shared__ int par[BAND_NODES], cnt[BAND_NODES];
    __shared__ unsigned long long fluid[BAND_GROUPS], pos[BAND_GROUPS], starts[BAND_GROUPS];
    const int run = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const RunGeom q = run_geom(rs, run);
    if (blockIdx.x == 0 && threadIdx.x < 2) m.best[2 * run + threadIdx.x] = 0ull;
    const int gb = (int)blockIdx.x * BAND_GROUPS;  // first group of the band
    if (gb >= q.groups) return;
#pragma unroll
    for (int k = 0; k < BAND_GROUPS / 16; ++k) {
        const int g = wave + 16 * k, a = (gb + g) * 64 + lane;
        const bool fl = gb + g < q.groups && a < q.N && !solid[q.off + a];
        const bool ph = fl && phase_positive(rho1 + q.off, rho2 + q.off, a);
        const unsigned long long f = __ballot(fl), p = __ballot(ph);
        const bool row0 = (unsigned)a % (unsigned)q.nx == 0;
        const bool start = lane == 0 || row0 || !((f >> (lane - 1)) & 1) || (((p >> (lane - 1)) & 1) != (ph ? 1u : 0u));
        const unsigned long long st = __ballot(start);
        // the last run start at or before this lane
        const unsigned long long upto = st & (~0ull >> (63 - lane));
        par[g * 64 + lane] = fl ? g * 64 + 63 - __clzll((long long)upto) : -1;
        cnt[g * 64 + lane] = 0;
        if (lane == 0) {
            fluid[g] = f;
            pos[g] = p;
            starts[g] = st;
            if (gb + g < q.groups) {
                m.fluid[q.g0 + gb + g] = f;
                m.pos[q.g0 + gb + g] = p;
            }
        }
    }
    __syncthreads();
    // along x only across words; along y and z one link per pair of runs that
    // touch (a link whose left neighbour is the same pair's is implied by it)
    for (int g = wave; g < BAND_GROUPS; g += 16) {
        const int l = g * 64 + lane, plane = q.nx * q.ny;
        bool ix, iy, iz;
        has_next(q, gb * 64 + l, ix, iy, iz);
        const unsigned long long lx = band_links(fluid, pos, g, 1, ix);
        const unsigned long long ly = q.nx < BAND_NODES ? band_links(fluid, pos, g, q.nx, iy) : 0ull;
        const unsigned long long lz = q.nz > 1 && plane < BAND_NODES ? band_links(fluid, pos, g, plane, iz) : 0ull;
        if (lane == 63 && (lx >> 63)) band_unite(par, l, l + 1);
        if (((ly & ~((lx & ly) << 1)) >> lane) & 1) band_unite(par, l, l + q.nx);
        if (((lz & ~((lx & lz) << 1)) >> lane) & 1) band_unite(par, l, l + plane);
    }
    __syncthreads();
    int root[BAND_GROUPS / 16];
#pragma unroll
    for (int k = 0; k < BAND_GROUPS / 16; ++k) {
        const int g = wave + 16 * k;
        int r = par[g * 64 + lane];
        if (r >= 0)
            for (int n = par[r]; n != r; n = par[r]) r = n;
        root[k] = r;
        // the run's nodes, counted by its first one
        const unsigned long long f = fluid[g], rest = lane == 63 ? 0ull : (starts[g] | ~f) >> (lane + 1);
        if (((starts[g] & f) >> lane) & 1) atomicAdd(cnt + r, rest ? __ffsll((long long)rest) : 64 - lane);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BAND_GROUPS / 16; ++k) {
        const int g = wave + 16 * k, a = (gb + g) * 64 + lane;
        if (gb + g < q.groups && a < q.N) {
            m.par[q.off + a] = root[k] >= 0 ? gb * 64 + root[k] : -1;
            m.cnt[2 * q.off + a] = cnt[g * 64 + lane];
        }
    }
}

// Join the bands' regions by the links between bands, one per pair of runs
// that touch (in two dimensions these leave the last nx nodes of a band, so the
// other groups are not looked at).  Grid of this and the next two kernels:
// blockIdx.y = run, the wavefronts of blockIdx.x stride over the run's groups.
static __global__ void __launch_bounds__(256) k_cc_join(RunSet rs, RegionMem m)
{
    const int lane = threadIdx.x & 63;
    const RunGeom q = run_geom(rs, blockIdx.y);
    int *par = m.par + q.off;
    // joins a and b in the lanes with `link` set, once per pair of labels
    auto join = [&](bool link, int a, int b) {
        link = link && ((a ^ b) & ~(BAND_NODES - 1)) != 0;
        if (!__ballot(link)) return;
        const int pa = link ? par[a] : -1, pb = link ? par[b] : -1;
        bool first = false;
        for (unsigned long long todo = __ballot(link); todo;) {
            const int lead = __ffsll((long long)todo) - 1;
            if (lane == lead) first = true;
            todo &= ~__ballot(pa == __shfl(pa, lead, 64) && pb == __shfl(pb, lead, 64));
        }
        if (first) cc_unite(par, pa, pb);
    };
    const int last = q.nz > 1 ? BAND_GROUPS : min(BAND_GROUPS, (q.nx + 63) / 64 + 1);  // groups of a band with such links
    const int bands = (q.groups + BAND_GROUPS - 1) / BAND_GROUPS;
    for (int k = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)); k < bands * last; k += (int)gridDim.x * 4) {
        const int g = k / last * BAND_GROUPS + BAND_GROUPS - last + k % last;
        if (g >= q.groups) continue;
        const int a = g * 64 + lane, plane = q.nx * q.ny;
        bool ix, iy, iz;
        has_next(q, a, ix, iy, iz);
        const unsigned long long lx = link_bits(q, m.fluid, m.pos, g, 1, ix, true);
        const unsigned long long ly = link_bits(q, m.fluid, m.pos, g, q.nx, iy, true);
        const unsigned long long lz = q.nz > 1 ? link_bits(q, m.fluid, m.pos, g, plane, iz, true) : 0ull;
        join(lane == 63 && (lx >> 63), a, a + 1);
        join(((ly & ~((lx & ly) << 1)) >> lane) & 1, a, a + q.nx);
        if (q.nz > 1) join(((lz & ~((lx & lz) << 1)) >> lane) & 1, a, a + plane);
    }
}

// After joining: every band region's size to the region's root, and
// par[root in the band] <- that root, so that the root of any fluid node a is
// par[par[a]].  (Sizes are nonzero at the bands' roots only, and only those
// have children, so a label read while another lane sets it is an ancestor
// either way.)
static __global__ void __launch_bounds__(256) k_cc_merge(RunSet rs, RegionMem m)
{
    const int lane = threadIdx.x & 63;
    const RunGeom q = run_geom(rs, blockIdx.y);
    int *par = m.par + q.off, *cnt = m.cnt + 2 * q.off;
    for (int g = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)); g < q.groups; g += (int)gridDim.x * 4) {
        const int a = g * 64 + lane;
        if (a >= q.N || cnt[a] == 0) continue;
        int r = par[a];
        if (r == a) continue;
        for (int n = par[r]; n != r; n = par[r]) r = n;
        atomicAdd(cnt + r, cnt[a]);
        par[a] = r;
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
                ok = par[par[a]] == best[ph] && par[par[a + step[d]]] == best[ph ^ 1] && pt.accept(q, a, d);
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
// wavefront, then the wavefronts in order, a thread per value); every thread
// gets the result.  Of each pair of lanes that a step of the butterfly adds,
// one goes on with one half of the values and one with the other, so that the
// 14 values of a sphere fit take 17 exchanges instead of 84: sixteen
// wavefronts share one LDS for them.
template <int NV, int NT> __device__ void block_sum(double (&v)[NV], double (*sh)[NT / 64])
{
    constexpr int P = NV > 8 ? 16 : NV > 4 ? 8 : NV > 2 ? 4 : 2;
    static_assert(NV <= 16, "at most 16 values");
    const int lane = threadIdx.x & 63;
    double w[P];
#pragma unroll
    for (int k = 0; k < P; ++k) w[k] = k < NV ? v[k] : 0.0;
#pragma unroll
    for (int h = P / 2, s = 32; s > 0; h /= 2, s >>= 1) {
        if (h > 0) {
            const bool up = lane & s;
#pragma unroll
            for (int k = 0; k < h; ++k) {
                const double mine = up ? w[k + h] : w[k], other = up ? w[k] : w[k + h];
                w[k] = mine + __shfl_xor(other, s, 64);
            }
        } else {
            w[0] += __shfl_xor(w[0], s, 64);
        }
    }
    constexpr int SHARE = 64 / P;  // lanes that hold the same value
    __syncthreads();
    if (lane % SHARE == 0 && lane / SHARE < NV) sh[lane / SHARE][threadIdx.x >> 6] = w[0];
    __syncthreads();
    if (threadIdx.x < NV) {
        double s = sh[threadIdx.x][0];
        for (int k = 1; k < NT / 64; ++k) s += sh[threadIdx.x][k];
        sh[threadIdx.x][0] = s;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = sh[k][0];
}

// The points of a fit, shared out over NT threads (thread t takes t, t + NT,
// ...): each thread keeps its first KEEP points in registers over the passes of
// the fit and finds the others again from the fields on every pass.  One
// compute unit does the fit, so its instructions count: with the points found
// again on every pass, all threads summing all wavefronts' sums and the pivot
// rows in memory, the sphere fit on 72 x 65 x 40 nodes took 97 us and the
// circle fit on 400 x 400 26; they take 41 and 17.
template <int ND, int NT, int KEEP, class Point> struct FitPoints {
    double kept[KEEP][ND];
    int n;
    Point point;
    __device__ __forceinline__ FitPoints(int count, const Point &pt) : n(count), point(pt)
    {
#pragma unroll
        for (int k = 0; k < KEEP; ++k)
            if ((int)threadIdx.x + k * NT < n) point((int)threadIdx.x + k * NT, kept[k]);
    }
    template <class F> __device__ __forceinline__ void each(F &&f) const
    {
#pragma unroll
        for (int k = 0; k < KEEP; ++k)
            if ((int)threadIdx.x + k * NT < n) f(kept[k]);
        for (int i = (int)threadIdx.x + KEEP * NT; i < n; i += NT) {
            double p[ND];
            point(i, p);
            f(p);
        }
    }
};

// Solve M x = b (ND unknowns, M with b as its last column) by elimination with
// row pivoting; false for a singular matrix.  Unrolled, with the pivot row
// exchanged by selection: rows picked by a runtime index would live in memory.
template <int ND> __device__ __forceinline__ bool solve_linear(double (&M)[ND][ND + 1], double (&x)[ND])
{
#pragma unroll
    for (int col = 0; col < ND; ++col) {
        int piv = col;
        double big = __builtin_fabs(M[col][col]);
#pragma unroll
        for (int r = col + 1; r < ND; ++r)
            if (__builtin_fabs(M[r][col]) > big) {
                piv = r;
                big = __builtin_fabs(M[r][col]);
            }
        if (big == 0.0) return false;
#pragma unroll
        for (int r = col + 1; r < ND; ++r)
#pragma unroll
            for (int q = 0; q <= ND; ++q) {
                const double a = M[col][q], b = M[r][q];
                M[col][q] = piv == r ? b : a;
                M[r][q] = piv == r ? a : b;
            }
#pragma unroll
        for (int r = col + 1; r < ND; ++r) {
            const double fct = M[r][col] / M[col][col];
#pragma unroll
            for (int q = col; q <= ND; ++q) M[r][q] -= fct * M[col][q];
        }
    }
#pragma unroll
    for (int r = ND - 1; r >= 0; --r) {
        double s = M[r][ND];
#pragma unroll
        for (int q = r + 1; q < ND; ++q) s -= M[r][q] * x[q];
        x[r] = s / M[r][r];
    }
    return true;
}

// Blocks of the labelling passes for runs of up to max_nodes nodes, and of the
// link passes: enough to fill the chip over all runs, at least a few per run
// (48 runs, 64 / 256 and 32 / 128 of them: links 60 / 40 us, joining 78 / 63).
inline dim3 region_grid(long long max_nodes, int nruns)
{
    long long bx = (max_nodes + 255) / 256;
    const long long cap = nruns > 1 ? (nruns < 192 ? 12288 / nruns : 64) : 2048;
    return dim3((unsigned)(bx > cap ? cap : bx < 1 ? 1 : bx), (unsigned)nruns);
}
inline dim3 link_grid(long long max_nodes, int nruns)
{
    long long bx = (max_nodes + 255) / 256;
    const long long cap = nruns <= 12 ? REGION_BLOCKS : nruns < 192 ? 6144 / nruns : 32;
    return dim3((unsigned)(bx > cap ? cap : bx < 1 ? 1 : bx), (unsigned)nruns);
}

// Label the phase regions and choose the largest of each phase.
static inline hipError_t launch_regions(hipStream_t st, const RunSet &rs, int nruns, long long max_nodes,
                                        const double *rho1, const double *rho2, const uint8_t *solid, const RegionMem &m)
{
    const dim3 grid = region_grid(max_nodes, nruns);
    const dim3 bands((unsigned)((max_nodes + BAND_NODES - 1) / BAND_NODES), (unsigned)nruns);
    hipLaunchKernelGGL(k_cc_band, bands, dim3(1024), 0, st, rs, m, rho1, rho2, solid);
    hipLaunchKernelGGL(k_cc_join, grid, dim3(256), 0, st, rs, m);
    hipLaunchKernelGGL(k_cc_merge, grid, dim3(256), 0, st, rs, m);
    hipLaunchKernelGGL(k_cc_pick, grid, dim3(256), 0, st, rs, m);
    return hipGetLastError();
}

}  // namespace lbm
