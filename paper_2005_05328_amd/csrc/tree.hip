// Oct-tree on Morton-sorted particles and the wavefront-cooperative short-range walk.
//
// Build (paper Sec. 2.1: root = box, each node split into its 8 octants while it holds more
// than one particle; here a node stops splitting at `leaf_size` particles): a node's particles
// are a contiguous range of the sorted order, so the nodes follow from the sorted keys without
// descending the tree (see the build section).  Nodes are stored level-major, children of a node
// contiguous and in Morton order.  Moments (mass, centre of mass, particle bounding box, largest
// softening) are accumulated bottom-up.
//
// Walk: one wave64 per target group (<= 64 Morton-contiguous particles inside one node,
// one target per lane).  The wave pops up to 64 nodes from its stack at a time; each lane
// classifies one node against the group's bounding box: skip (farther than r_cut),
// monopole (side < theta * distance of the node's centre of mass from the box), leaf, or
// open.  Opened nodes push their children; monopoles and leaf particles are appended,
// shifted to the periodic image nearest the group, to an interaction list staged in LDS.
// When the list fills, every lane sums its target's interactions with the whole list
// (LDS broadcast reads).
#include <type_traits>

#include "internal.h"

#define TB_THREADS 256
#define WALK_LIST 128
#define WALK_DEPTH 8192u
#define WALK_SLOTS_MAX 4096u

static inline uint32_t blocks_for(uint64_t n, uint32_t t) { return (uint32_t)((n + t - 1) / t); }

// ---------------------------------------------------------------------------------------
// build
// ---------------------------------------------------------------------------------------
// Particle i and the one before it share their first c_i octal digits (c_0 = -1), so a cube of
// every level above c_i starts at i.  The cube of level k holding i has more than `leaf`
// particles if and only if some window of leaf + 1 consecutive particles around i shares k
// digits; the deepest such level m_i is a sliding maximum.  A cube is a node when its parent
// splits, so the nodes holding i are those of levels 0 .. d_i = m_i + 1 (at most
// DZS_TREE_LEVELS): node k starts at i for c_i < k <= d_i, and the node of level k that holds
// i - 1 ends at i for c_i < k <= d_(i-1).  With the number E_k(i) of nodes of level k that start
// before i (a level-major scan of per-block counts), a node's index, its first child's (E_(k+1)
// where it starts) and the end of its children's (E_(k+1) where it ends) are all known where it
// starts and ends.  In place of a loop over the levels with five launches each and one for the moments the
// build is two kernels around a scan, a kernel for the moments inside blocks, one per tier of 32
// blocks for the others and three for the groups.  Build, moments and groups alone on the GPU:
// 20^3 270 -> 75 us, 128^3 408 -> 203 us, 256^3 1540 -> 1164 us.
//
// Build state in device memory (ctx->bstate): the counts stay on the device, so the build needs
// no host synchronisation (and can be graph-captured).
#define BS_NODES 1      // nodes
#define BS_GROUPS 2     // target groups
#define BS_OVERFLOW DZS_BS_OVERFLOW  // sticky: the tree needed more than the node capacity
#define BS_LMAX 7       // deepest level built (DZS_TREE_LEVELS unless the capacity cut it)
#define BS_LEVEL 8      // [BS_LEVEL + k]: first node of level k (k <= DZS_KEY_BITS + 1)
#define TREE_TILE 1024  // particles of a build block
#define TREE_NLEV (DZS_TREE_LEVELS + 1)
#define TREE_LEAF_MAX 64
#define TREE_TIER 32    // blocks (or tiers) that one workgroup joins

static inline uint64_t tree_blocks(uint64_t n) { return n / TREE_TILE + 1; }   // particles 0 .. n

uint64_t dzs_tree_scan_words(uint64_t n) { return TREE_NLEV * tree_blocks(n) + 1; }
uint64_t dzs_tree_span_words(uint64_t n) {
    uint64_t words = 0;
    for (uint64_t nb = tree_blocks(n);; nb = (nb + TREE_TIER - 1) / TREE_TIER) {
        words += TREE_NLEV * nb;
        if (nb == 1)
            return words;
    }
}
uint64_t dzs_tree_flag_tiles(uint64_t n) { return (n + 4095) / 4096; }

// octal digits that two keys share
__device__ __forceinline__ int tree_common(uint64_t a, uint64_t b) {
    return a == b ? DZS_KEY_BITS : (__clzll((long long)(a ^ b)) - 1) / 3;
}

// Per particle the first level that starts at it (c_i + 1, DZS_TREE_LEVELS + 1 = none) and the
// deepest node that holds it (d_i), packed as start | d_i << 8; per block and level the number of
// nodes that start in the block (level-major); the group flags cleared; and the block's first
// place where the coarsest cube starts (snap), which the moments take for the blocks' bounds:
// few levels of the tree then span them.  An input flagged out of
// order (DZS_BS_BADINPUT) starts nothing.  KB > 0: a batch whose keys carry the box in their top
// KB digits; the cubes above level KB always split.
__global__ __launch_bounds__(TB_THREADS) void k_tree_levels(
    uint32_t n, const uint64_t *__restrict__ key, int leaf, int KB,
    const uint32_t *__restrict__ bs, uint16_t *__restrict__ sd, uint32_t *__restrict__ cnt,
    uint8_t *__restrict__ flag, uint32_t *__restrict__ snap) {
    __shared__ uint64_t s_key[TREE_TILE + 2 * TREE_LEAF_MAX];
    __shared__ int8_t s_m[2][TREE_TILE + TREE_LEAF_MAX];
    __shared__ uint32_t s_cnt[TB_THREADS / 64][TREE_NLEV];
    __shared__ uint32_t s_snap;
    const uint32_t tid = threadIdx.x, nb = gridDim.x;
    if (tid == 0)
        s_snap = 0xffffffffu;
    const int64_t base = (int64_t)blockIdx.x * TREE_TILE;
    const int64_t N = bs[DZS_BS_BADINPUT] ? 0 : (int64_t)n;
    for (int e = (int)tid; e < TREE_TILE + 2 * leaf; e += TB_THREADS) {
        const int64_t j = base - leaf + e;
        s_key[e] = j >= 0 && j < N ? key[j] : 0ull;
    }
    __syncthreads();
    // m[e]: digits shared by the window of particles j .. j + leaf, j = base - leaf + e; then the
    // maximum over 2^p of them, the largest power of two within the leaf + 1 windows around i
    const int len = TREE_TILE + leaf;
    for (int e = (int)tid; e < len; e += TB_THREADS) {
        const int64_t j = base - leaf + e;
        s_m[0][e] = j >= 0 && j + leaf < N ? (int8_t)tree_common(s_key[e], s_key[e + leaf])
                                           : (int8_t)-1;
    }
    int cur = 0, span = 1;
    for (; 2 * span <= leaf + 1; span *= 2, cur ^= 1) {
        __syncthreads();
        for (int e = (int)tid; e < len; e += TB_THREADS) {
            const int8_t a = s_m[cur][e], b = e + span < len ? s_m[cur][e + span] : (int8_t)-1;
            s_m[cur ^ 1][e] = a > b ? a : b;
        }
    }
    __syncthreads();
    uint32_t c[TREE_NLEV];
#pragma unroll
    for (int k = 0; k < TREE_NLEV; ++k)
        c[k] = 0u;
    uint32_t best = 0xffffffffu;   // first level that starts * TREE_TILE + place
    for (int e = (int)tid; e < TREE_TILE; e += TB_THREADS) {
        const int64_t i = base + e;
        int start = TREE_NLEV, d = -1;
        if (i < N) {
            const int c_i = i == 0 ? -1 : tree_common(s_key[e + leaf - 1], s_key[e + leaf]);
            start = c_i + 1 < TREE_NLEV ? c_i + 1 : TREE_NLEV;
            const int8_t a = s_m[cur][e], b = s_m[cur][e + leaf + 1 - span];
            int m = a > b ? a : b;
            m = m > KB - 1 ? m : KB - 1;
            d = m + 1 < DZS_TREE_LEVELS ? m + 1 : DZS_TREE_LEVELS;
        }
        best = min(best, (uint32_t)start * TREE_TILE + (uint32_t)e);
        if (i < (int64_t)n) {
            sd[i] = (uint16_t)(start | ((d < 0 ? 0 : d) << 8));
            flag[i] = 0u;
        }
#pragma unroll
        for (int k = 0; k < TREE_NLEV; ++k)
            c[k] += (uint32_t)__popcll(__ballot(start <= k && k <= d));
    }
    if ((tid & 63u) == 0u)
#pragma unroll
        for (int k = 0; k < TREE_NLEV; ++k)
            s_cnt[tid >> 6][k] = c[k];
    atomicMin(&s_snap, best);
    __syncthreads();
    if (tid == 0) {
        const int64_t p = base + (int64_t)(s_snap % TREE_TILE);
        snap[blockIdx.x] = (uint32_t)(p < (int64_t)n ? p : (int64_t)n);
    }
    if (tid < TREE_NLEV) {
        uint32_t t = 0;
        for (int w = 0; w < TB_THREADS / 64; ++w)
            t += s_cnt[w][tid];
        cnt[(uint64_t)tid * nb + blockIdx.x] = t;
    }
}

// Nodes at the places where they start and end; E: the scanned counts.  A level that would take
// the nodes past the capacity is left out whole, with all below it: its parents are leaves (and
// the overflow is flagged).  The first block also writes the build state; an input flagged out
// of order gets an empty root.  snap_e: the same numbers at the moments' block bounds.
__global__ __launch_bounds__(TB_THREADS) void k_tree_emit(
    uint32_t n, const uint16_t *__restrict__ sd, const uint32_t *__restrict__ E, uint64_t cap,
    uint32_t *__restrict__ nd_first, uint32_t *__restrict__ nd_end,
    uint32_t *__restrict__ nd_child, uint32_t *__restrict__ nd_cend,
    uint8_t *__restrict__ nd_level, const uint32_t *__restrict__ snap,
    uint32_t *__restrict__ snap_e, uint32_t *__restrict__ bs) {
    constexpr int WAVES = TB_THREADS / 64, RUN = TREE_TILE / WAVES;
    __shared__ uint32_t s_cnt[WAVES][TREE_NLEV];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, nb = gridDim.x;
    const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const bool bad = bs[DZS_BS_BADINPUT] != 0u;
    int lmax = 0;   // the levels that fit (the root always does)
    {
        uint32_t upto[TREE_NLEV];
#pragma unroll
        for (int k = 0; k < TREE_NLEV; ++k)
            upto[k] = E[(uint64_t)(k + 1) * nb];
#pragma unroll
        for (int k = 1; k < TREE_NLEV; ++k)
            lmax += !bad && lmax == k - 1 && (uint64_t)upto[k] <= cap ? 1 : 0;
    }
    if (blockIdx.x == 0 && tid == 0) {
        const bool over = E[(uint64_t)TREE_NLEV * nb] > cap;
        if (over)
            bs[BS_OVERFLOW] = 1u;
        bs[BS_NODES] = bad ? 1u : E[(uint64_t)(lmax + 1) * nb];
        bs[BS_GROUPS] = 0u;
        bs[BS_LMAX] = (uint32_t)lmax;
        for (int k = 0; k <= DZS_KEY_BITS + 1; ++k)
            bs[BS_LEVEL + k] = bad ? (k == 0 ? 0u : 1u)
                                   : E[(uint64_t)(k <= lmax + 1 ? k : lmax + 1) * nb];
        if (bad) {
            nd_first[0] = nd_end[0] = nd_child[0] = nd_cend[0] = 0u;
            nd_level[0] = 0u;
        }
    }
    if (bad)
        return;
    const uint64_t base = (uint64_t)blockIdx.x * TREE_TILE + (uint64_t)wave * RUN;
    const uint32_t bound = snap[blockIdx.x];   // the moments' block starts here
    // the wave's particles (RUN / 64 rounds of 64): first level that starts, deepest node, and
    // the deepest node of the particle before
    constexpr int ROUNDS = RUN / 64;
    int start[ROUNDS], deep[ROUNDS], dprev[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint64_t i = base + (uint32_t)r * 64u + lane;
        const uint32_t v = i < n ? sd[i] : 0u, u = i > 0 && i <= n ? sd[i - 1] : 0u;
        // past the last particle (i = n) every node ends
        start[r] = i < n ? (int)(v & 0xffu) : (i == n ? 0 : TREE_NLEV);
        deep[r] = i < n ? min((int)(v >> 8), lmax) : -1;
        dprev[r] = i > 0 && i <= n ? min((int)(u >> 8), lmax) : -1;
    }
    // the wave's counts, then its first numbers
    uint32_t run[TREE_NLEV];
#pragma unroll
    for (int k = 0; k < TREE_NLEV; ++k) {
        run[k] = 0u;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            run[k] += (uint32_t)__popcll(__ballot(start[r] <= k && k <= deep[r]));
    }
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < TREE_NLEV; ++k)
            s_cnt[wave][k] = run[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TREE_NLEV; ++k) {
        run[k] = E[(uint64_t)k * nb + blockIdx.x];
        for (uint32_t w = 0; w < wave; ++w)
            run[k] += s_cnt[w][k];
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t i = (uint32_t)base + (uint32_t)r * 64u + lane;
        uint32_t below = 0u;   // E_(k+1)(i)
#pragma unroll
        for (int k = TREE_NLEV - 1; k >= 0; --k) {
            const bool open = start[r] <= k && k <= deep[r];
            const bool close = start[r] <= k && k <= dprev[r];
            const uint64_t m = __ballot(open);
            const uint32_t id = run[k] + (uint32_t)__popcll(m & lt_mask);
            if (close) {
                nd_end[id - 1u] = i;
                nd_cend[id - 1u] = k < dprev[r] ? below : 0u;
            }
            if (open) {
                nd_first[id] = i;
                nd_child[id] = k < deep[r] ? below : 0u;
                nd_level[id] = (uint8_t)k;
            }
            below = id;
            if (i == bound)
                snap_e[(uint64_t)k * nb + blockIdx.x] = id;
            run[k] += (uint32_t)__popcll(m);
        }
    }
}

// mult^(1/3), the softening factor of a particle of multiplicity mult (1 for an original
// particle without the library call: most particles)
__device__ __forceinline__ double mult_cbrt(uint32_t mult) {
    return mult == 1u ? 1.0 : cbrt((double)mult);
}

// Half extent of [mn, mx] about c, as an FP32 value rounded up: the box c +- h holds both ends.
__device__ __forceinline__ float half_up(double mn, double mx, double c) {
    return __double2float_ru(fmax(mx - c, c - mn));
}

// The nodes' topology as the build writes it: particles [first, end), children [child, cend).
struct tree_nodes {
    const uint32_t *first, *end, *child, *cend;
    const uint8_t *level;
};

// Moments of node v (mass, centre of mass, particle bounding box, largest softening): of its
// particles for a leaf, of its children (already complete) otherwise; with the node's
// topology its walk record.  child_rec(c) gives the record of child c.
template <typename Child>
__device__ __forceinline__ void node_moments(
    uint32_t v, const double *__restrict__ x, const double *__restrict__ y,
    const double *__restrict__ z, const uint32_t *__restrict__ mult, double m0, double h0,
    const tree_nodes &nd, const Child &child_rec, const uint64_t *__restrict__ key,
    const dzs_bbox *__restrict__ boxes, double L, int unwrap, dzs_node_rec &out) {
    const uint32_t first = nd.first[v], end = nd.end[v], child = nd.child[v],
                   nc = nd.cend[v] - child;
    if (boxes && nc == 0) {
        // a batch: the leaf's box (its key prefix) sets the mass unit and the softening
        const uint64_t b = key[first] >> DZS_BATCH_SHIFT;
        m0 = boxes[b].m0;
        h0 = boxes[b].h0;
    }
    double m = 0.0, sx = 0.0, sy = 0.0, sz = 0.0, hmax = 0.0;
    double mnx = 1e300, mny = 1e300, mnz = 1e300, mxx = -1e300, mxy = -1e300, mxz = -1e300;
    // kept tree: a member (child) more than half a box from the first one crossed a face of
    // the periodic box since the build; it is taken at the image next to the first one
    const double halfL = 0.5 * L;
    auto near = [&](double a, double a0) -> double {
        return a - a0 > halfL ? a - L : (a - a0 < -halfL ? a + L : a);
    };
    uint32_t crossed = 0u;
    if (nc == 0) {
        const uint32_t s = first, e = end;
        const double x0 = x[s], y0 = y[s], z0 = z[s];
        uint32_t mmax = 0;
        // four members are loaded before the first is added (in order: the same sums)
        for (uint32_t j0 = s; j0 < e; j0 += 4u) {
            double xs[4], ys[4], zs[4];
            uint32_t ms[4];
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                const uint32_t j = min(j0 + q, e - 1u);
                xs[q] = x[j];
                ys[q] = y[j];
                zs[q] = z[j];
                ms[q] = mult[j];
            }
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                if (j0 + q >= e)
                    break;
                const uint32_t mu = ms[q];
                const double mj = m0 * (double)mu;
                double xj = xs[q], yj = ys[q], zj = zs[q];
                if (unwrap) {
                    const double ux = near(xj, x0), uy = near(yj, y0), uz = near(zj, z0);
                    crossed |= (ux != xj || uy != yj || uz != zj) ? 1u : 0u;
                    xj = ux;
                    yj = uy;
                    zj = uz;
                }
                m += mj;
                sx += mj * xj;
                sy += mj * yj;
                sz += mj * zj;
                mnx = fmin(mnx, xj); mny = fmin(mny, yj); mnz = fmin(mnz, zj);
                mxx = fmax(mxx, xj); mxy = fmax(mxy, yj); mxz = fmax(mxz, zj);
                mmax = mu > mmax ? mu : mmax;
            }
        }
        hmax = h0 * mult_cbrt(mmax);  // the softening grows with the multiplicity
    } else {
        const uint32_t c0 = child;
        double x0 = 0.0, y0 = 0.0, z0 = 0.0;
        if (unwrap) {
            const dzs_node_rec r0 = child_rec(c0);
            x0 = r0.cx;
            y0 = r0.cy;
            z0 = r0.cz;
        }
        for (uint32_t cb = c0; cb < c0 + nc; cb += 4u) {
            dzs_node_rec rs[4];
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q)
                rs[q] = child_rec(min(cb + q, c0 + nc - 1u));
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                if (cb + q >= c0 + nc)
                    break;
                const dzs_node_rec &r = rs[q];
                const double mc = r.mass;
                double rcx = r.cx, rcy = r.cy, rcz = r.cz;
                double rmx = r.comx, rmy = r.comy, rmz = r.comz;
                if (unwrap) {
                    // the child's box and centre of mass move together, by the box's shift
                    const double dx = near(rcx, x0) - rcx, dy = near(rcy, y0) - rcy,
                                 dz = near(rcz, z0) - rcz;
                    rcx += dx; rcy += dy; rcz += dz;
                    rmx += dx; rmy += dy; rmz += dz;
                }
                m += mc;
                sx += mc * rmx;
                sy += mc * rmy;
                sz += mc * rmz;
                mnx = fmin(mnx, rcx - (double)r.hx); mny = fmin(mny, rcy - (double)r.hy);
                mnz = fmin(mnz, rcz - (double)r.hz);
                mxx = fmax(mxx, rcx + (double)r.hx); mxy = fmax(mxy, rcy + (double)r.hy);
                mxz = fmax(mxz, rcz + (double)r.hz);
                hmax = fmax(hmax, r.hmax);
            }
        }
    }
    out.cx = 0.5 * (mnx + mxx);
    out.cy = 0.5 * (mny + mxy);
    out.cz = 0.5 * (mnz + mxz);
    out.comx = sx / m;
    out.comy = sy / m;
    out.comz = sz / m;
    out.mass = m;
    out.hmax = hmax;
    out.hx = half_up(mnx, mxx, out.cx);
    out.hy = half_up(mny, mxy, out.cy);
    out.hz = half_up(mnz, mxz, out.cz);
    out.first = first;
    out.count = end - first;
    out.child = child;
    out.nl = nc | ((uint32_t)nd.level[v] << 8);
    out.pad = crossed;
}

struct moment_args {
    const double *x, *y, *z;
    const uint32_t *mult;
    double m0, h0, L;
    tree_nodes nd;
    dzs_node_rec *rec;
    const uint64_t *key;
    const dzs_bbox *boxes;
    int unwrap;
    const uint32_t *E;   // first node of each level and block (at the blocks' snapped starts)
    const uint32_t *snap;   // the blocks' starts
    uint32_t *span;      // [level][block] the level's node that starts in the block and ends
                         // past it (TREE_NONE: none)
    const uint32_t *bs;
    uint32_t n, nb;
};
#define TREE_NONE 0xffffffffu

template <typename Child>
__device__ __forceinline__ void moments_of(const moment_args &A, uint32_t v, const Child &child,
                                           dzs_node_rec &out) {
    node_moments(v, A.x, A.y, A.z, A.mult, A.m0, A.h0, A.nd, child, A.key, A.boxes, A.L,
                 A.unwrap, out);
}

// Target groups of node v: each node with more than G particles packs its consecutive children
// that hold at most G particles into bins of at most G (greedy, Morton order); a bin starts a
// group.  Leaves with more than G particles (coincident particles at the finest level) are cut
// into chunks of G.
__device__ __forceinline__ void node_groups(uint32_t v, const tree_nodes &nd, uint32_t G,
                                            uint8_t *__restrict__ flag, int KB) {
    const uint32_t first = nd.first[v], cnt = nd.end[v] - first;
    const uint32_t c0 = nd.child[v], c1 = nd.cend[v];
    if (KB > 0) {
        // a batch: nothing above the box nodes (level KB) is a group, and the box nodes of at
        // most G particles are groups of their own
        const int lev = nd.level[v];
        if (lev + 1 < KB)
            return;
        if (lev + 1 == KB) {
            for (uint32_t c = c0; c < c1; ++c)
                if (nd.end[c] - nd.first[c] <= G)
                    flag[nd.first[c]] = 1u;
            return;
        }
    }
    if (v == 0 && cnt <= G) {
        if (cnt > 0)
            flag[0] = 1u;
        return;
    }
    if (cnt <= G)
        return;
    if (c0 == c1) {
        for (uint32_t j = first; j < first + cnt; j += G)
            flag[j] = 1u;
        return;
    }
    uint32_t bin = 0;
    for (uint32_t c = c0; c < c1; ++c) {
        const uint32_t f = nd.first[c], cc = nd.end[c] - f;
        if (cc > G) {
            bin = 0;
        } else if (bin > 0 && bin + cc <= G) {
            bin += cc;
        } else {
            flag[f] = 1u;
            bin = cc;
        }
    }
}

// Moments of the nodes that lie inside the block's particles: first every leaf, then the other
// nodes level by level from the deepest (a node's children start and end inside it), whose
// children's records wait in LDS; and the group flags of all nodes that start in the block (flag
// null: the moments alone).  The levels are a chain of dependent steps, a few hundred
// nanoseconds each; the particles are read and the 96-byte records written once.
#define TREE_CACHE 320   // records in LDS (30 KB); a block with more nodes reads the rest back
__global__ __launch_bounds__(TB_THREADS) void k_tree_block(moment_args A, uint32_t G,
                                                           uint8_t *__restrict__ flag, int KB) {
    __shared__ uint32_t s_lo[TREE_NLEV], s_hi[TREE_NLEV], s_off[TREE_NLEV + 1];
    __shared__ dzs_node_rec s_rec[TREE_CACHE];
    const uint32_t tid = threadIdx.x;
    const uint32_t bend = blockIdx.x + 1u < A.nb ? A.snap[blockIdx.x + 1u] : A.n;
    if (A.bs[DZS_BS_BADINPUT]) {   // an empty root
        if (blockIdx.x == 0 && tid == 0) {
            dzs_node_rec out;
            moments_of(A, 0u, [&](uint32_t c) { return A.rec[c]; }, out);
            A.rec[0] = out;
        }
        return;
    }
    const int lmax = (int)A.bs[BS_LMAX];
    if (tid < TREE_NLEV) {
        const uint64_t at = (uint64_t)tid * A.nb + blockIdx.x;
        const uint32_t lo = A.E[at];
        const uint32_t hi = (int)tid > lmax ? lo
                            : (blockIdx.x + 1u < A.nb ? A.E[at + 1] : A.bs[BS_LEVEL + tid + 1u]);
        s_lo[tid] = lo;
        s_hi[tid] = hi;
        A.span[at] = hi > lo && A.nd.end[hi - 1u] > bend ? hi - 1u : TREE_NONE;
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t off = 0;
        for (int k = 0; k < TREE_NLEV; ++k) {
            s_off[k] = off;
            off += s_hi[k] - s_lo[k];
        }
        s_off[TREE_NLEV] = off;
    }
    __syncthreads();
    const uint32_t total = s_off[TREE_NLEV];
    for (uint32_t q = tid; q < total; q += TB_THREADS) {
        uint32_t k = 0;
        while (q >= s_off[k + 1])
            ++k;
        const uint32_t v = s_lo[k] + (q - s_off[k]);
        if (flag)
            node_groups(v, A.nd, G, flag, KB);
        if (A.nd.cend[v] == A.nd.child[v] && A.nd.end[v] <= bend) {
            dzs_node_rec out;
            moments_of(A, v, [&](uint32_t c) { return A.rec[c]; }, out);
            A.rec[v] = out;
            if (q < TREE_CACHE)
                s_rec[q] = out;
        }
    }
    for (int k = lmax; k >= 0; --k) {
        const uint32_t lo = s_lo[k], hi = s_hi[k];
        if (hi == lo)
            continue;
        __syncthreads();
        // children of level-k nodes: level k + 1, at this place of the block's list
        const uint32_t cshift = k < lmax ? s_off[k + 1] - s_lo[k + 1] : 0u;
        for (uint32_t v = lo + tid; v < hi; v += TB_THREADS) {
            if (A.nd.cend[v] == A.nd.child[v] || A.nd.end[v] > bend)
                continue;
            dzs_node_rec out;
            moments_of(A, v,
                       [&](uint32_t c) {
                           const uint32_t q = c + cshift;
                           return q < TREE_CACHE ? s_rec[q] : A.rec[c];
                       },
                       out);
            A.rec[v] = out;
            const uint32_t q = v - lo + s_off[k];
            if (q < TREE_CACHE)
                s_rec[q] = out;
        }
    }
}

// Moments of the nodes that span blocks.  A workgroup joins TREE_TIER blocks (or tiers of `size`
// blocks), in which at most one node of each level starts in each and ends past
// it (`in`): the nodes that end inside the tier are done, level by level from the deepest, those
// that span its end are handed on (`out`).  (One workgroup over all blocks took 287 us at 128^3:
// a single CU's bandwidth.)
__global__ __launch_bounds__(TREE_TIER *TREE_NLEV) void k_tree_tier(
    moment_args A, const uint32_t *__restrict__ in, uint32_t nb_in, uint32_t size,
    uint32_t *__restrict__ out, uint32_t nb_out) {
    __shared__ uint32_t s_out[TREE_NLEV];
    if (A.bs[DZS_BS_BADINPUT])
        return;
    const int level = (int)(threadIdx.x / TREE_TIER);
    const uint32_t b = blockIdx.x * TREE_TIER + threadIdx.x % TREE_TIER;
    if (threadIdx.x < TREE_NLEV)
        s_out[threadIdx.x] = TREE_NONE;
    const uint64_t next = (uint64_t)(blockIdx.x + 1u) * TREE_TIER * size;   // the next tier's block
    const uint32_t tend = next < A.nb ? A.snap[next] : A.n;
    const uint32_t v = b < nb_in ? in[(uint64_t)level * nb_in + b] : TREE_NONE;
    const bool here = v != TREE_NONE && A.nd.end[v] <= tend;
    __syncthreads();
    if (v != TREE_NONE && !here)
        s_out[level] = v;   // the level's last node of the tier
    for (int k = TREE_NLEV - 1; k >= 0; --k) {
        const bool mine = here && level == k;
        if (!__syncthreads_or(mine ? 1 : 0))   // (a barrier after each level that had one)
            continue;
        if (mine) {
            dzs_node_rec rec;
            moments_of(A, v, [&](uint32_t c) { return A.rec[c]; }, rec);
            A.rec[v] = rec;
        }
        __syncthreads();
    }
    if (out && threadIdx.x < TREE_NLEV)
        out[(uint64_t)threadIdx.x * nb_out + blockIdx.x] = s_out[threadIdx.x];
}

// Group starts from the flags: per tile of 4096 particles their number, then (after a scan of
// the numbers) their places.  A thread reads 16 flags at once.
__global__ __launch_bounds__(TB_THREADS) void k_flag_count(uint32_t n,
                                                           const uint8_t *__restrict__ flag,
                                                           uint32_t *__restrict__ cnt) {
    __shared__ uint32_t s_c[TB_THREADS / 64];
    const uint64_t i = (uint64_t)blockIdx.x * 4096u + threadIdx.x * 16u;
    uint32_t c = 0;
    if (i + 16u <= n) {
        const uint4 v = *(const uint4 *)(flag + i);
        c = (uint32_t)(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w));
    } else {
        for (uint64_t j = i; j < n; ++j)
            c += flag[j];
    }
    c = dzs_wave_last(dzs_wave_scan_add_full(c));
    if ((threadIdx.x & 63u) == 0u)
        s_c[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0)
        cnt[blockIdx.x] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
}

__global__ __launch_bounds__(TB_THREADS) void k_flag_place(uint32_t n,
                                                           const uint8_t *__restrict__ flag,
                                                           const uint32_t *__restrict__ scan,
                                                           const uint32_t *__restrict__ total,
                                                           uint32_t *__restrict__ grp_first) {
    __shared__ uint32_t s_c[TB_THREADS / 64];
    const uint64_t i = (uint64_t)blockIdx.x * 4096u + threadIdx.x * 16u;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if (i + 16u <= n) {
        const uint4 v = *(const uint4 *)(flag + i);
        w[0] = v.x;
        w[1] = v.y;
        w[2] = v.z;
        w[3] = v.w;
    } else {
        for (uint64_t j = i; j < n; ++j)
            w[(j - i) >> 2] |= (uint32_t)flag[j] << (8u * ((j - i) & 3u));
    }
    const uint32_t c = (uint32_t)(__popc(w[0]) + __popc(w[1]) + __popc(w[2]) + __popc(w[3]));
    const uint32_t incl = dzs_wave_scan_add_full(c);
    if ((threadIdx.x & 63u) == 63u)
        s_c[threadIdx.x >> 6] = incl;
    __syncthreads();
    uint32_t at = scan[blockIdx.x] + incl - c;
    for (uint32_t k = 0; k < (threadIdx.x >> 6); ++k)
        at += s_c[k];
    for (uint32_t k = 0; k < 16u; ++k)
        if ((w[k >> 2] >> (8u * (k & 3u))) & 1u)
            grp_first[at++] = (uint32_t)(i + k);
    if (i == 0)
        grp_first[*total] = n;
}

dzs_status dzs_flag_list(dzs_ctx *ctx, uint64_t n, const uint8_t *flag, uint32_t *cnt,
                         uint32_t *scan, uint32_t *total, uint32_t *list, hipStream_t s) {
    const uint32_t tiles = (uint32_t)dzs_tree_flag_tiles(n);
    hipLaunchKernelGGL(k_flag_count, dim3(tiles), dim3(TB_THREADS), 0, s, (uint32_t)n, flag, cnt);
    DZS_TRY(dzs_check_launch(ctx, "flag_count"));
    DZS_TRY(dzs_scan_u32(ctx, cnt, scan, tiles, total, s));
    hipLaunchKernelGGL(k_flag_place, dim3(tiles), dim3(TB_THREADS), 0, s, (uint32_t)n, flag,
                       (const uint32_t *)scan, (const uint32_t *)total, list);
    return dzs_check_launch(ctx, "flag_place");
}

__global__ __launch_bounds__(TB_THREADS) void k_fill_u32(uint64_t n, uint32_t *a, uint32_t v);

// flag[i] = 1 for a flagged target
__global__ __launch_bounds__(TB_THREADS) void k_target_flag(uint32_t n,
                                                            const uint8_t *__restrict__ active,
                                                            uint32_t *__restrict__ flag) {
    const uint32_t i = blockIdx.x * TB_THREADS + threadIdx.x;
    if (i < n)
        flag[i] = active[i] != 0 ? 1u : 0u;
}

__global__ __launch_bounds__(TB_THREADS) void k_target_list(uint32_t n,
                                                            const uint32_t *__restrict__ flag,
                                                            const uint32_t *__restrict__ scan,
                                                            uint32_t *__restrict__ list) {
    const uint32_t i = blockIdx.x * TB_THREADS + threadIdx.x;
    if (i < n && flag[i])
        list[scan[i]] = i;
}

// The tree's groups that hold a flagged target start a group of the target list at their
// first slot (the group then holds its flagged targets only; a group without one is left out).
__global__ __launch_bounds__(TB_THREADS) void k_target_groups(
    uint32_t n, const uint32_t *__restrict__ n_groups, const uint32_t *__restrict__ grp_first,
    const uint8_t *__restrict__ active, uint32_t *__restrict__ flag) {
    const uint32_t g = blockIdx.x * TB_THREADS + threadIdx.x;
    if (g >= n || g >= *n_groups)
        return;
    uint32_t any = 0u;
    for (uint32_t j = grp_first[g]; j < grp_first[g + 1] && !any; ++j)
        any = active[j] != 0 ? 1u : 0u;
    if (any)
        flag[grp_first[g]] = 1u;
}

// pos[k] = the target-list position where group k starts; pos[count] = the number of targets
__global__ __launch_bounds__(TB_THREADS) void k_target_group_pos(
    uint32_t n, const uint32_t *__restrict__ gflag, const uint32_t *__restrict__ gscan,
    const uint32_t *__restrict__ tscan, const uint32_t *__restrict__ n_tgt,
    const uint32_t *__restrict__ n_grp, uint32_t *__restrict__ pos) {
    const uint32_t i = blockIdx.x * TB_THREADS + threadIdx.x;
    if (i < n && gflag[i])
        pos[gscan[i]] = tscan[i];
    if (i == 0)
        pos[*n_grp] = *n_tgt;
}

dzs_status dzs_tree_active_targets(dzs_ctx *ctx, uint64_t n64, const uint8_t *active,
                                   hipStream_t s) {
    const uint32_t n = (uint32_t)n64;
    if (!ctx->grp_list || !ctx->tree_built || n != ctx->tree_n)
        return dzs_fail(ctx, DZS_EINVAL, "active targets: no target list or no tree");
    uint32_t *n_tgt = ctx->d_small + DZS_SMALL_GROUP_LIST;
    uint32_t *n_grp = ctx->d_small + DZS_SMALL_GROUP_LIST + 1;
    // the target list
    hipLaunchKernelGGL(k_target_flag, dim3(blocks_for(n, TB_THREADS)), dim3(TB_THREADS), 0, s, n,
                       active, ctx->tg_flag);
    DZS_TRY(dzs_check_launch(ctx, "target_flag"));
    DZS_TRY(dzs_scan_u32(ctx, ctx->tg_flag, ctx->tg_tscan, n, n_tgt, s));
    hipLaunchKernelGGL(k_target_list, dim3(blocks_for(n, TB_THREADS)), dim3(TB_THREADS), 0, s, n,
                       (const uint32_t *)ctx->tg_flag, (const uint32_t *)ctx->tg_tscan,
                       ctx->grp_list);
    DZS_TRY(dzs_check_launch(ctx, "target_list"));
    // their groups (the tree's, less the unflagged targets): flags at group-start slots, then
    // the list positions where they start
    hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(n, TB_THREADS)), dim3(TB_THREADS), 0, s,
                       (uint64_t)n, ctx->tg_flag, 0u);
    DZS_TRY(dzs_check_launch(ctx, "target_group_clear"));
    hipLaunchKernelGGL(k_target_groups, dim3(blocks_for(n, TB_THREADS)), dim3(TB_THREADS), 0, s,
                       n, (const uint32_t *)(ctx->bstate + BS_GROUPS),
                       (const uint32_t *)ctx->grp_first, active, ctx->tg_flag);
    DZS_TRY(dzs_check_launch(ctx, "target_groups"));
    DZS_TRY(dzs_scan_u32(ctx, ctx->tg_flag, ctx->tg_gscan, n, n_grp, s));
    hipLaunchKernelGGL(k_target_group_pos, dim3(blocks_for(n, TB_THREADS)), dim3(TB_THREADS), 0,
                       s, n, (const uint32_t *)ctx->tg_flag, (const uint32_t *)ctx->tg_gscan,
                       (const uint32_t *)ctx->tg_tscan, (const uint32_t *)n_tgt,
                       (const uint32_t *)n_grp, ctx->tg_pos);
    return dzs_check_launch(ctx, "target_group_pos");
}

dzs_status dzs_tree_build(dzs_ctx *ctx, const dzs_box *box, uint64_t n64, const double *x,
                          const double *y, const double *z, const uint32_t *mult, int leaf_size,
                          int group_size, hipStream_t s) {
    return dzs_tree_build_ex(ctx, box, n64, x, y, z, mult, leaf_size, group_size, 0, nullptr, s);
}

__global__ __launch_bounds__(TB_THREADS) void k_fill_u32(uint64_t n, uint32_t *a, uint32_t v) {
    const uint64_t i = (uint64_t)blockIdx.x * TB_THREADS + threadIdx.x;
    if (i < n)
        a[i] = v;
}

// Moments of every node of the last built tree (and, with G, the group flags).
static dzs_status tree_moments(dzs_ctx *ctx, const dzs_box *box, uint32_t n, const double *x,
                               const double *y, const double *z, const uint32_t *mult,
                               const dzs_bbox *boxes, int unwrap, uint32_t G, int KB,
                               hipStream_t s) {
    dzs_timed t(ctx, KC_TREE_MOMENTS, s);
    moment_args A;
    A.x = x; A.y = y; A.z = z; A.mult = mult;
    A.m0 = box->m0;
    A.h0 = 2.8 * box->eps0;
    A.L = box->L;
    A.nd = tree_nodes{ctx->nd_first, ctx->nd_end, ctx->nd_child, ctx->nd_cend, ctx->nd_level};
    A.rec = ctx->nd_rec;
    A.key = ctx->key;
    A.boxes = boxes;
    A.unwrap = unwrap;
    A.E = ctx->tree_snap_e;
    A.snap = ctx->tree_snap;
    A.span = ctx->tree_span;
    A.bs = ctx->bstate;
    A.n = n;
    A.nb = (uint32_t)tree_blocks(n);
    hipLaunchKernelGGL(k_tree_block, dim3(A.nb), dim3(TB_THREADS), 0, s, A, G,
                       G ? ctx->grp_flag : nullptr, KB);
    DZS_TRY(dzs_check_launch(ctx, "tree_block"));
    uint32_t size = 1;
    uint32_t *in = A.span;
    for (uint32_t nb = A.nb; nb > 1; size *= TREE_TIER) {
        const uint32_t nt = (nb + TREE_TIER - 1) / TREE_TIER;
        uint32_t *out = in + (uint64_t)TREE_NLEV * nb;
        hipLaunchKernelGGL(k_tree_tier, dim3(nt), dim3(TREE_TIER * TREE_NLEV), 0, s, A,
                           (const uint32_t *)in, nb, size, nt > 1 ? out : nullptr, nt);
        DZS_TRY(dzs_check_launch(ctx, "tree_tier"));
        in = out;
        nb = nt;
    }
    return DZS_OK;
}

dzs_status dzs_tree_refresh(dzs_ctx *ctx, const dzs_box *box, uint64_t n, const double *x,
                            const double *y, const double *z, const uint32_t *mult,
                            hipStream_t s) {
    if (!ctx->tree_built || n != ctx->tree_n)
        return dzs_fail(ctx, DZS_EINVAL, "tree refresh: no tree of %llu particles",
                        (unsigned long long)n);
    return tree_moments(ctx, box, (uint32_t)n, x, y, z, mult, nullptr, 1, 0u, 0, s);
}

dzs_status dzs_tree_build_ex(dzs_ctx *ctx, const dzs_box *box, uint64_t n64, const double *x,
                             const double *y, const double *z, const uint32_t *mult,
                             int leaf_size, int group_size, int KB, const dzs_bbox *boxes,
                             hipStream_t s) {
    const uint32_t n = (uint32_t)n64;
    ctx->tree_built = false;
    if (n == 0)
        return DZS_OK;
    uint32_t *bs = ctx->bstate;
    const uint32_t nb = (uint32_t)tree_blocks(n);
    const uint64_t words = (uint64_t)TREE_NLEV * nb;
    {
        dzs_timed t(ctx, KC_TREE_BUILD, s);
        hipLaunchKernelGGL(k_tree_levels, dim3(nb), dim3(TB_THREADS), 0, s, n,
                           (const uint64_t *)ctx->key, leaf_size, KB, (const uint32_t *)bs,
                           ctx->tree_sd, ctx->tree_cnt, ctx->grp_flag, ctx->tree_snap);
        DZS_TRY(dzs_check_launch(ctx, "tree_levels"));
        DZS_TRY(dzs_scan_u32(ctx, ctx->tree_cnt, ctx->tree_scan, words, ctx->tree_scan + words,
                             s));
        hipLaunchKernelGGL(k_tree_emit, dim3(nb), dim3(TB_THREADS), 0, s, n,
                           (const uint16_t *)ctx->tree_sd, (const uint32_t *)ctx->tree_scan,
                           ctx->cap_nodes, ctx->nd_first, ctx->nd_end, ctx->nd_child,
                           ctx->nd_cend, ctx->nd_level, (const uint32_t *)ctx->tree_snap,
                           ctx->tree_snap_e, bs);
        DZS_TRY(dzs_check_launch(ctx, "tree_emit"));
    }
    DZS_TRY(tree_moments(ctx, box, n, x, y, z, mult, boxes, 0, (uint32_t)group_size, KB, s));
    {
        dzs_timed t(ctx, KC_TREE_GROUPS, s);
        DZS_TRY(dzs_flag_list(ctx, n, ctx->grp_flag, ctx->grp_cnt, ctx->grp_scan, bs + BS_GROUPS,
                              ctx->grp_first, s));
    }
    ctx->tree_built = true;
    ctx->tree_n = n;
    return DZS_OK;
}

// The sticky overflow flags of the tree build (node capacity) and of the walk (stack depth),
// read back and cleared (synchronises the stream).
dzs_status dzs_tree_check(dzs_ctx *ctx, hipStream_t s) {
    DZS_HIP(ctx, hipMemcpyAsync(ctx->h_small + 8, ctx->bstate + BS_OVERFLOW, sizeof(uint32_t),
                                hipMemcpyDeviceToHost, s));
    DZS_HIP(ctx, hipMemcpyAsync(ctx->h_small + 9, ctx->walk_counter + 2, sizeof(uint32_t),
                                hipMemcpyDeviceToHost, s));
    DZS_HIP(ctx, hipMemcpyAsync(ctx->h_small + 11, ctx->bstate + DZS_BS_BADREPORT,
                                sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    DZS_HIP(ctx, hipStreamSynchronize(s));
    const uint32_t tree_over = ctx->h_small[8], walk_over = ctx->h_small[9];
    const uint32_t bad = ctx->h_small[11];
    if (tree_over || walk_over || bad) {
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(1), 0, s, (uint64_t)1,
                           ctx->bstate + BS_OVERFLOW, 0u);
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(1), 0, s, (uint64_t)1,
                           ctx->walk_counter + 2, 0u);
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(1), 0, s, (uint64_t)1,
                           ctx->bstate + DZS_BS_BADREPORT, 0u);
        DZS_HIP(ctx, hipStreamSynchronize(s));
    }
    if (bad)
        return dzs_fail(ctx, DZS_EINVAL, "tree_force: particles out of key order under "
                        "presorted, or a target index out of range (nothing was computed)");
    if (tree_over)
        return dzs_fail(ctx, DZS_ECAPACITY, "tree needs more than %llu nodes",
                        (unsigned long long)ctx->cap_nodes);
    if (walk_over)
        return dzs_fail(ctx, DZS_ECAPACITY, "tree walk stack overflow (depth %llu)",
                        (unsigned long long)ctx->walk_stack_depth);
    return DZS_OK;
}

// presorted input: keys (ctx->key) must ascend to the tree's depth; a descent flags the input
__global__ __launch_bounds__(TB_THREADS) void k_check_order(uint64_t n,
                                                            const uint64_t *__restrict__ key,
                                                            uint32_t *__restrict__ bad) {
    const int shift = 3 * (DZS_KEY_BITS - DZS_TREE_LEVELS);
    for (uint64_t i = (uint64_t)blockIdx.x * TB_THREADS + threadIdx.x; i + 1 < n;
         i += (uint64_t)gridDim.x * TB_THREADS)
        if ((key[i] >> shift) > (key[i + 1] >> shift))
            atomicOr(bad, 1u);
}

__global__ void k_latch_bad(uint32_t *bs) {
    bs[DZS_BS_BADREPORT] |= bs[DZS_BS_BADINPUT];
    bs[DZS_BS_BADINPUT] = 0u;
}

dzs_status dzs_latch_bad_input(dzs_ctx *ctx, hipStream_t s) {
    hipLaunchKernelGGL(k_latch_bad, dim3(1), dim3(1), 0, s, ctx->bstate);
    return dzs_check_launch(ctx, "latch_bad");
}

dzs_status dzs_check_order(dzs_ctx *ctx, uint64_t n, hipStream_t s) {
    if (n < 2)
        return DZS_OK;
    uint64_t nb = (n + TB_THREADS - 1) / TB_THREADS;
    nb = nb < 8192 ? nb : 8192;
    hipLaunchKernelGGL(k_check_order, dim3((uint32_t)nb), dim3(TB_THREADS), 0, s, n,
                       (const uint64_t *)ctx->key, ctx->bstate + DZS_BS_BADINPUT);
    return dzs_check_launch(ctx, "check_order");
}

// ---------------------------------------------------------------------------------------
// walk + pair evaluation (FP64)
//
// Lane layout: a wave holds G = 64/P targets; lane = t + G*s serves target t and evaluates
// every P-th list entry starting at s, so a group of G targets is served by all 64 lanes and
// a smaller G wastes fewer evaluations on sources inside the group's cutoff region but
// outside the target's cutoff sphere.  The P partial sums of a target are added in a fixed
// order at the end (deterministic).
//
// Split factor: S(u) = erfc(u/2) + u/sqrt(pi) exp(-u^2/4) = 1 - u w q(w), w = u^2, where
// q(w) = (erf(u/2) - u/sqrt(pi) e^{-u^2/4}) / u^3 is an entire function of w.  The host fits q
// on [0, (r_cut/r_s)^2] by a Chebyshev series (from its Taylor series in long double) and
// passes the monomial coefficients in t = 2 w / w_max - 1; the kernel evaluates it by Horner.
// The fit is checked on the host to 1e-12 relative error in S.
// ---------------------------------------------------------------------------------------
#define WALK_QN 18  // split-factor polynomial coefficients (Horner, fully unrolled): worst
                    // relative error in S 1.3e-13 at r_cut = 4.5 r_s, 7e-12 at 5 r_s
// FP32, outside the spline supports: F(w) = S(sqrt(w) / r_s) / w^1.5 from a table of cubics in
// w = r^2, one per interval of 1/32 of an octave of w (the interval is the exponent and the top
// five mantissa bits of w, so finding it takes no square root), over the 16 octaves up to the
// interval of r_cut^2, i.e. r from r_cut / 256.  The cubic of interval j sits in slot j mod 512,
// so any w finds a slot with one shift and one mask.  Its variable is the offset from the
// interval's low end over the power of two below it, y = (w - a) 2^-e, which is the low mantissa
// bits of w as they are: the coefficients are of the size of F in any unit of length (in powers of
// w - a the last one is some r^-9, past the FP32 range for r below 5.7e-5).  Cubics through the four Chebyshev nodes of the
// interval: worst error 2e-8 of F at small w, 1e-8 of the unsplit force near r_cut, before the
// FP32 rounding of the coefficients (the S table below with r^-3 from the hardware 1/sqrt:
// 8.5e-8 in S and four more roundings).  The walk's set-up kernel computes it for each call.
#define WALK_FT_BITS 5
#define WALK_FT_OCT 16
#define WALK_FT_N (WALK_FT_OCT << WALK_FT_BITS)
#define WALK_FT_SHIFT (23 - WALK_FT_BITS)
// the least interval of the table, w from 2^-83: the coefficients, up to some 4 F, are in the FP32
// range from there on (closer pairs take S and 1/sqrt)
#define WALK_FT_LEAST ((uint32_t)(127 - 83) << WALK_FT_BITS)
// FP32, close pairs (inside a spline support, or below the table of F): S(u) from a table of
// cubics, one per interval of u = r / r_s on [0, r_cut / r_s]: Hermite interpolation of S and
// dS/du at both ends of each interval (worst absolute error in S below 1e-7 at 64 intervals,
// FP32 coefficients included; checked on the host), plus an entry past the cutoff that extends
// the last one linearly.  The table rides in the kernel arguments; each workgroup stages both
// tables in LDS.
#define WALK_TAB_N 64
// list region / cutoff sphere below which an FP32 group evaluates densely: the one-pass loop
// wins even for wide groups (512^3 walk: 300 ms masked, 285 ms at 2.5, 282 ms at 3-4, 281 ms
// dense everywhere).  In FP64 the masked loop wins everywhere (128^3 walk: 2.38 ms masked, 2.40
// at 2.0, 2.81 dense everywhere), so the FP64 walk has no dense form.
#define WALK_DENSE_E 6.0
// waves of a walk workgroup: the FP32 form shares its tables among 8 waves (two workgroups of
// 67 KB fill a CU's 16 wave slots at 128 VGPRs); the waves work on their own groups and meet
// only once, when the tables are staged
template <typename T> struct walk_waves { static constexpr int N = 1; };
template <> struct walk_waves<float> { static constexpr int N = 8; };

struct walk_args {
    const uint32_t *grp_first;
    const uint32_t *n_groups;   // device: the build's group count
    const double *x, *y, *z;
    const uint32_t *mult;
    const dzs_node_rec *rec;  // the nodes as the walk reads them
    double L, halfL, rcut2, rcut, theta2, rs_inv, rs_inv2, G, m0, h0, t_scale;
    double *gx, *gy, *gz;
    int accumulate;
    int G_lanes;  // targets per wave (64 / phases)
    uint32_t *stack;
    uint32_t depth;
    uint32_t *counter;  // [0] next group, [2] overflow flag
    unsigned long long *pair_count;
    double q[WALK_QN];
    float4 stab[WALK_TAB_N + 1];  // FP32 form: the cubics of S(u), coefficients of f^0..f^3
    double stab_scale;            // intervals per unit of u (WALK_TAB_N r_s / r_cut)
    const float4 *ftab;           // FP32 form: the cubics of F(w), [WALK_FT_N] (device)
    float ft_lo;                  // the low end of the table of F (in w = r^2)
    // start cells: the walk of a group begins at the level-K nodes (and shallower leaves) of
    // the cells that meet its bounding box grown by r_cut, instead of at the root
    const uint32_t *cell_node;  // [8^K] node covering each level-K cell (Morton order)
    const uint8_t *cell_dl;     // [8^K] K - level of that node
    int cell_K;                 // 0: start at the root
    // a batch: the box of a group is its first particle's key prefix
    const uint64_t *key;
    const dzs_bbox *boxes;
    // relative opening criterion: previous |g| per target (nullptr: geometric) and
    // alpha_open / G (the walk's masses and distances carry no G)
    const float *aold;
    double alpha_g;
    // only flagged targets get a force (nullptr: every target); the force of tree slot i
    // goes to entry out_perm[i] (nullptr: i)
    const uint8_t *active;
    const uint32_t *out_perm;
    const uint32_t *bad;  // tree_force input rejected on the device: the walk does nothing
    // a kept, refreshed tree: targets are taken at the image next to the group's first one,
    // and a leaf flagged for members across a face keeps them all with minimum-image pairs;
    // the start cells are widened by the bound on every particle's displacement since the
    // build (device), since a node's particles may have left its cell
    int kept;
    const double *cell_extra;
    // only these targets (nullptr: the tree's groups): tgt[] in slot order, group g holding
    // tgt[tpos[g] .. tpos[g + 1]), g < *n_tgrp
    const uint32_t *tgt;
    const uint32_t *tpos;
    const uint32_t *n_tgrp;
};

// Geometry and constants of the box a group lives in.
struct walk_geom {
    double L, halfL, rcut, rcut2, rs_inv, rs_inv2, Gc, m0, h0, wide;
    uint32_t root;
};

// ---------------------------------------------------------------------------------------
// batch: the node of each box (the level-KB node with the box's key prefix)
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(TB_THREADS) void k_batch_roots(const uint32_t *__restrict__ bs,
                                                            int KB,
                                                            const uint64_t *__restrict__ key,
                                                            const uint32_t *__restrict__ nd_first,
                                                            dzs_bbox *__restrict__ boxes) {
    const uint32_t v = bs[BS_LEVEL + KB] + blockIdx.x * TB_THREADS + threadIdx.x;
    if (v < bs[BS_LEVEL + KB + 1])
        boxes[key[nd_first[v]] >> DZS_BATCH_SHIFT].root = v;
}

dzs_status dzs_batch_roots(dzs_ctx *ctx, dzs_bbox *boxes, hipStream_t s) {
    const int KB = DZS_BATCH_LEVELS;
    hipLaunchKernelGGL(k_batch_roots, dim3(blocks_for(1u << (3 * KB), TB_THREADS)),
                       dim3(TB_THREADS), 0, s, (const uint32_t *)ctx->bstate, KB,
                       (const uint64_t *)ctx->key, ctx->nd_first, boxes);
    return dzs_check_launch(ctx, "batch_roots");
}

// ---------------------------------------------------------------------------------------
// start cells
// ---------------------------------------------------------------------------------------
#define CELL_EMPTY 0xffffffffu

__global__ __launch_bounds__(TB_THREADS) void k_cell_clear(uint64_t n, uint32_t *cell_node) {
    const uint64_t i = (uint64_t)blockIdx.x * TB_THREADS + threadIdx.x;
    if (i < n)
        cell_node[i] = CELL_EMPTY;
}

// Every node at level K, and every leaf above level K, claims the level-K cells of its cube:
// in Morton order these form the contiguous range [P 8^(K-l), (P+1) 8^(K-l)), P = the node's
// key prefix.  The claimed ranges are disjoint; cells no node claims hold no particle.
__global__ __launch_bounds__(TB_THREADS) void k_cell_fill(
    const uint32_t *__restrict__ bs, int K, const uint64_t *__restrict__ key,
    const uint32_t *__restrict__ nd_first, const uint32_t *__restrict__ nd_child,
    const uint8_t *__restrict__ nd_level, uint32_t *__restrict__ cell_node,
    uint8_t *__restrict__ cell_dl) {
    const uint32_t node = blockIdx.x * TB_THREADS + threadIdx.x;
    if (node >= bs[BS_LEVEL + K + 1])  // the nodes of levels 0..K
        return;
    const int l = nd_level[node];
    if (l > K || (l < K && nd_child[node] != 0))   // (no node has the root for a child)
        return;
    const uint64_t P = key[nd_first[node]] >> (3 * (DZS_KEY_BITS - l));
    const int dl = K - l;
    const uint64_t lo = P << (3 * dl), hi = (P + 1) << (3 * dl);
    for (uint64_t m = lo; m < hi; ++m) {
        cell_node[m] = node;
        cell_dl[m] = (uint8_t)dl;
    }
}

// Arithmetic of the pair loop in the precision T of the form: FP64 (plain) or FP32
// (precision form; coordinates relative to the group centre, so FP32 keeps ~1e-7 of r_cut).
__device__ __forceinline__ double wfma(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float wfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double wmax(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ float wmax(float a, float b) { return fmaxf(a, b); }
template <typename T> __device__ __forceinline__ T wmin_image(T d, T L) {
    if (d >= T(0.5) * L)
        d -= L;
    else if (d < T(-0.5) * L)
        d += L;
    return d;
}

// Cubic-spline softened 1/r^3 (enclosed-mass force / r), r < h.
template <typename T> __device__ __forceinline__ T gsoft_inner(T r, T h) {
    const T hinv = T(1.0) / h;
    const T u = r * hinv;
    const T h3 = hinv * hinv * hinv;
    if (u < T(0.5))
        return h3 * (T(32.0 / 3.0) + u * u * (T(32.0) * u - T(192.0 / 5.0)));
    return h3 * (T(64.0 / 3.0) - T(48.0) * u + T(192.0 / 5.0) * u * u - T(32.0 / 3.0) * u * u * u -
                 T(1.0) / (T(15.0) * u * u * u));
}

// The interaction list in LDS: pm = position (shifted to the image nearest the group; in FP32
// relative to the group centre) and mass; hh = (hm2, h): the entry's spline support h and hm2 =
// max(h^2, the largest h_i^2 of the group's targets, the low end of the table of F), an upper
// bound of the pair's squared support that decides, with one comparison, whether the exact
// spline test is needed.  FP32: two arrays, one 16-byte and one 4-byte read per entry.
template <typename T> struct vec4_of;
template <> struct vec4_of<float> { typedef float4 type; typedef float2 half; };
struct dvec4 { double x, y, z, w; };
struct dvec2 { double x, y; };
template <> struct vec4_of<double> { typedef dvec4 type; typedef dvec2 half; };
struct dentry {   // 48 bytes: the masked loop's gathers spread over 16 bank offsets (8 at 32)
    dvec4 pm;
    dvec2 hh;
};
template <typename T> struct src_list;
template <> struct src_list<float> {
    float4 *p;
    float2 *h;
    __device__ __forceinline__ float4 &pm(uint32_t i) const { return p[i]; }
    __device__ __forceinline__ float2 &hh(uint32_t i) const { return h[i]; }
};
template <> struct src_list<double> {
    dentry *e;
    __device__ __forceinline__ dvec4 &pm(uint32_t i) const { return e[i].pm; }
    __device__ __forceinline__ dvec2 &hh(uint32_t i) const { return e[i].hh; }
};
template <typename T> struct list_lds;
template <> struct list_lds<float> {
    float4 p[WALK_LIST + 64];
    float2 h[WALK_LIST + 64];
    __device__ __forceinline__ src_list<float> list() { return {p, h}; }
};
template <> struct list_lds<double> {
    dentry e[WALK_LIST + 16];
    __device__ __forceinline__ src_list<double> list() { return {e}; }
};

// Ordering of LDS and stack accesses between the lanes of one wave (its LDS operations complete
// in order; only the compiler must keep them in place).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

template <typename T> struct split_coef;
template <> struct split_coef<double> {
    static constexpr int N = WALK_QN;
    static __device__ __forceinline__ double at(const walk_args &A, int k) { return A.q[k]; }
};

// 1/sqrt: the FP32 form takes the hardware approximation (about 1 ulp; its inputs are far
// from the denormal range).  The plain form refines the hardware FP64 estimate y by one
// third-order Newton step, y (1 + e/2 + 3 e^2/8) with e = 1 - a y^2, which takes a relative
// error eps to about (5/16) eps^3; a is a positive, normal squared separation here, so the
// special-value handling of the library's rsqrt is not needed.
__device__ __forceinline__ double pair_rsqrt(double a) {
    const double y = __builtin_amdgcn_rsq(a);
    const double e = __builtin_fma(-a * y, y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ float pair_rsqrt(float a) { return __builtin_amdgcn_rsqf(a); }
// The larger of two non-negative squared supports (no NaN canonicalisation needed).
__device__ __forceinline__ double pair_hmax(double a, double b) { return a > b ? a : b; }
__device__ __forceinline__ float pair_hmax(float a, float b) {
    return __uint_as_float(max(__float_as_uint(a), __float_as_uint(b)));
}

// Separation of a list entry from the target (minimum image for wide groups).
template <typename T, bool MINIMG, typename E>
__device__ __forceinline__ T pair_sep(const E &e, T xi, T yi, T zi, T L, T &dx, T &dy,
                                      T &dz) {
    dx = e.x - xi;
    dy = e.y - yi;
    dz = e.z - zi;
    if (MINIMG) {
        dx = wmin_image(dx, L);
        dy = wmin_image(dy, L);
        dz = wmin_image(dz, L);
    }
    return wfma(dx, dx, wfma(dy, dy, dz * dz));
}

// Pair force factor g (the force on the target is m r_ij g): g_soft(r) S(r/r_s) with
// S = 1 - u^3 q(u^2), u = r/r_s; outside the spline support g_soft = r^-3 and the product is
// r^-3 - r_s^-3 q, one fused operation.  (FP64; the FP32 form is pair_factor_tab.)
template <typename T>
__device__ __forceinline__ T pair_factor(const walk_args &A, T r2, T eh, T hm2, T hi, T hi2,
                                         T rs_inv2, T rs_inv3, T t_scale) {
    constexpr int QN = split_coef<T>::N;
    const T rinv = pair_rsqrt(r2);
    const T w = r2 * rs_inv2;
    const T t = wfma(w, t_scale, T(-1.0));
    T q = split_coef<T>::at(A, QN - 1);
#pragma unroll
    for (int c = QN - 2; c >= 0; --c)
        q = wfma(q, t, split_coef<T>::at(A, c));
    const T rq = rs_inv3 * q;
    T g = wfma(rinv * rinv, rinv, -rq);
    if (r2 < hm2 && r2 < pair_hmax(eh * eh, hi2)) {
        const T r = r2 * rinv;
        const T ks = gsoft_inner(r, wmax(eh, hi));
        g = ks - ks * (r2 * r) * rq;
    }
    return g;
}

// FP32 pair force factor g_soft(r) S(r/r_s) with S from the LDS table: x = u WALK_TAB_N / u_cut
// = r tscale, interval k = floor(x) (at most WALK_TAB_N, the entry past the cutoff), the cubic
// at f = x - k; in the spline only where r2 < hm2 (the entry's bound) and the exact test holds.
// x in [WALK_TAB_N, ...) (r at or past r_cut: only a pair within rounding of the cutoff is
// kept) takes the last entry at the fraction of x, a linear continuation from S(r_cut).
// r2 = 0 (the target itself) makes the factor NaN: the caller leaves the pair out.
__device__ __forceinline__ float pair_factor_tab(const float4 *__restrict__ tab, float r2,
                                                float hm2, const float *eh_ptr, float hi,
                                                float hi2, float tscale) {
    const float rinv = pair_rsqrt(r2);
    const float r = r2 * rinv;
    const float x = r * tscale;
    uint32_t k = (uint32_t)x;
    k = k < (uint32_t)WALK_TAB_N ? k : (uint32_t)WALK_TAB_N;
    const float f = __builtin_amdgcn_fractf(x);
    const float4 c = tab[k];
    const float S = __builtin_fmaf(__builtin_fmaf(__builtin_fmaf(c.w, f, c.z), f, c.y), f, c.x);
    float g = (rinv * rinv) * (rinv * S);
    if (r2 < hm2) {  // rare: the exact spline test
        const float eh = *eh_ptr;
        if (r2 < pair_hmax(eh * eh, hi2))
            g = gsoft_inner(r, fmaxf(eh, hi)) * S;
    }
    return g;
}

template <typename T, bool FT> struct pair_eval;
template <> struct pair_eval<double, false> {
    const walk_args *A;
    double rs_inv2, rs_inv3, t_scale;
    // hh: the entry's (hm2, h)
    __device__ __forceinline__ double operator()(double r2, const dvec2 *hh, double hi,
                                                 double hi2) const {
        const dvec2 v = *hh;
        return pair_factor<double>(*A, r2, v.y, v.x, hi, hi2, rs_inv2, rs_inv3, t_scale);
    }
};
template <> struct pair_eval<float, false> {
    const float4 *tab;
    float tscale;
    __device__ __forceinline__ float operator()(float r2, const float2 *hh, float hi,
                                                float hi2) const {
        return pair_factor_tab(tab, r2, hh->x, &hh->y, hi, hi2, tscale);
    }
};
// FP32 with far pairs' F from its table at w = r2.  The slot of a w outside the table holds
// another interval's cubic: such a w belongs to a close pair, a pair past the cutoff or a
// sentinel, whose F is not used.
template <> struct pair_eval<float, true> {
    const float4 *tab, *ftab;
    float tscale;
    __device__ __forceinline__ float far(float w) const {
        const uint32_t bits = __float_as_uint(w);
        const float4 c = ftab[(bits >> WALK_FT_SHIFT) & (uint32_t)(WALK_FT_N - 1)];
        const float y = __uint_as_float((bits & ((1u << WALK_FT_SHIFT) - 1u)) | 0x3f800000u) - 1.0f;
        return __builtin_fmaf(__builtin_fmaf(__builtin_fmaf(c.w, y, c.z), y, c.y), y, c.x);
    }
    // r2 = 0 (the target itself): any finite factor, its separation is zero
    __device__ __forceinline__ float close(float r2, const float *eh, float hi, float hi2) const {
        return r2 == 0.0f ? 0.0f
                          : pair_factor_tab(tab, r2, __builtin_inff(), eh, hi, hi2, tscale);
    }
    __device__ __forceinline__ float operator()(float r2, const float2 *hh, float hi,
                                                float hi2) const {
        float g = far(r2);
        if (r2 < hh->x)   // rare
            g = close(r2, &hh->y, hi, hi2);
        return g;
    }
};

// The lane's share of the list (entries s, s + P, s + 2P, ...) in two passes per block of 32
// of its entries: a cheap pass shifts one acceptance bit per entry (inside r_cut, not the
// target itself) into a 32-bit mask, first entry highest, then the lane evaluates only the
// marked pairs in ascending order.  A list culled against the group's box holds several
// times more entries than any one target's cutoff sphere; without the mask the whole wave
// would step through the force arithmetic for every entry some lane accepts.  The caller
// fills the P entries past the list with far-away sentinels, so the block bound is uniform.
template <typename T, bool MINIMG, typename Ev>
__device__ __forceinline__ void pair_loop(const Ev &ev, const walk_geom &W,
                                          const src_list<T> src, uint32_t nlist, uint32_t s,
                                          uint32_t P, T xi, T yi, T zi, T hi, T hi2, T &ax,
                                          T &ay, T &az, bool active, uint32_t &n_pairs) {
    const T rcut2 = T(W.rcut2), L = T(W.L);
    // entries per lane: uniform, so the block loops run on the scalar unit
    const uint32_t n_max = (uint32_t)__builtin_amdgcn_readfirstlane((int)((nlist + P - 1) / P));
    for (uint32_t kb = 0; kb < n_max; kb += 32u) {
        const uint32_t blk = s + kb * P;
        const uint32_t kmax =
            (uint32_t)__builtin_amdgcn_readfirstlane((int)(n_max - kb < 32u ? n_max - kb : 32u));
        uint32_t mask = 0;
        for (uint32_t k = 0; k < kmax; ++k) {
            T dx, dy, dz;
            const T r2 = pair_sep<T, MINIMG>(src.pm(blk + k * P), xi, yi, zi, L, dx, dy, dz);
            mask = mask + mask + ((r2 < rcut2 && r2 > T(0.0)) ? 1u : 0u);
        }
        mask = active ? mask << (32u - kmax) : 0u;   // targets nobody asked for: no pairs
        n_pairs += (uint32_t)__popc(mask);
        while (mask) {
            const uint32_t k = (uint32_t)__builtin_clz(mask);
            mask ^= 0x80000000u >> k;
            const auto e = src.pm(blk + k * P);
            T dx, dy, dz;
            const T r2 = pair_sep<T, MINIMG>(e, xi, yi, zi, L, dx, dy, dz);
            const T f = e.w * ev(r2, &src.hh(blk + k * P), hi, hi2);
            ax = wfma(f, dx, ax);
            ay = wfma(f, dy, ay);
            az = wfma(f, dz, az);
        }
    }
}

// 0 < r2 < rcut2 by one unsigned comparison of the bit patterns (r2 is a sum of squares: +0,
// positive, or +inf for the far sentinels), so the result is a single mask
__device__ __forceinline__ bool pair_inside(float r2, float rcut2) {
    return __float_as_uint(r2) - 1u < __float_as_uint(rcut2) - 1u;
}

// The dense loop with S and 1/sqrt for every pair, and minimum-image pairs: phase s takes the
// entries s, s + P, ...
template <bool MINIMG>
__device__ __forceinline__ void pair_dense_s(const pair_eval<float, false> &ev, float rcut2,
                                             float L, const src_list<float> src, uint32_t nlist,
                                             uint32_t s, uint32_t P, float xi, float yi, float zi,
                                             float hi, float hi2, float &ax, float &ay, float &az,
                                             uint64_t act_mask, uint32_t &np_wave) {
    const uint32_t n_max = (uint32_t)__builtin_amdgcn_readfirstlane((int)((nlist + P - 1) / P));
    uint32_t cnt = 0;   // wave-uniform, kept on the scalar unit
    for (uint32_t k = 0; k < n_max; ++k) {
        const float4 e = src.pm(s + k * P);
        float dx, dy, dz;
        const float r2 = pair_sep<float, MINIMG>(e, xi, yi, zi, L, dx, dy, dz);
        const bool in = pair_inside(r2, rcut2);
        // pairs of the flagged targets, counted on the scalar unit
        cnt = (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)(cnt + (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(in) & act_mask)));
        const float g = ev(r2, &src.hh(s + k * P), hi, hi2);
        // the factor of a pair outside (or of the target itself: r = 0) is not used
        const float f = in ? e.w * g : 0.0f;
        ax = wfma(f, dx, ax);
        ay = wfma(f, dy, ay);
        az = wfma(f, dz, az);
    }
    np_wave += cnt;
}

// The lane's share of the list (FP32) in one pass: every entry is evaluated and the pairs
// outside r_cut are multiplied by zero.  Phase s takes the entries s K .. s K + K - 1, K even,
// two per iteration; all lanes of a phase read the same entry and every lane works on every
// iteration, so when most of the list lies inside most targets' cutoff spheres (a compact group)
// this costs less than the masked two-pass loop.  The caller puts sentinels, or entries outside
// every target's cutoff, in the up to 2 P slots past the list.
//
// VALU-issue bound (the vector units of every SIMD are busy throughout), so its instructions
// per entry are its cost: 21 (6 separation, 2 slot, 2 offset in the interval, 3 cubic, 1 cutoff
// test, 1 close test, 5 mass, select and accumulation, the address) against 28 and a 1/sqrt at
// a quarter of the rate with S from a table of r.  With the list flushed at one place (the pair
// loops are in the kernel once, not three times) and short groups on fewer lanes: 256^3 walk
// 28.0 -> 22.2 ms, 512^3 193 -> 153 ms.
//
// The pairs inside r_cut are counted on the scalar unit; a pair at zero separation (the target
// itself) counts there too, always is a close pair and is taken off there (n_zero).
__device__ __forceinline__ void pair_dense(const pair_eval<float, true> &ev, float rcut2,
                                           const src_list<float> src, uint32_t nlist, uint32_t s,
                                           uint32_t P, float xi, float yi, float zi, float hi,
                                           float hi2, float &ax, float &ay, float &az,
                                           uint64_t act_mask, uint32_t &np_wave,
                                           uint32_t &n_zero) {
    const uint32_t K = ((nlist + P - 1) / P + 1u) & ~1u;
    const uint32_t n_max = (uint32_t)__builtin_amdgcn_readfirstlane((int)K);
    const float4 *pm = src.p + s * K;
    const float2 *hh = src.h + s * K;
    uint32_t cnt = 0;   // wave-uniform, kept on the scalar unit
    for (uint32_t k = 0; k < n_max; k += 2u, pm += 2, hh += 2) {
        const float4 e0 = pm[0], e1 = pm[1];
        const float b0 = hh[0].x, b1 = hh[1].x;
        float dx0, dy0, dz0, dx1, dy1, dz1;
        const float r0 = pair_sep<float, false>(e0, xi, yi, zi, 0.0f, dx0, dy0, dz0);
        const float r1 = pair_sep<float, false>(e1, xi, yi, zi, 0.0f, dx1, dy1, dz1);
        float g0 = ev.far(r0), g1 = ev.far(r1);
        const bool in0 = r0 < rcut2, in1 = r1 < rcut2;
        // pairs of the flagged targets
        cnt += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(in0) & act_mask) +
               (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(in1) & act_mask);
        const bool c0 = r0 < b0, c1 = r1 < b1;
        if (c0 || c1) {   // rare
            const uint32_t one = (uint32_t)(act_mask >> (threadIdx.x & 63u)) & 1u;
            if (c0) {
                g0 = ev.close(r0, &hh[0].y, hi, hi2);
                n_zero += r0 == 0.0f ? one : 0u;
            }
            if (c1) {
                g1 = ev.close(r1, &hh[1].y, hi, hi2);
                n_zero += r1 == 0.0f ? one : 0u;
            }
        }
        // the factor of a pair outside is not used
        const float f0 = in0 ? e0.w * g0 : 0.0f, f1 = in1 ? e1.w * g1 : 0.0f;
        ax = wfma(f0, dx0, ax);
        ay = wfma(f0, dy0, ay);
        az = wfma(f0, dz0, az);
        ax = wfma(f1, dx1, ax);
        ay = wfma(f1, dy1, ay);
        az = wfma(f1, dz1, az);
    }
    np_wave += (uint32_t)__builtin_amdgcn_readfirstlane((int)cnt);
}

// 4 waves per SIMD (128 VGPRs), at the price of spills around the pair loops: 10 to 18 VGPRs in
// FP64 with start cells or in a batch, 12 to 22 in FP32 (3 waves without them: 256^3 FP32 28.1 ms
// against 23.1 at the time).  The FP32 teams of two get 3: every two waves hold the tables (23.7
// KB a workgroup), so the LDS allows no more and the compiler takes 155 to 166 VGPRs.
//
// TEAM > 1: the workgroup's TEAM waves take every group together.  Each walks the tree and fills
// its own list (the same one), evaluates every TEAM-th of its entries, and the first adds the
// partial sums, wave by wave.  The walk proper is done TEAM times over, the pairs once: for the
// case that the groups are too few to keep every wave busy to the end, where one group of a
// dense clump can take as long as the whole launch.
//
// FT (FP32): far pairs from the table of F.  Not for a batch: its boxes' r_s differ, so F would
// need another scaling per pair; it keeps S, the order of its sums and with them the bits of
// its forces.
template <typename T, bool CELLS, bool BATCH, int TEAM, bool FT>
__global__ __launch_bounds__(64 * (TEAM > 1 ? TEAM : walk_waves<T>::N), 4) void k_tree_walk(
    walk_args A) {
    static_assert(!(CELLS && BATCH), "a batch walk starts at the box nodes");
    static_assert(sizeof(T) == 4 || !FT, "the table of F is FP32");
    static_assert(sizeof(T) == 8 || FT || TEAM == 1, "the order of the sums is kept");
    constexpr int KBL = BATCH ? DZS_BATCH_LEVELS : 0;  // tree levels above a box
    constexpr bool F32 = sizeof(T) == 4;
    constexpr bool COOP = TEAM > 1;
    constexpr int WAVES = COOP ? TEAM : walk_waves<T>::N;
    // each wave's own list, leaf queue and half boxes
    struct wave_lds {
        list_lds<T> list;
        double q_org[3][64];   // a queued leaf's origin in the list frame (image shift)
        uint32_t q_first[64], q_wide[64], q_mark[64], q_pref[64];
        uint32_t g;
        float hbox[F32 ? 12 : 1];
    };
    __shared__ float4 s_ftab[FT ? WALK_FT_N : 1];
    __shared__ float4 s_tab[F32 ? WALK_TAB_N + 1 : 1];
    __shared__ wave_lds s_wave[WAVES];

    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    wave_lds &S = s_wave[wave];
    const src_list<T> src = S.list.list();
    uint32_t *const q_first = S.q_first, *const q_pref = S.q_pref, *const q_wide = S.q_wide,
                    *const q_mark = S.q_mark;
    double(*const q_org)[64] = S.q_org;
    float *const s_hbox = S.hbox;
    const uint32_t team = (uint32_t)TEAM, member = COOP ? wave : 0u;
    const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    uint32_t *stk = A.stack + ((uint64_t)blockIdx.x * WAVES + wave) * A.depth;
    if (A.bad && *A.bad)
        return;
    if (F32) {
        for (uint32_t k = threadIdx.x; k <= WALK_TAB_N; k += 64 * WAVES)
            s_tab[k] = A.stab[k];
        if (FT)
            for (uint32_t k = threadIdx.x; k < WALK_FT_N; k += 64 * WAVES)
                s_ftab[k] = A.ftab[k];
        __syncthreads();
    }

    // A wave's first group follows from its place (neighbouring groups to different workgroups,
    // so that few groups spread over the chip), the others from the counter.
    const uint32_t n_first = gridDim.x * (COOP ? 1u : (uint32_t)WAVES);
    uint32_t g = (COOP ? 0u : wave * gridDim.x) + blockIdx.x;
    for (bool again = false;; again = true) {
        if (again && COOP) {   // every wave of the workgroup comes here once per group
            if (threadIdx.x == 0)
                s_wave[0].g = n_first + atomicAdd(&A.counter[0], 1u);
            __syncthreads();
            g = s_wave[0].g;
            __syncthreads();
        } else if (again) {
            if (lane == 0)
                S.g = n_first + atomicAdd(&A.counter[0], 1u);
            wave_sync();
            g = S.g;
            wave_sync();
        }
        // lanes: G targets, P phases (lane = target + G phase)
        uint32_t G = (uint32_t)A.G_lanes, P = 64u / G;
        uint32_t tl = lane % G, ph = lane / G;
        uint32_t first, cnt;
        if (A.tgt) {
            if (g >= *A.n_tgrp)
                break;
            first = A.tpos[g];
            cnt = A.tpos[g + 1] - first;
            if (cnt == 0u)
                continue;   // a group start with no flagged target before the next one
        } else {
            if (g >= *A.n_groups)
                break;
            first = A.grp_first[g];
            cnt = A.grp_first[g + 1] - first;
        }
        // a source node and the group may be wide enough that the image nearest the group
        // centre is not every pair's nearest image: an entry kept for the group lies within
        // 2 (h_node + h_group) + r_cut of any of its targets per axis, which must not exceed
        // L/2; above W.wide (half-extent sum (L/2 - r_cut) / 2) the pair loop reduces each
        // separation to the minimum image
        walk_geom W;
        if (BATCH) {
            const dzs_bbox &bx = A.boxes[A.key[first] >> DZS_BATCH_SHIFT];
            W = walk_geom{bx.L,      bx.halfL,   bx.r_cut, bx.rcut2, bx.rs_inv, bx.rs_inv2,
                          bx.G,      bx.m0,      bx.h0,    bx.wide_limit, bx.root};
        } else {
            W = walk_geom{A.L,  A.halfL, A.rcut, A.rcut2, A.rs_inv, A.rs_inv2,
                          A.G,  A.m0,    A.h0,   0.5 * (A.halfL - A.rcut), 0u};
        }
        bool valid = tl < cnt;
        uint32_t i = A.tgt ? A.tgt[valid ? first + tl : first] : (valid ? first + tl : first);
        bool active = valid && (!A.active || A.active[i] != 0);
        if (A.active && __ballot(active) == 0ull)
            continue;  // no target in this group
        double xi = A.x[i], yi = A.y[i], zi = A.z[i];
        if (A.kept) {
            const double x0 = __shfl(xi, 0, 64), y0 = __shfl(yi, 0, 64), z0 = __shfl(zi, 0, 64);
            xi = xi - x0 > W.halfL ? xi - W.L : (xi - x0 < -W.halfL ? xi + W.L : xi);
            yi = yi - y0 > W.halfL ? yi - W.L : (yi - y0 < -W.halfL ? yi + W.L : yi);
            zi = zi - z0 > W.halfL ? zi - W.L : (zi - z0 < -W.halfL ? zi + W.L : zi);
        }
        double hi = W.h0 * mult_cbrt(A.mult[i]);
        // group bounding box
        double mnx = xi, mny = yi, mnz = zi, mxx = xi, mxy = yi, mxz = zi;
        for (int o = 32; o >= 1; o >>= 1) {
            mnx = fmin(mnx, __shfl_xor(mnx, o, 64));
            mny = fmin(mny, __shfl_xor(mny, o, 64));
            mnz = fmin(mnz, __shfl_xor(mnz, o, 64));
            mxx = fmax(mxx, __shfl_xor(mxx, o, 64));
            mxy = fmax(mxy, __shfl_xor(mxy, o, 64));
            mxz = fmax(mxz, __shfl_xor(mxz, o, 64));
        }
        const double gcx = 0.5 * (mnx + mxx), gcy = 0.5 * (mny + mxy), gcz = 0.5 * (mnz + mxz);
        const double ghx = 0.5 * (mxx - mnx), ghy = 0.5 * (mxy - mny), ghz = 0.5 * (mxz - mnz);
        const double ghmax = fmax(ghx, fmax(ghy, ghz));
        // the list is culled to the group's box grown by r_cut (Steiner: volume, surface,
        // edge and ball terms); when that region is at most WALK_DENSE_E times one cutoff
        // sphere, enough entries are inside enough targets' spheres to evaluate densely
        const double rc = W.rcut, pi = 3.14159265358979323846;
        const double v_ball = (4.0 / 3.0) * pi * rc * rc * rc;
        const double v_list = 8.0 * ghx * ghy * ghz + 8.0 * rc * (ghx * ghy + ghy * ghz + ghz * ghx) +
                              2.0 * pi * rc * rc * (ghx + ghy + ghz) + v_ball;
        // (every lane holds the same group box: a wave-uniform choice)
        const bool dense = F32 && G >= 4u && __builtin_amdgcn_readfirstlane(
                                                 v_list <= WALK_DENSE_E * v_ball ? 1 : 0) != 0;
        // relative criterion: alpha / G times the smallest previous |g| of the group
        double alpha_a = 0.0;
        if (A.aold) {
            double a = valid ? (double)A.aold[i] : __builtin_inf();
            for (int o = 32; o >= 1; o >>= 1)
                a = fmin(a, __shfl_xor(a, o, 64));
            alpha_a = A.alpha_g * a;
        }
        // A group of at most half its G lanes' targets (cut short by the tree, or a short run of
        // listed targets) has fewer targets and more phases; lane t holds target t already.  (By
        // the group's count and not by its active targets: a target's force is the same bits
        // whichever others are asked for.)  The floor keeps the phases' sentinels inside the
        // list's spare slots.
        if (!F32 || FT) {
            uint32_t Ge = COOP ? (F32 ? 16u : 4u) : (F32 ? 4u : 2u);
            while (Ge < cnt)
                Ge <<= 1;
            if (Ge < G) {
                G = Ge;
                P = 64u / G;
                tl = lane % G;
                ph = lane / G;
                valid = tl < cnt;
                const int from = valid ? (int)tl : 0;
                active = __shfl((int)active, from, 64) != 0 && valid;
                i = (uint32_t)__shfl((int)i, from, 64);
                xi = __shfl(xi, from, 64);
                yi = __shfl(yi, from, 64);
                zi = __shfl(zi, from, 64);
                hi = __shfl(hi, from, 64);
            }
        }
        // list coordinates: absolute in FP64, relative to the group centre in FP32
        const bool rel = sizeof(T) == 4;
        const double ox = rel ? gcx : 0.0, oy = rel ? gcy : 0.0, oz = rel ? gcz : 0.0;
        const T txi = T(xi - ox), tyi = T(yi - oy), tzi = T(zi - oz), thi = T(hi);
        const T thi2 = thi * thi;
        // the largest squared support among the group's targets (the bound stored as hm2)
        T hg2 = valid ? thi2 : T(0.0);
        for (int o = 32; o >= 1; o >>= 1)
            hg2 = wmax(hg2, (T)__shfl_xor(hg2, o, 64));
        if constexpr (FT) {
            // pairs below the table of F are close pairs too (a few ulps above its low end)
            hg2 = wmax(hg2, 1.000001f * A.ft_lo);
        }
        const T m_unit = T(W.m0), h_unit = T(W.h0);
        const typename vec4_of<T>::half hh_unit = {wmax(h_unit * h_unit, hg2), h_unit};
        // A dense FP32 group is evaluated as two halves, A (its targets 0 .. G/2-1) and B
        // (G/2 .. G-1), compact in Morton order, each against the entries near its own box: at
        // every flush the list is reordered (stably) into the entries near A only, near both and
        // near B only, so that each half steps through a contiguous part of it with twice the
        // phases.  Entries farther than r_cut from both boxes are dropped.
        const uint32_t Gh = G >> 1;
        const uint32_t Ph = G >= 4u ? 64u / Gh : 1u;
        bool halves = false;        // the sums are the halves' (the group layout's otherwise)
        float rc_cls2 = 0.0f;
        if (F32 && dense) {
            const float inf = __builtin_inff();
            float b[6] = {valid ? float(txi) : inf, valid ? float(tyi) : inf,
                          valid ? float(tzi) : inf, valid ? float(txi) : -inf,
                          valid ? float(tyi) : -inf, valid ? float(tzi) : -inf};
            for (uint32_t o = 1; o < Gh; o <<= 1)
                for (int c = 0; c < 6; ++c) {
                    const float t = __shfl_xor(b[c], (int)o, 64);
                    b[c] = c < 3 ? fminf(b[c], t) : fmaxf(b[c], t);
                }
            // the halves' boxes (lo x, y, z, hi x, y, z in the group-centre frame) to LDS
            if (lane == 0u || lane == Gh)
                for (int c = 0; c < 6; ++c)
                    s_hbox[lane == 0u ? c : 6 + c] = b[c];
            // a few FP32 ulps of the largest coordinate above r_cut, so that the box test never
            // drops an entry the pair test would take
            const double rc_m = W.rcut * (1.0 + 1e-6) + 1e-6 * (W.rcut + 2.0 * ghmax);
            rc_cls2 = __double2float_ru(rc_m * rc_m);
        }

        pair_eval<T, FT> ev;
        if constexpr (F32) {
            ev.tab = s_tab;
            if constexpr (FT)
                ev.ftab = s_ftab;
            ev.tscale = float(A.stab_scale * W.rs_inv);
        } else {
            ev.A = &A;
            ev.rs_inv2 = W.rs_inv2;
            ev.rs_inv3 = W.rs_inv * W.rs_inv2;
            ev.t_scale = A.t_scale;
        }
        T ax = T(0.0), ay = T(0.0), az = T(0.0);   // the lane's partial sums (half A's)
        T bx = T(0.0), by = T(0.0), bz = T(0.0);   // half B's
        uint32_t nlist = 0;
        // the masked loop's P sentinels fit behind the list (16 slots in FP64)
        const uint32_t PT = P * team;
        const uint32_t list_cap = F32 || PT <= 16u ? WALK_LIST : WALK_LIST + 16u - PT;
        uint32_t n_pairs = 0;   // per lane (the masked loop)
        uint32_t np_wave = 0;   // the wave's (the dense loop)
        uint32_t n_zero = 0;    // per lane: pairs at zero separation it counted
        bool wide = false;

        // The halves' sums in the group layout: fixed-order sums of the Ph partial accelerations
        // of each half's targets, moved to the target's first lane.
        auto fold = [&]() {
            for (uint32_t o = Gh; o < 64; o <<= 1) {
                ax += __shfl_xor(ax, o, 64);
                ay += __shfl_xor(ay, o, 64);
                az += __shfl_xor(az, o, 64);
                bx += __shfl_xor(bx, o, 64);
                by += __shfl_xor(by, o, 64);
                bz += __shfl_xor(bz, o, 64);
            }
            const int sl = (int)(tl % Gh);
            const T ax2 = __shfl(ax, sl, 64), ay2 = __shfl(ay, sl, 64), az2 = __shfl(az, sl, 64);
            const T bx2 = __shfl(bx, sl, 64), by2 = __shfl(by, sl, 64), bz2 = __shfl(bz, sl, 64);
            const bool inA = tl < Gh;
            ax = ph == 0u ? (inA ? ax2 : bx2) : T(0.0);
            ay = ph == 0u ? (inA ? ay2 : by2) : T(0.0);
            az = ph == 0u ? (inA ? az2 : bz2) : T(0.0);
            halves = false;
        };

        // The list's interactions into the sums: compact lists by the dense halves, the others
        // (and the rare lists that need minimum-image pairs) by the masked loop.
        auto flush = [&]() {
            bool masked = true;
            if constexpr (F32) {
                if (dense && (!wide || !FT)) {
                    masked = false;
                    halves = true;
                    uint32_t n1 = 0u, n2 = nlist, n3 = 0u;
                    if (FT || !wide) {
                        // lane l holds entries l and l + 64 (the list holds at most 128)
                        static_assert(WALK_LIST <= 128, "two list entries per lane");
                        float hbA[6], hbB[6];
                        for (int c = 0; c < 6; ++c) {
                            hbA[c] = s_hbox[c];
                            hbB[c] = s_hbox[6 + c];
                        }
                        float4 p0 = {0.0f, 0.0f, 0.0f, 0.0f}, p1 = p0;
                        float2 q0 = {0.0f, 0.0f}, q1 = q0;
                        uint32_t c0 = 0u, c1 = 0u;   // 1 near A only, 2 near both, 3 near B only
                        auto cls = [&](const float4 &p) -> uint32_t {
                            auto d2 = [&](const float *bx_) {
                                const float dx = fmaxf(fmaxf(bx_[0] - p.x, p.x - bx_[3]), 0.0f);
                                const float dy = fmaxf(fmaxf(bx_[1] - p.y, p.y - bx_[4]), 0.0f);
                                const float dz = fmaxf(fmaxf(bx_[2] - p.z, p.z - bx_[5]), 0.0f);
                                return __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
                            };
                            const bool a = d2(hbA) < rc_cls2, b = d2(hbB) < rc_cls2;
                            return a ? (b ? 2u : 1u) : (b ? 3u : 0u);
                        };
                        if (lane < nlist) {
                            p0 = src.pm(lane);
                            q0 = src.hh(lane);
                            c0 = cls(p0);
                        }
                        if (lane + 64u < nlist) {
                            p1 = src.pm(lane + 64u);
                            q1 = src.hh(lane + 64u);
                            c1 = cls(p1);
                        }
                        const uint64_t m01 = __ballot(c0 == 1u), m02 = __ballot(c0 == 2u),
                                       m03 = __ballot(c0 == 3u), m11 = __ballot(c1 == 1u),
                                       m12 = __ballot(c1 == 2u), m13 = __ballot(c1 == 3u);
                        n1 = (uint32_t)(__popcll(m01) + __popcll(m11));
                        n2 = (uint32_t)(__popcll(m02) + __popcll(m12));
                        n3 = (uint32_t)(__popcll(m03) + __popcll(m13));
                        // stable destinations: class base, then the entries of the class before
                        const uint32_t s0 =
                            c0 == 1u ? (uint32_t)__popcll(m01 & lt_mask)
                                     : (c0 == 2u ? n1 + (uint32_t)__popcll(m02 & lt_mask)
                                                 : n1 + n2 + (uint32_t)__popcll(m03 & lt_mask));
                        const uint32_t r11 = (uint32_t)(__popcll(m01) + __popcll(m11 & lt_mask));
                        const uint32_t r12 = (uint32_t)(__popcll(m02) + __popcll(m12 & lt_mask));
                        const uint32_t r13 = (uint32_t)(__popcll(m03) + __popcll(m13 & lt_mask));
                        const uint32_t s1 = c1 == 1u ? r11 : (c1 == 2u ? n1 + r12 : n1 + n2 + r13);
                        wave_sync();   // every entry read before any is moved
                        if (c0 != 0u) {
                            src.pm(s0) = p0;
                            src.hh(s0) = q0;
                        }
                        if (c1 != 0u) {
                            src.pm(s1) = p1;
                            src.hh(s1) = q1;
                        }
                    }
                    // sentinels (2 Ph team <= 64): far outside every cutoff
                    if (lane < 2u * Ph * team) {
                        src.pm(n1 + n2 + n3 + lane) = {T(1e30), T(1e30), T(1e30), T(0.0)};
                        src.hh(n1 + n2 + n3 + lane) = {T(0.0), T(0.0)};
                    }
                    wave_sync();
                    const uint32_t sph = lane / Gh + Ph * member, t0 = lane % Gh;
                    {
                        const int ts = (int)t0;   // main-layout lane of the target (half A)
                        const T xs = __shfl(txi, ts, 64), ys = __shfl(tyi, ts, 64),
                                zs = __shfl(tzi, ts, 64), hs = __shfl(thi, ts, 64);
                        const uint64_t am = __ballot(__shfl((int)active, ts, 64) != 0);
                        if constexpr (FT)
                            pair_dense(ev, T(W.rcut2), src, n1 + n2, sph, Ph * team, xs, ys, zs,
                                       hs, hs * hs, ax, ay, az, am, np_wave, n_zero);
                        else if (wide)
                            pair_dense_s<true>(ev, T(W.rcut2), T(W.L), src, nlist, sph, Ph, xs, ys,
                                               zs, hs, hs * hs, ax, ay, az, am, np_wave);
                        else
                            pair_dense_s<false>(ev, T(W.rcut2), T(W.L), src, n1 + n2, sph, Ph, xs,
                                                ys, zs, hs, hs * hs, ax, ay, az, am, np_wave);
                    }
                    {
                        const int ts = (int)(Gh + t0);   // half B
                        const T xs = __shfl(txi, ts, 64), ys = __shfl(tyi, ts, 64),
                                zs = __shfl(tzi, ts, 64), hs = __shfl(thi, ts, 64);
                        const uint64_t am = __ballot(__shfl((int)active, ts, 64) != 0);
                        const src_list<T> sB{src.p + n1, src.h + n1};
                        if constexpr (FT)
                            pair_dense(ev, T(W.rcut2), sB, n2 + n3, sph, Ph * team, xs, ys, zs,
                                       hs, hs * hs, bx, by, bz, am, np_wave, n_zero);
                        else if (wide)
                            pair_dense_s<true>(ev, T(W.rcut2), T(W.L), sB, nlist, sph, Ph, xs, ys,
                                               zs, hs, hs * hs, bx, by, bz, am, np_wave);
                        else
                            pair_dense_s<false>(ev, T(W.rcut2), T(W.L), sB, n2 + n3, sph, Ph, xs,
                                                ys, zs, hs, hs * hs, bx, by, bz, am, np_wave);
                    }
                }
            }
            if (masked) {
                if (halves)
                    fold();   // the list has just become wide, and stays so
                if (lane < PT) {  // sentinels: far outside every cutoff, in any image
                    src.pm(nlist + lane) = {T(1e30), T(1e30), T(1e30), T(0.0)};
                    src.hh(nlist + lane) = {T(0.0), T(0.0)};
                }
                wave_sync();
                if (wide)
                    pair_loop<T, true>(ev, W, src, nlist, ph + P * member, PT, txi, tyi, tzi, thi, thi2, ax, ay,
                                       az, active, n_pairs);
                else
                    pair_loop<T, false>(ev, W, src, nlist, ph + P * member, PT, txi, tyi, tzi, thi, thi2, ax,
                                        ay, az, active, n_pairs);
            }
            nlist = 0;
            wave_sync();
        };

        uint32_t sp = 0;
        bool overflow = false;
        if (!CELLS) {
            if (lane == 0)
                stk[0] = W.root;
            sp = 1;
        } else {
            // cells of level K met by the bounding box grown by r_cut (plus a margin far above
            // rounding, so that every particle in it is found in a listed cell), wrapped
            const int K = A.cell_K;
            const int side = 1 << K, kmask = side - 1;
            const double inv = (double)side / W.L,
                         margin = 1e-9 * W.L + (A.cell_extra ? *A.cell_extra : 0.0);
            const int lox = (int)floor((mnx - W.rcut - margin) * inv);
            const int loy = (int)floor((mny - W.rcut - margin) * inv);
            const int loz = (int)floor((mnz - W.rcut - margin) * inv);
            const int nx = min((int)floor((mxx + W.rcut + margin) * inv) - lox + 1, side);
            const int ny = min((int)floor((mxy + W.rcut + margin) * inv) - loy + 1, side);
            const int nz = min((int)floor((mxz + W.rcut + margin) * inv) - loz + 1, side);
            const uint32_t nyz = (uint32_t)(ny * nz), total = (uint32_t)nx * nyz;
            for (uint32_t c0 = 0; c0 < total; c0 += 64) {
                const uint32_t c = c0 + lane;
                uint32_t node = CELL_EMPTY;
                if (c < total) {
                    const uint32_t cxo = c / nyz, rem = c - cxo * nyz;
                    const uint32_t cyo = rem / (uint32_t)nz, czo = rem - cyo * (uint32_t)nz;
                    const int cx = lox + (int)cxo, cy = loy + (int)cyo, cz = loz + (int)czo;
                    const uint32_t wx = (uint32_t)(cx & kmask), wy = (uint32_t)(cy & kmask),
                                   wz = (uint32_t)(cz & kmask);
                    const uint32_t m = (uint32_t)((dzs_spread3(wx) << 2) | (dzs_spread3(wy) << 1) |
                                                  dzs_spread3(wz));
                    node = A.cell_node[m];
                    const int dl = A.cell_dl[m];
                    if (node != CELL_EMPTY && dl > 0) {
                        // a leaf above level K covers 2^dl cells per axis: only the first
                        // listed cell inside its cube (per axis, in listing order) pushes it
                        const int span = 1 << dl;
                        auto first = [&](int lo, uint32_t w) -> int {
                            const int n0 = (int)w & ~(span - 1);
                            const int wlo = lo & kmask;
                            return ((wlo - n0) & kmask) < span ? lo : lo + ((n0 - wlo) & kmask);
                        };
                        if (cx != first(lox, wx) || cy != first(loy, wy) || cz != first(loz, wz))
                            node = CELL_EMPTY;
                    }
                }
                const uint32_t put = node != CELL_EMPTY ? 1u : 0u;
                const uint32_t incl = dzs_wave_scan_add_full(put);
                const uint32_t tot = dzs_wave_last(incl);
                if (sp + tot > A.depth) {
                    overflow = true;
                    break;
                }
                if (put)
                    stk[sp + incl - 1] = node;
                sp += tot;
            }
        }
        __threadfence_block();
        // Nodes until the stack is empty, then one more turn that flushes what is left (the list
        // is flushed at one place, which holds all of the pair code).
        for (bool last = false; !last;) {
            last = sp == 0 || overflow;
            const uint32_t take = last ? 0u : (sp < 64 ? sp : 64);
            sp -= take;
            const bool has = lane < take;
            const uint32_t node = has ? stk[sp + lane] : 0u;
            // classify: 0 skip, 1 leaf, 2 monopole, 3 open
            int act = 0;
            double shx = 0.0, shy = 0.0, shz = 0.0;
            uint32_t ncount = 0, nchild = 0, child = 0, nfirst = 0;
            double comx = 0.0, comy = 0.0, comz = 0.0, nmass = 0.0, nhmax = 0.0;
            bool node_wide = false;
            if (has) {
                // the node's record: one address, the fields read where they are needed
                const dzs_node_rec &nd = A.rec[node];
                comx = nd.comx;
                comy = nd.comy;
                comz = nd.comz;
                const uint32_t nl = nd.nl;
                const int nlev = (int)(nl >> 8);
                nchild = nl & 0xffu;
                ncount = nd.count;
                nfirst = nd.first;
                child = nd.child;
                double dcx = nd.cx - gcx, dcy = nd.cy - gcy, dcz = nd.cz - gcz;
                shx = dcx > W.halfL ? -W.L : (dcx < -W.halfL ? W.L : 0.0);
                shy = dcy > W.halfL ? -W.L : (dcy < -W.halfL ? W.L : 0.0);
                shz = dcz > W.halfL ? -W.L : (dcz < -W.halfL ? W.L : 0.0);
                dcx += shx; dcy += shy; dcz += shz;
                const double nhx = nd.hx, nhy = nd.hy, nhz = nd.hz;
                const double gx_ = fmax(0.0, fabs(dcx) - nhx - ghx);
                const double gy_ = fmax(0.0, fabs(dcy) - nhy - ghy);
                const double gz_ = fmax(0.0, fabs(dcz) - nhz - ghz);
                const double dist2 = gx_ * gx_ + gy_ * gy_ + gz_ * gz_;
                node_wide = fmax(nhx, fmax(nhy, nhz)) + ghmax > W.wide || nd.pad != 0u;
                if (dist2 >= W.rcut2) {
                    act = 0;
                } else if (nchild == 0) {
                    act = 1;
                } else {
                    act = 3;
                    if (A.theta2 > 0.0 || A.aold) {
                        const double cx = comx + shx - gcx;
                        const double cy = comy + shy - gcy;
                        const double cz = comz + shz - gcz;
                        const double ex = fmax(0.0, fabs(cx) - ghx);
                        const double ey = fmax(0.0, fabs(cy) - ghy);
                        const double ez = fmax(0.0, fabs(cz) - ghz);
                        const double d2 = ex * ex + ey * ey + ez * ez;
                        const double side = ldexp(W.L, -(nlev - KBL));
                        if (A.aold) {
                            // G M l^2 < alpha a_min d^4
                            if (nd.mass * (side * side) < alpha_a * (d2 * d2))
                                act = 2;
                        } else if (side * side < A.theta2 * d2) {
                            act = 2;
                        }
                        if (act == 2) {
                            nmass = nd.mass;
                            nhmax = nd.hmax;
                        }
                    }
                }
            }
            if (__ballot((act == 1 || act == 2) && node_wide) != 0ull)
                wide = true;
            // ---- pushes
            const uint32_t npush = act == 3 ? nchild : 0u;
            const uint32_t pincl = dzs_wave_scan_add_full(npush);
            const uint32_t ptot = dzs_wave_last(pincl);
            if (sp + ptot > A.depth) {
                overflow = true;   // what is left unvisited is flagged, as is its group's force
                act = 0;
            } else {
                for (uint32_t j = 0; j < npush; ++j)
                    stk[sp + pincl - npush + j] = child + j;
                sp += ptot;
            }
            __threadfence_block();
            const uint64_t mono = __ballot(act == 2);
            const uint32_t nmono = (uint32_t)__popcll(mono);
            // ---- leaves: queue
            const uint64_t lmask = __ballot(act == 1);
            const uint32_t nq = (uint32_t)__popcll(lmask);
            const uint32_t lc = act == 1 ? ncount : 0u;
            const uint32_t lincl = dzs_wave_scan_add_full(lc);
            const uint32_t Ptot = dzs_wave_last(lincl);
            const uint32_t lstart = lincl - lc;
            const uint32_t lq = (uint32_t)__popcll(lmask & lt_mask);
            if (nq > 0) {
                wave_sync();
                if (act == 1) {
                    q_first[lq] = nfirst;
                    q_pref[lq] = lstart;
                    q_org[0][lq] = ox - shx;
                    q_org[1][lq] = oy - shy;
                    q_org[2][lq] = oz - shz;
                    q_wide[lq] = node_wide ? 1u : 0u;
                }
                wave_sync();
            }
            // ---- passes: the monopoles, then the queued leaves' particles 64 at a time, keeping
            //      those within r_cut of the group's bounding box.  The list is flushed before a
            //      pass that might not fit, so that no candidate is held across a flush.
            uint32_t carry = 0;
            for (int done = (last || nmono > 0) ? -64 : 0; done < (int)Ptot; done += 64) {
                const uint32_t need =
                    last ? WALK_LIST + 1u : (done < 0 ? nmono : min(Ptot - (uint32_t)done, 64u));
                if (nlist + need > list_cap)
                    flush();
                if (done < 0) {
                    if (act == 2) {
                        const uint32_t slot = nlist + (uint32_t)__popcll(mono & lt_mask);
                        src.pm(slot) = {T(comx + shx - ox), T(comy + shy - oy),
                                        T(comz + shz - oz), T(nmass)};
                        const T hn = T(nhmax);
                        src.hh(slot) = {wmax(hn * hn, hg2), hn};
                    }
                    nlist += nmono;
                    continue;
                }
                // candidate f of a pass belongs to the last leaf starting at or before it: each
                // leaf marks its start in the pass's window, a wave max-scan spreads the marks
                // (the leaf of the window's first slot carries over from the pass before)
                const uint32_t f = (uint32_t)done + lane;
                q_mark[lane] = 0u;
                wave_sync();
                if (act == 1 && lstart >= (uint32_t)done && lstart - (uint32_t)done < 64u)
                    q_mark[lstart - (uint32_t)done] = lq + 1u;
                wave_sync();
                uint32_t v = q_mark[lane];
                if (lane == 0)
                    v = v > carry + 1u ? v : carry + 1u;
                v = dzs_wave_scan_max_full(v);
                const uint32_t lo = v - 1u;
                carry = dzs_wave_last(lo);
                bool keep = false;
                double ex_ = 0.0, ey_ = 0.0, ez_ = 0.0;
                uint32_t mj = 0;
                if (f < Ptot) {
                    const uint32_t j = q_first[lo] + (f - q_pref[lo]);
                    // the particle in the list frame: its nearest image, less the group
                    // centre in FP32 (then the offset from the centre is the coordinate)
                    ex_ = A.x[j] - q_org[0][lo];
                    ey_ = A.y[j] - q_org[1][lo];
                    ez_ = A.z[j] - q_org[2][lo];
                    mj = A.mult[j];
                    const double cx = fmax(0.0, fabs(rel ? ex_ : ex_ - gcx) - ghx);
                    const double cy = fmax(0.0, fabs(rel ? ey_ : ey_ - gcy) - ghy);
                    const double cz = fmax(0.0, fabs(rel ? ez_ : ez_ - gcz) - ghz);
                    keep = q_wide[lo] != 0u || cx * cx + cy * cy + cz * cz < W.rcut2;
                }
                const uint64_t kmask = __ballot(keep);
                const uint32_t nk = (uint32_t)__popcll(kmask);
                if (nk > 0) {
                    if (keep) {
                        const uint32_t slot = nlist + (uint32_t)__popcll(kmask & lt_mask);
                        // an original particle (multiplicity 1) takes the group's constants
                        T mj_mass = m_unit;
                        typename vec4_of<T>::half mj_hh = hh_unit;
                        if (mj != 1u) {
                            mj_mass = T(W.m0 * (double)mj);
                            const T hj = T(W.h0 * mult_cbrt(mj));
                            mj_hh = {wmax(hj * hj, hg2), hj};
                        }
                        src.pm(slot) = {T(ex_), T(ey_), T(ez_), mj_mass};
                        src.hh(slot) = mj_hh;
                    }
                    nlist += nk;
                }
            }
            wave_sync();
        }
        if (overflow) {
            if (lane == 0)
                atomicOr(&A.counter[2], 1u);   // sticky until checked
        }
        if (halves)
            fold();
        // fixed-order sum of the P partial accelerations of each target
        for (uint32_t o = G; o < 64; o <<= 1) {
            ax += __shfl_xor(ax, o, 64);
            ay += __shfl_xor(ay, o, 64);
            az += __shfl_xor(az, o, 64);
        }
        {
            uint64_t cnt_pairs = (active ? (uint64_t)n_pairs : 0ull) - n_zero;
            for (int o = 32; o >= 1; o >>= 1)
                cnt_pairs += __shfl_xor(cnt_pairs, o, 64);
            if (lane == 0)
                atomicAdd(A.pair_count, (unsigned long long)(cnt_pairs + np_wave));
        }
        if constexpr (COOP) {
            // the waves' partial sums, added in their order (every wave comes here; the
            // next group's fetch has a barrier before the rows are written again)
            T *const part = (T *)S.q_org;
            if (ph == 0) {
                part[lane] = ax;
                part[64u + lane] = ay;
                part[128u + lane] = az;
            }
            __syncthreads();
            if (wave == 0)
                for (int w = 1; w < WAVES; ++w) {
                    const T *const o = (const T *)s_wave[w].q_org;
                    ax += o[lane];
                    ay += o[64u + lane];
                    az += o[128u + lane];
                }
        }
        if (active && ph == 0 && (!COOP || wave == 0)) {
            const double gxv = W.Gc * (double)ax, gyv = W.Gc * (double)ay, gzv = W.Gc * (double)az;
            const uint32_t o = A.out_perm ? A.out_perm[i] : i;
            if (A.accumulate) {
                A.gx[o] += gxv;
                A.gy[o] += gyv;
                A.gz[o] += gzv;
            } else {
                A.gx[o] = gxv;
                A.gy[o] = gyv;
                A.gz[o] = gzv;
            }
        }
    }
}

// ---- host: the split-factor polynomial ------------------------------------------------
namespace {

// q(w) = (erf(u/2) - u/sqrt(pi) exp(-u^2/4)) / u^3 from its Taylor series:
// q(w) = (1/sqrt(pi)) sum_{n>=1} (-1)^(n+1) 2n w^(n-1) / ((2n+1) 4^n n!)
long double q_taylor(long double w) {
    const long double inv_sqrt_pi = 0.564189583547756286948079451560772586L;
    long double term = 1.0L;  // w^(n-1) / (4^n n!) * 4, starts at n = 1 as 1/4 * 4 ... kept as ratio
    long double sum = 0.0L;
    long double pw = 1.0L;     // w^(n-1)
    long double fac = 1.0L;    // 4^n n!
    for (int n = 1; n < 200; ++n) {
        fac *= 4.0L * n;
        term = (n % 2 ? 1.0L : -1.0L) * 2.0L * n * pw / ((2.0L * n + 1.0L) * fac);
        sum += term;
        if (n > 4 && fabsl(term) < 1e-24L * fabsl(sum))
            break;
        pw *= w;
    }
    return sum * inv_sqrt_pi;
}

// Chebyshev fit of q on [0, wmax] with n coefficients, converted to monomials in t.
void fit_q(long double wmax, int n, long double *mono) {
    const long double pi = 3.14159265358979323846264338327950288L;
    long double f[WALK_QN], c[WALK_QN];
    for (int j = 0; j < n; ++j) {
        long double t = cosl(pi * (j + 0.5L) / n);
        f[j] = q_taylor(0.5L * (t + 1.0L) * wmax);
    }
    for (int k = 0; k < n; ++k) {
        long double s = 0.0L;
        for (int j = 0; j < n; ++j)
            s += f[j] * cosl(pi * k * (j + 0.5L) / n);
        c[k] = s * (k == 0 ? 1.0L : 2.0L) / n;
    }
    // T_k as monomial vectors: T_0 = 1, T_1 = t, T_{k+1} = 2 t T_k - T_{k-1}
    long double Tm[WALK_QN], T0[WALK_QN], T1[WALK_QN];
    for (int i = 0; i < n; ++i)
        mono[i] = T0[i] = T1[i] = 0.0L;
    T0[0] = 1.0L;
    T1[1 < n ? 1 : 0] += (n > 1) ? 1.0L : 0.0L;
    for (int i = 0; i < n; ++i)
        mono[i] += c[0] * T0[i];
    if (n > 1)
        for (int i = 0; i < n; ++i)
            mono[i] += c[1] * T1[i];
    for (int k = 2; k < n; ++k) {
        for (int i = 0; i < n; ++i)
            Tm[i] = -T0[i] + (i > 0 ? 2.0L * T1[i - 1] : 0.0L);
        for (int i = 0; i < n; ++i) {
            mono[i] += c[k] * Tm[i];
            T0[i] = T1[i];
            T1[i] = Tm[i];
        }
    }
}

}  // namespace

// The WALK_QN-coefficient fit and its worst relative error in S on [0, wmax].
static double split_poly(double wmax, double *q) {
    long double mono[WALK_QN];
    fit_q(wmax, WALK_QN, mono);
    long double worst = 0.0L;
    for (int k = 0; k <= 800; ++k) {
        long double w = wmax * k / 800.0L;
        long double t = 2.0L * w / wmax - 1.0L;
        long double qa = 0.0L;
        for (int i = WALK_QN - 1; i >= 0; --i)
            qa = qa * t + mono[i];
        long double qe = q_taylor(w);
        long double u = sqrtl(w);
        long double S = 1.0L - u * w * qe;
        long double err = fabsl(u * w * (qa - qe)) / fabsl(S);
        worst = err > worst ? err : worst;
    }
    for (int i = 0; i < WALK_QN; ++i)
        q[i] = (double)mono[i];
    return (double)worst;
}

// The FP32 table of S(u) on [0, ucut] (WALK_TAB_N intervals): on interval j, with
// h = ucut / WALK_TAB_N and f in [0, 1], the cubic Hermite interpolant of S and h dS/du at
// both ends, in powers of f; entry WALK_TAB_N continues the last interval's end linearly.
// Returns the worst absolute error in S (FP32 coefficients, exact long double evaluation).
static double split_table_f32(double ucut, float4 *tab) {
    const long double pi = 3.14159265358979323846264338327950288L;
    auto S = [&](long double u) {
        return erfcl(0.5L * u) + u / sqrtl(pi) * expl(-0.25L * u * u);
    };
    auto dS = [&](long double u) { return -u * u / (2.0L * sqrtl(pi)) * expl(-0.25L * u * u); };
    const long double h = (long double)ucut / WALK_TAB_N;
    for (int j = 0; j <= WALK_TAB_N; ++j) {
        const long double u0 = h * j, u1 = h * (j + 1);
        const long double s0 = S(u0), d0 = h * dS(u0);
        if (j == WALK_TAB_N) {
            tab[j] = make_float4((float)s0, (float)d0, 0.0f, 0.0f);
            break;
        }
        const long double s1 = S(u1), d1 = h * dS(u1);
        tab[j] = make_float4((float)s0, (float)d0, (float)(3.0L * (s1 - s0) - 2.0L * d0 - d1),
                             (float)(2.0L * (s0 - s1) + d0 + d1));
    }
    long double worst = 0.0L;
    for (int j = 0; j < WALK_TAB_N; ++j)
        for (int k = 0; k <= 16; ++k) {
            const long double f = k / 16.0L;
            const float4 c = tab[j];
            const long double v = (long double)c.x +
                                  f * ((long double)c.y + f * ((long double)c.z + f * c.w));
            const long double e = fabsl(v - S(h * (j + f)));
            worst = e > worst ? e : worst;
        }
    return (double)worst;
}

// Before a walk: the work counter to zero and, for the FP32 form (tab non-null), the cubics of
// F(w) = S(sqrt(w) / r_s) / w^1.5 on each interval [a, a + h) of 2^-WALK_FT_BITS octave from index
// base: the polynomial through F at the four Chebyshev nodes (Newton's divided differences), in
// powers of y = 2^-WALK_FT_BITS (w - a) / h.
__global__ __launch_bounds__(64) void k_walk_setup(uint32_t *counter, float4 *tab, uint32_t base,
                                                   double r_s) {
    const uint32_t j = blockIdx.x * 64u + threadIdx.x;
    if (j == 0)
        counter[0] = 0u;
    if (!tab || j >= WALK_FT_N)
        return;
    const double a = (double)__uint_as_float((base + j) << WALK_FT_SHIFT);
    // (the octave's power of two: the end of the last one is past the FP32 range)
    const double h = (double)__uint_as_float((base + j) >> WALK_FT_BITS << 23) /
                     (double)(1 << WALK_FT_BITS);
    const double node[4] = {0.5 - 0.5 * 0.92387953251128674, 0.5 - 0.5 * 0.38268343236508977,
                            0.5 + 0.5 * 0.38268343236508977, 0.5 + 0.5 * 0.92387953251128674};
    double f[4];
    for (int k = 0; k < 4; ++k) {   // in units of h: x = (w - a) / h in [0, 1)
        const double w = a + h * node[k], r = sqrt(w), u = r / r_s;
        f[k] = (erfc(0.5 * u) + u * 0.56418958354775629 * exp(-0.25 * u * u)) / (w * r);
    }
    for (int o = 1; o < 4; ++o)
        for (int k = 3; k >= o; --k)
            f[k] = (f[k] - f[k - 1]) / (node[k] - node[k - o]);
    double c[4] = {f[3], 0.0, 0.0, 0.0};
    for (int k = 2; k >= 0; --k) {   // c <- c (x - node[k]) + f[k]
        for (int i = 3; i >= 1; --i)
            c[i] = c[i - 1] - node[k] * c[i];
        c[0] = f[k] - node[k] * c[0];
    }
    const double s = (double)(1 << WALK_FT_BITS);   // y = x / s
    tab[(base + j) & (uint32_t)(WALK_FT_N - 1)] =
        make_float4((float)c[0], (float)(c[1] * s), (float)(c[2] * s * s),
                    (float)(c[3] * s * s * s));
}

dzs_status dzs_tree_walk(dzs_ctx *ctx, const dzs_box *box, uint64_t n, const double *x,
                         const double *y, const double *z, const uint32_t *mult, double *gx,
                         double *gy, double *gz, const dzs_tree_params *prm, hipStream_t s,
                         const dzs_walk_io &io) {
    return dzs_tree_walk_ex(ctx, box, n, x, y, z, mult, gx, gy, gz, prm, nullptr, s, io);
}

// boxes != nullptr: a batch (device table of the boxes; the keys in ctx->key carry the box);
// every box must share r_cut / r_s, the ratio the split-factor polynomial is fitted for.
dzs_status dzs_tree_walk_ex(dzs_ctx *ctx, const dzs_box *box, uint64_t n, const double *x,
                            const double *y, const double *z, const uint32_t *mult, double *gx,
                            double *gy, double *gz, const dzs_tree_params *prm,
                            const dzs_bbox *boxes, hipStream_t s, const dzs_walk_io &io) {
    if (n == 0 || !ctx->tree_built)
        return DZS_OK;
    const float *aold = io.aold;
    const bool relative = prm->opening == DZS_OPEN_RELATIVE && aold && !boxes;
    walk_args A;
    memset(&A, 0, sizeof(A));
    A.grp_first = ctx->grp_first;
    A.n_groups = ctx->bstate + BS_GROUPS;
    A.x = x; A.y = y; A.z = z; A.mult = mult;
    A.rec = ctx->nd_rec;
    A.L = box->L;
    A.halfL = 0.5 * box->L;
    A.rcut = prm->r_cut;
    A.rcut2 = prm->r_cut * prm->r_cut;
    A.theta2 = prm->theta * prm->theta;
    A.rs_inv = 1.0 / prm->r_s;
    A.rs_inv2 = A.rs_inv * A.rs_inv;
    A.G = box->G;
    A.m0 = box->m0;
    A.h0 = 2.8 * box->eps0;
    A.gx = gx; A.gy = gy; A.gz = gz;
    A.accumulate = prm->accumulate;
    A.G_lanes = prm->group_size;
    A.aold = relative ? aold : nullptr;
    A.active = boxes ? nullptr : io.active;
    A.out_perm = boxes ? nullptr : io.out_perm;
    A.bad = ctx->bstate + DZS_BS_BADINPUT;
    A.kept = (io.kept_tree && !boxes) ? 1 : 0;
    A.cell_extra = A.kept ? (const double *)(ctx->d_small + DZS_SMALL_DRIFT_TOTAL) : nullptr;
    if (io.target_list && !boxes && ctx->grp_list) {
        A.tgt = ctx->grp_list;
        A.tpos = ctx->tg_pos;
        A.n_tgrp = ctx->d_small + DZS_SMALL_GROUP_LIST + 1;
    }
    A.alpha_g = relative ? prm->alpha_open / box->G : 0.0;
    const double wmax = (prm->r_cut / prm->r_s) * (prm->r_cut / prm->r_s);
    if (ctx->q_wmax != wmax) {
        ctx->q_err = split_poly(wmax, ctx->q_coef);
        ctx->qf_err = split_table_f32(sqrt(wmax), ctx->stab);
        ctx->q_wmax = wmax;
    }
    const bool fp32 = prm->precision == DZS_FP32;
    if (!(ctx->q_err < 1e-10) || (fp32 && !(ctx->qf_err < 2e-7)))
        return dzs_fail(ctx, DZS_EINVAL, "tree: split-factor fit error %.2e / %.2e (FP32) for "
                        "r_cut/r_s = %.3f", ctx->q_err, ctx->qf_err, sqrt(wmax));
    for (int k = 0; k < WALK_QN; ++k)
        A.q[k] = ctx->q_coef[k];
    for (int k = 0; k <= WALK_TAB_N; ++k)
        A.stab[k] = ctx->stab[k];
    A.stab_scale = WALK_TAB_N * prm->r_s / prm->r_cut;
    A.t_scale = 2.0 / wmax;
    A.stack = ctx->walk_stack;
    A.depth = (uint32_t)ctx->walk_stack_depth;
    A.counter = ctx->walk_counter;
    A.pair_count = (unsigned long long *)(ctx->walk_counter + 8);
    // start level K: the deepest level whose cells are at least r_cut wide, at most
    // DZS_CELL_K_MAX.  Every node above level K is opened: eq. 1 could accept some of them
    // (a group's box can lie up to r_cut + sqrt(3) l from the centre of mass of a node of
    // side l, farther than l / theta), so the walk is at least as accurate as eq. 1 alone
    A.key = (const uint64_t *)ctx->key;
    A.boxes = boxes;
    int K = 0;
    if ((prm->theta <= 1.0 || relative) && !boxes)
        while (K < DZS_CELL_K_MAX && ldexp(box->L, -(K + 1)) >= prm->r_cut)
            ++K;
    A.cell_K = K;
    A.cell_node = ctx->cell_node;
    A.cell_dl = ctx->cell_dl;
    if (K > 0) {
        dzs_timed t(ctx, KC_TREE_BUILD, s);
        const uint64_t n_cells = 1ull << (3 * K);
        hipLaunchKernelGGL(k_cell_clear, dim3(blocks_for(n_cells, TB_THREADS)), dim3(TB_THREADS),
                           0, s, n_cells, ctx->cell_node);
        DZS_TRY(dzs_check_launch(ctx, "cell_clear"));
        // at most (8^(K+1) - 1) / 7 nodes sit on levels 0..K
        uint64_t n_top = ((1ull << (3 * (K + 1))) - 1) / 7;
        n_top = n_top < ctx->cap_nodes ? n_top : ctx->cap_nodes;
        hipLaunchKernelGGL(k_cell_fill, dim3(blocks_for(n_top, TB_THREADS)), dim3(TB_THREADS), 0,
                           s, (const uint32_t *)ctx->bstate, K, (const uint64_t *)ctx->key,
                           ctx->nd_first, ctx->nd_child, ctx->nd_level, ctx->cell_node,
                           ctx->cell_dl);
        DZS_TRY(dzs_check_launch(ctx, "cell_fill"));
    }
    // persistent waves: each takes groups until the counter passes the device group count
    const bool ft = fp32 && !boxes;
    // Waves per group, by n / group_size, the least number of groups (the tree cuts about 1.5
    // times as many).  With 4096 resident waves (3072 in FP32 teams of two) a launch of few groups
    // lasts as long as its heaviest one: FP64, 110,592 clustered particles in groups of 32 (3456) 1.16 ms alone, 0.98
    // in twos, 1.01 in fours; 20^3 (250) 78, 63 and 58 us; FP32 in groups of 64, 100,000
    // clustered (1562) 1.42, 0.96 and 0.74 ms, near-uniform 32^3 (512) 286, 195 and 181 us, 48^3
    // (1728) 436, 446 and 489 us.  Where every wave has several groups the repeated walks only
    // cost: 64^3 (4096) 579, 698 and 897 us, FP64 200,003 in groups of 16 (12,500) 1.17 ms alone,
    // 1.41 in fours.  (Groups below 16 would need more sentinels than the list has spare slots.)
    const uint64_t least = n / (uint64_t)A.G_lanes;
    const int team = A.G_lanes < 16 || least >= 4096 || (fp32 && !ft) ? 1 : (least >= 1024 ? 2 : 4);
    uint32_t slots = (uint32_t)ctx->walk_stack_slots;   // waves
    if (n * team < slots)
        slots = (uint32_t)(n * team);   // there are at most n groups
    const float ft_top = (float)A.rcut2;
    uint32_t ft_bits;
    memcpy(&ft_bits, &ft_top, sizeof(ft_bits));
    ft_bits >>= WALK_FT_SHIFT;
    const uint32_t ft_base = ft_bits >= WALK_FT_LEAST + (WALK_FT_N - 1) ? ft_bits - (WALK_FT_N - 1)
                                                                        : WALK_FT_LEAST;
    const uint32_t ft_lo_bits = ft_base << WALK_FT_SHIFT;
    memcpy(&A.ft_lo, &ft_lo_bits, sizeof(A.ft_lo));
    A.ftab = (const float4 *)ctx->walk_ftab;
    hipLaunchKernelGGL(k_walk_setup, dim3(ft ? WALK_FT_N / 64 : 1), dim3(64), 0, s,
                       ctx->walk_counter, ft ? (float4 *)ctx->walk_ftab : nullptr, ft_base,
                       prm->r_s);
    DZS_TRY(dzs_check_launch(ctx, "walk_setup"));
    {
        dzs_timed t(ctx, KC_TREE_WALK, s);
        auto launch = [&](auto cells, auto batch, auto tm, auto far, auto real) {
            typedef decltype(real) T;
            constexpr uint32_t W = tm.value > 1 ? tm.value : walk_waves<T>::N;
            hipLaunchKernelGGL((k_tree_walk<T, cells.value, batch.value, tm.value, far.value>),
                               dim3((slots + W - 1) / W), dim3(64 * W), 0, s, A);
        };
        const std::true_type yes;
        const std::false_type no;
        const std::integral_constant<int, 1> one;
        const std::integral_constant<int, 2> two;
        const std::integral_constant<int, 4> four;
        auto pick = [&](auto cells, auto batch) {
            if (!fp32)
                team == 1 ? launch(cells, batch, one, no, 0.0)
                          : (team == 2 ? launch(cells, batch, two, no, 0.0)
                                       : launch(cells, batch, four, no, 0.0));
            else if constexpr (batch.value)
                launch(cells, batch, one, no, 0.0f);
            else
                team == 1 ? launch(cells, batch, one, yes, 0.0f)
                          : (team == 2 ? launch(cells, batch, two, yes, 0.0f)
                                       : launch(cells, batch, four, yes, 0.0f));
        };
        if (boxes)
            pick(no, yes);
        else if (K > 0)
            pick(yes, no);
        else
            pick(no, no);
        DZS_TRY(dzs_check_launch(ctx, "tree_walk"));
    }
    return DZS_OK;  // overflows stay on the device until dzs_check
}

static_assert(WALK_FT_N == DZS_WALK_FT_N, "the context's table of F(w) holds WALK_FT_N cubics");
static_assert(sizeof(((dzs_ctx *)nullptr)->stab) == sizeof(float4) * (WALK_TAB_N + 1),
              "the context's table of S(u) holds WALK_TAB_N + 1 cubics");
