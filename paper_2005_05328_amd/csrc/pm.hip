// Particle-mesh long-range force (paper Sec. 2.1: density on a uniform grid, Poisson
// equation in Fourier space, Gaussian split kernel).
//
//   deposit     cloud-in-cell, deterministic: each contribution mult * w_x w_y w_z is rounded
//               to 32.32 fixed point and added with 64-bit integer atomics, so the mesh does
//               not depend on the order the GPU adds in
//   FFT         3-D complex transform as three passes of 1-D line transforms, each line held
//               in LDS (mixed radix 4/2/3 Stockham, autosorting, twiddles from a host table);
//               the x pass reads the fixed-point mesh directly, the z pass multiplies by the
//               Green's function and transforms back in the same kernel, the last inverse x
//               pass writes the real potential
//   Green       -4 pi G exp(-k^2 r_s^2) / (k^2 W(k)^2) / N_g^3, separable per-axis tables
//   gradient +  the 4-point difference of the potential at the 8 cloud-in-cell corners of each
//   interp      particle, weighted with the same cloud-in-cell weights (one kernel)
// Particles in no order are brought into key order first (pm_force only; the steps' are).
//
// Mesh layout: index (ix * N_g + iy) * N_g + iz.  Mesh points at j * Delta, Delta = L / N_g.
#include <limits.h>
#include <math.h>
#include <vector>

#include "internal.h"

#define PM_THREADS 256
#define FFT_THREADS 256
#define FFT_ELEMS 2048       // complex elements per workgroup tile (32 KB in FP64)
#define FFT_MAX_STAGES 12
#define DEP_FRAC 4294967296.0  // 2^32: fixed-point scale of the deposit
#define DEP_TILE 4096          // mesh points of the LDS deposit tile (32 KB of 64-bit sums)

static inline uint32_t blocks_for(uint64_t n, uint32_t t) { return (uint32_t)((n + t - 1) / t); }

struct fft_plan {
    int n;                       // line length
    int n_stages;
    int radix[FFT_MAX_STAGES];
};

// A batch of boxes, each with its own mesh at its own offset of the mesh arrays.  Deposit and
// interpolation find a particle's box from its key prefix; the FFT kernels of one mesh-size
// class run blocks_per_mesh blocks for each member box.  boxes == nullptr: a single box.
struct pm_batch {
    const dzs_bbox *boxes;
    const uint32_t *members;
    int blocks_per_mesh;
    const uint64_t *key;
};

// Particles that the caller passed in no order, put in key order (copies in the context's
// arena): used when *ordered, which a kernel sets, is 0.  ordered == nullptr: none.
struct __align__(32) pm_row {
    double v[3];
    uint32_t mult, pad;
};

struct pm_sorted {
    const uint32_t *ordered;
    pm_row *out;                 // their forces, in the caller's order (accelerations in v)
    const double *x, *y, *z;
    const uint32_t *mult, *perm;
    __device__ __forceinline__ bool used() const { return ordered && *ordered == 0u; }
    __device__ __forceinline__ bool select(const double *&px, const double *&py,
                                           const double *&pz, const uint32_t *&pm) const {
        if (!used())
            return false;
        px = x;
        py = y;
        pz = z;
        pm = mult;
        return true;
    }
};

// ---------------------------------------------------------------------------------------
// LDS line FFT
// ---------------------------------------------------------------------------------------
// C is double2 (plain form) or float2 (precision form); R its component type.
template <typename C> __device__ __forceinline__ C cmul(C a, C b) {
    return C{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename C> __device__ __forceinline__ C cadd(C a, C b) { return C{a.x + b.x, a.y + b.y}; }
template <typename C> __device__ __forceinline__ C csub(C a, C b) { return C{a.x - b.x, a.y - b.y}; }

template <int R, bool INV, typename C>
__device__ __forceinline__ void dft_small(C *v) {
    typedef decltype(v[0].x) Rt;
    if (R == 2) {
        C a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if (R == 4) {
        C a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
        C c = cadd(v[1], v[3]), t = csub(v[1], v[3]);
        // forward: t * (-i) = (t.y, -t.x); inverse: t * (+i) = (-t.y, t.x)
        C d = INV ? C{-t.y, t.x} : C{t.y, -t.x};
        v[0] = cadd(a, c);
        v[1] = cadd(b, d);
        v[2] = csub(a, c);
        v[3] = csub(b, d);
    } else {  // R == 3
        const Rt s3 = Rt(0.86602540378443865);  // sqrt(3)/2
        C t = cadd(v[1], v[2]), s = csub(v[1], v[2]);
        C m = C{v[0].x - Rt(0.5) * t.x, v[0].y - Rt(0.5) * t.y};
        // forward: X1 = m - i s3 s, X2 = m + i s3 s ; inverse swaps the sign of i
        C is = INV ? C{-s3 * s.y, s3 * s.x} : C{s3 * s.y, -s3 * s.x};
        v[0] = cadd(v[0], t);
        v[1] = cadd(m, is);
        v[2] = csub(m, is);
    }
}

// b / d by a reciprocal, exact for 0 <= b < 2^21: (b + 1/2) / d is at least 1 / (2 d) from a
// whole number and the two roundings move it by less.  (The compiler's own division by a value
// it does not know is some 25 instructions; five index divisions a point and stage were most
// of what a line transform issued: five passes on 256^3 in FP64 480 -> 381 us, on 192^3 211 ->
// 171.)
struct fast_div {
    float r;
    __device__ __forceinline__ explicit fast_div(int d) : r(1.0f / (float)d) {}
    __device__ __forceinline__ int operator()(int b) const { return (int)(((float)b + 0.5f) * r); }
};

// One Stockham stage over TL = 2^lt lines held in LDS.  Element e of line l lives at
// buf[e * se + l * sl].  All loads of the stage complete before any store (barrier), so the
// stage runs in place.
template <int R, bool INV, typename C>
__device__ __forceinline__ void fft_stage(C *buf, const C *tw, int n, int lt, int se, int sl,
                                          int Ns) {
    constexpr int SLOTS = (FFT_ELEMS / R + FFT_THREADS - 1) / FFT_THREADS;
    const int nb = n / R;
    const int total = nb << lt;
    const int step = nb / Ns;
    const fast_div by_nb(nb), by_ns(Ns);
    C v[SLOTS][R];
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) {
        const int b = threadIdx.x + q * FFT_THREADS;
        if (b < total) {
            int l, j;
            if (sl == 1) {
                l = b & ((1 << lt) - 1);
                j = b >> lt;
            } else {
                l = by_nb(b);
                j = b - l * nb;
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
                v[q][r] = buf[(j + r * nb) * se + l * sl];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) {
        const int b = threadIdx.x + q * FFT_THREADS;
        if (b < total) {
            int l, j;
            if (sl == 1) {
                l = b & ((1 << lt) - 1);
                j = b >> lt;
            } else {
                l = by_nb(b);
                j = b - l * nb;
            }
            const int jq = by_ns(j), k = j - jq * Ns;
#pragma unroll
            for (int r = 1; r < R; ++r) {
                C w = tw[r * k * step];
                if (INV)
                    w.y = -w.y;
                v[q][r] = cmul(v[q][r], w);
            }
            dft_small<R, INV>(v[q]);
            const int idxD = jq * Ns * R + k;
#pragma unroll
            for (int r = 0; r < R; ++r)
                buf[(idxD + r * Ns) * se + l * sl] = v[q][r];
        }
    }
    __syncthreads();
}

template <bool INV, typename C>
__device__ __forceinline__ void fft_lines(C *buf, const C *tw, const fft_plan &P, int lt, int se,
                                          int sl) {
    int Ns = 1;
    for (int s = 0; s < P.n_stages; ++s) {
        const int R = P.radix[s];
        if (R == 4)
            fft_stage<4, INV>(buf, tw, P.n, lt, se, sl, Ns);
        else if (R == 2)
            fft_stage<2, INV>(buf, tw, P.n, lt, se, sl, Ns);
        else
            fft_stage<3, INV>(buf, tw, P.n, lt, se, sl, Ns);
        Ns *= R;
    }
}

// twiddles e^{-2 pi i m / n} from the FP64 host table, rounded to the form's precision
template <typename C>
__device__ __forceinline__ void load_twiddles(C *s_tw, const double2 *tw, int n) {
    typedef decltype(s_tw[0].x) Rt;
    for (int i = threadIdx.x; i < n; i += FFT_THREADS)
        s_tw[i] = C{Rt(tw[i].x), Rt(tw[i].y)};
}

// ---------------------------------------------------------------------------------------
// deposit
// ---------------------------------------------------------------------------------------
// Unwrapped cloud-in-cell base index floor(x / Delta) of one axis and the weights of the
// base point and the next one (x times the reciprocal of Delta: a loop over particles of one
// mesh computes the reciprocal once).
__device__ __forceinline__ int cic_base(double x, double delta, double &w0, double &w1) {
    const double u = x * (1.0 / delta);
    const double f = floor(u);
    w1 = u - f;
    w0 = 1.0 - w1;
    return (int)f;
}

__device__ __forceinline__ int wrap_index(int i, int ng) {
    i %= ng;
    return i < 0 ? i + ng : i;
}

// The same for an index within one period of the mesh, -ng <= i < 2 ng, by compares instead
// of a division: a stencil point i0 + d (|d| <= 3 < ng), or a point of a deposit tile (base
// indices in [0, ng] and the points after them; meshes have at least 8 points per side).
__device__ __forceinline__ int wrap_near(int i, int ng) {
    return i < 0 ? i + ng : (i >= ng ? i - ng : i);
}

__device__ __forceinline__ void cic_axis(double x, double delta, int ng, int &i0, int &i1,
                                         double &w0, double &w1) {
    const int i = wrap_index(cic_base(x, delta, w0, w1), ng);
    i0 = i;
    i1 = i + 1 == ng ? 0 : i + 1;
}

// One corner's contribution in 32.32 fixed point (the same expression on every path, so the
// integer sums, and with them the mesh, do not depend on which path adds them).
__device__ __forceinline__ unsigned long long dep_fixed(double m, double wx, double wy, double wz) {
    return (unsigned long long)llrint(m * wx * wy * wz);
}

// A particle's eight mesh points (offset 4 a + 2 b + c) and its contribution to each.
struct dep_points {
    int ix[2], iy[2], iz[2];
    double wx[2], wy[2], wz[2], m;
    __device__ __forceinline__ dep_points(double x, double y, double z, uint32_t mult,
                                          double delta, int ng) {
        cic_axis(x, delta, ng, ix[0], ix[1], wx[0], wx[1]);
        cic_axis(y, delta, ng, iy[0], iy[1], wy[0], wy[1]);
        cic_axis(z, delta, ng, iz[0], iz[1], wz[0], wz[1]);
        m = (double)mult * DEP_FRAC;
    }
    __device__ __forceinline__ uint64_t at(int e, int ng) const {
        return ((uint64_t)ix[e >> 2] * ng + iy[e >> 1 & 1]) * ng + iz[e & 1];
    }
    __device__ __forceinline__ unsigned long long part(int e) const {
        return dep_fixed(m, wx[e >> 2], wy[e >> 1 & 1], wz[e & 1]);
    }
};

// Direct deposit: eight 64-bit atomic adds per particle into the mesh.
__device__ __forceinline__ void dep_direct(const dep_points &D, int ng, unsigned long long *q) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const unsigned long long iv = D.part(e);
        if (iv)
            atomicAdd(&q[D.at(e, ng)], iv);
    }
}

// The same for a wave (every lane calls it; valid: the lane holds a particle): the lanes that share
// the base point of one of three lanes, where they are DEP_SHARED or more, add their contributions
// up (the same integers in another order) before one lane's atomics.  A particle among many of
// one mesh cell would wait for all their atomics on its eight points: 60,000 in no order, nine in
// ten in one cell of 64^3, 2.06 -> 0.08 ms, 131,072 on 162^3 4.05 -> 0.35; where no cell is shared
// (4099 on 32^3) 42.1 -> 42.4 us.
#define DEP_SHARED 12
__device__ __forceinline__ void dep_direct_wave(bool valid, const dep_points &D, int ng,
                                                unsigned long long *q,
                                                const unsigned long long *mesh) {
    // (fewer than 2^31 mesh points)
    const uint32_t point = valid ? (uint32_t)((uint64_t)(q - mesh) + D.at(0, ng)) : 0xffffffffu;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)point, 10 + 21 * r);
        const bool mine = valid && point == at;
        const uint64_t m = __ballot(mine);
        if (__popcll(m) < DEP_SHARED)
            continue;
        const bool first = mine && (threadIdx.x & 63u) == (uint32_t)__ffsll((long long)m) - 1u;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            unsigned long long v = mine ? D.part(e) : 0ull;
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1)
                v += __shfl_xor(v, o, 64);
            if (first && v)
                atomicAdd(&q[D.at(e, ng)], v);
        }
        valid = valid && !mine;
    }
    if (valid)
        dep_direct(D, ng, q);
}

__global__ __launch_bounds__(PM_THREADS) void k_pm_deposit(uint64_t n, const double *x,
                                                           const double *y, const double *z,
                                                           const uint32_t *mult, double delta,
                                                           int ng,
                                                           unsigned long long *__restrict__ q,
                                                           pm_batch B, pm_sorted S) {
    const uint64_t p = (uint64_t)blockIdx.x * PM_THREADS + threadIdx.x;
    if (p >= n)
        return;
    S.select(x, y, z, mult);
    if (B.boxes) {
        const dzs_bbox &bx = B.boxes[B.key[p] >> DZS_BATCH_SHIFT];
        delta = bx.delta;
        ng = bx.ng;
        q += bx.mesh_off;
    }
    dep_direct(dep_points(x[p], y[p], z[p], mult[p], delta, ng), ng, q);
}

// Boxes of the cloud-in-cell base indices.  The deposit and the interpolation hold a chunk's
// positions in registers; each run of 64 consecutive particles (one wave's registers) is a
// piece, whose box (unwrapped base indices, so a piece across the periodic boundary stays
// compact, and the range of its boxes of a batch) goes to LDS once.  The runs of pieces that
// fit a tile are then found from these boxes alone.
#define PM_PIECE 64
#define DEP_SPARSE 8                         // most tile points per particle, few particles
#define PM_ITEMS 4                           // particles per thread of a full chunk
#define PM_CHUNK (PM_ITEMS * PM_THREADS)     // 1024: what a workgroup holds at once
#define PM_PIECES (PM_CHUNK / PM_PIECE)      // 16: one row of a wave's lanes

// minimum over a wave's rows of 16 lanes, in every lane
__device__ __forceinline__ int row_min(int v) {
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x128, 0xf, 0xf, false));   // row_ror:8
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x124, 0xf, 0xf, false));   // row_ror:4
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x122, 0xf, 0xf, false));   // row_ror:2
    return min(v, __builtin_amdgcn_update_dpp(v, v, 0x121, 0xf, 0xf, false));  // row_ror:1
}
__device__ __forceinline__ int wave_min(int v) {
    v = row_min(v);
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// lo[0..2], -hi[3..5] of the base indices, the lowest and minus the highest box [6..7]
struct pm_span {
    int v[8];
};

__device__ __forceinline__ void span_none(pm_span &b) {
#pragma unroll
    for (int a = 0; a < 8; ++a)
        b.v[a] = INT_MAX;
}

// The box of the wave's 64 particles (valid: the lane holds one).
__device__ __forceinline__ void piece_span(bool valid, double x, double y, double z, double delta,
                                           const pm_batch &B, uint64_t p, int *out) {
    pm_span b;
    span_none(b);
    if (valid) {
        double d = delta;
        if (B.boxes) {
            const int bx = (int)(B.key[p] >> DZS_BATCH_SHIFT);
            d = B.boxes[bx].delta;
            b.v[6] = bx;
            b.v[7] = -bx;
        }
        double w0, w1;
        b.v[0] = cic_base(x, d, w0, w1);
        b.v[1] = cic_base(y, d, w0, w1);
        b.v[2] = cic_base(z, d, w0, w1);
#pragma unroll
        for (int a = 0; a < 3; ++a)
            b.v[3 + a] = b.v[a] == INT_MIN ? INT_MAX : -b.v[a];
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        const int m = wave_min(b.v[a]);
        if ((threadIdx.x & 63u) == 0u)
            out[a] = m;
    }
}

// The union of the boxes of pieces [s, s + len), the same in every thread.
__device__ __forceinline__ pm_span run_span(const int (*box)[8], uint32_t s, uint32_t len) {
    const uint32_t q = threadIdx.x & 15u;
    pm_span b;
#pragma unroll
    for (int a = 0; a < 8; ++a)
        b.v[a] = __builtin_amdgcn_readfirstlane(
            row_min(q >= s && q < s + len ? box[q][a] : INT_MAX));
    return b;
}

// Mesh points spanned (base .. base + 1 on each axis), or 0 where the run
// cannot use a tile of `cap` points: too many points, two boxes of a batch, or a base index
// outside [0, ng] (a position outside the box), which only the direct path folds.
__device__ __forceinline__ uint32_t run_points(const pm_span &b, int64_t cap, int ng,
                                               bool batch, uint32_t &ey, uint32_t &ez) {
    const int64_t ex = -(int64_t)b.v[3] - b.v[0] + 2,
                  fy = -(int64_t)b.v[4] - b.v[1] + 2,
                  fz = -(int64_t)b.v[5] - b.v[2] + 2;
    if ((batch && b.v[6] != -b.v[7]) || b.v[0] < 0 || b.v[1] < 0 || b.v[2] < 0 ||
        b.v[3] < -ng || b.v[4] < -ng || b.v[5] < -ng || ex > cap || fy > cap || fz > cap ||
        ex * fy * fz > cap)
        return 0;
    ey = (uint32_t)fy;
    ez = (uint32_t)fz;
    return (uint32_t)(ex * fy * fz);
}

// The coordinates (a, b, e) of tile point c = (a tey + b) tez + e, advanced by a fixed stride
// with carries instead of two integer divisions per point.
struct tile_walk {
    uint32_t a, b, e, da, db, de, tey, tez;
    __device__ __forceinline__ tile_walk(uint32_t c0, uint32_t stride, uint32_t tey_,
                                         uint32_t tez_)
        : tey(tey_), tez(tez_) {
        const uint32_t pyz = tey * tez;
        a = c0 / pyz;
        const uint32_t r = c0 - a * pyz;
        b = r / tez;
        e = r - b * tez;
        da = stride / pyz;
        const uint32_t q = stride - da * pyz;
        db = q / tez;
        de = q - db * tez;
    }
    __device__ __forceinline__ void next() {
        e += de;
        b += db;
        a += da;
        if (e >= tez) {
            e -= tez;
            ++b;
        }
        if (b >= tey) {
            b -= tey;
            ++a;
        }
    }
};

// LDS-binned deposit.  A workgroup takes `chunk` consecutive particles (in key order they
// fill a compact region), PM_CHUNK at a time in registers, in runs of pieces: a run whose box
// holds at most DEP_TILE points sums its contributions into an LDS tile with 64-bit LDS
// atomics, then adds each non-zero tile point to the mesh (wrapped) with one global atomic.  A
// run whose box is too large is halved; pieces that do not fit alone add directly.  The mesh
// is the same integer sum either way.  Bound by the atomics: a mesh point that several
// particles share is added once per tile, and the lanes of a flush add to whole mesh lines
// (128^3 particles on 256^3, directly 371 us; 60000 clustered ones wait for each other's points
// ten times as long).  The positions are read once; earlier every halving read them again.
// A single wave (few particles) uses the tile only where it holds at most DEP_SPARSE points per
// particle: clearing and flushing more takes longer than its 8 atomics a particle.
template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_pm_deposit_tiled(
    uint64_t n, const double *x, const double *y, const double *z, const uint32_t *mult,
    double delta, int ng, unsigned long long *__restrict__ q, pm_batch B, pm_sorted S, uint32_t chunk) {
    S.select(x, y, z, mult);
    __shared__ unsigned long long s_tile[DEP_TILE];
    __shared__ int s_box[PM_PIECES][8];
    const uint64_t c0 = (uint64_t)blockIdx.x * chunk;
    const uint64_t c1 = c0 + chunk < n ? c0 + chunk : n;
    const uint32_t tid = threadIdx.x;
    for (uint64_t b0 = c0; b0 < c1; b0 += ITEMS * THREADS) {
        double px[ITEMS] = {}, py[ITEMS] = {}, pz[ITEMS] = {};
        uint32_t pm[ITEMS] = {};
        const uint32_t np = (uint32_t)(c1 - b0 < ITEMS * THREADS ? c1 - b0
                                                                    : ITEMS * THREADS);
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t o = tid + (uint32_t)i * THREADS;
            if (o < np) {
                px[i] = x[b0 + o];
                py[i] = y[b0 + o];
                pz[i] = z[b0 + o];
                pm[i] = mult[b0 + o];
            }
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t o = tid + (uint32_t)i * THREADS;
            piece_span(o < np, px[i], py[i], pz[i], delta, B, b0 + o, s_box[o / PM_PIECE]);
        }
        __syncthreads();
        const uint32_t pieces = (np + PM_PIECE - 1) / PM_PIECE;
        uint32_t direct = 0;   // pieces that add directly
        uint32_t len = ITEMS * THREADS / PM_PIECE;
        for (uint32_t s = 0; s < pieces;) {
            // the same in every thread: the choices are uniform over the workgroup
            const pm_span sp = run_span(s_box, s, len);
            int gn = ng;
            if (B.boxes && sp.v[6] == -sp.v[7])
                gn = B.boxes[sp.v[6]].ng;
            uint32_t tey, tez;
            const uint32_t cells = run_points(sp, DEP_TILE, gn, B.boxes != nullptr, tey, tez);
            const bool tile = cells && (THREADS > 64 || cells <= DEP_SPARSE * PM_PIECE);
            if (!tile && len > 1) {
                len >>= 1;
                continue;
            }
            if (!tile) {
                direct |= 1u << s;
                ++s;
                continue;
            }
            double dl = delta;
            unsigned long long *qb = q;
            if (B.boxes) {
                const dzs_bbox &bx = B.boxes[sp.v[6]];
                dl = bx.delta;
                qb = q + bx.mesh_off;
            }
            for (uint32_t c = tid; c < cells; c += THREADS)
                s_tile[c] = 0ull;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const uint32_t o = tid + (uint32_t)i * THREADS, pc = o / PM_PIECE;
                if (o >= np || pc < s || pc >= s + len)
                    continue;
                double wx[2], wy[2], wz[2];
                const uint32_t ti = (uint32_t)(cic_base(px[i], dl, wx[0], wx[1]) - sp.v[0]);
                const uint32_t tj = (uint32_t)(cic_base(py[i], dl, wy[0], wy[1]) - sp.v[1]);
                const uint32_t tk = (uint32_t)(cic_base(pz[i], dl, wz[0], wz[1]) - sp.v[2]);
                const double m = (double)pm[i] * DEP_FRAC;
#pragma unroll
                for (uint32_t a = 0; a < 2; ++a)
#pragma unroll
                    for (uint32_t b = 0; b < 2; ++b)
#pragma unroll
                        for (uint32_t c = 0; c < 2; ++c) {
                            const unsigned long long iv = dep_fixed(m, wx[a], wy[b], wz[c]);
                            if (iv)
                                atomicAdd(&s_tile[((ti + a) * tey + (tj + b)) * tez + (tk + c)],
                                          iv);
                        }
            }
            __syncthreads();
            tile_walk w(tid, THREADS, tey, tez);
            for (uint32_t c = tid; c < cells; c += THREADS, w.next()) {
                const unsigned long long v = s_tile[c];
                if (!v)
                    continue;
                const int ix = wrap_near(sp.v[0] + (int)w.a, gn),
                          iy = wrap_near(sp.v[1] + (int)w.b, gn),
                          iz = wrap_near(sp.v[2] + (int)w.e, gn);
                atomicAdd(&qb[((uint64_t)ix * gn + iy) * gn + iz], v);
            }
            __syncthreads();   // the tile is read before the next run clears it
            s += len;
        }
        if (direct) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const uint32_t o = tid + (uint32_t)i * THREADS;
                if (!(direct >> (o / PM_PIECE) & 1u))   // (a wave's lanes are one piece)
                    continue;
                double d = delta;
                int g = ng;
                unsigned long long *qq = q;
                if (B.boxes) {
                    const dzs_bbox &bx = B.boxes[B.key[b0 + min(o, np - 1)] >> DZS_BATCH_SHIFT];
                    d = bx.delta;
                    g = bx.ng;
                    qq = q + bx.mesh_off;
                }
                // (lanes past the last particle hold position 0: its points are not used)
                dep_direct_wave(o < np, dep_points(px[i], py[i], pz[i], pm[i], d, g), g, qq, q);
            }
        }
        __syncthreads();   // the boxes are read before the next particles' are written
    }
}

// ---------------------------------------------------------------------------------------
// x passes, real <-> half spectrum.  The density and the potential are real, so only the
// planes k_x = 0 .. N_g/2 of the transform are kept (the others are their conjugates): the
// y and z passes run on N_g/2 + 1 planes.  A tile is 2 CL consecutive iz values for a fixed
// iy; lines iz0 + t and iz0 + t + CL travel as the real and imaginary parts of one complex
// line of length N_g, and their spectra are separated (forward) or combined (inverse) with
// the conjugate symmetry of a real line's transform.  The complex mesh keeps the layout
// (k_x N_g + iy) N_g + iz.
// ---------------------------------------------------------------------------------------
template <typename C>
__global__ __launch_bounds__(FFT_THREADS) void k_fft_x_r2c(const unsigned long long *q, C *c,
                                                           const double2 *__restrict__ tw,
                                                           fft_plan P, int CL, double q_scale,
                                                           pm_batch B) {
    // q and c may be the same memory (meshes for the precision form only): the tile writes
    // only cells it has read, after all of its loads
    typedef decltype(C::x) Rt;
    extern __shared__ __align__(16) unsigned char s_fft[];
    C *s_buf = (C *)s_fft, *s_tw = s_buf + P.n * CL;   // the tile's lines, the twiddles
    const int n = P.n;
    const int TZ = 2 * CL, lt = 31 - __clz(CL);
    const int tiles_z = n / TZ;
    uint32_t blk = blockIdx.x;
    if (B.boxes) {
        const dzs_bbox &bx = B.boxes[B.members[blk / (uint32_t)B.blocks_per_mesh]];
        blk %= (uint32_t)B.blocks_per_mesh;
        q += bx.mesh_off;
        c += bx.mesh_off;
        q_scale = bx.q_scale;
    }
    const int iy = blk / tiles_z;
    const int iz0 = (blk % tiles_z) * TZ;
    const uint64_t sx = (uint64_t)n * n;
    const uint64_t base = (uint64_t)iy * n + iz0;
    load_twiddles(s_tw, tw, n);
    for (int e = threadIdx.x; e < n * CL; e += FFT_THREADS) {
        const int t = e & (CL - 1), a = e >> lt;
        const uint64_t gi = base + (uint64_t)a * sx + t;
        s_buf[e] = C{Rt((double)(long long)q[gi] * q_scale),
                     Rt((double)(long long)q[gi + CL] * q_scale)};
    }
    __syncthreads();
    fft_lines<false>(s_buf, s_tw, P, lt, CL, 1);
    // Z = A + i B with A, B the spectra of the two real lines: A[k] = (Z[k] + conj Z[n-k]) / 2,
    // B[k] = (Z[k] - conj Z[n-k]) / 2i
    const int nh = n / 2 + 1;
    for (int e = threadIdx.x; e < nh * CL; e += FFT_THREADS) {
        const int t = e & (CL - 1), k = e >> lt;
        const C z = s_buf[e];
        const C w = s_buf[(k == 0 ? 0 : n - k) * CL + t];
        const uint64_t gi = base + (uint64_t)k * sx + t;
        c[gi] = C{Rt(0.5) * (z.x + w.x), Rt(0.5) * (z.y - w.y)};
        c[gi + CL] = C{Rt(0.5) * (z.y + w.y), Rt(-0.5) * (z.x - w.x)};
    }
}

template <typename C>
__global__ __launch_bounds__(FFT_THREADS) void k_fft_x_c2r(const C *__restrict__ c,
                                                           decltype(C::x) *__restrict__ phi,
                                                           const double2 *__restrict__ tw,
                                                           fft_plan P, int CL, pm_batch B) {
    typedef decltype(C::x) Rt;
    extern __shared__ __align__(16) unsigned char s_fft[];
    C *s_buf = (C *)s_fft, *s_tw = s_buf + P.n * CL;   // the tile's lines, the twiddles
    const int n = P.n;
    const int TZ = 2 * CL, lt = 31 - __clz(CL);
    const int tiles_z = n / TZ;
    uint32_t blk = blockIdx.x;
    if (B.boxes) {
        const dzs_bbox &bx = B.boxes[B.members[blk / (uint32_t)B.blocks_per_mesh]];
        blk %= (uint32_t)B.blocks_per_mesh;
        c += bx.mesh_off;
        phi += bx.mesh_off;
    }
    const int iy = blk / tiles_z;
    const int iz0 = (blk % tiles_z) * TZ;
    const uint64_t sx = (uint64_t)n * n;
    const uint64_t base = (uint64_t)iy * n + iz0;
    load_twiddles(s_tw, tw, n);
    // Z[k] = A[k] + i B[k], Z[n-k] = conj A[k] + i conj B[k]; the k_x = 0 and N_g/2 values of
    // a real line's spectrum are real (their imaginary rounding is dropped, as the real part
    // of a full inverse transform drops it)
    const int nh = n / 2 + 1;
    for (int e = threadIdx.x; e < nh * CL; e += FFT_THREADS) {
        const int t = e & (CL - 1), k = e >> lt;
        const uint64_t gi = base + (uint64_t)k * sx + t;
        C a = c[gi], b = c[gi + CL];
        const bool edge = k == 0 || 2 * k == n;
        if (edge)
            a.y = b.y = Rt(0.0);
        s_buf[e] = C{a.x - b.y, a.y + b.x};
        if (!edge)
            s_buf[(n - k) * CL + t] = C{a.x + b.y, b.x - a.y};
    }
    __syncthreads();
    fft_lines<true>(s_buf, s_tw, P, lt, CL, 1);
    for (int e = threadIdx.x; e < n * CL; e += FFT_THREADS) {
        const int t = e & (CL - 1), a = e >> lt;
        const uint64_t gi = base + (uint64_t)a * sx + t;
        const C z = s_buf[e];
        phi[gi] = z.x;
        phi[gi + CL] = z.y;
    }
}

// ---------------------------------------------------------------------------------------
// y passes: a tile is TZ consecutive iz values x all N_g values of iy, for a fixed k_x plane.
// ---------------------------------------------------------------------------------------
template <bool INV, typename C>
__global__ __launch_bounds__(FFT_THREADS) void k_fft_y(C *__restrict__ c,
                                                       const double2 *__restrict__ tw,
                                                       fft_plan P, int TZ, pm_batch B) {
    extern __shared__ __align__(16) unsigned char s_fft[];
    C *s_buf = (C *)s_fft, *s_tw = s_buf + P.n * TZ;   // the tile's lines, the twiddles
    const int n = P.n, lt = 31 - __clz(TZ);
    const int tiles_z = n / TZ;
    uint32_t blk = blockIdx.x;
    if (B.boxes) {
        const dzs_bbox &bx = B.boxes[B.members[blk / (uint32_t)B.blocks_per_mesh]];
        blk %= (uint32_t)B.blocks_per_mesh;
        c += bx.mesh_off;
    }
    const int ix = blk / tiles_z;
    const int iz0 = (blk % tiles_z) * TZ;
    const uint64_t base = (uint64_t)ix * n * n + iz0;
    load_twiddles(s_tw, tw, n);
    const int total = n * TZ;
    for (int e = threadIdx.x; e < total; e += FFT_THREADS) {
        const int t = e & (TZ - 1), a = e >> lt;
        s_buf[e] = c[base + (uint64_t)a * n + t];
    }
    __syncthreads();
    fft_lines<INV>(s_buf, s_tw, P, lt, TZ, 1);
    for (int e = threadIdx.x; e < total; e += FFT_THREADS) {
        const int t = e & (TZ - 1), a = e >> lt;
        c[base + (uint64_t)a * n + t] = s_buf[e];
    }
}

// z pass: TL whole contiguous lines (fixed k_x plane, consecutive iy): forward FFT, Green's
// function, inverse FFT.
template <typename C>
__global__ __launch_bounds__(FFT_THREADS) void k_fft_z_green(C *__restrict__ c,
                                                              const double2 *__restrict__ tw,
                                                              const double *__restrict__ gt,
                                                              const double *__restrict__ k2t,
                                                              fft_plan P, int TL, double gconst,
                                                              pm_batch B) {
    typedef decltype(C::x) Rt;
    extern __shared__ __align__(16) unsigned char s_fft[];
    C *s_buf = (C *)s_fft, *s_tw = s_buf + P.n * TL;   // the tile's lines, the twiddles
    const int n = P.n, lt = 31 - __clz(TL);
    const fast_div by_n(n);
    const int tiles_y = n / TL;
    uint32_t blk = blockIdx.x;
    if (B.boxes) {
        const dzs_bbox &bx = B.boxes[B.members[blk / (uint32_t)B.blocks_per_mesh]];
        blk %= (uint32_t)B.blocks_per_mesh;
        c += bx.mesh_off;
        gt += bx.tab_off;
        k2t += bx.tab_off + (uint64_t)n;
    }
    const int ix = blk / tiles_y;
    const int iy0 = (blk % tiles_y) * TL;
    const uint64_t base = ((uint64_t)ix * n + iy0) * n;
    load_twiddles(s_tw, tw, n);
    const int total = n * TL;
    for (int e = threadIdx.x; e < total; e += FFT_THREADS)
        s_buf[e] = c[base + e];
    __syncthreads();
    fft_lines<false>(s_buf, s_tw, P, lt, 1, n);
    for (int e = threadIdx.x; e < total; e += FFT_THREADS) {
        const int l = by_n(e), iz = e - l * n;
        const int iy = iy0 + l;
        const double k2 = k2t[ix] + k2t[iy] + k2t[iz];
        double gk = 0.0;
        if (k2 > 0.0)
            gk = gconst * gt[ix] * gt[iy] * gt[iz] / k2;
        const Rt g = Rt(gk);
        C v = s_buf[e];
        s_buf[e] = C{v.x * g, v.y * g};
    }
    __syncthreads();
    fft_lines<true>(s_buf, s_tw, P, lt, 1, n);
    for (int e = threadIdx.x; e < total; e += FFT_THREADS)
        c[base + e] = s_buf[e];
}

// ---------------------------------------------------------------------------------------
// gradient + interpolation
// ---------------------------------------------------------------------------------------
// The potential values of one particle's stencils, by rows along z: all six points of the four
// rows through the cloud-in-cell points, and the two cloud points of the sixteen rows beside
// them.  Two neighbours along z come with one load: 28 loads instead of 56, and the direct
// path, bound by the cache lines its loads look up (a wave's 64 lanes lie in nearly as many
// lines at each of them), takes little more than half the time.
template <typename Rt> struct stencil {
    Rt ctr[2][2][6];   // (a, b) in {0, 1}^2, c = -2 .. 3
    Rt xr[4][2][2];    // a = -2, -1, 2, 3; b, c in {0, 1}
    Rt yr[2][4][2];    // b = -2, -1, 2, 3; a, c in {0, 1}
    // load(a, b, c, v): the points (a, b, c) and (a, b, c + 1) into v[0], v[1]
    template <typename Load> __device__ __forceinline__ void read(const Load &load) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    load(a, b, 2 * c - 2, &ctr[a][b][2 * c]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                load(e < 2 ? e - 2 : e, b, 0, xr[e][b]);
                load(b, e < 2 ? e - 2 : e, 0, yr[b][e]);
            }
    }
    __device__ __forceinline__ Rt x(int a, int b, int c) const {
        return a == 0 || a == 1 ? ctr[a][b][c + 2] : xr[a < 0 ? a + 2 : a][b][c];
    }
    __device__ __forceinline__ Rt y(int a, int b, int c) const {
        return b == 0 || b == 1 ? ctr[a][b][c + 2] : yr[a][b < 0 ? b + 2 : b][c];
    }
    __device__ __forceinline__ Rt z(int a, int b, int c) const { return ctr[a][b][c + 2]; }
};

// The 4-point difference of the potential at the 8 cloud-in-cell points of one particle,
// weighted with the cloud-in-cell weights; every path runs this same arithmetic, so they give
// the same bits.
template <typename Rt>
__device__ __forceinline__ void cic_gradient(const stencil<Rt> &v, const double *wx,
                                             const double *wy, const double *wz, Rt &sx, Rt &sy,
                                             Rt &sz) {
    const Rt c1 = Rt(2.0 / 3.0), c2 = Rt(1.0 / 12.0);
    sx = sy = sz = Rt(0.0);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const Rt w = Rt(wx[a] * wy[b] * wz[c]);
                const Rt dxp = c1 * (v.x(a + 1, b, c) - v.x(a - 1, b, c)) -
                               c2 * (v.x(a + 2, b, c) - v.x(a - 2, b, c));
                const Rt dyp = c1 * (v.y(a, b + 1, c) - v.y(a, b - 1, c)) -
                               c2 * (v.y(a, b + 2, c) - v.y(a, b - 2, c));
                const Rt dzp = c1 * (v.z(a, b, c + 1) - v.z(a, b, c - 1)) -
                               c2 * (v.z(a, b, c + 2) - v.z(a, b, c - 2));
                sx += w * dxp;
                sy += w * dyp;
                sz += w * dzp;
            }
}

template <typename Rt>
__device__ __forceinline__ void interp_store(uint64_t p, double delta, Rt sx, Rt sy, Rt sz,
                                             double *__restrict__ gx, double *__restrict__ gy,
                                             double *__restrict__ gz, int accumulate) {
    const double s = -1.0 / delta;
    if (accumulate) {
        gx[p] += s * (double)sx;
        gy[p] += s * (double)sy;
        gz[p] += s * (double)sz;
    } else {
        gx[p] = s * (double)sx;
        gy[p] = s * (double)sy;
        gz[p] = s * (double)sz;
    }
}

// Two neighbouring values, aligned only as one value is (the hardware needs no more).
template <typename Rt> struct value_pair;
template <> struct value_pair<double> {
    typedef double t __attribute__((ext_vector_type(2), aligned(8)));
};
template <> struct value_pair<float> {
    typedef float t __attribute__((ext_vector_type(2), aligned(4)));
};

// The potential read from the mesh (wrapped indices), row by row.  Bound by the cache lines
// looked up, which an LDS tile of the same values does not improve on: 2e6 particles in key order
// on 64^3 56 us against 78 from tiles, 256^3 on 256^3 in FP32 535 against 567 (699 with single
// loads and tiles), 128^3 on 256^3 in FP64 128 against 202 with single loads.
template <typename Rt>
__device__ __forceinline__ void interp_direct(double x, double y, double z,
                                              const Rt *__restrict__ phi, double delta, int ng,
                                              Rt &sx, Rt &sy, Rt &sz) {
    double wx[2], wy[2], wz[2];
    const int i = wrap_index(cic_base(x, delta, wx[0], wx[1]), ng);
    const int j = wrap_index(cic_base(y, delta, wy[0], wy[1]), ng);
    const int k = wrap_index(cic_base(z, delta, wz[0], wz[1]), ng);
    const uint32_t N = (uint32_t)ng;
    uint32_t ox[6], oy[6];   // rows and planes i - 2 .. i + 3 (meshes have at most 2^30 points)
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        ox[a] = (uint32_t)wrap_near(i + a - 2, ng) * N * N;
        oy[a] = (uint32_t)wrap_near(j + a - 2, ng) * N;
    }
    stencil<Rt> v;
    if (k >= 2 && k + 3 < ng) {
        v.read([&](int a, int b, int c, Rt *d) {
            typedef typename value_pair<Rt>::t pair;
            const pair r = *(const pair *)(phi + (ox[a + 2] + oy[b + 2] + (uint32_t)(k + c)));
            d[0] = r.x;
            d[1] = r.y;
        });
    } else {
        v.read([&](int a, int b, int c, Rt *d) {
            const uint32_t o = ox[a + 2] + oy[b + 2];
            d[0] = phi[o + (uint32_t)wrap_near(k + c, ng)];
            d[1] = phi[o + (uint32_t)wrap_near(k + c + 1, ng)];
        });
    }
    cic_gradient<Rt>(v, wx, wy, wz, sx, sy, sz);
}

template <typename Rt>
__global__ __launch_bounds__(PM_THREADS) void k_pm_interp(
    uint64_t n, const double *x, const double *y, const double *z, const Rt *__restrict__ phi,
    double delta, int ng, double *__restrict__ gx, double *__restrict__ gy,
    double *__restrict__ gz, int accumulate, pm_batch B, pm_sorted S) {
    const uint64_t p = (uint64_t)blockIdx.x * PM_THREADS + threadIdx.x;
    if (p >= n)
        return;
    const uint32_t *mult;
    const bool sorted = S.select(x, y, z, mult);
    if (B.boxes) {
        const dzs_bbox &bx = B.boxes[B.key[p] >> DZS_BATCH_SHIFT];
        delta = bx.delta;
        ng = bx.ng;
        phi += bx.mesh_off;
    }
    Rt sx, sy, sz;
    interp_direct<Rt>(x[p], y[p], z[p], phi, delta, ng, sx, sy, sz);
    if (sorted) {
        // one row instead of a line of each of three arrays
        const double s = -1.0 / delta;
        pm_row &r = S.out[S.perm[p]];
        r.v[0] = s * (double)sx;
        r.v[1] = s * (double)sy;
        r.v[2] = s * (double)sz;
    } else {
        interp_store<Rt>(p, delta, sx, sy, sz, gx, gy, gz, accumulate);
    }
}

// The forces of sorted particles to (or onto) the caller's arrays.
__global__ __launch_bounds__(PM_THREADS) void k_pm_out(uint64_t n, pm_sorted S,
                                                       double *__restrict__ gx,
                                                       double *__restrict__ gy,
                                                       double *__restrict__ gz, int accumulate) {
    const uint64_t p = (uint64_t)blockIdx.x * PM_THREADS + threadIdx.x;
    if (p >= n || !S.used())
        return;
    const pm_row r = S.out[p];
    if (accumulate) {
        gx[p] += r.v[0];
        gy[p] += r.v[1];
        gz[p] += r.v[2];
    } else {
        gx[p] = r.v[0];
        gy[p] = r.v[1];
        gz[p] = r.v[2];
    }
}


// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
static bool make_plan(int n, fft_plan *P) {
    P->n = n;
    P->n_stages = 0;
    int m = n;
    while (m % 4 == 0 && P->n_stages < FFT_MAX_STAGES) {
        P->radix[P->n_stages++] = 4;
        m /= 4;
    }
    while (m % 2 == 0 && P->n_stages < FFT_MAX_STAGES) {
        P->radix[P->n_stages++] = 2;
        m /= 2;
    }
    while (m % 3 == 0 && P->n_stages < FFT_MAX_STAGES) {
        P->radix[P->n_stages++] = 3;
        m /= 3;
    }
    return m == 1;
}

// largest power of two t <= cap with t * ng <= FFT_ELEMS and t dividing ng
static int tile_lines(int ng, int cap) {
    int t = 1;
    while (2 * t <= cap && 2 * t * ng <= FFT_ELEMS && ng % (2 * t) == 0)
        t *= 2;
    return t;
}

// complex lines per x tile: each carries two real lines, so 2 CL must divide N_g
static int pair_lines(int ng) {
    int t = 1;
    while (2 * t <= 16 && 2 * t * ng <= FFT_ELEMS && ng % (4 * t) == 0)
        t *= 2;
    return t;
}

// even 2^a 3^b sides (the x passes pair real lines and keep N_g/2 + 1 planes)
bool dzs_pm_mesh_ok(int ng) {
    fft_plan P;
    return ng >= 8 && ng <= 1024 && ng % 2 == 0 && make_plan(ng, &P);
}

// tables at ctx->pm_tables: [0, 2n) twiddles (double2), [2n, 3n) gt, [3n, 4n) k^2
static dzs_status upload_tables(dzs_ctx *ctx, int ng, double L, double r_s, hipStream_t s) {
    // staged in the context's host table when it has one (the allocation-free entry point),
    // else in a temporary
    std::vector<double> tmp(ctx->pm_host_tab ? 0 : 4 * (size_t)ng);
    double *h = ctx->pm_host_tab ? ctx->pm_host_tab : tmp.data();
    const long double pi = 3.14159265358979323846264338327950288L;
    for (int m = 0; m < ng; ++m) {
        long double ang = -2.0L * pi * m / ng;
        h[2 * m] = (double)cosl(ang);
        h[2 * m + 1] = (double)sinl(ang);
    }
    const double delta = L / ng;
    for (int m = 0; m < ng; ++m) {
        const int nn = m < ng / 2 ? m : m - ng;  // frequency index in [-ng/2, ng/2)
        const long double k = 2.0L * pi * nn / L;
        long double hh = 0.5L * k * delta;
        long double sinc = hh == 0.0L ? 1.0L : sinl(hh) / hh;
        long double w2 = sinc * sinc * sinc * sinc;  // W^2 per axis: sinc^4
        h[2 * ng + m] = (double)(expl(-k * k * (long double)r_s * r_s) / w2);
        h[3 * ng + m] = (double)(k * k);
    }
    DZS_HIP(ctx, hipMemcpyAsync(ctx->pm_tables, h, sizeof(double) * 4 * (size_t)ng,
                                hipMemcpyHostToDevice, s));
    DZS_HIP(ctx, hipStreamSynchronize(s));
    return DZS_OK;
}

// The Poisson solve (x, y passes forward, z pass with the Green's function, y, x passes
// inverse) over n_meshes meshes of side P.n, in the complex type C of the form.
template <typename C>
static dzs_status pm_solve(dzs_ctx *ctx, const fft_plan &P, const double2 *tw, const double *gt,
                           const double *k2t, double q_scale, double gconst, uint32_t n_meshes,
                           pm_batch B, hipStream_t s) {
    typedef decltype(C::x) Rt;
    const int ng = P.n;
    const int nkx = ng / 2 + 1;                  // k_x planes kept
    const int CL = pair_lines(ng);               // complex lines per x tile (2 CL real lines)
    const int TZ = tile_lines(ng, 16);           // lines per y tile
    const int TL = tile_lines(ng, FFT_ELEMS);    // lines per z tile
    const uint32_t x_per = (uint32_t)((uint64_t)ng * (ng / (2 * CL)));
    const uint32_t y_per = (uint32_t)((uint64_t)nkx * (ng / TZ));
    const uint32_t z_per = (uint32_t)((uint64_t)nkx * (ng / TL));
    const unsigned long long *mq = (const unsigned long long *)ctx->mesh_q;
    C *mc = (C *)ctx->mesh_c;
    Rt *phi = (Rt *)ctx->mesh_phi;
    // a tile's lines and the twiddles, so that small meshes leave LDS for more workgroups
    const auto lds = [&](int lines) { return (uint32_t)(sizeof(C) * ng * (lines + 1)); };
    pm_batch Bx = B, By = B, Bz = B;
    Bx.blocks_per_mesh = (int)x_per;
    By.blocks_per_mesh = (int)y_per;
    Bz.blocks_per_mesh = (int)z_per;
    const dim3 gx(x_per * n_meshes), gy(y_per * n_meshes), gz(z_per * n_meshes);
    {
        dzs_timed t(ctx, KC_PM_FFT_X, s);
        hipLaunchKernelGGL(k_fft_x_r2c<C>, gx, dim3(FFT_THREADS), lds(CL), s, mq, mc, tw, P, CL,
                           q_scale, Bx);
        DZS_TRY(dzs_check_launch(ctx, "fft_x_fwd"));
    }
    {
        dzs_timed t(ctx, KC_PM_FFT_Y, s);
        hipLaunchKernelGGL((k_fft_y<false, C>), gy, dim3(FFT_THREADS), lds(TZ), s, mc, tw, P, TZ, By);
        DZS_TRY(dzs_check_launch(ctx, "fft_y_fwd"));
    }
    {
        dzs_timed t(ctx, KC_PM_FFT_Z_GREEN, s);
        hipLaunchKernelGGL(k_fft_z_green<C>, gz, dim3(FFT_THREADS), lds(TL), s, mc, tw, gt, k2t, P, TL,
                           gconst, Bz);
        DZS_TRY(dzs_check_launch(ctx, "fft_z_green"));
    }
    {
        dzs_timed t(ctx, KC_PM_FFT_Y, s);
        hipLaunchKernelGGL((k_fft_y<true, C>), gy, dim3(FFT_THREADS), lds(TZ), s, mc, tw, P, TZ, By);
        DZS_TRY(dzs_check_launch(ctx, "fft_y_inv"));
    }
    {
        dzs_timed t(ctx, KC_PM_FFT_X, s);
        hipLaunchKernelGGL(k_fft_x_c2r<C>, gx, dim3(FFT_THREADS), lds(CL), s, mc, phi, tw, P, CL, Bx);
        DZS_TRY(dzs_check_launch(ctx, "fft_x_inv"));
    }
    return DZS_OK;
}

// The default chunk (a power of two).  Few particles: waves of 64 particles on their own, so
// that a piece waits for no other (8000 particles on 48^3 77 -> 12 us).  Then 256, four pieces
// that share a tile (128^3 on 256^3, key order: 230 us, 1024 at a time 251, and 277 before), and
// with more particles longer chunks, whose tiles' shared lines stay in one L2 (256^3 on 256^3:
// 783 us by 256, 589 by 1024, 518 by 4096; 671 before).
#define PM_SMALL 65536

static int32_t default_chunk(uint64_t n) {
    if (n < PM_SMALL)
        return 64;
    int32_t c = 256;
    while (c < 4096 && (uint64_t)c * 2 * 4096 <= n)
        c *= 2;
    return c;
}

// Order of the particles as they come, from neighbours in memory at 256 places: for three in four
// of them, is the neighbour less than a quarter as far as another sample, from anywhere?  (Pairs
// of pairs at equal separations, coincident particles, say nothing.)  In key order it is for 19 in
// 20, in lattice order for 9 in 10.  Without an order the two separations are alike whatever the
// set, so it is for half at the most: one dense clump, whose random pairs are all close, as well as
// a uniform set.  (Separations measured against L / 16 instead took a shuffled set with nine in
// ten in a clump of L / 200 for ordered: 131,072 on 64^3 4.09 ms.)
#define PM_ORDER_SAMPLES 256
__global__ __launch_bounds__(PM_ORDER_SAMPLES) void k_pm_order(uint64_t n, const double *__restrict__ x,
                                                   const double *__restrict__ y,
                                                   const double *__restrict__ z,
                                                   uint32_t *__restrict__ ordered) {
    __shared__ double s_p[3][PM_ORDER_SAMPLES];
    __shared__ uint32_t s_near, s_cnt;
    if (threadIdx.x == 0)
        s_near = s_cnt = 0u;
    // (multiples of the golden ratio: even steps would meet the row ends of a lattice of 2^k a side)
    const uint64_t p = ((uint64_t)(threadIdx.x * 2654435769u) * (n - 1)) >> 32;
    const double px = s_p[0][threadIdx.x] = x[p], py = s_p[1][threadIdx.x] = y[p],
                 pz = s_p[2][threadIdx.x] = z[p];
    const double next = fmax(fabs(x[p + 1] - px), fmax(fabs(y[p + 1] - py), fabs(z[p + 1] - pz)));
    __syncthreads();
    const uint32_t o = (threadIdx.x * 101u + 53u) % PM_ORDER_SAMPLES;   // (never the sample itself)
    const double other =
        fmax(fabs(s_p[0][o] - px), fmax(fabs(s_p[1][o] - py), fabs(s_p[2][o] - pz)));
    const uint64_t near = __ballot(4.0 * next < other), cnt = __ballot(next != other);
    if ((threadIdx.x & 63u) == 0u) {
        atomicAdd(&s_near, (uint32_t)__popcll(near));
        atomicAdd(&s_cnt, (uint32_t)__popcll(cnt));
    }
    __syncthreads();
    if (threadIdx.x == 0)
        *ordered = 4u * s_near >= 3u * s_cnt;
}

// Keys, and the particles as rows, so that each is gathered from one line instead of four.
__global__ __launch_bounds__(PM_THREADS) void k_pm_rows(uint64_t n, const double *__restrict__ x,
                                                        const double *__restrict__ y,
                                                        const double *__restrict__ z,
                                                        const uint32_t *__restrict__ mult,
                                                        double scale,
                                                        const uint32_t *__restrict__ ordered,
                                                        uint64_t *__restrict__ key,
                                                        uint32_t *__restrict__ idx,
                                                        pm_row *__restrict__ row) {
    const uint64_t i = (uint64_t)blockIdx.x * PM_THREADS + threadIdx.x;
    if (i >= n || *ordered)
        return;
    const pm_row r = {{x[i], y[i], z[i]}, mult[i], 0u};
    key[i] = dzs_morton(r.v[0], r.v[1], r.v[2], scale);
    idx[i] = (uint32_t)i;
    row[i] = r;
}

__global__ __launch_bounds__(PM_THREADS) void k_pm_gather(uint64_t n,
                                                          const pm_row *__restrict__ row,
                                                          const uint32_t *__restrict__ perm,
                                                          const uint32_t *__restrict__ ordered,
                                                          double *__restrict__ sx,
                                                          double *__restrict__ sy,
                                                          double *__restrict__ sz,
                                                          uint32_t *__restrict__ smult) {
    const uint64_t i = (uint64_t)blockIdx.x * PM_THREADS + threadIdx.x;
    if (i >= n || *ordered)
        return;
    const pm_row r = row[perm[i]];
    sx[i] = r.v[0];
    sy[i] = r.v[1];
    sz[i] = r.v[2];
    smult[i] = r.mult;
}

// Particles in no order: sorted by the top 15 bits of their Morton keys, two passes (32 cells a
// side; on finer meshes than 256 points four passes, 1290 cells a side), so that neighbours
// in memory share mesh lines.  As they come, every one of a particle's 8 atomics and 28 loads
// is a mesh line of its own, and the atomics of a clump queue on the same points.  Deposit and
// interpolation with the sort against without: 1e6 clustered particles on 192^3 312 against
// 708 us, 2e6 clustered on 64^3 318 against 2170, 8e6 uniform on 384^3 2.43 against 6.10 ms.
// From where it starts to pay: 1.4e5 particles on 64^3 clustered 98 against 129 us, on 32^3
// uniform 89 against 81; 7e4 on 64^3 97 against 76.  Not on meshes of more than 32 points a
// particle, where neighbours share few lines in any order: 1.4e5 on 192^3 161 against 126.
// Positions go to their place and forces back as rows of 32 bytes, one line each: gathered from
// four arrays and scattered to three, 1e6 took 66 instead of 25 us and 110 instead of 89, 8e6
// 0.61 instead of 0.20 ms and 1.17 instead of 0.91.
// Particles in order pay for the look and a dozen kernels that exit at once: 131,072 on 64^3 90 us
// against 68 with a chunk given (which never sorts), 2e6 on 128^3 240 against 212, 1.7e7 on 256^3
// 1.36 ms against 1.32.  Nine in ten of 131,072 in a clump of L / 200, shuffled: 4.09 -> 0.12 ms.
#define PM_SORT_MIN 131072
static const pm_sorted NO_SORT{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
static dzs_status pm_sort(dzs_ctx *ctx, const dzs_particles *p, double L, int ng, pm_sorted *S,
                          hipStream_t s) {
    const uint64_t n = p->n;
    // (a context shell without scratch of its own passes the particles as they are)
    if (n < PM_SORT_MIN || n > 0xffffffffull || (uint64_t)ng * ng * ng > 32 * n || !ctx->arena ||
        ctx->arena_bytes < 60 * n + 64)
        return DZS_OK;
    ctx->tree_built = false;   // the arena is the tree's
    // (the rows are free again once gathered: the forces' rows take their place)
    pm_row *row = (pm_row *)ctx->arena;
    double *sx = (double *)(row + n), *sy = sx + n, *sz = sy + n;
    uint32_t *sm = (uint32_t *)(sz + n), *ordered = sm + n;
    {
        dzs_timed t(ctx, KC_KEYS, s);
        hipLaunchKernelGGL(k_pm_order, dim3(1), dim3(PM_ORDER_SAMPLES), 0, s, n, (const double *)p->x,
                           (const double *)p->y, (const double *)p->z, ordered);
        DZS_TRY(dzs_check_launch(ctx, "pm_order"));
        hipLaunchKernelGGL(k_pm_rows, dim3(blocks_for(n, PM_THREADS)), dim3(PM_THREADS), 0, s, n,
                           (const double *)p->x, (const double *)p->y, (const double *)p->z,
                           (const uint32_t *)p->mult, DZS_KEY_SIDE / L,
                           (const uint32_t *)ordered, ctx->key, ctx->idx, row);
        DZS_TRY(dzs_check_launch(ctx, "pm_rows"));
    }
    DZS_TRY(dzs_radix_sort(ctx, n, s, ng > 256 ? 4 : 6, ordered));
    dzs_timed t(ctx, KC_PERMUTE, s);
    hipLaunchKernelGGL(k_pm_gather, dim3(blocks_for(n, PM_THREADS)), dim3(PM_THREADS), 0, s, n,
                       (const pm_row *)row, (const uint32_t *)ctx->idx,
                       (const uint32_t *)ordered, sx, sy, sz, sm);
    DZS_TRY(dzs_check_launch(ctx, "pm_gather"));
    *S = pm_sorted{ordered, row, sx, sy, sz, sm, ctx->idx};
    return DZS_OK;
}

template <typename Rt>
static dzs_status pm_interp(dzs_ctx *ctx, const dzs_particles *p, int accumulate, double delta,
                            int ng, pm_batch B, pm_sorted S, hipStream_t s) {
    if (p->n == 0)
        return DZS_OK;
    dzs_timed t(ctx, KC_PM_INTERP, s);
    hipLaunchKernelGGL(k_pm_interp<Rt>, dim3(blocks_for(p->n, PM_THREADS)), dim3(PM_THREADS), 0,
                       s, p->n, (const double *)p->x, (const double *)p->y, (const double *)p->z,
                       (const Rt *)ctx->mesh_phi, delta, ng, p->gx, p->gy, p->gz, accumulate, B,
                       S);
    DZS_TRY(dzs_check_launch(ctx, "pm_interp"));
    if (!S.ordered)
        return DZS_OK;
    hipLaunchKernelGGL(k_pm_out, dim3(blocks_for(p->n, PM_THREADS)), dim3(PM_THREADS), 0, s, p->n,
                       S, p->gx, p->gy, p->gz, accumulate);
    return dzs_check_launch(ctx, "pm_out");
}

// zero fill by a kernel (a memset node in a captured graph is avoided)
__global__ __launch_bounds__(PM_THREADS) void k_zero_u64(uint64_t n, unsigned long long *a) {
    for (uint64_t i = (uint64_t)blockIdx.x * PM_THREADS + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * PM_THREADS)
        a[i] = 0ull;
}

// chunk: particles per LDS tile (a power of two in [DZS_PM_CHUNK_MIN, _MAX]), 0 for the
// default, -1 for the direct deposit.
static dzs_status pm_deposit(dzs_ctx *ctx, const dzs_particles *p, uint64_t cells, double delta,
                             int ng, pm_batch B, pm_sorted S, int32_t chunk, hipStream_t s) {
    dzs_timed t(ctx, KC_PM_DEPOSIT, s);
    const uint64_t zb = (cells + PM_THREADS - 1) / PM_THREADS;
    hipLaunchKernelGGL(k_zero_u64, dim3((uint32_t)(zb < 65536 ? zb : 65536)), dim3(PM_THREADS), 0,
                       s, cells, (unsigned long long *)ctx->mesh_q);
    DZS_TRY(dzs_check_launch(ctx, "mesh_clear"));
    if (p->n == 0)
        return DZS_OK;
    if (chunk == 0)
        chunk = default_chunk(p->n);
    const dim3 grid(blocks_for(p->n, chunk < 0 ? PM_THREADS : (uint32_t)chunk));
#define DEPOSIT(KERNEL, THREADS, ...)                                                            \
    hipLaunchKernelGGL(KERNEL, grid, dim3(THREADS), 0, s, p->n, (const double *)p->x,            \
                       (const double *)p->y, (const double *)p->z, (const uint32_t *)p->mult,    \
                       delta, ng, (unsigned long long *)ctx->mesh_q, B, __VA_ARGS__)
    if (chunk < 0)
        DEPOSIT(k_pm_deposit, PM_THREADS, S);
    else if (chunk == 64)
        DEPOSIT((k_pm_deposit_tiled<64, 1>), 64, S, (uint32_t)chunk);
    else if (chunk == 256)
        DEPOSIT((k_pm_deposit_tiled<PM_THREADS, 1>), PM_THREADS, S, (uint32_t)chunk);
    else if (chunk == 512)
        DEPOSIT((k_pm_deposit_tiled<PM_THREADS, 2>), PM_THREADS, S, (uint32_t)chunk);
    else
        DEPOSIT((k_pm_deposit_tiled<PM_THREADS, PM_ITEMS>), PM_THREADS, S, (uint32_t)chunk);
#undef DEPOSIT
    return dzs_check_launch(ctx, "pm_deposit");
}

// The potential on the mesh (deposit, forward FFT, Green's function, inverse FFT).
static dzs_status pm_mesh(dzs_ctx *ctx, const dzs_box *box, const dzs_particles *p,
                          const dzs_pm_params *prm, pm_sorted S, hipStream_t s) {
    const int ng = prm->ng;
    fft_plan P;
    if (!dzs_pm_mesh_ok(ng) || !make_plan(ng, &P))
        return dzs_fail(ctx, DZS_EINVAL, "pm_force: mesh side %d is not an even 2^a 3^b", ng);
    const uint64_t ng3 = (uint64_t)ng * ng * ng;
    const double delta = box->L / ng;
    if (ctx->pm_tab_ng != ng || ctx->pm_tab_L != box->L || ctx->pm_tab_rs != prm->r_s) {
        DZS_TRY(upload_tables(ctx, ng, box->L, prm->r_s, s));
        ctx->pm_tab_ng = ng;
        ctx->pm_tab_L = box->L;
        ctx->pm_tab_rs = prm->r_s;
    }
    const double2 *tw = (const double2 *)ctx->pm_tables;
    const double *gt = ctx->pm_tables + 2 * ng;
    const double *k2t = ctx->pm_tables + 3 * ng;
    const pm_batch none{nullptr, nullptr, 0, nullptr};
    DZS_TRY(pm_deposit(ctx, p, ng3, delta, ng, none, S, prm->tile_chunk, s));
    const double q_scale = box->m0 / (DEP_FRAC * delta * delta * delta);
    const double gconst = -4.0 * 3.14159265358979323846 * box->G / (double)ng3;
    if (prm->precision == DZS_FP32)
        return pm_solve<float2>(ctx, P, tw, gt, k2t, q_scale, gconst, 1, none, s);
    return pm_solve<double2>(ctx, P, tw, gt, k2t, q_scale, gconst, 1, none, s);
}

// The long-range force at the particles from the potential pm_mesh left on the mesh
// (same box, particles, order and parameters).
static dzs_status pm_force_at(dzs_ctx *ctx, const dzs_box *box, const dzs_particles *p,
                              const dzs_pm_params *prm, pm_sorted S, hipStream_t s) {
    const int ng = prm->ng;
    const double delta = box->L / ng;
    const pm_batch none{nullptr, nullptr, 0, nullptr};
    if (prm->precision == DZS_FP32)
        return pm_interp<float>(ctx, p, prm->accumulate, delta, ng, none, S, s);
    return pm_interp<double>(ctx, p, prm->accumulate, delta, ng, none, S, s);
}

// The same in two calls for particles in key order (the steps), with other work between.
dzs_status dzs_pm_solve(dzs_ctx *ctx, const dzs_box *box, const dzs_particles *p,
                        const dzs_pm_params *prm, hipStream_t s) {
    return pm_mesh(ctx, box, p, prm, NO_SORT, s);
}

dzs_status dzs_pm_apply(dzs_ctx *ctx, const dzs_box *box, const dzs_particles *p,
                        const dzs_pm_params *prm, hipStream_t s) {
    return pm_force_at(ctx, box, p, prm, NO_SORT, s);
}

dzs_status dzs_pm_run(dzs_ctx *ctx, const dzs_box *box, const dzs_particles *p,
                      const dzs_pm_params *prm, hipStream_t s) {
    pm_sorted S = NO_SORT;
    if (prm->tile_chunk == 0)
        DZS_TRY(pm_sort(ctx, p, box->L, prm->ng, &S, s));
    DZS_TRY(pm_mesh(ctx, box, p, prm, S, s));
    return pm_force_at(ctx, box, p, prm, S, s);
}

// A batch: every box's mesh at its offset of the mesh arrays.  dzs_pm_batch_prepare fills
// each box's mesh offset, spacing, deposit scale and table offset in the host table hb[] and
// uploads the twiddle and Green's function tables of every box and mesh size; the caller
// uploads hb[] to the device table.  Boxes of one mesh size share each FFT launch.
dzs_status dzs_pm_batch_prepare(dzs_ctx *ctx, uint32_t nb, dzs_bbox *hb, hipStream_t s) {
    ctx->batch_sides.clear();
    uint64_t cells = 0;
    for (uint32_t b = 0; b < nb; ++b) {
        if (!dzs_pm_mesh_ok(hb[b].ng))
            return dzs_fail(ctx, DZS_EINVAL, "batch: box %u mesh side %d is not an even 2^a 3^b "
                            "in [8, 1024]", b, hb[b].ng);
        hb[b].mesh_off = cells;
        cells += (uint64_t)hb[b].ng * hb[b].ng * hb[b].ng;
        bool seen = false;
        for (int v : ctx->batch_sides)
            seen |= v == hb[b].ng;
        if (!seen)
            ctx->batch_sides.push_back(hb[b].ng);
    }
    const uint64_t cap_cells = (uint64_t)ctx->cap_ng * ctx->cap_ng * ctx->cap_ng;
    if (cells > cap_cells)
        return dzs_fail(ctx, DZS_ECAPACITY, "batch: meshes need %llu cells, the context holds %llu",
                        (unsigned long long)cells, (unsigned long long)cap_cells);
    ctx->batch_cells = cells;
    // tables: per box [Green factor (ng), k^2 (ng)], then per mesh side twiddles (2 ng)
    std::vector<double> tab;
    const long double pi = 3.14159265358979323846264338327950288L;
    for (uint32_t b = 0; b < nb; ++b) {
        const int ng = hb[b].ng;
        const double L = hb[b].L, delta = L / ng;
        hb[b].delta = delta;
        hb[b].q_scale = hb[b].m0 / (DEP_FRAC * delta * delta * delta);
        hb[b].tab_off = tab.size();
        tab.resize(tab.size() + 2 * (size_t)ng);
        double *gt = tab.data() + hb[b].tab_off, *k2 = gt + ng;
        for (int m = 0; m < ng; ++m) {
            const int nn = m < ng / 2 ? m : m - ng;
            const long double k = 2.0L * pi * nn / L;
            const long double hh = 0.5L * k * delta;
            const long double sinc = hh == 0.0L ? 1.0L : sinl(hh) / hh;
            const long double w2 = sinc * sinc * sinc * sinc;
            gt[m] = (double)(expl(-k * k * (long double)hb[b].r_s * hb[b].r_s) / w2);
            k2[m] = (double)(k * k);
        }
    }
    ctx->batch_tw_off.clear();
    ctx->batch_cls_first.clear();
    std::vector<uint32_t> members;
    for (int ng : ctx->batch_sides) {
        ctx->batch_tw_off.push_back(tab.size());
        tab.resize(tab.size() + 2 * (size_t)ng);
        for (int m = 0; m < ng; ++m) {
            const long double ang = -2.0L * pi * m / ng;
            tab[ctx->batch_tw_off.back() + 2 * m] = (double)cosl(ang);
            tab[ctx->batch_tw_off.back() + 2 * m + 1] = (double)sinl(ang);
        }
        ctx->batch_cls_first.push_back((uint32_t)members.size());
        for (uint32_t b = 0; b < nb; ++b)
            if (hb[b].ng == ng)
                members.push_back(b);
    }
    ctx->batch_cls_first.push_back((uint32_t)members.size());
    // per box 2 ng and per distinct side 2 ng doubles: within the 4 max_boxes max_mesh_side
    // the context holds
    if (tab.size() > ctx->batch_tab_cap)
        return dzs_fail(ctx, DZS_ECAPACITY, "batch: tables of %llu doubles exceed the context's "
                        "%llu", (unsigned long long)tab.size(),
                        (unsigned long long)ctx->batch_tab_cap);
    DZS_HIP(ctx, hipMemcpyAsync(ctx->batch_tab, tab.data(), sizeof(double) * tab.size(),
                                hipMemcpyHostToDevice, s));
    DZS_HIP(ctx, hipMemcpyAsync(ctx->batch_members, members.data(),
                                sizeof(uint32_t) * members.size(), hipMemcpyHostToDevice, s));
    // the staging vectors die here: wait for the copies
    DZS_HIP(ctx, hipStreamSynchronize(s));
    return DZS_OK;
}

// The long-range force of every box of a prepared batch into g (g = g_long); db is the device
// box table and ctx->key the sorted keys (box in the top digits) of the particles.
dzs_status dzs_pm_run_batch(dzs_ctx *ctx, const dzs_particles *p, int precision,
                            int32_t tile_chunk, const dzs_bbox *db, double G, hipStream_t s) {
    const pm_batch all{db, nullptr, 0, (const uint64_t *)ctx->key};
    DZS_TRY(pm_deposit(ctx, p, ctx->batch_cells, 0.0, 0, all, NO_SORT, tile_chunk, s));
    for (size_t c = 0; c < ctx->batch_sides.size(); ++c) {
        const int ng = ctx->batch_sides[c];
        fft_plan P;
        make_plan(ng, &P);
        const uint32_t nm = ctx->batch_cls_first[c + 1] - ctx->batch_cls_first[c];
        const pm_batch B{db, ctx->batch_members + ctx->batch_cls_first[c], 0,
                         (const uint64_t *)ctx->key};
        const double2 *tw = (const double2 *)(ctx->batch_tab + ctx->batch_tw_off[c]);
        const double gconst = -4.0 * 3.14159265358979323846 * G / ((double)ng * ng * ng);
        if (precision == DZS_FP32)
            DZS_TRY(pm_solve<float2>(ctx, P, tw, ctx->batch_tab, ctx->batch_tab, 0.0, gconst, nm,
                                     B, s));
        else
            DZS_TRY(pm_solve<double2>(ctx, P, tw, ctx->batch_tab, ctx->batch_tab, 0.0, gconst, nm,
                                      B, s));
    }
    if (precision == DZS_FP32)
        return pm_interp<float>(ctx, p, 0, 0.0, 0, all, NO_SORT, s);
    return pm_interp<double>(ctx, p, 0, 0.0, 0, all, NO_SORT, s);
}
