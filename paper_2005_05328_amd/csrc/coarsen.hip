// DZS coarsening on the GPU (paper Sec. 2.2 and 2.2.1, eqs. 1 and 3).
//
// The paper walks the tree from the root and replaces every node that meets the merging
// criterion by one particle, without descending further.  Equivalently, every particle joins
// its shallowest qualifying ancestor.  On the GPU the levels go from k_min down: at level
// k the first particle of each level-k cube (a contiguous run of the (key, id)-sorted state)
// that holds two or more stands for its cube.  Its members are summed in order — mult, mult*x
// and mult*p with Neumaier compensation —, the criterion is tested, and if it holds the members
// are stamped with the first one's index and the sum takes the first one's row.  Particles
// stamped at a shallower level are skipped.  A compaction then keeps the rows of survivors and
// of first members, in sorted order.
//
// The node sums, the centre of mass, the minimum-image distance and the threshold comparison
// use the exact operation sequence of the definition (no contraction), so the grouping is
// bit-identical to any implementation that follows the same definition.
//
// Two criteria (Sec. 2.2.1): the geometric one (eq. 1 with eq. 3) compares |d|^2 with a
// per-level threshold; the dynamical one (eq. 2 with eq. 3) compares G m0 K l_k^2 with
// alpha a_min D^4, where a_min, the smallest previous acceleration inside the lightcone plus
// buffer, is reduced on the device beforehand (an order-independent minimum, so exact).
#include "internal.h"

#define DZ_THREADS 256
#define DZ_NONE 0xffffffffu

static inline uint32_t blocks_for(uint64_t n, uint32_t t) { return (uint32_t)((n + t - 1) / t); }

struct neumaier {
    double sum, comp;
};

// (the larger of sum and v first, by selects: a branch here costs more than the sum)
__device__ __forceinline__ void nm_add(neumaier &a, double v) {
    const double t = a.sum + v;
    const bool big = fabs(a.sum) >= fabs(v);
    const double hi = big ? a.sum : v, lo = big ? v : a.sum;
    a.comp += (hi - t) + lo;
    a.sum = t;
}

__device__ __forceinline__ double nm_value(const neumaier &a) { return a.sum + a.comp; }

struct dz_level_args {
    uint64_t n;
    int k0, k1, crit;                 // the levels of this launch
    double L, iL;                     // box side, 1 / L
    double T2[DZS_KEY_BITS + 1], T2_max;   // levels whose threshold exceeds T2_max merge nothing
    double Gm0, Rb, alpha;            // dynamical criterion
    const unsigned long long *amin2;  // bits of min g.g inside the lightcone (device)
    double xo[3];
    const uint64_t *key;
    double *f[6];                     // x, y, z, px, py, pz
    uint32_t *mult, *id;
    uint8_t *type;
    uint32_t *head;
    uint8_t *keep;                    // 0: a member of a group, not its first
    int fresh;                        // no row is a member of a group yet
    uint32_t *stat;                   // groups made, over DZ_STATS words a cache line apart
};

// Largest minimum-image |x - x_obs| along one axis over the cube [a, a + l), widened by a
// margin far above the rounding of the keys and of the centre of mass.
// (iL = 1/L: its rounding is far below the margin too.)
__device__ __forceinline__ double dz_axis_far(double a, double l, double xo, double L, double iL) {
    const double m = 1e-9 * L;
    const double u = a - m - xo, v = a + l + m - xo;
    // the farthest offset, L/2 (mod L), lies inside [u, v]
    if (ceil((u - 0.5 * L) * iL) <= floor((v - 0.5 * L) * iL))
        return 0.5 * L;
    const double wu = u - L * floor(u * iL + 0.5), wv = v - L * floor(v * iL + 0.5);
    return fmax(fabs(wu), fabs(wv));
}

#define DZ_TILE 256          // particles of a workgroup, whose cubes it owns
#define DZ_LT 128            // threads: 16 cubes at a time
#define DZ_WINDOW 336        // rows held in LDS: the tile and what its last cube has past it
#define DZ_UNROLL 4          // members loaded together from LDS
#define DZ_UNROLL_MEM 16     // and from memory, where a load takes a hundred times as long as a sum
#define DZ_MARK 512          // every DZ_MARK-th particle is a mark: cubes with two marks are large
#define DZ_MARKS 32          // marks that a workgroup of k_dz_large looks at
#define DZ_LARGE 512         // its threads: 64 cubes at a time
#define DZ_ONE 256           // particles a cube from which a level takes its own launch
#define DZ_STATS 16          // counters of groups, a cache line apart

// Rows t0 .. t0 + len - 1 of the state, keys one more on either side (where there are any), and
// which rows are members of a group already.  Rows behind are read from memory.
struct dz_window {
    double f[6][DZ_WINDOW + 1];
    uint64_t key[DZ_WINDOW + 2];   // key[1] is row t0's
    uint32_t mult[DZ_WINDOW], id[DZ_WINDOW];
    uint8_t done[DZ_WINDOW];
};

struct dz_sum {
    neumaier S;
    uint64_t K;
    uint32_t min_id;
};

// One lane's sum over members 0 .. n - 1, in their order.  (Past the last, zeros: they change
// neither the sum nor its compensation, which are never -0.)
template <uint32_t U>
__device__ __forceinline__ void dz_members(uint32_t n, const double *src, const uint32_t *mult,
                                           const uint32_t *id, dz_sum &a) {
    for (uint32_t r = 0; r < n; r += U) {
        double v[U];
        uint32_t mu[U], ids[U];
#pragma unroll
        for (uint32_t q = 0; q < U; ++q) {
            const uint32_t j = min(r + q, n - 1);
            v[q] = src[j];
            mu[q] = mult[j];
            ids[q] = id[j];
        }
#pragma unroll
        for (uint32_t q = 0; q < U; ++q) {
            const bool in = r + q < n;
            const uint32_t m = in ? mu[q] : 0u;
            a.K += m;
            a.min_id = min(a.min_id, ids[q]);
            nm_add(a.S, in ? (double)m * v[q] : 0.0);
        }
    }
}

// Largest squared distance from the observer over the level-k cube of key prefix pk.
__device__ __forceinline__ double dz_far2(const dz_level_args &A, int k, uint64_t pk) {
    const double l = ldexp(A.L, -k);
    const double fx = dz_axis_far((double)dzs_compact3(pk >> 2) * l, l, A.xo[0], A.L, A.iL);
    const double fy = dz_axis_far((double)dzs_compact3(pk >> 1) * l, l, A.xo[1], A.L, A.iL);
    const double fz = dz_axis_far((double)dzs_compact3(pk) * l, l, A.xo[2], A.L, A.iL);
    return fx * fx + fy * fy + fz * fz;
}

// True where no level-k cube whose points all lie within far2 can merge: such cubes are skipped
// before their members are visited.
__device__ __forceinline__ bool dz_near(const dz_level_args &A, int k, double far2) {
    if (A.crit == DZS_CRIT_GEOMETRIC)
        return far2 * (1.0 + 1e-12) <= A.T2[k];
    const double Dmax = sqrt(far2) * (1.0 + 1e-12) - A.Rb;
    if (!(Dmax > 0.0))
        return true;
    const double l = ldexp(A.L, -k);
    const double amin = sqrt(__longlong_as_double((long long)*A.amin2));
    const double D2 = Dmax * Dmax;
    return (A.Gm0 * 2.0) * (l * l) >= (A.alpha * amin) * (D2 * D2) * (1.0 + 1e-9);
}

// Octal digits that two keys share.
__device__ __forceinline__ int dz_common(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;
    return x ? DZS_KEY_BITS - 1 - (63 - (int)__clzll((long long)x)) / 3 : DZS_KEY_BITS;
}

// Key of row i >= t0 - 1.
__device__ __forceinline__ uint64_t dz_key(const dz_level_args &A, const dz_window &W, uint64_t t0,
                                           uint64_t i) {
    const uint64_t o = i + 1 - t0;
    return o < DZ_WINDOW + 2 ? W.key[o] : A.key[i];
}

// One cube at level k whose first member is i, worked on by 8 lanes: each of the six sums, the
// multiplicity and the lowest id is one lane's, in the members' order.  WINDOW: rows t0 ..
// t0 + len - 1 are in W.
template <bool WINDOW>
__device__ __forceinline__ void dz_cube(const dz_level_args &A, int k, uint64_t i, dz_window *W,
                                        uint64_t t0, uint32_t len, uint32_t *s_groups) {
    const uint32_t lane = threadIdx.x & 7u, shift = threadIdx.x & 56u;
    const int sh = 3 * (DZS_KEY_BITS - k);
    const auto key = [&](uint64_t r) { return WINDOW ? dz_key(A, *W, t0, r) : A.key[r]; };
    const uint64_t pk = key(i) >> sh;
    const double l = ldexp(A.L, -k), lk2 = l * l;
    // the last member: strides of 8, then longer while they stay inside, then shorter
    uint64_t e = i;
    for (uint64_t stride = 8;;) {
        const uint64_t r = e + stride * (lane + 1u);
        const bool in = r < A.n && (key(r) >> sh) == pk;
        const uint32_t m = (uint32_t)__popc((uint32_t)(__ballot(in) >> shift) & 0xffu);
        e += stride * m;
        if (m == 8u) {
            stride *= 8;
        } else {
            if (stride == 1)
                break;
            stride /= 8;
        }
    }
    ++e;
    const uint32_t ax = lane < 6u ? lane : 5u;
    dz_sum a = {{0.0, 0.0}, 0, 0xffffffffu};
    if (!WINDOW)
        dz_members<DZ_UNROLL_MEM>((uint32_t)(e - i), A.f[ax] + i, A.mult + i, A.id + i, a);
    else if (e - t0 <= len)
        dz_members<DZ_UNROLL>((uint32_t)(e - i), W->f[ax] + (i - t0), W->mult + (i - t0),
                              W->id + (i - t0), a);
    else
        dz_members<DZ_UNROLL>((uint32_t)(e - i), A.f[ax] + i, A.mult + i, A.id + i, a);
    const uint64_t K = a.K;
    const double Kd = (double)K;
    double val = nm_value(a.S) / Kd;
    if (lane < 3u)
        val = dzs_wrap(val, A.L);
    const double dd = dzs_min_image(
        val - (lane == 0u ? A.xo[0] : lane == 1u ? A.xo[1] : A.xo[2]), A.L);
    const double dx = __shfl(dd, 0, 8), dy = __shfl(dd, 1, 8), dz = __shfl(dd, 2, 8);
    const double d2 = dx * dx + dy * dy + dz * dz;
    if (A.crit == DZS_CRIT_GEOMETRIC) {
        if (!(d2 > A.T2[k]))
            return;
    } else {
        const double D = sqrt(d2) - A.Rb;
        if (!(D > 0.0))
            return;
        const double amin = sqrt(__longlong_as_double((long long)*A.amin2));
        const double lhs = (A.Gm0 * Kd) * lk2;
        const double rhs = (A.alpha * amin) * ((D * D) * (D * D));
        if (!(lhs < rhs))
            return;
    }
    for (uint64_t r = i + lane; r < e; r += 8) {
        A.head[r] = (uint32_t)i;
        A.keep[r] = r == i;
        if (WINDOW && r - t0 < len)
            W->done[r - t0] = 1u;
    }
    if (lane < 6u) {
        A.f[lane][i] = val;
    } else if (lane == 6u) {
        A.mult[i] = (uint32_t)K;
        A.type[i] = 1u;
    } else {
        A.id[i] = a.min_id;
        atomicAdd(s_groups, 1u);
    }
}

// The large cubes of levels k0 .. k1: those that hold two marks (and so every cube of 1024
// particles or more, and none below 514).  k_dz_levels works on the others, a workgroup on all
// levels of what begins in its tile; a clump's cubes would keep one workgroup for themselves.  The
// level-k0 cube of the first mark inside belongs to a workgroup here, with all large cubes in it:
// their first marks follow from the marks' keys alone, level by level, so it visits particles only
// where a cube may merge.  Bound by the loads of the longest sum (one cube's members in their
// order).  1e6 particles, most of them in 8 clumps of scale L/40, that merge at levels well below
// k0: 2.34 -> 0.71 ms against the clumps in k_dz_levels (1.62 with a thread a cube and a launch a
// level); 9e5 of 1e6 in a clump of L/200 that is too near to merge 7.0 -> 0.67 (1.0).
__global__ __launch_bounds__(DZ_LARGE) void k_dz_large(dz_level_args A) {
    __shared__ uint32_t s_own[DZ_MARKS], s_work[DZ_LARGE];
    __shared__ uint32_t s_n, s_cnt, s_groups;
    const uint32_t tid = threadIdx.x;
    const uint32_t marks = (uint32_t)((A.n + DZ_MARK - 1) / DZ_MARK);
    const auto mark = [&](uint32_t j) { return A.key[(uint64_t)j * DZ_MARK]; };
    const auto common = [&](uint32_t a, uint32_t b) { return dz_common(mark(a), mark(b)); };
    if (tid == 0)
        s_n = s_groups = 0u;
    __syncthreads();
    if (tid < DZ_MARKS) {
        const uint32_t m = blockIdx.x * DZ_MARKS + tid;
        if (m + 1 < marks && common(m, m + 1) >= A.k0 && (m == 0 || common(m - 1, m) < A.k0))
            s_own[atomicAdd(&s_n, 1u)] = m;
    }
    __syncthreads();
    const uint32_t owned = s_n;
    for (uint32_t w = 0; w < owned; ++w) {
        const uint32_t m = s_own[w];
        uint32_t in = m + 1, end = marks;   // the last mark inside, the first behind
        while (end - in > 1) {
            const uint32_t mid = in + (end - in) / 2;
            if (common(m, mid) >= A.k0)
                in = mid;
            else
                end = mid;
        }
        for (int k = A.k0; k <= A.k1; ++k) {
            if (A.crit == DZS_CRIT_GEOMETRIC && A.T2[k] > A.T2_max)
                continue;
            const int sh = 3 * (DZS_KEY_BITS - k);
            bool live = false;   // a large cube of this level that is in no group
            for (uint32_t b = m; b < end; b += DZ_LARGE) {
                __syncthreads();   // the stamps and the queue of the cubes before
                if (tid == 0)
                    s_cnt = 0u;
                __syncthreads();
                const uint32_t j = b + tid;
                if (j + 1 < end && common(j, j + 1) >= k &&
                    A.head[(uint64_t)j * DZ_MARK] == DZ_NONE) {
                    live = true;
                    if ((j == m || common(j - 1, j) < k) &&
                        !dz_near(A, k, dz_far2(A, k, mark(j) >> sh)))
                        s_work[atomicAdd(&s_cnt, 1u)] = j;
                }
                __syncthreads();
                const uint32_t cnt = s_cnt;
                for (uint32_t c = tid >> 3; c < cnt; c += DZ_LARGE / 8) {
                    const uint32_t q = s_work[c];
                    // the first member: after the mark before (outside), at most this one
                    const uint64_t pk = mark(q) >> sh;
                    int64_t out = q ? (int64_t)(q - 1) * DZ_MARK : -1, i = (int64_t)q * DZ_MARK;
                    while (i - out > 1) {
                        const int64_t mid = out + (i - out) / 2;
                        if ((A.key[mid] >> sh) == pk)
                            i = mid;
                        else
                            out = mid;
                    }
                    dz_cube<false>(A, k, (uint64_t)i, nullptr, 0, 0, &s_groups);
                }
            }
            if (!__syncthreads_or(live ? 1 : 0))
                break;
        }
    }
    __syncthreads();
    if (tid == 0 && s_groups)
        atomicAdd(&A.stat[(blockIdx.x % DZ_STATS) * 16u], s_groups);
}

// Levels k0 .. k1 (k1 > k0: without the large cubes of k_dz_large, which ran before).  A workgroup
// owns the cubes that begin in its tile of DZ_TILE particles, each from the first level on, k0 or
// deeper, at which it is not large, to the end of the last (less than two marks, so less than 1024
// particles, past the tile), and with them every cube of the deeper levels inside: the levels
// follow each other without another launch.  At each level
// the first members of cubes of two or more are queued in LDS and worked on densely, 8 lanes a
// cube; the levels end with the deepest that two neighbouring keys share.
//
// Bound by latency: finding the cubes, their distances, the rows and the sums (in the members'
// order) follow each other, and 14 waves a CU hide a third of it.  Small workgroups, so that
// many are at different places: 256 particles by 128 threads 67 us on 884736 particles (27 a
// cube at k_min) and 150 us on 128^3, 512 by 256 79 and 172, 1024 by 256 85 and 185; rows from
// memory instead of LDS 75 and 163.  One thread a cube, every lane between two first members
// idle, and a launch a level took 282 us (17 levels) and 700 us (21).
__global__ __launch_bounds__(DZ_LT, 4) void k_dz_levels(dz_level_args A) {
    __shared__ dz_window W;
    __shared__ uint16_t s_queue[DZ_TILE], s_work[DZ_TILE / 2];
    __shared__ uint8_t s_own[DZ_TILE];
    __shared__ uint32_t s_cnt, s_n, s_groups, s_first, s_last, s_live;
    __shared__ int s_deep, s_top;
    __shared__ unsigned long long s_far;
    const uint32_t tid = threadIdx.x;
    const uint64_t t0 = (uint64_t)blockIdx.x * DZ_TILE;
    const uint64_t t1 = t0 + DZ_TILE < A.n ? t0 + DZ_TILE : A.n;
    const uint32_t wlen = (uint32_t)(A.n - t0 < DZ_WINDOW ? A.n - t0 : DZ_WINDOW);
    const bool multi = A.k1 > A.k0;
    static_assert(DZ_MARK % DZ_TILE == 0, "no mark inside a tile but its first particle");
    // digits shared by the mark at or before the tile and the next, the one before, and of the
    // next two: a particle's cube of level k is large where k digits are shared by one of these
    // pairs and by the particle
    int big0 = -1, big1 = -1, big2 = -1;
    uint64_t mark0 = 0, mark1 = 0;
    if (multi) {
        const uint64_t q = t0 / DZ_MARK * DZ_MARK;
        mark0 = A.key[q];
        if (q)
            big0 = dz_common(A.key[q - DZ_MARK], mark0);
        if (q + DZ_MARK < A.n) {
            mark1 = A.key[q + DZ_MARK];
            big1 = dz_common(mark0, mark1);
            if (q + 2 * DZ_MARK < A.n)
                big2 = dz_common(mark1, A.key[q + 2 * DZ_MARK]);
        }
    }
    const bool large = multi && max(big0, max(big1, big2)) >= A.k0;
    if (tid == 0) {
        s_groups = 0u;
        s_first = s_last = 0xffffffffu;
        s_deep = 0;
        s_top = A.k0;
        s_far = 0ull;
    }
    for (uint32_t o = tid; o < wlen + 2; o += DZ_LT)
        if (t0 + o >= 1 && t0 + o - 1 < A.n)
            W.key[o] = A.key[t0 + o - 1];
    for (uint32_t o = tid; o < wlen; o += DZ_LT)
        W.done[o] = A.fresh && !large ? 0u : A.head[t0 + o] != DZ_NONE;
    __syncthreads();
    const auto key = [&](uint64_t i) { return dz_key(A, W, t0, i); };
    // first level of the tile's particle o (DZS_KEY_BITS + 1: none, its cubes are all large)
    const auto own = [&](uint32_t o) -> int {
        if (!large)
            return A.k0;
        const uint64_t ki = W.key[o + 1];
        return max(A.k0, 1 + max(big1, max(min(big0, dz_common(mark0, ki)),
                                           min(big2, dz_common(mark1, ki)))));
    };
    uint64_t s0 = t0, s1 = t1;
    int last_own = A.k0;
    if (multi) {
        // from the first cube that begins in the tile to the first that begins after it
        if (large && tid == 0)
            s_top = DZS_KEY_BITS + 1;
        if (large)
            __syncthreads();
        for (uint32_t o = tid; o < (uint32_t)(t1 - t0); o += DZ_LT) {
            const int ow = own(o);
            if (large)
                s_own[o] = (uint8_t)ow;
            if (ow <= DZS_KEY_BITS && (t0 + o == 0 || dz_common(W.key[o], W.key[o + 1]) < ow)) {
                atomicMin(&s_first, o);
                if (!large)
                    break;
                atomicMin(&s_top, ow);
            }
        }
        __syncthreads();
        if (s_first == 0xffffffffu)
            return;
        s0 = t0 + s_first;
        last_own = own((uint32_t)(t1 - t0) - 1u);
        const int shl = 3 * (DZS_KEY_BITS - last_own);
        while (last_own <= DZS_KEY_BITS && s1 < A.n) {
            const uint64_t last = key(t1 - 1) >> shl;
            const uint64_t i = s1 + tid;
            if (i >= A.n || (key(i) >> shl) != last)
                atomicMin(&s_last, tid);
            __syncthreads();
            const uint32_t f = s_last;
            __syncthreads();   // read by all before the next round writes it
            s1 += f == 0xffffffffu ? DZ_LT : f;
            if (f != 0xffffffffu)
                break;
        }
    }
    // first level of particle i of the range (those past the tile are in the last cube)
    const auto own_at = [&](uint64_t i) -> int {
        return !large ? A.k0 : (i < t1 ? (int)s_own[i - t0] : last_own);
    };
    // the deepest level that two neighbours of the range share, and the largest distance of the
    // owned cubes (every cube of a deeper level lies in one of them): levels at which that is
    // too close to merge are skipped, all of them inside the lightcone
    int deep = 0;
    for (uint64_t b0 = s0; b0 < s1; b0 += DZ_TILE) {
        if (tid == 0)
            s_cnt = 0u;
        __syncthreads();
        const uint32_t len = (uint32_t)(s1 - b0 < DZ_TILE ? s1 - b0 : DZ_TILE);
        for (uint32_t o = tid; o < len; o += DZ_LT) {
            const uint64_t i = b0 + o, ki = key(i);
            if (i + 1 < A.n)
                deep = max(deep, dz_common(ki, key(i + 1)));
            const int ow = own_at(i);
            if (i < t1 && ow <= DZS_KEY_BITS && (i == 0 || dz_common(key(i - 1), ki) < ow))
                s_queue[atomicAdd(&s_cnt, 1u)] = (uint16_t)o;
        }
        __syncthreads();
        const uint32_t cnt = s_cnt;
        double far2 = 0.0;
        for (uint32_t c = tid; c < cnt; c += DZ_LT) {
            const uint64_t i = b0 + s_queue[c];
            const int ow = own_at(i);
            far2 = fmax(far2, dz_far2(A, ow, key(i) >> (3 * (DZS_KEY_BITS - ow))));
        }
        if (far2 > 0.0)
            atomicMax(&s_far, (unsigned long long)__double_as_longlong(far2));
        __syncthreads();
    }
    if (deep)
        atomicMax(&s_deep, deep);
    __syncthreads();
    const int k1 = min(A.k1, s_deep);
    const double range_far2 = __longlong_as_double((long long)s_far) * (1.0 + 1e-9);
    const auto skipped = [&](int k) {
        return (A.crit == DZS_CRIT_GEOMETRIC && A.T2[k] > A.T2_max) || dz_near(A, k, range_far2);
    };
    int k = s_top;
    while (k <= k1 && skipped(k))
        ++k;
    if (k > k1)
        return;   // no two particles share a cube that could merge
    for (uint32_t o = tid; o < wlen; o += DZ_LT) {
#pragma unroll
        for (int f = 0; f < 6; ++f)
            W.f[f][o] = A.f[f][t0 + o];
        W.mult[o] = A.mult[t0 + o];
        W.id[o] = A.id[t0 + o];
    }
    for (; k <= k1; ++k) {
        if (skipped(k))
            continue;
        const int sh = 3 * (DZS_KEY_BITS - k);
        if (tid == 0)
            s_live = 0u;
        bool live = false;   // a particle was in no group before this level
        for (uint64_t b0 = s0; b0 < s1; b0 += DZ_TILE) {
            const uint32_t len = (uint32_t)(s1 - b0 < DZ_TILE ? s1 - b0 : DZ_TILE);
            __syncthreads();   // the stamps and the queue of the cubes before
            if (tid == 0)
                s_cnt = s_n = 0u;
            __syncthreads();
            for (uint32_t o = tid; o < len; o += DZ_LT) {
                const uint64_t i = b0 + o;
                if (i - t0 < wlen ? W.done[i - t0] != 0u : A.head[i] != DZ_NONE)
                    continue;
                const int ow = own_at(i);
                if (ow > DZS_KEY_BITS)
                    continue;
                live = true;
                if (i + 1 >= A.n || k < ow)
                    continue;
                const uint64_t pk = key(i) >> sh;
                if ((key(i + 1) >> sh) == pk && (i == 0 || (key(i - 1) >> sh) != pk))
                    s_queue[atomicAdd(&s_cnt, 1u)] = (uint16_t)o;
            }
            __syncthreads();
            const uint32_t cnt = s_cnt;
            for (uint32_t c = tid; c < cnt; c += DZ_LT)
                if (!dz_near(A, k, dz_far2(A, k, key(b0 + s_queue[c]) >> sh)))
                    s_work[atomicAdd(&s_n, 1u)] = s_queue[c];
            __syncthreads();
            const uint32_t work = s_n;
            for (uint32_t c = tid >> 3; c < work; c += DZ_LT / 8)
                dz_cube<true>(A, k, b0 + s_work[c], &W, t0, wlen, &s_groups);
        }
        if (live)
            s_live = 1u;
        __syncthreads();
        if (s_live == 0u)
            break;
        __syncthreads();   // read before the next level clears it
    }
    __syncthreads();
    if (tid == 0 && s_groups)
        atomicAdd(&A.stat[(blockIdx.x % DZ_STATS) * 16u], s_groups);
}

// The smallest g.g among particles strictly inside R_lc + b of the observer (minimum image);
// its bit pattern orders like the value because g.g >= 0, so blocks combine by an integer
// atomic minimum on a slot preset to +inf.
__global__ __launch_bounds__(1) void k_dz_amin_init(unsigned long long *out) {
    *out = 0x7ff0000000000000ull;
}

__global__ __launch_bounds__(DZ_THREADS) void k_dz_amin(uint64_t n, const double *__restrict__ x,
                                                       const double *__restrict__ y,
                                                       const double *__restrict__ z,
                                                       const double *__restrict__ gx,
                                                       const double *__restrict__ gy,
                                                       const double *__restrict__ gz, double L,
                                                       double xo0, double xo1, double xo2,
                                                       double Rb,
                                                       const uint32_t *__restrict__ perm,
                                                       unsigned long long *out) {
    __shared__ double red[DZ_THREADS];
    double best = __builtin_inf();
    const uint64_t stride = (uint64_t)gridDim.x * DZ_THREADS;
    for (uint64_t i = (uint64_t)blockIdx.x * DZ_THREADS + threadIdx.x; i < n; i += stride) {
        const double dx = dzs_min_image(x[i] - xo0, L);
        const double dy = dzs_min_image(y[i] - xo1, L);
        const double dz = dzs_min_image(z[i] - xo2, L);
        if (!(sqrt(dx * dx + dy * dy + dz * dz) < Rb))
            continue;
        const uint64_t j = perm ? perm[i] : i;
        const double g2 = gx[j] * gx[j] + gy[j] * gy[j] + gz[j] * gz[j];
        best = g2 < best ? g2 : best;
    }
    red[threadIdx.x] = best;
    __syncthreads();
    for (int h = DZ_THREADS / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            const double o = red[threadIdx.x + h];
            red[threadIdx.x] = o < red[threadIdx.x] ? o : red[threadIdx.x];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        atomicMin(out, (unsigned long long)__double_as_longlong(red[0]));
}

dzs_status dzs_coarsen_amin(dzs_ctx *ctx, const dzs_box *box, const dzs_particles *p,
                            const dzs_coarsen_params *prm, hipStream_t s,
                            const uint32_t *perm) {
    unsigned long long *slot = (unsigned long long *)(ctx->d_small + DZS_SMALL_AMIN);
    hipLaunchKernelGGL(k_dz_amin_init, dim3(1), dim3(1), 0, s, slot);
    DZS_TRY(dzs_check_launch(ctx, "dz_amin_init"));
    if (p->n == 0)
        return DZS_OK;
    const uint64_t want = (p->n + DZ_THREADS - 1) / DZ_THREADS;
    const uint32_t blocks = (uint32_t)(want < 2048 ? want : 2048);
    hipLaunchKernelGGL(k_dz_amin, dim3(blocks), dim3(DZ_THREADS), 0, s, p->n,
                       (const double *)p->x, (const double *)p->y, (const double *)p->z,
                       (const double *)p->gx, (const double *)p->gy, (const double *)p->gz,
                       box->L, prm->x_obs[0], prm->x_obs[1], prm->x_obs[2], prm->R_lc + prm->b,
                       perm, slot);
    return dzs_check_launch(ctx, "dz_amin");
}

// After a merge the state stays in key order (a merged particle takes its cube's first slot
// and its centre of mass lies in that cube), unless rounding put a centre of mass on the
// cube's far face: flag any descent.
__global__ __launch_bounds__(1) void k_dz_flag_clear(uint32_t *flag) { *flag = 0u; }

__global__ __launch_bounds__(DZ_THREADS) void k_dz_unsorted(uint64_t n, const uint64_t *key,
                                                           uint32_t *flag) {
    const uint64_t i = (uint64_t)blockIdx.x * DZ_THREADS + threadIdx.x;
    if (i + 1 < n && key[i] > key[i + 1])
        atomicOr(flag, 1u);
}

dzs_status dzs_coarsen_rekey(dzs_ctx *ctx, const dzs_box *box, const dzs_particles *p,
                             bool *sorted, hipStream_t s) {
    *sorted = true;
    if (p->n < 2)
        return dzs_launch_keys(ctx, p->x, p->y, p->z, p->n, box->L, ctx->key, nullptr, s);
    DZS_TRY(dzs_launch_keys(ctx, p->x, p->y, p->z, p->n, box->L, ctx->key, nullptr, s));
    uint32_t *flag = ctx->d_small + DZS_SMALL_UNSORTED;
    hipLaunchKernelGGL(k_dz_flag_clear, dim3(1), dim3(1), 0, s, flag);
    DZS_TRY(dzs_check_launch(ctx, "dz_flag_clear"));
    hipLaunchKernelGGL(k_dz_unsorted, dim3(blocks_for(p->n, DZ_THREADS)), dim3(DZ_THREADS), 0, s,
                       p->n, (const uint64_t *)ctx->key, flag);
    DZS_TRY(dzs_check_launch(ctx, "dz_unsorted"));
    DZS_HIP(ctx, hipMemcpyAsync(ctx->h_small + DZS_SMALL_UNSORTED, flag, sizeof(uint32_t),
                                hipMemcpyDeviceToHost, s));
    DZS_HIP(ctx, hipStreamSynchronize(s));
    *sorted = ctx->h_small[DZS_SMALL_UNSORTED] == 0u;
    return DZS_OK;
}

__global__ __launch_bounds__(DZ_THREADS) void k_dz_init(uint64_t n, uint32_t *head, uint8_t *keep,
                                                        uint32_t *stat) {
    const uint64_t i = (uint64_t)blockIdx.x * DZ_THREADS + threadIdx.x;
    if (i < n) {
        head[i] = DZ_NONE;
        keep[i] = 1u;
    }
    if (i < DZ_STATS)
        stat[i * 16u] = 0u;
}

// The place after the compaction of each kept row, then of every entry particle's group.
__global__ __launch_bounds__(DZ_THREADS) void k_dz_rank(const uint32_t *__restrict__ n_new,
                                                        const uint32_t *__restrict__ list,
                                                        uint32_t *__restrict__ rank) {
    const uint64_t j = (uint64_t)blockIdx.x * DZ_THREADS + threadIdx.x;
    if (j < *n_new)
        rank[list[j]] = (uint32_t)j;
}

__global__ __launch_bounds__(DZ_THREADS) void k_dz_groupmap(uint64_t n, const uint32_t *head,
                                                            const uint32_t *rank,
                                                            const uint32_t *perm,
                                                            uint32_t *group_of) {
    const uint64_t i = (uint64_t)blockIdx.x * DZ_THREADS + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t h = head[i];
    group_of[perm[i]] = rank[h == DZ_NONE ? (uint32_t)i : h];
}

// State already sorted by (key, id) with ctx->key holding the sorted keys and ctx->idx the
// entry index of each sorted slot.
dzs_status dzs_coarsen_sorted(dzs_ctx *ctx, const dzs_box *box, dzs_particles *p,
                              const dzs_coarsen_params *prm, uint32_t *group_of,
                              dzs_coarsen_report *report, hipStream_t s) {
    const uint64_t n = p->n;
    const bool dyn = prm->criterion == DZS_CRIT_DYNAMICAL;
    if (report) {
        report->n_before = n;
        report->n_after = n;
        report->n_groups = 0;
        report->a_min = dyn ? __builtin_inf() : __builtin_nan("");
    }
    if (n == 0)
        return DZS_OK;
    dz_level_args A;
    dzs_merge_thresholds(box->L, prm->R_lc, prm->b, dyn ? 1.0 : prm->theta, A.T2);
    // geometric: no centre of mass lies beyond sqrt(3)/2 L (minimum image), so a level whose
    // threshold exceeds it cannot merge anything
    A.T2_max = 0.75 * box->L * box->L * (1.0 + 1e-9);
    A.n = n;
    A.L = box->L;
    A.iL = 1.0 / box->L;
    A.crit = dyn ? DZS_CRIT_DYNAMICAL : DZS_CRIT_GEOMETRIC;
    A.Gm0 = box->G * box->m0;
    A.Rb = prm->R_lc + prm->b;
    A.alpha = prm->alpha_dyn;
    A.amin2 = (const unsigned long long *)(ctx->d_small + DZS_SMALL_AMIN);
    for (int d = 0; d < 3; ++d)
        A.xo[d] = prm->x_obs[d];
    A.key = ctx->key;
    double *const f[6] = {p->x, p->y, p->z, p->px, p->py, p->pz};
    for (int k = 0; k < 6; ++k)
        A.f[k] = f[k];
    A.mult = p->mult;
    A.id = p->id;
    A.type = p->type;
    A.head = ctx->dz_head;
    A.keep = ctx->dz_keep;
    A.stat = ctx->dz_stat;
    uint32_t *total = ctx->dz_stat + 16 * DZ_STATS;
    const uint32_t blocks = blocks_for(n, DZ_THREADS);
    {
        dzs_timed t(ctx, KC_DZS_LEVELS, s);
        hipLaunchKernelGGL(k_dz_init, dim3(blocks), dim3(DZ_THREADS), 0, s, n, ctx->dz_head,
                           ctx->dz_keep, ctx->dz_stat);
        DZS_TRY(dzs_check_launch(ctx, "dz_init"));
        // The levels whose cubes hold more than DZ_ONE particles on average take a launch each
        // (a workgroup that owned such a cube would work on everything in it alone); all deeper
        // ones share one.
        for (int k = prm->k_min; k <= DZS_KEY_BITS;) {
            A.k0 = k;
            A.k1 = (n >> (3 * k)) > DZ_ONE ? k : DZS_KEY_BITS;
            A.fresh = k == prm->k_min;
            k = A.k1 + 1;
            if (!dyn && A.k0 == A.k1 && A.T2[A.k0] > A.T2_max)
                continue;
            if (A.k1 > A.k0 && n > DZ_MARK) {
                hipLaunchKernelGGL(k_dz_large, dim3(blocks_for(n, DZ_MARK * DZ_MARKS)),
                                   dim3(DZ_LARGE), 0, s, A);
                DZS_TRY(dzs_check_launch(ctx, "dz_large"));
            }
            hipLaunchKernelGGL(k_dz_levels, dim3(blocks_for(n, DZ_TILE)), dim3(DZ_LT), 0, s, A);
            DZS_TRY(dzs_check_launch(ctx, "dz_levels"));
        }
    }
    uint64_t n_new, n_heads = 0;
    {
        dzs_timed t(ctx, KC_DZS_COMPACT, s);
        DZS_TRY(dzs_flag_list(ctx, n, ctx->dz_keep, ctx->dz_cnt, ctx->dz_scan, total, ctx->dz_list,
                              s));
        if (group_of) {
            // (the counters' copy below waits for these as well)
            hipLaunchKernelGGL(k_dz_rank, dim3(blocks), dim3(DZ_THREADS), 0, s,
                               (const uint32_t *)total, (const uint32_t *)ctx->dz_list,
                               ctx->dz_rank);
            DZS_TRY(dzs_check_launch(ctx, "dz_rank"));
            hipLaunchKernelGGL(k_dz_groupmap, dim3(blocks), dim3(DZ_THREADS), 0, s, n,
                               (const uint32_t *)ctx->dz_head, (const uint32_t *)ctx->dz_rank,
                               (const uint32_t *)ctx->idx, group_of);
            DZS_TRY(dzs_check_launch(ctx, "dz_groupmap"));
        }
        uint32_t *h = ctx->h_small + 64;
        DZS_HIP(ctx, hipMemcpyAsync(h, ctx->dz_stat, DZS_STAT_WORDS * sizeof(uint32_t),
                                    hipMemcpyDeviceToHost, s));
        if (dyn)
            DZS_HIP(ctx, hipMemcpyAsync(ctx->h_small + DZS_SMALL_AMIN,
                                        ctx->d_small + DZS_SMALL_AMIN, 2 * sizeof(uint32_t),
                                        hipMemcpyDeviceToHost, s));
        DZS_HIP(ctx, hipStreamSynchronize(s));
        n_new = h[16 * DZ_STATS];
        for (int k = 0; k < DZ_STATS; ++k)
            n_heads += h[16 * k];
        if (dyn && report) {
            unsigned long long bits;
            memcpy(&bits, ctx->h_small + DZS_SMALL_AMIN, sizeof(bits));
            double g2;
            memcpy(&g2, &bits, sizeof(g2));
            report->a_min = sqrt(g2);
        }
    }
    p->n = n_new;
    if (n_new != n)
        DZS_TRY(dzs_permute_state(ctx, p, ctx->dz_list, 0, s));
    if (report) {
        report->n_after = n_new;
        report->n_groups = n_heads;
    }
    return DZS_OK;
}
