// Exclusive prefix scan (u32) and stable LSD radix sort of (u64 Morton key, u32 index)
// pairs for gfx950.
//
// Sort: 8 passes of 8-bit digits (the sort before a tree build skips the lowest two: the tree
// reads the keys' order to level 15 only).  Per pass: (1) each workgroup counts the digits of its
// 4096-key tile in LDS into a row of a table [tile][256]; (2) the table's columns are scanned,
// in segments of tiles, so that a row holds the keys of each digit in the tiles before it, and
// the columns' totals kept; (3) each workgroup ranks its tile stably — each wave its own part
// by wave-level digit matching through eight ballots, then the waves' counts become offsets —
// stages the tile in LDS in local digit order and writes it out so that consecutive lanes write
// consecutive addresses of the same digit run.  Three launches of a pass up to 64 tiles, four
// above.  At most 32768 keys: each key's place is counted against all others, in two launches.
#include "internal.h"

#define SCAN_THREADS 256
#define SCAN_ITEMS 16
#define SCAN_TILE (SCAN_THREADS * SCAN_ITEMS)

#define SORT_THREADS 512
#define SORT_ITEMS 8
#define SORT_TILE (SORT_THREADS * SORT_ITEMS)
#define SORT_SEG 64        // tiles of a column segment (more above 512 segments)
#define SORT_SMALL 32768   // keys whose places are counted

// ---------------------------------------------------------------------------------------
// block-wide exclusive scan of one value per thread (256 threads = 4 wave64)
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t block_excl_scan_256(uint32_t v, uint32_t *s_wave,
                                                       uint32_t *total) {
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t incl = dzs_wave_incl_scan(v);
    if (lane == 63)
        s_wave[wave] = incl;
    __syncthreads();
    uint32_t off = 0;
    for (uint32_t w = 0; w < wave; ++w)
        off += s_wave[w];
    uint32_t tot = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    __syncthreads();
    if (total)
        *total = tot;
    return off + incl - v;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_reduce(const uint32_t *__restrict__ in,
                                                              uint64_t n,
                                                              uint32_t *__restrict__ part) {
    __shared__ uint32_t s_wave[4];
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_TILE;
    uint32_t sum = 0;
    for (int r = 0; r < SCAN_ITEMS; ++r) {
        uint64_t e = base + (uint64_t)r * SCAN_THREADS + threadIdx.x;
        if (e < n)
            sum += in[e];
    }
    uint32_t tot;
    block_excl_scan_256(sum, s_wave, &tot);
    if (threadIdx.x == 0)
        part[blockIdx.x] = tot;
}

// Offset of tile b from the unscanned tile sums part[0..b) (b <= SCAN_TILE), summed by the
// block; every thread returns it.
__device__ __forceinline__ uint32_t tile_offset(const uint32_t *__restrict__ part, uint32_t b,
                                                uint32_t *s_wave) {
    uint32_t sum = 0;
    for (uint32_t i = threadIdx.x; i < b; i += SCAN_THREADS)
        sum += part[i];
    uint32_t tot;
    block_excl_scan_256(sum, s_wave, &tot);
    return tot;
}

// scan one tile (blocked: thread t owns items t*16 .. t*16+15), adding the tile offset: the
// scanned tile sums offs[b], or the unscanned tile sums part[0..b) (two-launch scan), or 0
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_tile(const uint32_t *__restrict__ in,
                                                            uint32_t *__restrict__ out,
                                                            uint64_t n,
                                                            const uint32_t *__restrict__ offs,
                                                            const uint32_t *__restrict__ part,
                                                            uint32_t *__restrict__ total) {
    __shared__ uint32_t s_wave[4];
    const uint64_t base = (uint64_t)blockIdx.x * SCAN_TILE + (uint64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS];
    uint32_t sum = 0;
#pragma unroll
    for (int r = 0; r < SCAN_ITEMS; ++r) {
        uint64_t e = base + r;
        v[r] = e < n ? in[e] : 0u;
        sum += v[r];
    }
    uint32_t tot;
    uint32_t run = block_excl_scan_256(sum, s_wave, &tot);
    if (offs)
        run += offs[blockIdx.x];
    else if (part)
        run += tile_offset(part, blockIdx.x, s_wave);
#pragma unroll
    for (int r = 0; r < SCAN_ITEMS; ++r) {
        uint64_t e = base + r;
        if (e < n)
            out[e] = run;
        run += v[r];
    }
    if (total && threadIdx.x == SCAN_THREADS - 1 && blockIdx.x == gridDim.x - 1)
        *total = run;
}

uint64_t dzs_scan_tmp_words(uint64_t n) {
    uint64_t words = 0;
    while (n > SCAN_TILE) {
        uint64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
        words += 2 * nb;
        n = nb;
    }
    return words + 64;
}

// One tile: one launch.  Up to SCAN_TILE tiles: tile sums, then the tiles, each adding the
// sum of the tile sums before it (two launches).  More: the tile sums are scanned recursively.
static dzs_status scan_rec(dzs_ctx *ctx, const uint32_t *in, uint32_t *out, uint64_t n,
                           uint32_t *total_dev, uint32_t *tmp, hipStream_t s) {
    uint64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (nb <= 1) {
        hipLaunchKernelGGL(k_scan_tile, dim3(1), dim3(SCAN_THREADS), 0, s, in, out, n,
                           (const uint32_t *)nullptr, (const uint32_t *)nullptr, total_dev);
        return dzs_check_launch(ctx, "scan_tile");
    }
    uint32_t *part = tmp, *part_scan = tmp + nb;
    hipLaunchKernelGGL(k_scan_reduce, dim3((uint32_t)nb), dim3(SCAN_THREADS), 0, s, in, n, part);
    DZS_TRY(dzs_check_launch(ctx, "scan_reduce"));
    if (nb <= SCAN_TILE) {
        hipLaunchKernelGGL(k_scan_tile, dim3((uint32_t)nb), dim3(SCAN_THREADS), 0, s, in, out, n,
                           (const uint32_t *)nullptr, (const uint32_t *)part, total_dev);
        return dzs_check_launch(ctx, "scan_tile");
    }
    DZS_TRY(scan_rec(ctx, part, part_scan, nb, nullptr, tmp + 2 * nb, s));
    hipLaunchKernelGGL(k_scan_tile, dim3((uint32_t)nb), dim3(SCAN_THREADS), 0, s, in, out, n,
                       (const uint32_t *)part_scan, (const uint32_t *)nullptr, total_dev);
    return dzs_check_launch(ctx, "scan_tile");
}

dzs_status dzs_scan_u32(dzs_ctx *ctx, const uint32_t *in, uint32_t *out, uint64_t n,
                        uint32_t *total_dev, hipStream_t s) {
    if (n == 0) {
        if (total_dev)
            DZS_HIP(ctx, hipMemsetAsync(total_dev, 0, sizeof(uint32_t), s));
        return DZS_OK;
    }
    if (dzs_scan_tmp_words(n) > ctx->scan_tmp_cap)
        return dzs_fail(ctx, DZS_ECAPACITY, "scan of %llu elements exceeds scratch",
                        (unsigned long long)n);
    return scan_rec(ctx, in, out, n, total_dev, ctx->scan_tmp, s);
}

// ---------------------------------------------------------------------------------------
// radix sort
// ---------------------------------------------------------------------------------------
uint64_t dzs_sort_hist_words(uint64_t n) {
    uint64_t tiles = (n + SORT_TILE - 1) / SORT_TILE;
    if (tiles < 2)
        tiles = 2;
    return 256 * tiles;
}

// The tile's digit counts, row [tile][256].  HBM-bound (8 bytes read per key).
__global__ __launch_bounds__(SORT_THREADS) void k_radix_hist(const uint64_t *__restrict__ key,
                                                             uint64_t n, int shift,
                                                             uint32_t *__restrict__ tab,
                                                             const uint32_t *skip) {
    if (skip && *skip)
        return;
    __shared__ uint32_t s_h[256];
    if (threadIdx.x < 256)
        s_h[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * SORT_TILE;
    uint64_t k[SORT_ITEMS];
#pragma unroll
    for (int r = 0; r < SORT_ITEMS; ++r) {
        const uint64_t e = base + (uint64_t)r * SORT_THREADS + threadIdx.x;
        k[r] = e < n ? key[e] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < SORT_ITEMS; ++r) {
        const uint64_t e = base + (uint64_t)r * SORT_THREADS + threadIdx.x;
        const uint32_t d = (uint32_t)(k[r] >> shift) & 255u;
        // keys of one digit throughout the wave (the upper digits of nearly sorted keys): one add
        const uint64_t in = __ballot(e < n);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
        if (__ballot(e < n && d != d0) == 0ull) {
            if ((threadIdx.x & 63u) == 0u)
                atomicAdd(&s_h[d0], (uint32_t)__popcll(in));
        } else if (e < n) {
            atomicAdd(&s_h[d], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < 256)
        tab[(uint64_t)blockIdx.x * 256u + threadIdx.x] = s_h[threadIdx.x];
}

// Column sums of each segment of `seg` rows, then (k_col_scan) the rows of each segment to the
// sums of the rows before them, the last segment also writing the columns' totals.  A thread
// owns a column; rows are read eight at a time.
__global__ __launch_bounds__(256) void k_col_sum(const uint32_t *__restrict__ tab, uint32_t tiles,
                                                 uint32_t seg, uint32_t *__restrict__ segsum,
                                                 const uint32_t *skip) {
    if (skip && *skip)
        return;
    const uint32_t t0 = blockIdx.x * seg, t1 = min(t0 + seg, tiles);
    uint32_t sum = 0;
#pragma unroll 8
    for (uint32_t t = t0; t < t1; ++t)
        sum += tab[(uint64_t)t * 256u + threadIdx.x];
    segsum[(uint64_t)blockIdx.x * 256u + threadIdx.x] = sum;
}

__global__ __launch_bounds__(256) void k_col_scan(uint32_t *__restrict__ tab, uint32_t tiles,
                                                  uint32_t seg,
                                                  const uint32_t *__restrict__ segsum,
                                                  uint32_t *__restrict__ totals,
                                                  const uint32_t *skip) {
    if (skip && *skip)
        return;
    const uint32_t t0 = blockIdx.x * seg, t1 = min(t0 + seg, tiles);
    uint32_t run = 0;
#pragma unroll 8
    for (uint32_t q = 0; q < blockIdx.x; ++q)
        run += segsum[(uint64_t)q * 256u + threadIdx.x];
    uint32_t t = t0;
    for (; t + 8u <= t1; t += 8u) {
        uint32_t v[8];
#pragma unroll
        for (uint32_t r = 0; r < 8u; ++r)
            v[r] = tab[(uint64_t)(t + r) * 256u + threadIdx.x];
#pragma unroll
        for (uint32_t r = 0; r < 8u; ++r) {
            tab[(uint64_t)(t + r) * 256u + threadIdx.x] = run;
            run += v[r];
        }
    }
    for (; t < t1; ++t) {
        const uint32_t v = tab[(uint64_t)t * 256u + threadIdx.x];
        tab[(uint64_t)t * 256u + threadIdx.x] = run;
        run += v;
    }
    if (blockIdx.x == gridDim.x - 1)
        totals[threadIdx.x] = run;
}

// Stable rank of one wave's key among the wave's keys of its digit so far (running counts in
// LDS, no block barrier): lanes holding the same digit are found with eight ballots, the lowest
// of them advances the wave's count.
__device__ __forceinline__ uint32_t wave_rank(uint32_t d, bool valid, uint64_t lt_mask,
                                              uint32_t *wcnt) {
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
        const uint64_t bal = __ballot(((d >> bit) & 1u) != 0u);
        m &= ((d >> bit) & 1u) ? bal : ~bal;
    }
    const uint32_t rank = (uint32_t)__popcll(m & lt_mask);
    // every lane reads the wave's count before the lowest lane of the digit advances it (LDS
    // operations of one wave complete in order)
    const uint32_t prev = wcnt[d];
    if (valid && rank == 0)
        wcnt[d] = prev + (uint32_t)__popcll(m);
    return prev + rank;
}

// exclusive scan of v over the first 256 threads of the workgroup (every thread calls it)
__device__ __forceinline__ uint32_t excl_scan_256(uint32_t v, uint32_t *s_wave) {
    const uint32_t tid = threadIdx.x;
    const uint32_t incl = dzs_wave_scan_add_full(tid < 256u ? v : 0u);
    if (tid < 256u && (tid & 63u) == 63u)
        s_wave[tid >> 6] = incl;
    __syncthreads();
    uint32_t off = 0;
    for (uint32_t w = 0; w < ((tid >> 6) & 3u); ++w)
        off += s_wave[w];
    __syncthreads();
    return off + incl - v;
}

// Each wave ranks its own contiguous part of the tile (rounds of 64 keys, in input order); the
// waves' counts become offsets (wave 0's keys of a digit first); equal digits keep their order.
// Bound by the LDS traffic of the ranks and the staging (two workgroups of eight waves a CU)
// and by HBM: 24 bytes per key and pass.  Neighbouring tiles write neighbouring parts of each
// digit's run, so an XCD takes tiles that follow each other: six passes of 1.7e7 keys 968 -> 742
// us (2e6 keys, which the caches hold, 193 either way).
__global__ __launch_bounds__(SORT_THREADS) void k_radix_scatter(
    const uint64_t *__restrict__ key_in, const uint32_t *__restrict__ idx_in,
    uint64_t *__restrict__ key_out, uint32_t *__restrict__ idx_out, uint64_t n, int shift,
    const uint32_t *__restrict__ tab, const uint32_t *__restrict__ totals, const uint32_t *skip) {
    if (skip && *skip)
        return;
    const uint32_t blk = dzs_xcd_block();
    constexpr int WAVES = SORT_THREADS / 64;
    constexpr int ROUNDS = SORT_ITEMS;  // rounds of 64 keys per wave
    __shared__ uint64_t s_key[SORT_TILE];
    __shared__ uint32_t s_idx[SORT_TILE];
    __shared__ uint32_t s_lstart[256], s_gstart[256];
    __shared__ uint32_t s_wcnt[WAVES][256];
    __shared__ uint32_t s_wave[4];

    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t base = (uint64_t)blk * SORT_TILE;
    const uint32_t cnt = (uint32_t)((n - base) < SORT_TILE ? (n - base) : SORT_TILE);
    const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const uint32_t q0 = wave * (ROUNDS * 64);

    uint64_t k[ROUNDS];
    uint32_t id[ROUNDS], pos[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t local = q0 + (uint32_t)r * 64u + lane;
        k[r] = local < cnt ? key_in[base + local] : 0ull;
        id[r] = local < cnt ? idx_in[base + local] : 0u;
    }
    // the tile's global start of each digit: the digits below it, and its keys in earlier tiles
    const uint32_t before = tid < 256u ? tab[(uint64_t)blk * 256u + tid] : 0u;
    const uint32_t total = tid < 256u ? totals[tid] : 0u;
    for (uint32_t e = tid; e < WAVES * 256u; e += SORT_THREADS)
        (&s_wcnt[0][0])[e] = 0u;
    const uint32_t digit0 = excl_scan_256(total, s_wave);
    if (tid < 256u)
        s_gstart[tid] = digit0 + before;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
        pos[r] = wave_rank((uint32_t)(k[r] >> shift) & 255u, q0 + (uint32_t)r * 64u + lane < cnt,
                           lt_mask, s_wcnt[wave]);
    __syncthreads();
    {
        // the tile's count of digit tid (the waves' counts), its start inside the tile, and
        // the offsets of each wave's run of it
        uint32_t c = 0;
        if (tid < 256u)
            for (int w = 0; w < WAVES; ++w)
                c += s_wcnt[w][tid];
        const uint32_t ls = excl_scan_256(c, s_wave);
        if (tid < 256u) {
            s_lstart[tid] = ls;
            uint32_t run = ls;
            for (int w = 0; w < WAVES; ++w) {
                const uint32_t t = s_wcnt[w][tid];
                s_wcnt[w][tid] = run;
                run += t;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t local = q0 + (uint32_t)r * 64u + lane;
        if (local < cnt) {
            const uint32_t d = (uint32_t)(k[r] >> shift) & 255u;
            const uint32_t lp = s_wcnt[wave][d] + pos[r];
            s_key[lp] = k[r];
            s_idx[lp] = id[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t i = (uint32_t)r * SORT_THREADS + tid;
        if (i < cnt) {
            const uint64_t kk = s_key[i];
            const uint32_t d = (uint32_t)(kk >> shift) & 255u;
            const uint64_t gp = (uint64_t)s_gstart[d] + (i - s_lstart[d]);
            key_out[gp] = kk;
            idx_out[gp] = s_idx[i];
        }
    }
}

// At most SORT_SMALL keys: the place of each is counted, against all others, over the whole GPU,
// and a second launch puts them there.  The passes of a radix sort are a chain of short launches
// at these sizes (one workgroup for all passes of 8000 keys took 47 us on one CU of 256, from
// 190 by launches); n^2 comparisons spread evenly.  Bound by latency, then by the comparisons:
// 4000 keys 16 us, 8000 19, 16384 33, 32768 87, where six passes take as long (40000: 103).
// Segments of 128 keys are as fast up to 16384 and slower above (116), of 512 slower below (27).
#define RANK_THREADS 256
#define RANK_SEG 256       // keys that a workgroup compares its RANK_THREADS keys with
__global__ __launch_bounds__(RANK_THREADS) void k_rank_count(const uint64_t *__restrict__ key,
                                                             const uint32_t *__restrict__ idx,
                                                             uint32_t n, int shift,
                                                             uint32_t *__restrict__ part,
                                                             uint64_t *__restrict__ key_in,
                                                             uint32_t *__restrict__ idx_in) {
    __shared__ __align__(16) uint64_t s_key[RANK_SEG];
    const uint32_t i = blockIdx.x * RANK_THREADS + threadIdx.x, j0 = blockIdx.y * RANK_SEG;
    const uint32_t cnt = min(n - j0, (uint32_t)RANK_SEG);
    // (keys that fill the segment up are above every other: counted nowhere)
    for (uint32_t j = threadIdx.x; j < RANK_SEG; j += RANK_THREADS)
        s_key[j] = j < cnt ? key[j0 + j] >> shift : ~0ull;
    uint64_t k = 0;
    if (i < n) {
        k = key[i];
        if (blockIdx.y == 0) {
            key_in[i] = k;
            idx_in[i] = idx[i];
        }
        k >>= shift;
    }
    __syncthreads();
    // equal keys keep their order: those of segments before the thread's block come first, those
    // of segments after it behind
    uint32_t rank = 0;
    const uint32_t b0 = blockIdx.x * RANK_THREADS;
    const auto count = [&](const auto &before) {
        for (uint32_t j = 0; j < RANK_SEG; j += 16) {
            ulonglong2 v[8];   // read together, then compared
#pragma unroll
            for (int q = 0; q < 8; ++q)
                v[q] = *(const ulonglong2 *)(s_key + j + 2 * q);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                rank += (uint32_t)before(v[q].x, j + 2 * q) + (uint32_t)before(v[q].y, j + 2 * q + 1);
        }
    };
    if (j0 + RANK_SEG <= b0)
        count([&](uint64_t v, uint32_t) { return v <= k; });
    else if (j0 >= b0 + RANK_THREADS)
        count([&](uint64_t v, uint32_t) { return v < k; });
    else
        count([&](uint64_t v, uint32_t j) { return v < k || (v == k && j0 + j < i); });
    if (i < n)
        part[blockIdx.y * n + i] = rank;
}

__global__ __launch_bounds__(RANK_THREADS) void k_rank_place(const uint64_t *__restrict__ key_in,
                                                             const uint32_t *__restrict__ idx_in,
                                                             uint32_t n, uint32_t segs,
                                                             const uint32_t *__restrict__ part,
                                                             uint64_t *__restrict__ key,
                                                             uint32_t *__restrict__ idx) {
    const uint32_t i = blockIdx.x * RANK_THREADS + threadIdx.x;
    if (i >= n)
        return;
    uint32_t rank = 0;
#pragma unroll 8
    for (uint32_t g = 0; g < segs; ++g)
        rank += part[g * n + i];
    key[rank] = key_in[i];
    idx[rank] = idx_in[i];
}

dzs_status dzs_radix_sort(dzs_ctx *ctx, uint64_t n, hipStream_t s, int first_pass,
                          const uint32_t *skip) {
    if (n <= 1)
        return DZS_OK;
    if (n > 0xffffffffull)
        return dzs_fail(ctx, DZS_EINVAL, "radix sort: n exceeds 2^32-1");
    if (first_pass < 0 || first_pass > 6 || (first_pass & 1))
        return dzs_fail(ctx, DZS_EINVAL, "radix sort: first pass %d", first_pass);
    dzs_timed t(ctx, KC_SORT, s);
    // By counting up to where that takes as long as the passes (see k_rank_count).  Above, 1.1e5
    // keys 265 -> 92 us, 2.1e6 371 -> 190, 1.7e7 1576 -> 742, against a
    // digit-major table scanned as one array and transposed, and four waves a workgroup.
    if (n <= SORT_SMALL && !skip) {
        // scratch: the walk's stacks, which hold nothing outside the walk
        const uint32_t segs = (uint32_t)((n + RANK_SEG - 1) / RANK_SEG);
        uint64_t *key_in = (uint64_t *)ctx->walk_stack;
        uint32_t *idx_in = (uint32_t *)(key_in + n), *part = idx_in + n;
        static_assert(SORT_SMALL * (3 + (SORT_SMALL + RANK_SEG - 1) / RANK_SEG) <= 4096 * 8192,
                      "the keys, their indices and the counts fit the walk's stacks");
        const dim3 blocks((uint32_t)((n + RANK_THREADS - 1) / RANK_THREADS));
        hipLaunchKernelGGL(k_rank_count, dim3(blocks.x, segs), dim3(RANK_THREADS), 0, s,
                           (const uint64_t *)ctx->key, (const uint32_t *)ctx->idx, (uint32_t)n,
                           8 * first_pass, part, key_in, idx_in);
        DZS_TRY(dzs_check_launch(ctx, "rank_count"));
        hipLaunchKernelGGL(k_rank_place, blocks, dim3(RANK_THREADS), 0, s,
                           (const uint64_t *)key_in, (const uint32_t *)idx_in, (uint32_t)n, segs,
                           (const uint32_t *)part, ctx->key, ctx->idx);
        return dzs_check_launch(ctx, "rank_place");
    }
    const uint32_t tiles = (uint32_t)((n + SORT_TILE - 1) / SORT_TILE);
    if (256ull * tiles > ctx->hist_cap)
        return dzs_fail(ctx, DZS_ECAPACITY, "radix sort histogram exceeds scratch");
    // at most 512 segments; the segment sums and the totals are in the second table
    const uint32_t seg = tiles <= 512u * SORT_SEG ? SORT_SEG : (tiles + 511u) / 512u;
    const uint32_t nseg = (tiles + seg - 1) / seg;
    uint32_t *tab = ctx->hist, *totals = ctx->hist_scan, *segsum = ctx->hist_scan + 256;
    uint64_t *kin = ctx->key, *kout = ctx->key_alt;
    uint32_t *iin = ctx->idx, *iout = ctx->idx_alt;
    for (int pass = first_pass; pass < 8; ++pass) {
        const int shift = 8 * pass;
        hipLaunchKernelGGL(k_radix_hist, dim3(tiles), dim3(SORT_THREADS), 0, s, kin, n, shift,
                           tab, skip);
        DZS_TRY(dzs_check_launch(ctx, "radix_hist"));
        if (nseg > 1) {
            hipLaunchKernelGGL(k_col_sum, dim3(nseg), dim3(256), 0, s, (const uint32_t *)tab,
                               tiles, seg, segsum, skip);
            DZS_TRY(dzs_check_launch(ctx, "col_sum"));
        }
        hipLaunchKernelGGL(k_col_scan, dim3(nseg), dim3(256), 0, s, tab, tiles, seg,
                           (const uint32_t *)segsum, totals, skip);
        DZS_TRY(dzs_check_launch(ctx, "col_scan"));
        hipLaunchKernelGGL(k_radix_scatter, dim3(tiles), dim3(SORT_THREADS), 0, s, kin, iin,
                           kout, iout, n, shift, (const uint32_t *)tab,
                           (const uint32_t *)totals, skip);
        DZS_TRY(dzs_check_launch(ctx, "radix_scatter"));
        uint64_t *tk = kin; kin = kout; kout = tk;
        uint32_t *ti = iin; iin = iout; iout = ti;
    }
    // an even number of passes: the result is back in ctx->key / ctx->idx
    return DZS_OK;
}

// Equal keys keep their input order (the sort is stable); where a canonical order is
// needed, runs of equal keys are re-ordered by ascending particle id (runs are short).
__global__ void k_fix_ties(const uint64_t *__restrict__ key, uint32_t *__restrict__ idx,
                           const uint32_t *__restrict__ id, uint64_t n) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i + 1 >= n)
        return;
    if (key[i] != key[i + 1] || (i > 0 && key[i - 1] == key[i]))
        return;
    uint64_t e = i + 1;
    while (e < n && key[e] == key[i])
        ++e;
    for (uint64_t a = i + 1; a < e; ++a) {
        uint32_t v = idx[a];
        uint32_t vid = id[v];
        uint64_t b = a;
        while (b > i && id[idx[b - 1]] > vid) {
            idx[b] = idx[b - 1];
            --b;
        }
        idx[b] = v;
    }
}

dzs_status dzs_fix_ties(dzs_ctx *ctx, uint64_t n, const uint32_t *id, hipStream_t s) {
    if (n <= 1)
        return DZS_OK;
    dzs_timed t(ctx, KC_SORT, s);
    uint32_t blocks = (uint32_t)((n + 255) / 256);
    hipLaunchKernelGGL(k_fix_ties, dim3(blocks), dim3(256), 0, s, ctx->key, ctx->idx, id, n);
    return dzs_check_launch(ctx, "fix_ties");
}
