// Tile binning: ordered compaction of the visible (view, Gaussian) pairs, a stable LSD radix sort
// of them by float32 depth bits, depth-ordered emission of (view-tile, pair) instances and a
// stable LSD radix sort of the instances by view-tile.  The result equals a lexicographic sort by
// (view, tile, depth bits, Gaussian index) while the expensive instance sort only moves the
// ceil(log2(V*T)) tile bits (two 8-bit passes for up to 65,536 view-tiles) instead of all 47+.
//
// Every kernel reads the live element count from device memory and is launched over the
// capacity, so the whole pipeline runs without a host round-trip (and can be graph-captured).
#include "gsr_internal.h"

namespace gsr {

__device__ __forceinline__ uint32_t dev_count(const uint32_t *n_dev, uint32_t n_host, uint32_t cap) {
    const uint32_t n = n_dev ? *n_dev : n_host;
    return n < cap ? n : cap;
}

// ---- generic helpers -------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t *__restrict__ dst, uint32_t value, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = value;
}

// Exclusive scan in place of nb (small) block sums by one 1024-thread block; writes the total.
// With lim, only the first ceil(*lim / per) sums are scanned (the rest are zero and unread).
__global__ __launch_bounds__(1024) void k_scan_small(uint32_t *__restrict__ v, int nb, uint32_t *__restrict__ total,
                                                     const uint32_t *__restrict__ lim = nullptr, uint32_t per = 1) {
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_carry;
    if (lim) {
        const uint32_t used = (*lim + per - 1) / per;
        nb = used < (uint32_t)nb ? (int)used : nb;
    }
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int base = 0; base < nb; base += 1024) {
        const int idx = base + threadIdx.x;
        const uint32_t x = idx < nb ? v[idx] : 0u;
        uint32_t inc = wave_incl_scan(x);
        const int w = threadIdx.x >> 6;
        if (__lane_id() == 63) s_w[w] = inc;
        __syncthreads();
        uint32_t wb = 0, tot = 0;
        for (int k = 0; k < 16; k++) {
            wb += k < w ? s_w[k] : 0u;
            tot += s_w[k];
        }
        const uint32_t carry = s_carry;
        if (idx < nb) v[idx] = carry + wb + inc - x;
        __syncthreads();
        if (threadIdx.x == 0) s_carry = carry + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = s_carry;
}

// ---- ordered compaction of visible pairs ---------------------------------------------------------
// Block b covers pairs [b*4096, (b+1)*4096) in round-major order: pair b*4096 + r*256 + t is read by
// thread t in round r, so every load is coalesced; (round, wave, lane) order is pair order.
// Also clears the tile ranges (VT2 words), which k_tile_ranges writes for tiles with instances only.
__global__ __launch_bounds__(256) void k_vis_count(const uint32_t *__restrict__ ntiles, uint32_t VN,
                                                   uint32_t *__restrict__ bsum, uint32_t *__restrict__ ranges,
                                                   uint32_t VT2) {
    __shared__ uint32_t s_w[4];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < VT2; i += gridDim.x * 256) ranges[i] = 0u;
    const uint32_t base = blockIdx.x * kSortTile;
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        const uint32_t e = base + r * kSortThreads + threadIdx.x;
        c += (e < VN && ntiles[e] > 0) ? 1u : 0u;
    }
    uint32_t tot;
    block_excl_scan256(c, s_w, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Sum of v[0 .. n) over a 256-thread block (four words of LDS).
__device__ __forceinline__ uint32_t block_sum_of(const uint32_t *__restrict__ v, uint32_t n, uint32_t *s_w) {
    uint32_t c = 0;
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < n; i += 256) c += v[i];
    uint32_t tot;
    block_excl_scan256(c, s_w, &tot);
    return tot;
}

// SELF: boff holds the blocks' plain counts; every block adds up those before it (they fit a few loads
// per thread), which saves the launch that would scan them, and the last one writes the total.
template <bool SELF>
__global__ __launch_bounds__(256) void k_vis_compact(const uint32_t *__restrict__ info, uint32_t VN,
                                                     const uint32_t *__restrict__ boff, uint32_t *__restrict__ keys,
                                                     uint32_t *__restrict__ vals, uint32_t *__restrict__ n_vis) {
    __shared__ uint32_t s_cnt[kSortItems * 4];
    __shared__ uint32_t s_w[4];
    const uint32_t base = blockIdx.x * kSortTile;
    const int w = threadIdx.x >> 6, lane = __lane_id();
    uint64_t m[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        const uint32_t e = base + r * kSortThreads + threadIdx.x;
        m[r] = __ballot(e < VN && info[e] > 0);
        if (lane == 0) s_cnt[r * 4 + w] = (uint32_t)__popcll(m[r]);
    }
    __syncthreads();
    // exclusive prefix of the 64 (round, wave) counts, in that order
    if (threadIdx.x < kSortItems * 4) {
        const uint32_t c = s_cnt[threadIdx.x];
        s_cnt[threadIdx.x] = wave_incl_scan(c) - c;
    }
    __syncthreads();
    uint32_t b0;
    if (SELF) {
        b0 = block_sum_of(boff, blockIdx.x, s_w);
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *n_vis = b0 + boff[blockIdx.x];
    } else {
        b0 = boff[blockIdx.x];
    }
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        if ((m[r] >> lane) & 1ull) {
            const uint32_t e = base + r * kSortThreads + threadIdx.x;
            const uint32_t pos = b0 + s_cnt[r * 4 + w] + (uint32_t)__popcll(m[r] & lt);
            keys[pos] = info[VN + e];
            vals[pos] = e;
        }
    }
}

// ---- exclusive scan of a long uint32 array (the stored-contributor offsets) ------------------
// The kSortItems consecutive words of one thread, in 16-byte accesses where they are whole and aligned (1.5M
// words: the write took 12.5 us in single words, 5.5 us so).
__device__ __forceinline__ bool whole_items(const uint32_t *p, int64_t base, int64_t n) {
    return base + kSortItems <= n && (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
}
__device__ __forceinline__ void load_items(const uint32_t *__restrict__ in, int64_t base, int64_t n,
                                           uint32_t x[kSortItems]) {
    if (whole_items(in, base, n)) {
#pragma unroll
        for (int k = 0; k < kSortItems / 4; k++) {
            const uint4 q = reinterpret_cast<const uint4 *>(in + base)[k];
            x[4 * k] = q.x, x[4 * k + 1] = q.y, x[4 * k + 2] = q.z, x[4 * k + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kSortItems; k++) x[k] = base + k < n ? in[base + k] : 0u;
    }
}

__global__ __launch_bounds__(256) void k_scan_sum(const uint32_t *__restrict__ in, int64_t n,
                                                  uint32_t *__restrict__ bsum) {
    __shared__ uint32_t s_w[4];
    uint32_t x[kSortItems], c = 0;
    load_items(in, (int64_t)blockIdx.x * kSortTile + threadIdx.x * kSortItems, n, x);
#pragma unroll
    for (int k = 0; k < kSortItems; k++) c += x[k];
    uint32_t tot;
    block_excl_scan256(c, s_w, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void k_scan_write(const uint32_t *__restrict__ in, int64_t n,
                                                    const uint32_t *__restrict__ boff, uint32_t *__restrict__ out) {
    __shared__ uint32_t s_w[4];
    const int64_t base = (int64_t)blockIdx.x * kSortTile + threadIdx.x * kSortItems;
    uint32_t x[kSortItems], c = 0;
    load_items(in, base, n, x);
#pragma unroll
    for (int k = 0; k < kSortItems; k++) c += x[k];
    uint32_t run = boff[blockIdx.x] + block_excl_scan256(c, s_w, nullptr);
#pragma unroll
    for (int k = 0; k < kSortItems; k++) {
        const uint32_t v = x[k];
        x[k] = run;
        run += v;
    }
    if (whole_items(out, base, n)) {
#pragma unroll
        for (int k = 0; k < kSortItems / 4; k++)
            reinterpret_cast<uint4 *>(out + base)[k] = make_uint4(x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < kSortItems; k++)
            if (base + k < n) out[base + k] = x[k];
    }
}

// ---- stable LSD radix sort, 8-bit digits -----------------------------------------------------
// Block b sorts items [b*tile, (b+1)*tile), tile = 256 * ITEMS; the histogram counts each block's
// digits, and the scatter ranks them stably (input order) inside the block.
//
// Long sorts take 12 keys per thread: a block's run of one digit is then 12 keys long on average, so
// the scattered writes stay wide.  Short ones are bound by one block's latency (dependent loads, then
// a chain of ITEMS rank rounds) on a chip they do not fill, and take 4.  The choice follows the live
// count, which only the device knows: a capacity says little (a registration sorts 240k targets of a map of
// 1.5M rows: 14 us of its 632 less with 4).  The line is the largest sort that the two-launch form takes on
// the host: four passes over 1.1M keys take 83 us either way, over 2M 121 with 4 and 109 with 12, over 4.1M
// 224 and 187.
constexpr int kRadixItems = 12, kShortItems = 4;
constexpr uint32_t kShortSort = 1 << 20;  // live keys
constexpr int kRadixTile = kSortThreads * kRadixItems, kShortTile = kSortThreads * kShortItems;
inline int64_t radix_blocks(int64_t cap) {
    const int64_t few = ceil_div(cap < (int64_t)kShortSort ? cap : (int64_t)kShortSort, kShortTile), all = ceil_div(cap, kRadixTile);
    return all > few ? all : few;
}

template <int ITEMS>
__device__ __forceinline__ void radix_hist_block(const uint32_t *__restrict__ keys, uint32_t n, uint32_t cap, int shift,
                                                 int nblocks, uint32_t *__restrict__ hist, uint32_t *cnt) {
    // Counts are order-free: each thread takes ITEMS consecutive keys (16-byte loads) and adds a run
    // of equal digits to the block's LDS count in one atomic, so nearly sorted input (long runs)
    // costs one add per run and shuffled input one per key.
    // blocks past the live count write nothing: the row scan and the scatter skip them
    if (blockIdx.x * (uint32_t)(kSortThreads * ITEMS) >= n) return;
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t first = blockIdx.x * (kSortThreads * ITEMS) + threadIdx.x * ITEMS;
    if (first < n) {
        uint32_t k[ITEMS];
        if (first + ITEMS <= cap && (reinterpret_cast<uintptr_t>(keys) & 15u) == 0) {
#pragma unroll
            for (int q = 0; q < ITEMS / 4; q++) {
                const uint4 x = *reinterpret_cast<const uint4 *>(keys + first + 4 * q);
                k[4 * q] = x.x, k[4 * q + 1] = x.y, k[4 * q + 2] = x.z, k[4 * q + 3] = x.w;
            }
        } else {
#pragma unroll
            for (int r = 0; r < ITEMS; r++) k[r] = first + r < cap ? keys[first + r] : 0u;
        }
        const uint32_t m = n - first < (uint32_t)ITEMS ? n - first : (uint32_t)ITEMS;
        uint32_t d = (k[0] >> shift) & (kRadix - 1), run = 1;
#pragma unroll
        for (int r = 1; r < ITEMS; r++) {
            if ((uint32_t)r >= m) break;
            const uint32_t dr = (k[r] >> shift) & (kRadix - 1);
            if (dr != d) {
                atomicAdd(&cnt[d], run);
                d = dr;
                run = 0;
            }
            run++;
        }
        atomicAdd(&cnt[d], run);
    }
    __syncthreads();
    hist[threadIdx.x * nblocks + blockIdx.x] = cnt[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_radix_hist(const uint32_t *__restrict__ keys, const uint32_t *n_dev,
                                                    uint32_t n_host, uint32_t cap, int shift, int nblocks,
                                                    uint32_t *__restrict__ hist) {
    __shared__ uint32_t cnt[kRadix];
    const uint32_t n = dev_count(n_dev, n_host, cap);
    if (n <= kShortSort) radix_hist_block<kShortItems>(keys, n, cap, shift, nblocks, hist, cnt);
    else radix_hist_block<kRadixItems>(keys, n, cap, shift, nblocks, hist, cnt);
}

// Row d of hist (one row per digit, row stride nblocks) is scanned exclusively in place over the
// blocks that hold live items; the row total goes to totals[d].
__global__ __launch_bounds__(256) void k_radix_scan_rows(uint32_t *__restrict__ hist, int nblocks,
                                                         uint32_t *__restrict__ totals, const uint32_t *n_dev,
                                                         uint32_t n_host, uint32_t cap) {
    // one digit's row per workgroup; each thread owns a contiguous run of the row: sum it, one
    // workgroup scan of the run sums, then rewrite the run as exclusive prefixes.  Runs of up to
    // 16 entries (up to 4096 live blocks) stay in registers, loaded all at once.
    __shared__ uint32_t s_w[4];
    uint32_t *row = hist + (int64_t)blockIdx.x * nblocks;
    const uint32_t n = dev_count(n_dev, n_host, cap);
    const uint32_t tile = n <= kShortSort ? kShortTile : kRadixTile;
    const int live = (int)((n + tile - 1) / tile);
    const int nb = live < nblocks ? live : nblocks;
    const int per = (nb + 255) / 256;
    const int b0 = threadIdx.x * per;
    const int b1 = b0 + per < nb ? b0 + per : nb;
    if (per <= 16) {
        uint32_t x[16];
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < 16; k++) {
            x[k] = b0 + k < b1 ? row[b0 + k] : 0u;
            sum += x[k];
        }
        uint32_t tot;
        uint32_t run = block_excl_scan256(sum, s_w, &tot);
#pragma unroll
        for (int k = 0; k < 16; k++) {
            if (b0 + k < b1) row[b0 + k] = run;
            run += x[k];
        }
        if (threadIdx.x == 0) totals[blockIdx.x] = tot;
        return;
    }
    uint32_t sum = 0;
    for (int idx = b0; idx < b1; idx++) sum += row[idx];
    uint32_t tot;
    uint32_t run = block_excl_scan256(sum, s_w, &tot);
    for (int idx = b0; idx < b1; idx++) {
        const uint32_t x = row[idx];
        row[idx] = run;
        run += x;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = tot;
}

// Block b sorts its tile: wave w owns a quarter of it, 64 items per round, so (wave, round, lane)
// order is input order and each wave ranks its items with its own running digit counts, without a
// workgroup barrier per round; the four waves' counts then give every digit's local start and each
// wave's offset inside it.
template <int ITEMS>
__device__ __forceinline__ void radix_scatter_block(const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                    uint32_t *__restrict__ kout, uint32_t *__restrict__ vout,
                                                    const uint32_t *__restrict__ vin2, uint32_t *__restrict__ vout2,
                                                    uint32_t n, int shift, int nblocks,
                                                    const uint32_t *__restrict__ hist,
                                                    const uint32_t *__restrict__ totals, uint32_t *s_keys,
                                                    uint32_t *s_vals, uint32_t (*s_wcnt)[kRadix], uint32_t *s_gbase,
                                                    uint32_t *s_w) {
    constexpr int kTile = kSortThreads * ITEMS, kWaveItems = kTile / 4;
    const uint32_t base = blockIdx.x * kTile;
    if (base >= n) return;
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    // all loads first: the items, and digit t's counts
    uint32_t mk[ITEMS], mv[ITEMS], mv2[ITEMS], mrank[ITEMS];
    const uint32_t wbase = base + w * kWaveItems;
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const uint32_t idx = wbase + r * 64 + lane;
        const bool valid = idx < n;
        mk[r] = valid ? kin[idx] : 0u;
        mv[r] = valid ? vin[idx] : 0u;
        mv2[r] = vin2 ? (valid ? vin2[idx] : 0u) : idx;
    }
    const uint32_t dtot = totals[t], before_blocks = hist[t * nblocks + blockIdx.x];
    for (int k = 0; k < 4; k++) s_wcnt[k][t] = 0;
    __syncthreads();
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const bool valid = wbase + r * 64 + lane < n;
        const uint32_t d = (mk[r] >> shift) & (kRadix - 1);
        const uint64_t peers = match_digit8(d, valid);
        const uint32_t rank = (uint32_t)__popcll(peers & lt);
        // the wave's count of digit d so far (read by every lane before its leader adds)
        const uint32_t before = s_wcnt[w][d];
        mrank[r] = before + rank;
        if (valid && rank == 0) s_wcnt[w][d] = before + (uint32_t)__popcll(peers);
    }
    // global start of digit t for this block
    const uint32_t gstart = block_excl_scan256(dtot, s_w, nullptr) + before_blocks;
    {
        const uint32_t c0 = s_wcnt[0][t], c1 = s_wcnt[1][t], c2 = s_wcnt[2][t], c3 = s_wcnt[3][t];
        const uint32_t ls = block_excl_scan256(c0 + c1 + c2 + c3, s_w, nullptr);
        s_gbase[t] = gstart - ls;
        s_wcnt[0][t] = ls;
        s_wcnt[1][t] = ls + c0;
        s_wcnt[2][t] = ls + c0 + c1;
        s_wcnt[3][t] = ls + c0 + c1 + c2;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        if (wbase + r * 64 + lane < n) {
            mrank[r] += s_wcnt[w][(mk[r] >> shift) & (kRadix - 1)];
            s_keys[mrank[r]] = mk[r];
            s_vals[mrank[r]] = mv[r];
        }
    }
    __syncthreads();
    const uint32_t bn = (n - base) < (uint32_t)kTile ? (n - base) : (uint32_t)kTile;
    uint32_t dst[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const uint32_t p = r * kSortThreads + t;
        if (p < bn) {
            const uint32_t k = s_keys[p];
            dst[r] = s_gbase[(k >> shift) & (kRadix - 1)] + p;
            kout[dst[r]] = k;
            vout[dst[r]] = s_vals[p];
        }
    }
    if (vout2) {
        // the second payload takes the same permutation through the same LDS staging (without
        // vin2 it is each item's input position)
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; r++)
            if (wbase + r * 64 + lane < n) s_vals[mrank[r]] = mv2[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; r++) {
            const uint32_t p = r * kSortThreads + t;
            if (p < bn) vout2[dst[r]] = s_vals[p];
        }
    }
}

__global__ __launch_bounds__(256) void k_radix_scatter(const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                       uint32_t *__restrict__ kout, uint32_t *__restrict__ vout,
                                                       const uint32_t *__restrict__ vin2, uint32_t *__restrict__ vout2,
                                                       const uint32_t *n_dev, uint32_t n_host, uint32_t cap, int shift,
                                                       int nblocks, const uint32_t *__restrict__ hist,
                                                       const uint32_t *__restrict__ totals) {
    __shared__ uint32_t s_keys[kRadixTile];
    __shared__ uint32_t s_vals[kRadixTile];
    __shared__ uint32_t s_wcnt[4][kRadix];  // per-wave running counts, then per-wave starts
    __shared__ uint32_t s_gbase[kRadix];    // global minus local start of the digit
    __shared__ uint32_t s_w[4];
    const uint32_t n = dev_count(n_dev, n_host, cap);
    if (n <= kShortSort)
        radix_scatter_block<kShortItems>(kin, vin, kout, vout, vin2, vout2, n, shift, nblocks, hist, totals, s_keys, s_vals,
                                         s_wcnt, s_gbase, s_w);
    else
        radix_scatter_block<kRadixItems>(kin, vin, kout, vout, vin2, vout2, n, shift, nblocks, hist, totals, s_keys, s_vals,
                                         s_wcnt, s_gbase, s_w);
}

// ---- instance emission in depth order --------------------------------------------------------
// Instance count of each block of 256 depth-ordered visible pairs.
__global__ __launch_bounds__(256) void k_inst_count(const uint32_t *__restrict__ sorted_gid, const uint32_t *n_vis,
                                                    uint32_t cap, const uint32_t *__restrict__ ntiles,
                                                    uint32_t *__restrict__ bsum) {
    __shared__ uint32_t s_w[4];
    const uint32_t n = dev_count(n_vis, 0, cap);
    // blocks of 256 pairs up to the visible count (grid-stride; later sums are never read)
    for (uint32_t b = blockIdx.x; b * 256 < n; b += gridDim.x) {
        const uint32_t idx = b * 256 + threadIdx.x;
        const uint32_t c = idx < n ? ntiles[sorted_gid[idx]] : 0u;
        uint32_t tot;
        block_excl_scan256(c, s_w, &tot);
        if (threadIdx.x == 0) bsum[b] = tot;
    }
}

// Emission of the instances of 256 depth-ordered visible pairs per block, load-balanced: the
// block's instances are spread over its threads (instance k of the block goes to thread
// k mod 256, which finds its pair by binary search over the pairs' offsets in LDS), so the
// writes are coalesced.  A pair's tiles are emitted row-major and consecutively ("emission
// order").  With pair_gid: the emission-ordered list of visible pairs and the emission index of
// each pair's first instance.  (Each instance's emission index is its position here: the sort's
// first pass generates it as the second payload.)  SELF: as in k_vis_compact; the block of the last
// pairs writes the instance count.
// The nearest pairs come first and cover most tiles: the first kSplitPairs blocks of pairs are shared by
// kEmitSplit workgroups each, every one emitting its share of the block's instances.  One workgroup
// alone held the launch up (room of 300k Gaussians: 56 us, now 15; three 640x360 views: 22 us, now 11;
// the corridor step's 87 us are bound by its 2.8M pairs).  They come first in the grid: at its end they
// started last and cost the corridor 10 us.
constexpr uint32_t kSplitPairs = 32, kEmitSplit = 8;
template <bool SELF>
__global__ __launch_bounds__(256) void k_inst_emit(const uint32_t *__restrict__ sorted_gid, const uint32_t *n_vis,
                                                   uint32_t cap_vis, const uint32_t *__restrict__ info, uint32_t VN,
                                                   uint32_t n, uint32_t T, uint32_t ntx,
                                                   const uint32_t *__restrict__ boff, uint32_t *__restrict__ ikey,
                                                   uint32_t *__restrict__ ival,
                                                   uint32_t *__restrict__ pair_gid, uint32_t *__restrict__ pair_first,
                                                   uint32_t *__restrict__ n_pairs, uint32_t *__restrict__ n_inst,
                                                   uint32_t cap, uint32_t nb_p) {
    // block of pairs and this workgroup's share of its instances; the shared blocks come first
    const uint32_t split = nb_p < kSplitPairs ? nb_p : kSplitPairs;
    const bool shared = blockIdx.x < split * kEmitSplit;
    const uint32_t blk = shared ? blockIdx.x / kEmitSplit : blockIdx.x - split * (kEmitSplit - 1);
    const uint32_t share = shared ? blockIdx.x % kEmitSplit : 0u;
    const uint32_t shares = blk < kSplitPairs ? kEmitSplit : 1u;
    __shared__ uint32_t s_w[4];
    __shared__ uint32_t s_off[256], s_gid[256], s_r0[256], s_r1[256];
    const uint32_t nv = dev_count(n_vis, 0, cap_vis);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (n_pairs) *n_pairs = nv;
        if (SELF && nv == 0) *n_inst = 0u;
    }
    if (blk * 256 >= nv) return;
    const uint32_t idx = blk * 256 + threadIdx.x;
    const bool valid = idx < nv;
    const uint32_t gid = valid ? sorted_gid[idx] : 0u;
    const uint32_t c = valid ? info[gid] : 0u;
    uint32_t tot;
    const uint32_t excl = block_excl_scan256(c, s_w, &tot);
    const uint32_t base = SELF ? block_sum_of(boff, blk, s_w) : boff[blk];
    if (SELF && share == 0 && (blk + 1) * 256 >= nv && threadIdx.x == 0) *n_inst = base + tot;
    s_off[threadIdx.x] = excl;
    s_gid[threadIdx.x] = gid;
    s_r0[threadIdx.x] = valid ? info[2 * VN + gid] : 0u;
    s_r1[threadIdx.x] = valid ? info[3 * VN + gid] : 0u;
    if (valid && pair_gid && share == 0) {
        pair_gid[idx] = gid;
        pair_first[idx] = base + excl;
    }
    __syncthreads();
    for (uint32_t k = share * 256 + threadIdx.x; k < tot; k += shares * 256) {
        // the last pair whose offset is <= k (pairs without instances share the next one's offset)
        uint32_t lo = 0, hi = 256;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (s_off[mid] <= k) lo = mid;
            else hi = mid;
        }
        const uint32_t g = s_gid[lo], r0 = s_r0[lo], r1 = s_r1[lo];
        const uint32_t local = k - s_off[lo];
        const uint32_t tx0 = r0 & 0xffffu, ty0 = r0 >> 16, tx1 = r1 & 0xffffu;
        const uint32_t wdt = tx1 - tx0 + 1;
        const uint32_t ly = local / wdt, lx = local - ly * wdt;
        const uint32_t pos = base + k;
        if (pos < cap) {
            ikey[pos] = (g / n) * T + (ty0 + ly) * ntx + tx0 + lx;
            ival[pos] = g;
        }
    }
}

// LPT key of every view-tile, one byte: the instance count as a small float (the exponent
// floor(log2 c) times 16 plus the next four bits below the leading one, so the key grows with the
// count and resolves it to 1/16 of an octave; empty tiles share the key of a single instance,
// counts of 2^16 and more the key of the top step below 2^16), stored as 255 minus that so that an
// ascending stable sort puts the longest tiles first, ties by index.
__device__ __forceinline__ uint32_t lpt_key(uint32_t c) {
    if (c == 0) return 255u;
    const uint32_t e = 31u - (uint32_t)__builtin_clz(c);  // 0 .. 31
    if (e >= 16u) return 0u;
    const uint32_t m = e >= 4u ? (c >> (e - 4u)) & 15u : (c << (4u - e)) & 15u;
    return 255u - (e * 16u + m);
}

__global__ void k_tile_keys(const uint32_t *__restrict__ ranges, uint32_t VT, uint32_t *__restrict__ keys,
                            uint32_t *__restrict__ vals) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < VT; i += gridDim.x * blockDim.x) {
        keys[i] = lpt_key(ranges[2 * i + 1] - ranges[2 * i]);
        vals[i] = i;
    }
}

// [start, end) of every view-tile with instances (ranges were cleared before).  An instance count
// above the capacity leaves incomplete lists.  Rather than render them, the frame is emptied: no
// pair visible (tile_info row 0 cleared), every tile range empty and no emitted pair, so the render,
// backward, pair sums, projection backward, fused Adam and visible list that follow on the stream do
// nothing.
__global__ void k_tile_ranges(const uint32_t *__restrict__ keys, const uint32_t *__restrict__ n_inst, uint32_t cap,
                              uint32_t *__restrict__ ranges, uint32_t *__restrict__ ntiles, uint32_t VN,
                              uint32_t *__restrict__ n_pairs) {
    const uint32_t m = *n_inst, stride = gridDim.x * blockDim.x;
    if (m > cap) {
        for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < VN; i += stride) ntiles[i] = 0u;
        if (n_pairs && blockIdx.x == 0 && threadIdx.x == 0) *n_pairs = 0u;
        return;
    }
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const uint32_t k = keys[i];
        if (i == 0 || keys[i - 1] != k) ranges[2 * k] = i;
        if (i + 1 == m || keys[i + 1] != k) ranges[2 * k + 1] = i + 1;
    }
}

// ---- small problems: one workgroup -------------------------------------------------------------
// Up to kSmallSort items fit one 1024-thread block's LDS.  A launch of the general path costs 2 to 5
// us on an idle chip whatever its work, so the 17 launches from the visible pairs to the emission
// offsets (compaction, four radix passes, instance scan) become one, and the tile order's four one.
constexpr int kSmallThreads = 1024, kSmallRounds = 8, kSmallSort = kSmallThreads * kSmallRounds;

// Exclusive prefix of one value per thread over the 1024-thread block; *total its sum.
__device__ __forceinline__ uint32_t block_excl_scan1024(uint32_t v, uint32_t *s_w, uint32_t *total) {
    const int w = threadIdx.x >> 6;
    const uint32_t inc = wave_incl_scan(v);
    if (__lane_id() == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < 16; k++) {
        base += k < w ? s_w[k] : 0u;
        tot += s_w[k];
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

// Stable positions of n items by their 8-bit digits.  Thread t of wave w holds items w * rounds * 64 +
// r * 64 + lane, r < rounds = ceil(n / 1024), so that (wave, round, lane) order is item order.
__device__ __forceinline__ void small_positions(const uint32_t d[kSmallRounds], uint32_t n, int rounds,
                                                uint32_t (*s_cnt)[kRadix], uint32_t *s_w,
                                                uint32_t pos[kSmallRounds]) {
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    for (int q = t; q < 16 * kRadix; q += kSmallThreads) s_cnt[q >> kRadixBits][q & (kRadix - 1)] = 0u;
    __syncthreads();
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < kSmallRounds; r++) {
        if (r >= rounds) break;
        const bool valid = (uint32_t)((w * rounds + r) * 64 + lane) < n;
        const uint64_t peers = match_digit8(d[r], valid);
        const uint32_t rank = (uint32_t)__popcll(peers & lt);
        const uint32_t before = s_cnt[w][d[r]];
        pos[r] = before + rank;
        if (valid && rank == 0) s_cnt[w][d[r]] = before + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    uint32_t c[16], sum = 0, tot;
    if (t < kRadix) {
#pragma unroll
        for (int k = 0; k < 16; k++) sum += c[k] = s_cnt[k][t];
    }
    uint32_t run = block_excl_scan1024(sum, s_w, &tot);
    if (t < kRadix) {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            s_cnt[k][t] = run;
            run += c[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallRounds; r++) {
        if (r >= rounds) break;
        pos[r] += s_cnt[w][d[r]];
    }
}

// Visible pairs of VN <= kSmallSort, stably sorted by depth bits: their rows, count, the exclusive
// instance offset of every 256 of them and the instance count.  Clears the tile ranges.
__global__ __launch_bounds__(kSmallThreads) void k_bin_small(const uint32_t *__restrict__ info, uint32_t VN,
                                                             uint32_t *__restrict__ sorted_gid,
                                                             uint32_t *__restrict__ boff, uint32_t *__restrict__ n_vis,
                                                             uint32_t *__restrict__ n_inst,
                                                             uint32_t *__restrict__ ranges, uint32_t VT2) {
    __shared__ uint32_t s_k[kSmallSort], s_v[kSmallSort];
    __shared__ uint32_t s_cnt[16][kRadix];
    __shared__ uint32_t s_w[16];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    for (uint32_t i = t; i < VT2; i += kSmallThreads) ranges[i] = 0u;
    // ordered compaction: thread t reads pairs r * 1024 + t
    uint32_t nt[kSmallRounds], z[kSmallRounds];
#pragma unroll
    for (int r = 0; r < kSmallRounds; r++) {
        const uint32_t e = r * kSmallThreads + t;
        nt[r] = e < VN ? info[e] : 0u;
        z[r] = e < VN ? info[VN + e] : 0u;  // (unwritten where no tile is, and not used then)
    }
    uint32_t n = 0;
#pragma unroll
    for (int r = 0; r < kSmallRounds; r++) {
        if ((uint32_t)(r * kSmallThreads) >= VN) break;
        uint32_t tot;
        const uint32_t p = n + block_excl_scan1024(nt[r] ? 1u : 0u, s_w, &tot);
        if (nt[r]) {
            s_k[p] = z[r];
            s_v[p] = r * kSmallThreads + t;
        }
        n += tot;
    }
    __syncthreads();
    const int rounds = (int)((n + kSmallThreads - 1) / kSmallThreads);
    const uint32_t first = (uint32_t)(w * rounds * 64 + lane);
    for (int shift = 0; shift < 32; shift += kRadixBits) {
        uint32_t k[kSmallRounds], v[kSmallRounds], d[kSmallRounds], pos[kSmallRounds];
#pragma unroll
        for (int r = 0; r < kSmallRounds; r++) {
            if (r >= rounds) break;
            const uint32_t i = first + r * 64;
            k[r] = i < n ? s_k[i] : 0u;
            v[r] = i < n ? s_v[i] : 0u;
            d[r] = (k[r] >> shift) & (kRadix - 1);
        }
        small_positions(d, n, rounds, s_cnt, s_w, pos);  // (barriers inside: every item has been read)
#pragma unroll
        for (int r = 0; r < kSmallRounds; r++) {
            if (r >= rounds) break;
            if (first + r * 64 < n) {
                s_k[pos[r]] = k[r];
                s_v[pos[r]] = v[r];
            }
        }
        __syncthreads();
    }
    uint32_t run = 0;
    for (int r = 0; r < rounds; r++) {
        const uint32_t i = r * kSmallThreads + t;
        const uint32_t g = i < n ? s_v[i] : 0u, c = i < n ? info[g] : 0u;
        uint32_t tot;
        const uint32_t p = run + block_excl_scan1024(c, s_w, &tot);
        if (i < n) {
            sorted_gid[i] = g;
            if ((i & 255u) == 0) boff[i >> 8] = p;
        }
        run += tot;
    }
    if (t == 0) {
        *n_vis = n;
        *n_inst = run;
    }
}

// Longest-first order of VT <= kSmallSort view-tiles.
__global__ __launch_bounds__(kSmallThreads) void k_tile_order_small(const uint32_t *__restrict__ ranges, uint32_t VT,
                                                                    uint32_t *__restrict__ order) {
    __shared__ uint32_t s_cnt[16][kRadix];
    __shared__ uint32_t s_w[16];
    const int rounds = (int)((VT + kSmallThreads - 1) / kSmallThreads);
    const uint32_t first = (uint32_t)((threadIdx.x >> 6) * rounds * 64 + (threadIdx.x & 63));
    uint32_t d[kSmallRounds], pos[kSmallRounds];
#pragma unroll
    for (int r = 0; r < kSmallRounds; r++) {
        if (r >= rounds) break;
        const uint32_t i = first + r * 64;
        d[r] = i < VT ? lpt_key(ranges[2 * i + 1] - ranges[2 * i]) : 0u;
    }
    small_positions(d, VT, rounds, s_cnt, s_w, pos);
#pragma unroll
    for (int r = 0; r < kSmallRounds; r++) {
        if (r >= rounds) break;
        if (first + r * 64 < VT) order[pos[r]] = first + r * 64;
    }
}

// ---- few keys: two launches per pass ------------------------------------------------------------
// Each of the general path's three launches per pass costs its 3 to 5 us at some hundred thousand keys
// whatever it does, and the host as much again where the launches are not captured.  Up to kFewSort
// keys the live ones are cut into at most kFewRows chunks, few enough for every workgroup of the scatter
// to add up the counts of all chunks itself (one row of 256 counts per chunk, read coalesced), and the
// row scan goes.  (Counting the next digit in the scatter by atomics, one launch per pass, was slower:
// atomics to one cache line follow each other in 26 ns, and a digit of few values has one line a chunk.)
// A pass over 40k depth keys: 3.3 + 3.5 + 6.0 -> 2.6 + 6.8 us; a scan's two voxel sorts of 100k points,
// with the rest of the initialisation, 156 -> 147 us.  Instances of 600k with two payloads break even
// (3.7 + 4 + 8 -> 4 + 13 us), and 1.5M keys lose (22 -> 28 us): the line lies at 8 keys per thread.
constexpr int kFewThreads = 1024, kFewRows = 128, kFewItems = 8;
constexpr int64_t kFewSort = (int64_t)kFewThreads * kFewRows * kFewItems;

// Keys per thread of n live keys; a chunk is kFewThreads times that.
__device__ __forceinline__ uint32_t few_rounds(uint32_t n) {
    return n ? (n + kFewThreads * kFewRows - 1) / (kFewThreads * kFewRows) : 1u;
}

// Digit counts of every chunk, one row each.
__global__ __launch_bounds__(kFewThreads) void k_few_hist(const uint32_t *__restrict__ keys, const uint32_t *n_dev,
                                                          uint32_t n_host, uint32_t cap, int shift,
                                                          uint32_t *__restrict__ hist) {
    __shared__ uint32_t s_cnt[4][kRadix];
    const uint32_t n = dev_count(n_dev, n_host, cap), chunk = few_rounds(n) * kFewThreads;
    const uint32_t base = blockIdx.x * chunk, t = threadIdx.x;
    if (base >= n) return;
    s_cnt[t >> kRadixBits][t & (kRadix - 1)] = 0u;
    __syncthreads();
    const uint32_t end = n - base < chunk ? n : base + chunk;
    uint32_t *cnt = s_cnt[(t >> 6) & 3u];
    for (uint32_t i = base + t; i < end; i += kFewThreads) {
        const uint32_t d = (keys[i] >> shift) & (kRadix - 1);
        // a wave of one digit (sorted input, high digits) adds once instead of 64 times to one word
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
        const uint64_t same = __ballot(d == d0), on = __ballot(true);
        if (same == on) {
            if (__lane_id() == (int)__builtin_ctzll(on)) atomicAdd(&cnt[d0], (uint32_t)__popcll(on));
        } else {
            atomicAdd(&cnt[d], 1u);
        }
    }
    __syncthreads();
    if (t < kRadix) hist[blockIdx.x * kRadix + t] = s_cnt[0][t] + s_cnt[1][t] + s_cnt[2][t] + s_cnt[3][t];
}

// One pass: chunk b's keys go to their places, in input order within a digit.  Loads, ranks and LDS staging as in k_radix_scatter.
template <int ITEMS>
__global__ __launch_bounds__(kFewThreads) void k_few_pass(const uint32_t *__restrict__ kin,
                                                          const uint32_t *__restrict__ vin,
                                                          uint32_t *__restrict__ kout, uint32_t *__restrict__ vout,
                                                          const uint32_t *__restrict__ vin2,
                                                          uint32_t *__restrict__ vout2, const uint32_t *n_dev,
                                                          uint32_t n_host, uint32_t cap, int shift,
                                                          const uint32_t *__restrict__ hist) {
    __shared__ __align__(16) uint32_t s_stage[kFewThreads * ITEMS > 32 * kRadix ? kFewThreads * ITEMS : 32 * kRadix];
    __shared__ uint32_t s_cnt[16][kRadix];
    __shared__ uint32_t s_gbase[kRadix];  // global minus local start of the digit
    __shared__ uint32_t s_w[16];
    const uint32_t n = dev_count(n_dev, n_host, cap), rounds = few_rounds(n), chunk = rounds * kFewThreads;
    const uint32_t base = blockIdx.x * chunk;
    if (base >= n) return;
    const uint32_t t = threadIdx.x, w = t >> 6, lane = t & 63u;
    const uint32_t first = base + w * rounds * 64 + lane;  // this thread's keys: first + 64 r
    uint32_t mk[ITEMS], mv[ITEMS], mv2[ITEMS], pos[ITEMS];
#pragma unroll
    for (uint32_t r = 0; r < ITEMS; r++) {
        if (r >= rounds) continue;
        const uint32_t i = first + r * 64;
        mk[r] = i < n ? kin[i] : 0u;
        mv[r] = i < n ? vin[i] : 0u;
        mv2[r] = vin2 ? (i < n ? vin2[i] : 0u) : i;
    }
    // wave w adds up the counts of chunks w, w + 16, ...: all of them, and those before this one
    const uint32_t rows = (n + chunk - 1) / chunk;
    {
        uint4 tot = make_uint4(0, 0, 0, 0), before = tot;
#pragma unroll
        for (uint32_t k = 0; k < kFewRows / 16; k++) {
            const uint32_t row = k * 16 + w;
            const uint4 c = row < rows ? reinterpret_cast<const uint4 *>(hist + row * kRadix)[lane] : make_uint4(0, 0, 0, 0);
            const uint32_t m = row < blockIdx.x ? 0xffffffffu : 0u;
            tot.x += c.x, tot.y += c.y, tot.z += c.z, tot.w += c.w;
            before.x += c.x & m, before.y += c.y & m, before.z += c.z & m, before.w += c.w & m;
        }
        reinterpret_cast<uint4 *>(s_stage)[t] = tot;
        reinterpret_cast<uint4 *>(s_stage)[kFewThreads + t] = before;
    }
    for (uint32_t q = t; q < 16 * kRadix; q += kFewThreads) s_cnt[q >> kRadixBits][q & (kRadix - 1)] = 0u;
    __syncthreads();
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (uint32_t r = 0; r < ITEMS; r++) {
        if (r >= rounds) continue;
        const bool valid = first + r * 64 < n;
        const uint32_t d = (mk[r] >> shift) & (kRadix - 1);
        const uint64_t peers = match_digit8(d, valid);
        const uint32_t rank = (uint32_t)__popcll(peers & lt);
        const uint32_t seen = s_cnt[w][d];
        pos[r] = seen + rank;
        if (valid && rank == 0) s_cnt[w][d] = seen + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    uint32_t c[16], sum = 0, dtot = 0, before = 0, all;
    if (t < kRadix) {
#pragma unroll
        for (uint32_t k = 0; k < 16; k++) sum += c[k] = s_cnt[k][t];
#pragma unroll
        for (uint32_t k = 0; k < 16; k++) {
            dtot += s_stage[k * kRadix + t];
            before += s_stage[(16 + k) * kRadix + t];
        }
    }
    uint32_t run = block_excl_scan1024(sum, s_w, &all);
    const uint32_t gstart = block_excl_scan1024(dtot, s_w, &all) + before;
    if (t < kRadix) {
        s_gbase[t] = gstart - run;
#pragma unroll
        for (uint32_t k = 0; k < 16; k++) {
            s_cnt[k][t] = run;
            run += c[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < ITEMS; r++) {
        if (r >= rounds) continue;
        pos[r] += s_cnt[w][(mk[r] >> shift) & (kRadix - 1)];
        if (first + r * 64 < n) s_stage[pos[r]] = mk[r];
    }
    __syncthreads();
    const uint32_t bn = n - base < chunk ? n - base : chunk;
    uint32_t dst[ITEMS];
#pragma unroll
    for (uint32_t r = 0; r < ITEMS; r++) {
        if (r >= rounds) continue;
        const uint32_t p = r * kFewThreads + t;
        if (p < bn) {
            const uint32_t k = s_stage[p];
            dst[r] = s_gbase[(k >> shift) & (kRadix - 1)] + p;
            kout[dst[r]] = k;
        }
    }
    // the payloads take the same permutation through the same staging
    const auto move = [&](const uint32_t *x, uint32_t *out) {
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < ITEMS; r++) {
            if (r >= rounds) continue;
            if (first + r * 64 < n) s_stage[pos[r]] = x[r];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < ITEMS; r++) {
            if (r >= rounds) continue;
            if (r * kFewThreads + t < bn) out[dst[r]] = s_stage[r * kFewThreads + t];
        }
    };
    move(mv, vout);
    if (vout2) move(mv2, vout2);
}

}  // namespace gsr

using namespace gsr;

namespace {

// rows and words of the histogram of a sort of up to cap keys (never fewer words for more keys)
int64_t few_rows(int64_t cap) { return ceil_div(cap, kFewThreads) < kFewRows ? ceil_div(cap, kFewThreads) : kFewRows; }
int64_t hist_words(int64_t cap) {
    cap = cap > 0 ? cap : 1;
    return kRadix * (cap <= kFewSort ? few_rows(cap) : radix_blocks(cap));
}

struct BinWs {
    uint32_t *zk0, *zv0, *zk1, *zv1;  // depth sort ping-pong [VN]
    uint32_t *vis_b, *cnt_b;          // block sums [nb_vn], [VN / 256]
    uint32_t *n_vis;                  // 1
    uint32_t *ik0, *ik1, *iv1, *iw1;  // instance sort [cap]
    uint32_t *tk0, *tk1, *tv1;        // tile-order sort [VT]
    uint32_t *hist;                   // hist_words of the largest sort
    uint32_t *totals;                 // [256]
    size_t bytes;
};

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

BinWs layout(void *base, int64_t VN, int64_t cap, int64_t VT) {
    BinWs w{};
    const int64_t nb_vn = ceil_div(VN > 0 ? VN : 1, kSortTile);
    // the largest sort's histogram
    int64_t hw = hist_words(VN);
    hw = hw > hist_words(cap) ? hw : hist_words(cap);
    hw = hw > hist_words(VT) ? hw : hist_words(VT);
    char *p = static_cast<char *>(base);
    size_t off = 0;
    auto take = [&](size_t words) {
        uint32_t *r = reinterpret_cast<uint32_t *>(p ? p + off : nullptr);
        off += al(words * 4);
        return r;
    };
    w.zk0 = take(VN); w.zv0 = take(VN); w.zk1 = take(VN); w.zv1 = take(VN);
    w.vis_b = take(nb_vn); w.cnt_b = take(ceil_div(VN > 0 ? VN : 1, 256)); w.n_vis = take(1);
    w.ik0 = take(cap); w.ik1 = take(cap); w.iv1 = take(cap); w.iw1 = take(cap);
    w.tk0 = take(VT); w.tk1 = take(VT); w.tv1 = take(VT);
    w.hist = take((size_t)hw); w.totals = take(kRadix);
    w.bytes = off;
    return w;
}

gsr_status radix_sort(uint32_t *&k, uint32_t *&v, uint32_t *&k2, uint32_t *&v2, const uint32_t *n_dev,
                      uint32_t n_host, uint32_t cap, int bits, uint32_t *hist, uint32_t *totals, hipStream_t st,
                      uint32_t **w = nullptr, uint32_t **w2 = nullptr, bool w_is_position = false) {
    const bool few = cap <= kFewSort;
    const int rows = (int)few_rows(cap), nb = (int)radix_blocks(cap);
    for (int shift = 0; shift < bits; shift += kRadixBits) {
        // w_is_position: the second payload starts as each item's input position, generated by
        // the first pass instead of read
        const uint32_t *win = w && !(w_is_position && shift == 0) ? *w : nullptr;
        if (few) {
            k_few_hist<<<rows, kFewThreads, 0, st>>>(k, n_dev, n_host, cap, shift, hist);
            const auto pass = cap <= kFewThreads * kFewRows * 4 ? k_few_pass<4> : k_few_pass<kFewItems>;
            pass<<<rows, kFewThreads, 0, st>>>(k, v, k2, v2, win, w ? *w2 : nullptr, n_dev, n_host, cap, shift, hist);
        } else {
            k_radix_hist<<<nb, kSortThreads, 0, st>>>(k, n_dev, n_host, cap, shift, nb, hist);
            k_radix_scan_rows<<<kRadix, 256, 0, st>>>(hist, nb, totals, n_dev, n_host, cap);
            k_radix_scatter<<<nb, kSortThreads, 0, st>>>(k, v, k2, v2, win, w ? *w2 : nullptr, n_dev, n_host, cap,
                                                         shift, nb, hist, totals);
        }
        uint32_t *tk = k, *tv = v;
        k = k2; v = v2; k2 = tk; v2 = tv;
        if (w) {
            uint32_t *tw = *w;
            *w = *w2;
            *w2 = tw;
        }
    }
    return last_launch();
}

int bit_length(uint64_t x) {
    int b = 0;
    while (x) { b++; x >>= 1; }
    return b;
}

}  // namespace

extern "C" size_t gsr_bin_sort_ws_bytes(int64_t VN, int64_t cap, int64_t VT) { return layout(nullptr, VN, cap, VT).bytes; }

extern "C" gsr_status gsr_bin_sort_launch(uint32_t *info, int64_t n, int V, int ntx, int nty,
                                          uint32_t *inst_gid, const gsr_emission *em, int64_t cap,
                                          uint32_t *ranges, uint32_t *n_inst, uint32_t *tile_order, void *ws,
                                          hipStream_t st) {
    const int64_t VN = (int64_t)V * n;
    const uint32_t T = (uint32_t)(ntx * nty);
    const int64_t VT = (int64_t)V * T;
    BinWs w = layout(ws, VN, cap, VT);
    const int nb_vn = (int)ceil_div(VN > 0 ? VN : 1, kSortTile), nb_p = (int)ceil_div(VN > 0 ? VN : 1, 256);
    const uint32_t capv = (uint32_t)(VN > 0 ? VN : 1);
    // block counts few enough for every block to add up those before it (at most eight 4-byte loads per
    // thread); beyond, the quadratic work would outgrow the launch it saves
    const bool self = nb_p <= 2048;
    const bool small = VN <= kSmallSort && 2 * VT <= 4 * kSmallSort;
    uint32_t *k = w.zk0, *v = w.zv0, *k2 = w.zk1, *v2 = w.zv1;
    gsr_status s;
    if (small) {
        k_bin_small<<<1, kSmallThreads, 0, st>>>(info, (uint32_t)VN, v, w.cnt_b, w.n_vis, n_inst, ranges,
                                                 (uint32_t)(2 * VT));
    } else {
        // 1. ordered compaction of visible pairs: keys = depth bits, values = v*n + i
        k_vis_count<<<nb_vn, 256, 0, st>>>(info, (uint32_t)VN, w.vis_b, ranges, (uint32_t)(2 * VT));
        if (self) {
            k_vis_compact<true><<<nb_vn, 256, 0, st>>>(info, (uint32_t)VN, w.vis_b, w.zk0, w.zv0, w.n_vis);
        } else {
            k_scan_small<<<1, 1024, 0, st>>>(w.vis_b, nb_vn, w.n_vis);
            k_vis_compact<false><<<nb_vn, 256, 0, st>>>(info, (uint32_t)VN, w.vis_b, w.zk0, w.zv0, w.n_vis);
        }
        // 2. stable sort by depth bits (32 bits, 4 passes: result back in zk0 / zv0)
        s = radix_sort(k, v, k2, v2, w.n_vis, 0, capv, 32, w.hist, w.totals, st);
        if (s != GSR_OK) return s;
        // 3. instance counts in depth order, scan, emission
        k_inst_count<<<nb_p < 4096 ? nb_p : 4096, 256, 0, st>>>(v, w.n_vis, capv, info, w.cnt_b);
        if (!self) k_scan_small<<<1, 1024, 0, st>>>(w.cnt_b, nb_p, n_inst, w.n_vis, 256u);
    }
    // the instance sort runs ceil(bits/8) passes; emit into the buffer that makes the last
    // pass land in the sorted-values output (inst_emit when asked for, else inst_gid)
    const int tbits = bit_length((uint64_t)V * T - 1) > 0 ? bit_length((uint64_t)V * T - 1) : 1;
    const int passes = (tbits + kRadixBits - 1) / kRadixBits;
    uint32_t *ek = w.ik0, *ev = (passes % 2 == 0) ? inst_gid : w.iv1;
    uint32_t *ok = w.ik1, *ov = (passes % 2 == 0) ? w.iv1 : inst_gid;
    uint32_t *inst_emit = em ? em->inst_emit : nullptr;
    uint32_t *ew = inst_emit ? ((passes % 2 == 0) ? inst_emit : w.iw1) : nullptr;
    uint32_t *ow = inst_emit ? ((passes % 2 == 0) ? w.iw1 : inst_emit) : nullptr;
    // (the small path has scanned the offsets)
    const auto emit = self && !small ? k_inst_emit<true> : k_inst_emit<false>;
    const int extra = (int)((nb_p < (int)kSplitPairs ? nb_p : (int)kSplitPairs) * (kEmitSplit - 1));
    emit<<<nb_p + extra, 256, 0, st>>>(v, w.n_vis, capv, info, (uint32_t)VN, (uint32_t)n, T, (uint32_t)ntx, w.cnt_b, ek, ev,
                               em ? em->pair_gid : nullptr, em ? em->pair_first : nullptr, em ? em->n_pairs : nullptr,
                               n_inst, (uint32_t)cap, (uint32_t)nb_p);
    // 4. stable sort by view-tile (carrying the emission index along when asked for)
    s = radix_sort(ek, ev, ok, ov, n_inst, 0, (uint32_t)cap, passes * kRadixBits, w.hist, w.totals, st,
                   inst_emit ? &ew : nullptr, inst_emit ? &ow : nullptr, true);
    if (s != GSR_OK) return s;
    // 5. per view-tile [start, end), or an empty frame when the instances do not fit
    const int nr = (int)(ceil_div(cap, 256) < 8192 ? ceil_div(cap, 256) : 8192);
    k_tile_ranges<<<nr, 256, 0, st>>>(ek, n_inst, (uint32_t)cap, ranges, info, (uint32_t)VN, em ? em->n_pairs : nullptr);
    // 6. longest-processing-time order of the view-tiles (descending instance count, to 1/16 of
    // an octave): one 8-bit pass, whose values land in tile_order
    if (tile_order && VT <= kSmallSort) {
        k_tile_order_small<<<1, kSmallThreads, 0, st>>>(ranges, (uint32_t)VT, tile_order);
    } else if (tile_order) {
        const int nt = (int)(ceil_div(VT, 256) < 4096 ? ceil_div(VT, 256) : 4096);
        k_tile_keys<<<nt, 256, 0, st>>>(ranges, (uint32_t)VT, w.tk0, w.tv1);
        uint32_t *a = w.tk0, *b = w.tv1, *c = w.tk1, *d = tile_order;
        s = radix_sort(a, b, c, d, nullptr, (uint32_t)VT, (uint32_t)VT, 8, w.hist, w.totals, st);
        if (s != GSR_OK) return s;
    }
    return last_launch();
}

extern "C" gsr_status gsr_fill_u32_launch(void *dst, uint32_t value, int64_t n, hipStream_t st) {
    if (n <= 0) return GSR_OK;
    const int nb = (int)(ceil_div(n, 256) < 8192 ? ceil_div(n, 256) : 8192);
    k_fill_u32<<<nb, 256, 0, st>>>(static_cast<uint32_t *>(dst), value, n);
    return last_launch();
}

__global__ void k_iota_u32(uint32_t *__restrict__ dst, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = (uint32_t)i;
}

extern "C" gsr_status gsr_tile_order_identity(uint32_t *dst, int64_t n, hipStream_t st) {
    if (n <= 0) return GSR_OK;
    const int nb = (int)(ceil_div(n, 256) < 4096 ? ceil_div(n, 256) : 4096);
    k_iota_u32<<<nb, 256, 0, st>>>(dst, n);
    return last_launch();
}

extern "C" size_t gsr_scan_ws_bytes(int64_t n) { return (size_t)(ceil_div(n > 0 ? n : 1, kSortTile) * 4 + 256); }

// out[i] = sum of in[0..i) (in and out may not alias), *total = sum of all; ws: gsr_scan_ws_bytes.
extern "C" gsr_status gsr_scan_launch(const uint32_t *in, int64_t n, uint32_t *out, uint32_t *total, void *ws,
                                      hipStream_t st) {
    if (n <= 0) return gsr_fill_u32_launch(total, 0u, 1, st);
    const int nb = (int)ceil_div(n, kSortTile);
    uint32_t *bsum = static_cast<uint32_t *>(ws);
    k_scan_sum<<<nb, 256, 0, st>>>(in, n, bsum);
    k_scan_small<<<1, 1024, 0, st>>>(bsum, nb, total);
    k_scan_write<<<nb, 256, 0, st>>>(in, n, bsum, out);
    return last_launch();
}

// Stable LSD radix sort of n (key, value) pairs by the low `bits` key bits (host-side count),
// ping-ponging between (k, v) and (k2, v2): the result is in (k, v) when ceil(bits / 8) is even,
// else in (k2, v2).  ws: gsr_sort_pairs_ws_bytes(n).
extern "C" size_t gsr_sort_pairs_ws_bytes(int64_t n) {
    return (size_t)(hist_words(n) * 4 + kRadix * 4 + 512);
}

// The histogram in a sort's workspace: k_few_pass reads its rows 16 bytes at a time (the 512 spare bytes leave room).
static uint32_t *sort_hist(void *ws) {
    return reinterpret_cast<uint32_t *>((reinterpret_cast<uintptr_t>(ws) + 15) & ~(uintptr_t)15);
}

// As gsr_sort_pairs_launch with the count read on the device (*n_dev, at most cap).
extern "C" gsr_status gsr_sort_pairs_dev_launch(uint32_t *k, uint32_t *v, uint32_t *k2, uint32_t *v2,
                                                const uint32_t *n_dev, uint32_t cap, int bits, void *ws,
                                                hipStream_t st) {
    if (cap == 0) return GSR_OK;
    uint32_t *hist = sort_hist(ws);
    uint32_t *totals = hist + (size_t)hist_words(cap);
    return radix_sort(k, v, k2, v2, n_dev, cap, cap, bits, hist, totals, st);
}

extern "C" gsr_status gsr_sort_pairs_launch(uint32_t *k, uint32_t *v, uint32_t *k2, uint32_t *v2, uint32_t n, int bits,
                                            void *ws, hipStream_t st) {
    if (n == 0) return GSR_OK;
    uint32_t *hist = sort_hist(ws);
    uint32_t *totals = hist + (size_t)hist_words(n);
    return radix_sort(k, v, k2, v2, nullptr, n, n, bits, hist, totals, st);
}


// Stable LSD radix sort of n keys by their low `bits`, carrying a payload v and the items' input
// positions w: k[0], v[0] in, k[1], v[1], w[0], w[1] buffers; on return [0] of each is the result.
extern "C" gsr_status gsr_sort_positions_launch(uint32_t *k[2], uint32_t *v[2], uint32_t *w[2], uint32_t n, int bits,
                                                void *ws, hipStream_t st) {
    if (n == 0) return GSR_OK;
    uint32_t *hist = sort_hist(ws);
    uint32_t *totals = hist + (size_t)hist_words(n);
    return radix_sort(k[0], v[0], k[1], v[1], nullptr, n, n, bits, hist, totals, st, &w[0], &w[1], true);
}

// v[0 .. nb) replaced by its exclusive prefix sums, *total their sum (one block).
extern "C" gsr_status gsr_exclusive_scan_small_launch(uint32_t *v, int nb, uint32_t *total, hipStream_t st) {
    k_scan_small<<<1, 1024, 0, st>>>(v, nb, total);
    return last_launch();
}
