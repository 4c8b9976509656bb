// Gaussian-based loop registration (Sec. III-D, Eq. 13-16).
//
// Prepare: the source set (the loopframe's segment) and the target set of Eq. 13 (Gaussians that
// some query keyframe sees inside its image with its centre within d_max) are flagged per row and
// compacted in row order; every listed Gaussian gets its planar regularised covariance (eigenvalues
// replaced by 1, 1, 1e-3, the small one on the smallest-scale axis: I - 0.999 a a^T); the target
// means go into a hashed cell grid of edge slightly above d_corr.
//
// Iterate (Gauss-Newton, all on the device): sixteen lanes per source Gaussian move its mean by the
// current pose and find the nearest target mean within d_corr among the 27 neighbouring cells; one
// lane then forms r = mu_n - q, C = S_n + R S_m R^T, W = C^-1 and J = [-I, [q]x], and accumulates
// J^T W J, J^T W r, r^T W r and |r|^2 in float64.  Blocks write partials; one block adds them in a
// fixed order, solves the 6x6 system by Cholesky and applies the left update (R, t) <- (Exp(phi) R,
// Exp(phi) t + rho).  Converged or failed iterations turn the remaining launches into no-ops, so a
// fixed number of iterations can be queued without host round trips.
//
// The geometric decisions (frustum test, distances, nearest neighbour) use float64 operations
// rounded one by one in a stated order, so another implementation can reproduce them exactly.
#include "grid.h"

extern "C" gsr_status gsr_scan_launch(const uint32_t *, int64_t, uint32_t *, uint32_t *, void *, hipStream_t);
extern "C" size_t gsr_scan_ws_bytes(int64_t);
extern "C" size_t gsr_sort_pairs_ws_bytes(int64_t);
extern "C" gsr_status gsr_fill_u32_launch(void *, uint32_t, int64_t, hipStream_t);

namespace gsr {

constexpr int kGicpAcc = 30;  // H (21, upper triangle row-major), g (6), cost, |r|^2, count
enum { kStCost = 27, kStSq = 28, kStCount = 29, kStXi = 30, kStConv = 36, kStIters = 37, kStFailed = 38 };
constexpr int kGicpSub = 9;         // low key bits: Morton index of the 1/8 cell inside the cell
constexpr int kRunSteps = 4;       // runs of a bucket stepped through before it is searched
constexpr int kGicpChunk = 64;     // sources per block and turn
constexpr int kGicpBlocks = 2048;  // most blocks of an iteration: eight per CU
constexpr double kRegSmall = 1e-3;
constexpr double kEpsRho = 2.5e-3, kEpsPhi = 2.5e-4;

__device__ __forceinline__ double dmadd3(double a0, double b0, double a1, double b1, double a2, double b2) {
    // ((a0 b0 + a1 b1) + a2 b2), each operation rounded
    return __dadd_rn(__dadd_rn(__dmul_rn(a0, b0), __dmul_rn(a1, b1)), __dmul_rn(a2, b2));
}

__global__ void k_gicp_flags(const float *__restrict__ means, const int32_t *__restrict__ seg, int64_t n,
                             int32_t src_segment, const gsr_camera *__restrict__ cams, int n_cams, double dd_max,
                             uint32_t *__restrict__ f_src, uint32_t *__restrict__ f_tgt) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const bool src = seg[i] == src_segment;
    bool tgt = false;
    const double mx = means[i], my = means[n + i], mz = means[2 * n + i];
    for (int k = 0; k < n_cams && !src && !tgt; k++) {
        const gsr_camera &c = cams[k];
        double R[9], t[3];
        for (int e = 0; e < 9; e++) R[e] = c.R[e];
        for (int e = 0; e < 3; e++) t[e] = c.t[e];
        const double x = __dadd_rn(dmadd3(R[0], mx, R[1], my, R[2], mz), t[0]);
        const double y = __dadd_rn(dmadd3(R[3], mx, R[4], my, R[5], mz), t[1]);
        const double z = __dadd_rn(dmadd3(R[6], mx, R[7], my, R[8], mz), t[2]);
        if (!(z > (double)c.z_near)) continue;
        const double u = __dadd_rn(__dmul_rn((double)c.fx, __ddiv_rn(x, z)), (double)c.cx);
        const double v = __dadd_rn(__dmul_rn((double)c.fy, __ddiv_rn(y, z)), (double)c.cy);
        if (!(u >= 0.0 && u < (double)c.width && v >= 0.0 && v < (double)c.height)) continue;
        // centre -R^T t
        const double cx = -dmadd3(R[0], t[0], R[3], t[1], R[6], t[2]);
        const double cy = -dmadd3(R[1], t[0], R[4], t[1], R[7], t[2]);
        const double cz = -dmadd3(R[2], t[0], R[5], t[1], R[8], t[2]);
        tgt = sqdist_rn(mx, my, mz, cx, cy, cz) < dd_max;
    }
    f_src[i] = src ? 1u : 0u;
    f_tgt[i] = tgt ? 1u : 0u;
}

__global__ void k_gicp_compact(const uint32_t *__restrict__ flag, const uint32_t *__restrict__ off, int64_t n,
                               uint32_t *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && flag[i]) out[off[i]] = (uint32_t)i;
}

// cov [6][cap] (xx, xy, xz, yy, yz, zz) of the listed Gaussians
__global__ void k_gicp_cov(const uint32_t *__restrict__ list, const uint32_t *__restrict__ count, int64_t cap,
                           const float *__restrict__ quats, const float *__restrict__ log_scales, int64_t n,
                           double *__restrict__ cov) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= (int64_t)*count || j >= cap) return;
    const int64_t i = list[j];
    double w = quats[i], x = quats[n + i], y = quats[2 * n + i], z = quats[3 * n + i];
    const double inv = 1.0 / sqrt(w * w + x * x + y * y + z * z);
    w *= inv, x *= inv, y *= inv, z *= inv;
    const float s0 = log_scales[i], s1 = log_scales[n + i], s2 = log_scales[2 * n + i];
    const int a = (s1 < s0 && s1 <= s2) ? 1 : ((s2 < s0 && s2 < s1) ? 2 : 0);  // first smallest
    double ax, ay, az;  // column a of the rotation
    if (a == 0) ax = 1 - 2 * (y * y + z * z), ay = 2 * (x * y + w * z), az = 2 * (x * z - w * y);
    else if (a == 1) ax = 2 * (x * y - w * z), ay = 1 - 2 * (x * x + z * z), az = 2 * (y * z + w * x);
    else ax = 2 * (x * z + w * y), ay = 2 * (y * z - w * x), az = 1 - 2 * (x * x + y * y);
    const double k = 1.0 - kRegSmall;
    cov[j] = 1.0 - k * ax * ax;
    cov[cap + j] = -k * ax * ay;
    cov[2 * cap + j] = -k * ax * az;
    cov[3 * cap + j] = 1.0 - k * ay * ay;
    cov[4 * cap + j] = -k * ay * az;
    cov[5 * cap + j] = 1.0 - k * az * az;
}

// Smallest box of 16 (and of 256) consecutive target means in grid order.
struct Box {
    float4 lo, hi;
};

// Target means in grid order (x, y, z as float, list position as bits), so that a probe scans a
// cell's candidates contiguously instead of gathering them through two index arrays, with the
// boxes of every 16 and every 256 of them (a block's 256).  The first entry of every cell's run
// also gets the run's end, so that a probe steps through a bucket run by run.
__global__ __launch_bounds__(256) void k_gicp_grid_points(
    const float *__restrict__ means, int64_t n, const uint32_t *__restrict__ tgt_list,
    const uint32_t *__restrict__ counts, const uint32_t *__restrict__ key, const uint32_t *__restrict__ val,
    const uint32_t *__restrict__ bucket, float4 *__restrict__ gp, Box *__restrict__ box16, Box *__restrict__ box256,
    uint32_t *__restrict__ run_end) {
    __shared__ Box s_box[16];
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, cnt = counts[1];
    if ((int64_t)blockIdx.x * blockDim.x >= cnt) return;
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (e < cnt) {
        const uint32_t p = val[e];
        const int64_t i = tgt_list[p];
        for (int a = 0; a < 3; a++) v[a] = v[3 + a] = means[a * n + i];
        gp[e] = make_float4(v[0], v[1], v[2], __uint_as_float(p));
        const uint32_t h = key[e] >> kGicpSub;
        if (e == 0 || key[e - 1] >> kGicpSub != h) {
            uint32_t lo = (uint32_t)e + 1, hi = bucket[(key[e] >> (32 - kBucketBits)) + 1];
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (key[mid] >> kGicpSub == h) lo = mid + 1;
                else hi = mid;
            }
            run_end[e] = lo;
        }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1)
        for (int a = 0; a < 3; a++) {
            v[a] = fminf(v[a], __shfl_xor(v[a], off));
            v[3 + a] = fmaxf(v[3 + a], __shfl_xor(v[3 + a], off));
        }
    if ((threadIdx.x & 15) == 0) {
        const Box b = {make_float4(v[0], v[1], v[2], 0.f), make_float4(v[3], v[4], v[5], 0.f)};
        s_box[threadIdx.x >> 4] = b;
        if (e < cnt) box16[e >> 4] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        Box b = s_box[0];
        for (int k = 1; k < 16; k++) {
            const Box o = s_box[k];
            b.lo = make_float4(fminf(b.lo.x, o.lo.x), fminf(b.lo.y, o.lo.y), fminf(b.lo.z, o.lo.z), 0.f);
            b.hi = make_float4(fmaxf(b.hi.x, o.hi.x), fmaxf(b.hi.y, o.hi.y), fmaxf(b.hi.z, o.hi.z), 0.f);
        }
        box256[blockIdx.x] = b;
    }
}

__device__ __forceinline__ int tri(int i, int j) { return i * 6 - i * (i - 1) / 2 + (j - i); }  // i <= j

__device__ __forceinline__ bool gicp_stopped(const double *stats) {
    return stats[kStConv] != 0.0 || stats[kStFailed] != 0.0;
}

// Nearest target of sixteen lanes' common query q, strictly within sqrt(dd_corr), ties to the
// lowest list position (0xFFFFFFFF: none).  Every lane looks up two of the 27 cells around q (its
// own first, then faces, edges and corners), so the dependent loads of the lookups overlap; a lookup
// steps through its bucket run by run, which finds a crowded cell among few at once, and searches it
// beyond kRunSteps runs (1.4M targets in cells of their own, 22 to a bucket: an iteration takes 218 us
// so, 320 by steps alone and 130 by search alone, but with 240k in crowded cells the search alone costs a registration 40 of 713); the
// lanes then share each cell's candidates.  A LiDAR map holds thousands of means in the cells near
// a sensor, so candidates are tested by boxes of 256, of 16 and one by one (inside a cell they are
// in Morton order of 1/8 cells, so the boxes are small), starting from the closest box.  What lies
// farther than the best candidate so far is skipped.  A box's distance is computed with the same
// rounded operations as its candidates' and each is monotone, so it never exceeds theirs; a cell's
// is taken a micrometre (and the rounding of the coordinates) short.  No tie is lost.
__constant__ int8_t kCellOrder[27][3] = {
    {0, 0, 0},   {-1, 0, 0},  {1, 0, 0},   {0, -1, 0},  {0, 1, 0},   {0, 0, -1},  {0, 0, 1},   {-1, -1, 0}, {1, -1, 0},
    {-1, 1, 0},  {1, 1, 0},   {-1, 0, -1}, {1, 0, -1},  {-1, 0, 1},  {1, 0, 1},   {0, -1, -1}, {0, 1, -1},  {0, -1, 1},
    {0, 1, 1},   {-1, -1, -1}, {1, -1, -1}, {-1, 1, -1}, {1, 1, -1},  {-1, -1, 1}, {1, -1, 1},  {-1, 1, 1},  {1, 1, 1}};

struct GicpGrid {
    const uint32_t *key, *bucket, *run_end;
    const float4 *gp;
    const Box *box16, *box256;
    double cell, inv_cell;
};

__device__ __forceinline__ double box_gap(int o, double x, int64_t c, double cell, double slack) {
    const double g = o < 0 ? x - (double)c * cell : (double)(c + 1) * cell - x;
    return o == 0 || !(g > slack) ? 0.0 : g - slack;
}

// squared distance of q to a box (0 inside), the operations of sqdist_rn
__device__ __forceinline__ double box_sqdist(const Box *__restrict__ p, const double q[3]) {
    const Box b = *p;
    const double dx = fmax(fmax(__dsub_rn(b.lo.x, q[0]), __dsub_rn(q[0], b.hi.x)), 0.0);
    const double dy = fmax(fmax(__dsub_rn(b.lo.y, q[1]), __dsub_rn(q[1], b.hi.y)), 0.0);
    const double dz = fmax(fmax(__dsub_rn(b.lo.z, q[2]), __dsub_rn(q[2], b.hi.z)), 0.0);
    return __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
}

// One query's search state, the same in its sixteen lanes but for (best, bi) between two merges.
struct Nearest {
    const GicpGrid &g;
    const double *q;
    double best;
    uint32_t bi;
    int sub, sh;  // lane in the group, the group's first lane in the wave

    __device__ __forceinline__ uint32_t group(bool v) const { return (uint32_t)(__ballot(v) >> sh) & 0xFFFFu; }
    __device__ __forceinline__ void test(uint32_t i) {
        const float4 a = g.gp[i];
        const double d = sqdist_rn(a.x, a.y, a.z, q[0], q[1], q[2]);
        const uint32_t p = __float_as_uint(a.w);
        if (d < best || (d == best && p < bi && bi != 0xFFFFFFFFu)) best = d, bi = p;
    }
    __device__ __forceinline__ void merge() {
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) {
            const double ob = __shfl_xor(best, off);
            const uint32_t oi = __shfl_xor(bi, off);
            if (ob < best || (ob == best && oi < bi)) best = ob, bi = oi;
        }
    }
    // the closest of the boxes [b, e), the first on ties
    __device__ __forceinline__ uint32_t closest(const Box *__restrict__ boxes, uint32_t b, uint32_t e) const {
        double d = INFINITY;
        uint32_t at = b;
        for (uint32_t k = b + sub; k < e; k += 16) {
            const double dk = box_sqdist(boxes + k, q);
            if (dk < d) d = dk, at = k;
        }
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) {
            const double od = __shfl_xor(d, off);
            const uint32_t oa = __shfl_xor(at, off);
            if (od < d || (od == d && oa < at)) d = od, at = oa;
        }
        return at;
    }
    // candidates [s, e) of one cell
    __device__ __forceinline__ void cell(uint32_t s, uint32_t e) {
        if (e - s <= 64) {
            for (uint32_t i = s + sub; i < e; i += 16) test(i);
            merge();
            return;
        }
        const uint32_t b0 = s >> 4, b1 = ((e - 1) >> 4) + 1, c1 = ((e - 1) >> 8) + 1;
        if (bi == 0xFFFFFFFFu) {  // a first bound from the closest box of the closest 256
            const uint32_t c = closest(g.box256, s >> 8, c1);
            const uint32_t k = closest(g.box16, max(c * 16, b0), min(c * 16 + 16, b1)) * 16 + sub;
            if (k >= s && k < e) test(k);
            merge();
        }
        for (uint32_t c = s >> 8; c < c1; c += 16) {
            uint32_t open = group(c + sub < c1 && box_sqdist(g.box256 + min(c + sub, c1 - 1), q) <= best);
            while (open) {
                const uint32_t b = (c + __builtin_ctz(open)) * 16 + sub;
                open &= open - 1;
                uint32_t hit = group(b >= b0 && b < b1 && box_sqdist(g.box16 + min(max(b, b0), b1 - 1), q) <= best);
                if (!hit) continue;
                while (hit) {
                    const uint32_t k = (b - sub + __builtin_ctz(hit)) * 16 + sub;
                    hit &= hit - 1;
                    if (k >= s && k < e) test(k);
                }
                merge();
            }
        }
    }
};

__device__ __forceinline__ uint32_t gicp_nearest(const double q[3], const GicpGrid &g, double dd_corr) {
    const int lane = lane_id(), sub = lane & 15, sh = lane & 48;
    const int64_t c[3] = {cell_of(q[0], g.inv_cell), cell_of(q[1], g.inv_cell), cell_of(q[2], g.inv_cell)};
    const double slack = 1e-6 + 1e-12 * fmax(fabs(q[0]), fmax(fabs(q[1]), fabs(q[2])));
    uint32_t first[2], last[2];
    float gap[2];
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const int slot = sub + 16 * k;
        first[k] = last[k] = 0;
        gap[k] = 0.f;
        if (slot < 27) {
            const int o0 = kCellOrder[slot][0], o1 = kCellOrder[slot][1], o2 = kCellOrder[slot][2];
            const uint32_t hash = cell_hash(c[0] + o0, c[1] + o1, c[2] + o2), h = hash >> kGicpSub;
            uint32_t e = g.bucket[hash >> (32 - kBucketBits)];
            const uint32_t hi = g.bucket[(hash >> (32 - kBucketBits)) + 1];
            auto at = [&](uint32_t i) { return i < hi ? g.key[i] >> kGicpSub : 0xFFFFFFFFu; };
            uint32_t ke = at(e);
            for (int r = 0; ke < h; r++) {
                if (r < kRunSteps) {
                    e = g.run_end[e];
                } else {  // the first entry of hash h or above lies in (e, hi]
                    uint32_t top = hi;
                    while (top - e > 1) {
                        const uint32_t mid = (e + top) >> 1;
                        if (g.key[mid] >> kGicpSub < h) e = mid;
                        else top = mid;
                    }
                    e = top;
                }
                ke = at(e);
            }
            if (ke == h) first[k] = e, last[k] = g.run_end[e];
            const double gx = box_gap(o0, q[0], c[0], g.cell, slack), gy = box_gap(o1, q[1], c[1], g.cell, slack),
                         gz = box_gap(o2, q[2], c[2], g.cell, slack);
            gap[k] = (float)((gx * gx + gy * gy + gz * gz) * (1.0 - 1e-6));
        }
    }
    Nearest s{g, q, dd_corr, 0xFFFFFFFFu, sub, sh};
    // the nearest-first cells that are not empty, not visited and not farther than the best so far
    uint32_t left = 0x7FFFFFFu;
    for (;;) {  // every turn clears at least one of the 27 bits
        const uint32_t cells = (s.group(last[0] > first[0] && (double)gap[0] <= s.best) |
                                s.group(last[1] > first[1] && (double)gap[1] <= s.best) << 16) & left;
        if (!cells) break;
        const int k = __builtin_ctz(cells);
        left &= ~0u << k << 1;
        const int from = sh | (k & 15);
        s.cell(__shfl(k < 16 ? first[0] : first[1], from), __shfl(k < 16 ? last[0] : last[1], from));
    }
    return s.bi;
}

// Adds the 64 pairs of a wave (lane = source position j, bi = its target position or none) to
// s_sum: H, g, cost, |r|^2 and the count of Eq. 16 linearised at (R, t).
__device__ __forceinline__ void gicp_pair_sums(uint32_t bi, int64_t j, const float *__restrict__ means, int64_t n,
                                               const uint32_t *__restrict__ src_list,
                                               const uint32_t *__restrict__ tgt_list,
                                               const double *__restrict__ src_cov,
                                               const double *__restrict__ tgt_cov, int64_t cap, const double R[9],
                                               const double t[3], double *s_sum) {
    if (__ballot(bi != 0xFFFFFFFFu) == 0) return;  // most chunks lie outside the overlap
    double acc[kGicpAcc];
#pragma unroll
    for (int e = 0; e < kGicpAcc; e++) acc[e] = 0.0;
    if (bi != 0xFFFFFFFFu) {
        const int64_t i = src_list[j];
        const double mx = means[i], my = means[n + i], mz = means[2 * n + i];
        const double q[3] = {__dadd_rn(dmadd3(R[0], mx, R[1], my, R[2], mz), t[0]),
                             __dadd_rn(dmadd3(R[3], mx, R[4], my, R[5], mz), t[1]),
                             __dadd_rn(dmadd3(R[6], mx, R[7], my, R[8], mz), t[2])};
        const int64_t it = tgt_list[bi];
        const double r[3] = {means[it] - q[0], means[n + it] - q[1], means[2 * n + it] - q[2]};
        // C = S_n + R S_m R^T
        const double Sm[9] = {src_cov[j], src_cov[cap + j], src_cov[2 * cap + j],
                              src_cov[cap + j], src_cov[3 * cap + j], src_cov[4 * cap + j],
                              src_cov[2 * cap + j], src_cov[4 * cap + j], src_cov[5 * cap + j]};
        double RS[9], C[9];
        for (int a = 0; a < 3; a++)
            for (int b = 0; b < 3; b++)
                RS[3 * a + b] = R[3 * a] * Sm[b] + R[3 * a + 1] * Sm[3 + b] + R[3 * a + 2] * Sm[6 + b];
        for (int a = 0; a < 3; a++)
            for (int b = 0; b < 3; b++)
                C[3 * a + b] = RS[3 * a] * R[3 * b] + RS[3 * a + 1] * R[3 * b + 1] + RS[3 * a + 2] * R[3 * b + 2];
        const int64_t pb = bi;
        C[0] += tgt_cov[pb], C[1] += tgt_cov[cap + pb], C[2] += tgt_cov[2 * cap + pb];
        C[3] += tgt_cov[cap + pb], C[4] += tgt_cov[3 * cap + pb], C[5] += tgt_cov[4 * cap + pb];
        C[6] += tgt_cov[2 * cap + pb], C[7] += tgt_cov[4 * cap + pb], C[8] += tgt_cov[5 * cap + pb];
        // W = C^-1 (adjugate over determinant)
        double W[9];
        W[0] = C[4] * C[8] - C[5] * C[7];
        W[1] = C[2] * C[7] - C[1] * C[8];
        W[2] = C[1] * C[5] - C[2] * C[4];
        W[3] = C[5] * C[6] - C[3] * C[8];
        W[4] = C[0] * C[8] - C[2] * C[6];
        W[5] = C[2] * C[3] - C[0] * C[5];
        W[6] = C[3] * C[7] - C[4] * C[6];
        W[7] = C[1] * C[6] - C[0] * C[7];
        W[8] = C[0] * C[4] - C[1] * C[3];
        const double id = 1.0 / (C[0] * W[0] + C[1] * W[3] + C[2] * W[6]);
        for (int e = 0; e < 9; e++) W[e] *= id;
        // J = [-I, [q]x]: column c of J
        double J[3][6];
        for (int a = 0; a < 3; a++)
            for (int b = 0; b < 3; b++) J[a][b] = a == b ? -1.0 : 0.0;
        J[0][3] = 0.0, J[0][4] = -q[2], J[0][5] = q[1];
        J[1][3] = q[2], J[1][4] = 0.0, J[1][5] = -q[0];
        J[2][3] = -q[1], J[2][4] = q[0], J[2][5] = 0.0;
        double WJ[3][6], Wr[3];
        for (int a = 0; a < 3; a++) {
            for (int c = 0; c < 6; c++) WJ[a][c] = W[3 * a] * J[0][c] + W[3 * a + 1] * J[1][c] + W[3 * a + 2] * J[2][c];
            Wr[a] = W[3 * a] * r[0] + W[3 * a + 1] * r[1] + W[3 * a + 2] * r[2];
        }
        for (int a = 0; a < 6; a++) {
            for (int b = a; b < 6; b++) acc[tri(a, b)] = J[0][a] * WJ[0][b] + J[1][a] * WJ[1][b] + J[2][a] * WJ[2][b];
            acc[21 + a] = J[0][a] * Wr[0] + J[1][a] * Wr[1] + J[2][a] * Wr[2];
        }
        acc[kStCost] = r[0] * Wr[0] + r[1] * Wr[1] + r[2] * Wr[2];
        acc[kStSq] = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
        acc[kStCount] = 1.0;
    }
#pragma unroll
    for (int e = 0; e < kGicpAcc; e++) {
        const double v = wave_sum_d(acc[e]);
        if (lane_id() == e) s_sum[e] += v;
    }
}

// One Gauss-Newton iteration.  Each block takes chunks of 64 sources: four passes of sixteen
// sixteen-lane searches, then its first wave linearises the 64 pairs.  The per-block sums go to
// partial[e][block]; k_gicp_solve, a launch of its own, adds them and updates the pose.
//
// The search is bound by the latency of its dependent loads, not by bytes or FLOPs.  One lane per
// source walked 27 cells and every candidate in them one after another, 1.1 waves per SIMD, in 1.46
// ms per iteration at 75k sources and 240k targets, and the sum of 5,859 partials (mostly of empty
// blocks) took another 0.2 ms.
__global__ __launch_bounds__(256) void k_gicp_linearise(
    const float *__restrict__ means, int64_t n, const uint32_t *__restrict__ src_list,
    const uint32_t *__restrict__ tgt_list, const uint32_t *__restrict__ counts, const double *__restrict__ src_cov,
    const double *__restrict__ tgt_cov, int64_t cap, GicpGrid grid, double dd_corr,
    const double *__restrict__ pose, const double *__restrict__ stats, double *__restrict__ partial,
    int32_t *__restrict__ corr) {
    __shared__ uint32_t s_hit[kGicpChunk];
    __shared__ double s_sum[kGicpAcc];
    if (gicp_stopped(stats)) return;
    const int64_t n_src = counts[0];
    const int64_t chunks = (n_src + kGicpChunk - 1) / kGicpChunk;
    if (blockIdx.x >= chunks) return;
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    double R[9], tr[3];
    for (int e = 0; e < 9; e++) R[e] = pose[e];
    for (int e = 0; e < 3; e++) tr[e] = pose[9 + e];
    if (t < kGicpAcc) s_sum[t] = 0.0;
    for (int64_t ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
        for (int p = 0; p < kGicpChunk / 16; p++) {
            const int slot = p * 16 + (t >> 4);
            const int64_t j = slot * chunks + ch;
            uint32_t bi = 0xFFFFFFFFu;
            if (j < n_src) {
                const int64_t i = src_list[j];
                const double mx = means[i], my = means[n + i], mz = means[2 * n + i];
                const double q[3] = {__dadd_rn(dmadd3(R[0], mx, R[1], my, R[2], mz), tr[0]),
                                     __dadd_rn(dmadd3(R[3], mx, R[4], my, R[5], mz), tr[1]),
                                     __dadd_rn(dmadd3(R[6], mx, R[7], my, R[8], mz), tr[2])};
                bi = gicp_nearest(q, grid, dd_corr);
                if (corr && (t & 15) == 0) corr[j] = bi == 0xFFFFFFFFu ? -1 : (int32_t)bi;
            }
            if ((t & 15) == 0) s_hit[slot] = bi;
        }
        __syncthreads();
        if (w == 0) {
            const int64_t j = lane * chunks + ch;
            gicp_pair_sums(s_hit[lane], j, means, n, src_list, tgt_list, src_cov, tgt_cov, cap, R, tr, s_sum);
        }
        __syncthreads();
    }
    if (w == 0 && lane < kGicpAcc) partial[(int64_t)lane * kGicpBlocks + blockIdx.x] = s_sum[lane];
}

__device__ void so3_exp(const double phi[3], double E[9]) {
    const double th2 = phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2];
    const double th = sqrt(th2);
    const double K[9] = {0.0, -phi[2], phi[1], phi[2], 0.0, -phi[0], -phi[1], phi[0], 0.0};
    double a = 1.0, b = 0.0;
    if (th >= 1e-12) {
        a = sin(th) / th;
        b = (1.0 - cos(th)) / th2;
    }
    for (int r = 0; r < 3; r++)
        for (int c = 0; c < 3; c++) {
            const double KK = K[3 * r] * K[c] + K[3 * r + 1] * K[3 + c] + K[3 * r + 2] * K[6 + c];
            E[3 * r + c] = (r == c ? 1.0 : 0.0) + a * K[3 * r + c] + b * KK;
        }
}

// Fixed-order sum of the active blocks' partials, then the Gauss-Newton update of the pose (one
// block).  A launch of its own: counting the blocks off inside the iteration's kernel cost every
// block a write-back of its XCD's L2 (__threadfence), 65 us per iteration more than this launch.
__global__ __launch_bounds__(1024) void k_gicp_solve(const double *__restrict__ partial,
                                                     const uint32_t *__restrict__ counts, int grid,
                                                     double *__restrict__ pose, double *__restrict__ stats) {
    __shared__ double s[kGicpAcc];
    if (gicp_stopped(stats)) return;
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const int64_t chunks = ((int64_t)counts[0] + kGicpChunk - 1) / kGicpChunk;
    const int active = chunks < grid ? (int)chunks : grid;
    for (int e = w; e < kGicpAcc; e += 16) {
        double a = 0.0;
#pragma unroll 4
        for (int b = lane; b < active; b += 64) a += partial[(int64_t)e * kGicpBlocks + b];
        a = wave_sum_d(a);
        if (lane == 0) s[e] = a;
    }
    __syncthreads();
    if (t < kGicpAcc) stats[t] = s[t];
    if (t != 0) return;
    stats[kStIters] += 1.0;
    if (s[kStCount] < 6.0) {
        stats[kStFailed] = 1.0;
        return;
    }
    double H[6][6], L[6][6] = {}, x[6];
    for (int a = 0; a < 6; a++)
        for (int b = a; b < 6; b++) H[a][b] = H[b][a] = s[tri(a, b)];
    // Cholesky H = L L^T, then L y = -g, L^T xi = y
    for (int c = 0; c < 6; c++) {
        double d = H[c][c];
        for (int k = 0; k < c; k++) d -= L[c][k] * L[c][k];
        if (!(d > 0.0)) {
            stats[kStFailed] = 1.0;
            return;
        }
        L[c][c] = sqrt(d);
        for (int r = c + 1; r < 6; r++) {
            double v = H[r][c];
            for (int k = 0; k < c; k++) v -= L[r][k] * L[c][k];
            L[r][c] = v / L[c][c];
        }
    }
    for (int r = 0; r < 6; r++) {
        double v = -s[21 + r];
        for (int k = 0; k < r; k++) v -= L[r][k] * x[k];
        x[r] = v / L[r][r];
    }
    for (int r = 5; r >= 0; r--) {
        double v = x[r];
        for (int k = r + 1; k < 6; k++) v -= L[k][r] * x[k];
        x[r] = v / L[r][r];
    }
    for (int e = 0; e < 6; e++) stats[kStXi + e] = x[e];
    double E[9], R[9], tt[3];
    so3_exp(x + 3, E);
    for (int e = 0; e < 9; e++) R[e] = pose[e];
    for (int e = 0; e < 3; e++) tt[e] = pose[9 + e];
    for (int r = 0; r < 3; r++) {
        for (int c = 0; c < 3; c++) pose[3 * r + c] = E[3 * r] * R[c] + E[3 * r + 1] * R[3 + c] + E[3 * r + 2] * R[6 + c];
        pose[9 + r] = E[3 * r] * tt[0] + E[3 * r + 1] * tt[1] + E[3 * r + 2] * tt[2] + x[r];
    }
    const double nr = sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]);
    const double np = sqrt(x[3] * x[3] + x[4] * x[4] + x[5] * x[5]);
    if (nr < kEpsRho && np < kEpsPhi) stats[kStConv] = 1.0;
}

size_t a256g(size_t b) { return (b + 255) & ~(size_t)255; }

struct GicpWs {
    double *src_cov, *tgt_cov, *partial;
    float4 *gp;
    Box *box16, *box256;
    uint32_t *f_src, *f_tgt, *off, *key, *val, *k2, *v2, *bucket;
    void *scan, *sort;
    size_t bytes;
};

int nblk256(int64_t n) { return (int)ceil_div(n > 0 ? n : 1, 256); }

GicpWs gicp_layout(void *base, int64_t n) {
    GicpWs w;
    char *p = static_cast<char *>(base);
    size_t off = 0;
    auto take = [&](size_t b) {
        void *r = p ? p + off : nullptr;
        off += a256g(b);
        return r;
    };
    const size_t nn = (size_t)(n > 0 ? n : 1);
    w.src_cov = (double *)take(6 * nn * 8);
    w.tgt_cov = (double *)take(6 * nn * 8);
    w.partial = (double *)take((size_t)kGicpBlocks * kGicpAcc * 8);
    w.gp = (float4 *)take(nn * 16);
    w.box16 = (Box *)take((nn / 16 + 1) * sizeof(Box));
    w.box256 = (Box *)take((nn / 256 + 1) * sizeof(Box));
    w.f_src = (uint32_t *)take(nn * 4);
    w.f_tgt = (uint32_t *)take(nn * 4);
    w.off = (uint32_t *)take(nn * 4);
    w.key = (uint32_t *)take(nn * 4);
    w.val = (uint32_t *)take(nn * 4);
    w.k2 = (uint32_t *)take(nn * 4);
    w.v2 = (uint32_t *)take(nn * 4);
    w.bucket = (uint32_t *)take((size_t)(kBuckets + 1) * 4);
    w.scan = take(gsr_scan_ws_bytes(n));
    w.sort = take(gsr_sort_pairs_ws_bytes(n));
    w.bytes = off;
    return w;
}

double grid_cell(float d_corr) { return (double)d_corr * (1.0 + 1.0 / (1 << 20)); }

}  // namespace gsr

using namespace gsr;

extern "C" size_t gsr_gicp_ws_bytes(int64_t n) { return gicp_layout(nullptr, n).bytes; }

extern "C" gsr_status gsr_gicp_prepare_launch(const gsr_gaussians *g, const int32_t *seg, int32_t src_segment,
                                              const gsr_camera *cams, int n_cams, float d_max, float d_corr,
                                              uint32_t *src_index, uint32_t *tgt_index, uint32_t *counts,
                                              double *stats, void *ws, hipStream_t st) {
    const int64_t n = g->n;
    GicpWs w = gicp_layout(ws, n);
    gsr_status s = gsr_fill_u32_launch(stats, 0u, 2 * 40, st);
    if (s != GSR_OK) return s;
    if (n == 0) return gsr_fill_u32_launch(counts, 0u, 2, st);
    const double dd = (double)d_max * (double)d_max;
    k_gicp_flags<<<nblk256(n), 256, 0, st>>>(g->means, seg, n, src_segment, cams, n_cams, dd, w.f_src, w.f_tgt);
    s = gsr_scan_launch(w.f_src, n, w.off, counts, w.scan, st);
    if (s != GSR_OK) return s;
    k_gicp_compact<<<nblk256(n), 256, 0, st>>>(w.f_src, w.off, n, src_index);
    s = gsr_scan_launch(w.f_tgt, n, w.off, counts + 1, w.scan, st);
    if (s != GSR_OK) return s;
    k_gicp_compact<<<nblk256(n), 256, 0, st>>>(w.f_tgt, w.off, n, tgt_index);
    k_gicp_cov<<<nblk256(n), 256, 0, st>>>(src_index, counts, n, g->quats, g->log_scales, n, w.src_cov);
    k_gicp_cov<<<nblk256(n), 256, 0, st>>>(tgt_index, counts + 1, n, g->quats, g->log_scales, n, w.tgt_cov);
    s = gsr_grid_build_launch(g->means, n, tgt_index, counts + 1, n, grid_cell(d_corr), w.key, w.val, w.k2, w.v2,
                              w.bucket, w.sort, kGicpSub, st);
    if (s != GSR_OK) return s;
    // the sort's second key buffer is free again: it takes the run ends
    k_gicp_grid_points<<<nblk256(n), 256, 0, st>>>(g->means, n, tgt_index, counts, w.key, w.val, w.bucket, w.gp,
                                                   w.box16, w.box256, w.k2);
    return last_launch();
}

extern "C" gsr_status gsr_gicp_iterate_launch(const gsr_gaussians *g, const uint32_t *src_index,
                                              const uint32_t *tgt_index, const uint32_t *counts, float d_corr,
                                              double *pose, double *stats, int32_t *corr, int n_iter, void *ws,
                                              hipStream_t st) {
    const int64_t n = g->n;
    if (n == 0) return GSR_OK;
    GicpWs w = gicp_layout(ws, n);
    const double dd = (double)d_corr * (double)d_corr;
    const GicpGrid grid = {w.key, w.bucket, w.k2, w.gp, w.box16, w.box256, grid_cell(d_corr), 1.0 / grid_cell(d_corr)};
    const int64_t chunks = ceil_div(n, kGicpChunk);
    const int nb = (int)(chunks < kGicpBlocks ? chunks : kGicpBlocks);
    for (int it = 0; it < n_iter; it++) {
        k_gicp_linearise<<<nb, 256, 0, st>>>(g->means, n, src_index, tgt_index, counts, w.src_cov, w.tgt_cov, n, grid,
                                             dd, pose, stats, w.partial, corr);
        k_gicp_solve<<<1, 1024, 0, st>>>(w.partial, counts, nb, pose, stats);
    }
    return last_launch();
}

// ---- propagation of a corrected pose to a segment ------------------------------------------------
// The segment moves rigidly by (R, t): means R mu + t, orientations q_R (x) q (so R_q' = R R_q),
// and each SH degree l >= 1 turns with D_l, D_ab = integral of Y_a(d) Y_b(R^T d) over the sphere, so
// that the colour seen along R d afterwards is the colour seen along d before.  The integrand is
// a spherical polynomial of degree <= 6; the product rule of the 4-point Gauss-Legendre rule in
// z = cos(theta) with 8 equally spaced azimuths integrates it exactly.
namespace gsr {

constexpr int kShRotEntries = 9 + 25 + 49;  // D_1, D_2, D_3 row-major, then q_R (w, x, y, z)

// Real orthonormal SH without Condon-Shortley phase, degree <= 3, in float64 (index k = l^2 + l + m)
__device__ double sh_basis_d(int k, double x, double y, double z) {
    const double pi = 3.141592653589793;
    switch (k) {
        case 1: return sqrt(3.0 / (4.0 * pi)) * y;
        case 2: return sqrt(3.0 / (4.0 * pi)) * z;
        case 3: return sqrt(3.0 / (4.0 * pi)) * x;
        case 4: return sqrt(15.0 / (4.0 * pi)) * x * y;
        case 5: return sqrt(15.0 / (4.0 * pi)) * y * z;
        case 6: return sqrt(5.0 / (16.0 * pi)) * (3.0 * z * z - 1.0);
        case 7: return sqrt(15.0 / (4.0 * pi)) * x * z;
        case 8: return sqrt(15.0 / (16.0 * pi)) * (x * x - y * y);
        case 9: return sqrt(35.0 / (32.0 * pi)) * y * (3.0 * x * x - y * y);
        case 10: return sqrt(105.0 / (4.0 * pi)) * x * y * z;
        case 11: return sqrt(21.0 / (32.0 * pi)) * y * (5.0 * z * z - 1.0);
        case 12: return sqrt(7.0 / (16.0 * pi)) * z * (5.0 * z * z - 3.0);
        case 13: return sqrt(21.0 / (32.0 * pi)) * x * (5.0 * z * z - 1.0);
        case 14: return sqrt(105.0 / (16.0 * pi)) * z * (x * x - y * y);
        case 15: return sqrt(35.0 / (32.0 * pi)) * x * (x * x - 3.0 * y * y);
        default: return 0.28209479177387814;
    }
}

__global__ void k_sh_rotation(const double *__restrict__ pose, double *__restrict__ out) {
    const int e = threadIdx.x;
    double R[9];
    for (int i = 0; i < 9; i++) R[i] = pose[i];
    if (e < kShRotEntries) {
        int l, a, b;
        if (e < 9) l = 1, a = e / 3, b = e % 3;
        else if (e < 34) l = 2, a = (e - 9) / 5, b = (e - 9) % 5;
        else l = 3, a = (e - 34) / 7, b = (e - 34) % 7;
        const int ka = l * l + a, kb = l * l + b;
        // 4-point Gauss-Legendre nodes: roots of 35 z^4 - 30 z^2 + 3, weights 2 / ((1 - z^2) P4'(z)^2)
        const double r30 = sqrt(30.0);
        const double zs[2] = {sqrt((15.0 - 2.0 * r30) / 35.0), sqrt((15.0 + 2.0 * r30) / 35.0)};
        const double pi = 3.141592653589793;
        double acc = 0.0;
        for (int zi = 0; zi < 4; zi++) {
            const double z = zi < 2 ? zs[zi] : -zs[zi - 2];
            const double dp = (140.0 * z * z * z - 60.0 * z) / 8.0;  // P4'(z)
            const double wz = 2.0 / ((1.0 - z * z) * dp * dp);
            const double rho = sqrt(1.0 - z * z);
            for (int j = 0; j < 8; j++) {
                const double ph = 2.0 * pi * j / 8.0;
                const double x = rho * cos(ph), y = rho * sin(ph);
                // R^T d
                const double rx = R[0] * x + R[3] * y + R[6] * z;
                const double ry = R[1] * x + R[4] * y + R[7] * z;
                const double rz = R[2] * x + R[5] * y + R[8] * z;
                acc += wz * (2.0 * pi / 8.0) * sh_basis_d(ka, x, y, z) * sh_basis_d(kb, rx, ry, rz);
            }
        }
        out[e] = acc;
    } else if (e == kShRotEntries) {
        // q_R by Shepperd's method, sign with w >= 0
        double w, x, y, z;
        const double tr = R[0] + R[4] + R[8];
        if (tr > 0.0) {
            const double s = 2.0 * sqrt(tr + 1.0);
            w = 0.25 * s, x = (R[7] - R[5]) / s, y = (R[2] - R[6]) / s, z = (R[3] - R[1]) / s;
        } else if (R[0] > R[4] && R[0] > R[8]) {
            const double s = 2.0 * sqrt(1.0 + R[0] - R[4] - R[8]);
            w = (R[7] - R[5]) / s, x = 0.25 * s, y = (R[1] + R[3]) / s, z = (R[2] + R[6]) / s;
        } else if (R[4] > R[8]) {
            const double s = 2.0 * sqrt(1.0 + R[4] - R[0] - R[8]);
            w = (R[2] - R[6]) / s, x = (R[1] + R[3]) / s, y = 0.25 * s, z = (R[5] + R[7]) / s;
        } else {
            const double s = 2.0 * sqrt(1.0 + R[8] - R[0] - R[4]);
            w = (R[3] - R[1]) / s, x = (R[2] + R[6]) / s, y = (R[5] + R[7]) / s, z = 0.25 * s;
        }
        const double sg = w < 0.0 ? -1.0 : 1.0;
        out[kShRotEntries] = sg * w, out[kShRotEntries + 1] = sg * x;
        out[kShRotEntries + 2] = sg * y, out[kShRotEntries + 3] = sg * z;
    }
}

__global__ void k_transform_rows(float *__restrict__ means, float *__restrict__ quats, float *__restrict__ sh,
                                 int64_t n, int deg, const int32_t *__restrict__ seg, int32_t segment,
                                 const double *__restrict__ pose, const double *__restrict__ rot) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || seg[i] != segment) return;
    double R[9], t[3];
    for (int e = 0; e < 9; e++) R[e] = pose[e];
    for (int e = 0; e < 3; e++) t[e] = pose[9 + e];
    const double mx = means[i], my = means[n + i], mz = means[2 * n + i];
    means[i] = (float)(R[0] * mx + R[1] * my + R[2] * mz + t[0]);
    means[n + i] = (float)(R[3] * mx + R[4] * my + R[5] * mz + t[1]);
    means[2 * n + i] = (float)(R[6] * mx + R[7] * my + R[8] * mz + t[2]);
    const double aw = rot[kShRotEntries], ax = rot[kShRotEntries + 1], ay = rot[kShRotEntries + 2],
                 az = rot[kShRotEntries + 3];
    const double bw = quats[i], bx = quats[n + i], by = quats[2 * n + i], bz = quats[3 * n + i];
    quats[i] = (float)(aw * bw - ax * bx - ay * by - az * bz);
    quats[n + i] = (float)(aw * bx + ax * bw + ay * bz - az * by);
    quats[2 * n + i] = (float)(aw * by - ax * bz + ay * bw + az * bx);
    quats[3 * n + i] = (float)(aw * bz + ax * by - ay * bx + az * bw);
    int off = 0;
    for (int l = 1; l <= deg; l++) {
        const int w = 2 * l + 1;
        const double *D = rot + off;
        for (int ch = 0; ch < 3; ch++) {
            double c[7], o[7];
            for (int b = 0; b < w; b++) c[b] = sh[(int64_t)((l * l + b) * 3 + ch) * n + i];
            for (int a = 0; a < w; a++) {
                double v = 0.0;
                for (int b = 0; b < w; b++) v += D[a * w + b] * c[b];
                o[a] = v;
            }
            for (int a = 0; a < w; a++) sh[(int64_t)((l * l + a) * 3 + ch) * n + i] = (float)o[a];
        }
        off += w * w;
    }
}

// world -> camera of a moved segment: R_c R^T, t_c - R_c R^T t
__global__ void k_transform_cams(gsr_camera *__restrict__ cams, int n_cams, const uint8_t *__restrict__ mask,
                                 const double *__restrict__ pose) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_cams || (mask && !mask[k])) return;
    double R[9], t[3], Rc[9], tc[3], M[9];
    for (int e = 0; e < 9; e++) R[e] = pose[e], Rc[e] = cams[k].R[e];
    for (int e = 0; e < 3; e++) t[e] = pose[9 + e], tc[e] = cams[k].t[e];
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) M[3 * a + b] = Rc[3 * a] * R[3 * b] + Rc[3 * a + 1] * R[3 * b + 1] + Rc[3 * a + 2] * R[3 * b + 2];
    for (int e = 0; e < 9; e++) cams[k].R[e] = (float)M[e];
    for (int a = 0; a < 3; a++) cams[k].t[a] = (float)(tc[a] - (M[3 * a] * t[0] + M[3 * a + 1] * t[1] + M[3 * a + 2] * t[2]));
}

}  // namespace gsr

extern "C" gsr_status gsr_transform_segment_launch(const gsr_params *p, int64_t n, int deg, const int32_t *seg,
                                                   int32_t segment, const double *pose, double *ws, hipStream_t st) {
    k_sh_rotation<<<1, 128, 0, st>>>(pose, ws);
    if (n > 0)
        k_transform_rows<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(p->means, p->quats, p->sh, n, deg, seg, segment,
                                                                     pose, ws);
    return last_launch();
}

extern "C" gsr_status gsr_transform_cameras_launch(gsr_camera *cams, int n_cams, const uint8_t *mask,
                                                   const double *pose, hipStream_t st) {
    if (n_cams > 0) k_transform_cams<<<(unsigned)ceil_div(n_cams, 64), 64, 0, st>>>(cams, n_cams, mask, pose);
    return last_launch();
}
