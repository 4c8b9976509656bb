// Initialisation path: voxel-PCA geometric fitting (Sec. III-A, Eq. 1-2) and the cascaded
// Gaussian initialisation (Sec. III-B, Eq. 3, 5, 6).
//
// Voxel PCA: every point gets a packed 32-bit voxel key and a 64-bit SplitMix64 hash of
// (seed XOR index); two stable radix sorts (the hash's leading bits, then the key) group the points
// by voxel in ascending key order and, inside a voxel, by those bits; the few points of one voxel
// that share them are put in order of the whole hash when the voxels are numbered.  One thread per
// voxel then fits its first (at most 32) points in double precision: mean, biased covariance, cyclic Jacobi eigensystem, canonical
// frame, planar / linear / unreliable class, and the trace of the descriptor's direction
// covariance, which Eq. 1-2 with isotropic point covariance sigma^2 I reduce to
// sigma^2 / N * sum_{m != k} (l_m + l_k) / (l_k - l_m)^2.  Given per-point world covariances,
// the same thread sums Eq. 2 itself, J_i Sigma_i J_i^T over the fitting points, for the full 6x6
// descriptor covariance and its trace.
#include "gsr_internal.h"

namespace gsr {

constexpr float kVoxel = 0.5f;
constexpr int kMaxPts = 32;
constexpr double kTauP = 2.5e-3, kTauL = 4.0, kLamFloor = 0.005 * 0.005, kSigma = 0.02, kRelTrace = 0.01;
constexpr int kMinPts = 5;
constexpr uint32_t kOutside = 0xffffffffu;

__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// packed key: (kx + 1024) << 21 | (ky + 1024) << 10 | (kz + 511); kx, ky in [-1024, 1023],
// kz in [-511, 511] (so the all-ones word never names a voxel and marks points outside)
__global__ void k_vox_prep(const float *__restrict__ pts, int64_t n, uint64_t seed, int hash_bits,
                           uint32_t *__restrict__ key, uint32_t *__restrict__ hash, uint32_t *__restrict__ n_outside) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_outside = 0u;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float x = pts[i], y = pts[n + i], z = pts[2 * n + i];
        const float kxf = floorf(x / kVoxel), kyf = floorf(y / kVoxel), kzf = floorf(z / kVoxel);
        const bool in = kxf >= -1024.f && kxf <= 1023.f && kyf >= -1024.f && kyf <= 1023.f && kzf >= -511.f &&
                        kzf <= 511.f;
        key[i] = in ? ((uint32_t)((int)kxf + 1024) << 21) | ((uint32_t)((int)kyf + 1024) << 10) |
                          (uint32_t)((int)kzf + 511)
                    : kOutside;
        hash[i] = (uint32_t)(splitmix64(seed ^ (uint64_t)i) >> (64 - hash_bits));
    }
}

// Voxel heads per block of 256 ROUNDS sorted points (round-major, coalesced).
template <int ROUNDS>
__global__ __launch_bounds__(256) void k_vox_heads(const uint32_t *__restrict__ skey, int64_t n,
                                                   uint32_t *__restrict__ bsum) {
    __shared__ uint32_t s_w[4];
    const int64_t base = (int64_t)blockIdx.x * (256 * ROUNDS);
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        const int64_t e = base + r * kSortThreads + threadIdx.x;
        if (e < n) {
            const uint32_t k = skey[e];
            c += k != kOutside && (e == 0 || k != skey[e - 1]) ? 1u : 0u;
        }
    }
    uint32_t tot;
    block_excl_scan256(c, s_w, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// A lane's 64-bit value, and the number of ones below the lowest zero.
__device__ __forceinline__ uint64_t lane64(uint64_t x, int lane) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane) << 32;
}
__device__ __forceinline__ int ones_below(uint64_t m) { return ~m ? __builtin_ctzll(~m) : 64; }

constexpr int kNear = 3;

// Numbers the voxels, writes the points' order and voxels.  Points of one voxel whose leading hash bits
// agree form a run that the sort left in index order: each of them counts the run's smaller whole hashes
// (distinct: SplitMix64 is a bijection), a lane alone within kNear points and its wave beyond.  bsum: the blocks' head counts, scanned when
// `scanned`, else added up here (the last block then writes the voxel count).
template <int ROUNDS>
__global__ __launch_bounds__(256) void k_vox_assign(const uint32_t *__restrict__ skey, const uint32_t *__restrict__ sidx,
                                                    int64_t n, uint64_t seed, int hash_bits,
                                                    const uint32_t *__restrict__ bsum, bool scanned, gsr_voxels V) {
    __shared__ uint32_t s_cnt[ROUNDS * 4];
    __shared__ uint32_t s_w[4];
    const int64_t base = (int64_t)blockIdx.x * (256 * ROUNDS);
    const int w = threadIdx.x >> 6, lane = __lane_id();
    uint32_t b0;
    if (scanned) {
        b0 = bsum[blockIdx.x];
    } else {
        uint32_t c = 0;
#pragma unroll 4
        for (uint32_t i = threadIdx.x; i < blockIdx.x; i += 256) c += bsum[i];
        block_excl_scan256(c, s_w, &b0);
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *V.n_voxels = b0 + bsum[blockIdx.x];
    }
    uint64_t m[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; r++) {
        const int64_t e = base + r * 256 + threadIdx.x;
        const uint32_t k = e < n ? skey[e] : kOutside;
        m[r] = __ballot(k != kOutside && (e == 0 || k != skey[e - 1]));
        if (lane == 0) s_cnt[r * 4 + w] = (uint32_t)__popcll(m[r]);
    }
    __syncthreads();
    if (threadIdx.x < ROUNDS * 4) {
        const uint32_t c = s_cnt[threadIdx.x];
        s_cnt[threadIdx.x] = wave_incl_scan(c) - c;
    }
    __syncthreads();
    const int sh = 64 - hash_bits;
#pragma unroll 4
    for (int r = 0; r < ROUNDS; r++) {
        const int64_t e = base + r * 256 + threadIdx.x;
        const bool in = e < n;
        const uint32_t k = in ? skey[e] : 0u, p = in ? sidx[e] : 0u;
        const uint64_t out = __ballot(in && k == kOutside);
        if (out && lane == __builtin_ctzll(out)) atomicAdd(V.n_outside, (uint32_t)__popcll(out));
        const bool head = (m[r] >> lane) & 1ull;
        if (in && k == kOutside) {
            V.point_voxel[p] = kOutside;
        } else if (in) {
            const uint32_t v = b0 + s_cnt[r * 4 + w] + (uint32_t)__popcll(m[r] & lanemask_lt()) + (head ? 1u : 0u) - 1u;
            V.point_voxel[p] = v;
            if (head) {
                V.start[v] = (uint32_t)e;
                V.key[v] = k;
            }
        }
        const uint64_t h = splitmix64(seed ^ (uint64_t)p);
        auto hash = [&](int64_t q) { return splitmix64(seed ^ (uint64_t)sidx[q]); };
        auto member = [&](int64_t q, uint32_t kr, uint64_t hr, uint64_t &hq) {  // of the run of key kr and leading bits hr
            if (q < 0 || q >= n || skey[q] != kr) return false;
            hq = hash(q);
            return hq >> sh == hr;
        };
        // a lane walks a few points to either side by itself
        uint64_t hq;
        int64_t b = e - 1, f = e + 1, at = e;
        for (; in && e - b <= kNear && member(b, k, h >> sh, hq); b--) at -= hq > h ? 1 : 0;
        for (; in && f - e <= kNear && member(f, k, h >> sh, hq); f++) at += hq < h ? 1 : 0;
        const bool run = in && (e - b > kNear || f - e > kNear);
        if (in && !run) V.point_order[at] = p;
        uint64_t left = __ballot(run);
        while (left) {  // the run of the first lane left, by the whole wave
            const int lead = __builtin_ctzll(left);
            const uint32_t kr = (uint32_t)__builtin_amdgcn_readlane((int)k, lead);
            const uint64_t hr = lane64(h, lead) >> sh;
            int64_t lo = e - lane + lead, hi = lo + 1;
            for (int c = 64; c == 64; lo -= c) c = ones_below(__ballot(member(lo - 1 - lane, kr, hr, hq)));
            for (int c = 64; c == 64; hi += c) c = ones_below(__ballot(member(hi + lane, kr, hr, hq)));
            uint32_t rank = 0;
            for (int64_t q = lo; q < hi; q += 64) {
                hq = q + lane < hi ? hash(q + lane) : 0u;
                const int c = hi - q < 64 ? (int)(hi - q) : 64;
                for (int i = 0; i < c; i++) rank += lane64(hq, i) < h ? 1u : 0u;
            }
            const bool mine = run && e >= lo && e < hi;
            if (mine) V.point_order[lo + rank] = p;
            left &= ~__ballot(mine);
        }
    }
}

// The points as records, so that a fit gathers one cache line per point and not one per component:
// (x, y, z, 0), or with covariances (x, y, z, xx, xy, xz, yy, yz); zz stays where it is.
template <bool COV>
__global__ void k_vox_records(const float *__restrict__ pts, const float *__restrict__ pcov, int64_t n,
                              float4 *__restrict__ rec) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float x = pts[i], y = pts[n + i], z = pts[2 * n + i];
        if (COV) {
            rec[2 * i] = make_float4(x, y, z, pcov[i]);
            rec[2 * i + 1] = make_float4(pcov[n + i], pcov[2 * n + i], pcov[3 * n + i], pcov[4 * n + i]);
        } else {
            rec[i] = make_float4(x, y, z, 0.f);
        }
    }
}

// 3x3 row-major products
__device__ __forceinline__ void mm3(const double *a, const double *b, double *c) {
    for (int i = 0; i < 3; i++)
        for (int j = 0; j < 3; j++) c[i * 3 + j] = a[i * 3] * b[j] + a[i * 3 + 1] * b[3 + j] + a[i * 3 + 2] * b[6 + j];
}

// Cyclic Jacobi on a symmetric 3x3 (row-major a): plane rotations J over (0,1), (0,2), (1,2)
// that zero a_pq, a <- J^T a J, eigenvectors accumulated as the columns of w <- w J.
__device__ void jacobi3(double a[9], double w[9]) {
    for (int k = 0; k < 9; k++) w[k] = (k % 4 == 0) ? 1.0 : 0.0;
    const int pp[3] = {0, 0, 1}, qq[3] = {1, 2, 2};
    for (int sweep = 0; sweep < 60; sweep++) {
        const double off = a[1] * a[1] + a[2] * a[2] + a[5] * a[5];
        const double sc = a[0] * a[0] + a[4] * a[4] + a[8] * a[8];
        if (off <= 1e-30 * fmax(sc, 1e-300)) break;
        for (int r = 0; r < 3; r++) {
            const int p = pp[r], q = qq[r];
            const double apq = a[p * 3 + q];
            if (!(fabs(apq) > 1e-300)) continue;
            // tan(2 theta) = 2 a_pq / (a_qq - a_pp)
            const double th = 0.5 * atan2(2.0 * apq, a[q * 3 + q] - a[p * 3 + p]);
            const double c = cos(th), s = sin(th);
            double J[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1}, Jt[9], t[9];
            J[p * 3 + p] = c;
            J[q * 3 + q] = c;
            J[p * 3 + q] = s;
            J[q * 3 + p] = -s;
            for (int u = 0; u < 3; u++)
                for (int v = 0; v < 3; v++) Jt[u * 3 + v] = J[v * 3 + u];
            mm3(Jt, a, t);
            mm3(t, J, a);
            mm3(w, J, t);
            for (int k = 0; k < 9; k++) w[k] = t[k];
        }
    }
}

// f(point, record) for the m points of a voxel in order, the records loaded N at a time (two dependent
// loads each, so a fit waits out m / N round trips instead of m).  Records of HALVES float4.
template <int N, int HALVES, typename F>
__device__ __forceinline__ void each_record(const uint32_t *__restrict__ order, const float4 *__restrict__ rec, int m,
                                            F &&f) {
#pragma unroll 1
    for (int j0 = 0; j0 < m; j0 += N) {
        uint32_t p[N];
        float4 r[N];
#pragma unroll
        for (int q = 0; q < N; q++) p[q] = order[j0 + q < m ? j0 + q : m - 1];
#pragma unroll
        for (int q = 0; q < N; q++) r[q] = rec[(int64_t)HALVES * p[q]];
#pragma unroll
        for (int q = 0; q < N; q++)
            if (j0 + q < m) f(p[q], r[q]);
    }
}

// One thread per voxel, its sums in the order of the points: the same bits however they are fetched
// (where eigenvalues coincide the eigenvectors follow the last bit).  Bound by the gather: 6.4M points in
// random order, 32 per voxel, with covariances take 535 us (and 70 for the records) against 1760 with one component and one
// point at a time.
//
// COV: Eq. 1-2 with the per-point world covariances pcov [6][n] (xx, xy, xz, yy, yz, zz) instead
// of sigma^2 I; the full descriptor covariance goes to sg [21][n] (upper triangle, row-major)
// when sg is not null.
template <bool COV>
__global__ __launch_bounds__(64) void k_vox_pca(const float4 *__restrict__ rec, int64_t n, gsr_voxels V,
                                                const float *__restrict__ pcov, float *__restrict__ sg) {
    constexpr int kStep = COV ? 2 : 1;
    const uint32_t nv = *V.n_voxels;
    const uint32_t nvalid = (uint32_t)n - *V.n_outside;
    for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
        const uint32_t s0 = V.start[v];
        const uint32_t e0 = v + 1 < nv ? V.start[v + 1] : nvalid;
        const uint32_t cnt = e0 - s0;
        const int m = cnt < (uint32_t)kMaxPts ? (int)cnt : kMaxPts;
        V.count[v] = cnt;
        double mu[3] = {0, 0, 0};
        const uint32_t *order = V.point_order + s0;
        each_record<8, kStep>(order, rec, m, [&](uint32_t, const float4 &x) {
            mu[0] += x.x;
            mu[1] += x.y;
            mu[2] += x.z;
        });
        for (int c = 0; c < 3; c++) mu[c] /= m;
        double C[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        each_record<8, kStep>(order, rec, m, [&](uint32_t, const float4 &x) {
            const double d[3] = {x.x - mu[0], x.y - mu[1], x.z - mu[2]};
            for (int a = 0; a < 3; a++)
                for (int b = 0; b < 3; b++) C[a * 3 + b] += d[a] * d[b];
        });
        for (int k = 0; k < 9; k++) C[k] /= m;
        double A[9], W[9];
        for (int k = 0; k < 9; k++) A[k] = C[k];
        jacobi3(A, W);
        // ascending eigenvalues (stable order on ties), eigenvectors as W's columns
        double lam[3] = {A[0], A[4], A[8]};
        int ord[3] = {0, 1, 2};
        for (int i = 1; i < 3; i++)
            for (int j = i; j > 0 && lam[ord[j]] < lam[ord[j - 1]]; j--) {
                const int t = ord[j];
                ord[j] = ord[j - 1];
                ord[j - 1] = t;
            }
        const double l[3] = {lam[ord[0]], lam[ord[1]], lam[ord[2]]};
        // R_pca columns (v_max, v_mid, v_min): largest |component| positive, then det = +1
        double R[9];
        for (int c = 0; c < 3; c++) {
            const int src = ord[2 - c];
            int big = 0;
            for (int r = 1; r < 3; r++)
                if (fabs(W[r * 3 + src]) > fabs(W[big * 3 + src])) big = r;
            const double sg = W[big * 3 + src] < 0 ? -1.0 : 1.0;
            for (int r = 0; r < 3; r++) R[r * 3 + c] = sg * W[r * 3 + src];
        }
        const double det = R[0] * (R[4] * R[8] - R[5] * R[7]) - R[1] * (R[3] * R[8] - R[5] * R[6]) +
                           R[2] * (R[3] * R[7] - R[4] * R[6]);
        if (det < 0)
            for (int r = 0; r < 3; r++) R[r * 3 + 2] = -R[r * 3 + 2];
        uint8_t cls = 2;
        if (l[0] < kTauP) cls = 0;
        else if (l[2] / l[0] > kTauL) cls = 1;
        if (m < kMinPts) cls = 2;
        double tr = INFINITY;
        if (cls != 2 && !COV) {
            const int k = cls == 0 ? 0 : 2;
            double t = 0.0;
            for (int q = 0; q < 3; q++)
                if (q != k) t += (l[q] + l[k]) / ((l[k] - l[q]) * (l[k] - l[q]));
            tr = kSigma * kSigma / m * t;
        }
        if (COV) {
            double G[21];
#pragma unroll
            for (int e = 0; e < 21; e++) G[e] = 0.0;
            if (cls != 2) {
                // eigenvectors ascending (v_min, v_mid, v_max) = R_pca columns 2, 1, 0
                const int k = cls == 0 ? 0 : 2;
                double ev[3][3];
#pragma unroll
                for (int q = 0; q < 3; q++)
#pragma unroll
                    for (int r = 0; r < 3; r++) ev[q][r] = R[r * 3 + (2 - q)];
                double vk[3], lk = k == 0 ? l[0] : l[2];
#pragma unroll
                for (int r = 0; r < 3; r++) vk[r] = k == 0 ? ev[0][r] : ev[2][r];
                // (one point at a time, the next one's loads in flight: the body is too wide for more)
                uint32_t p = order[0];
                float4 x = rec[2 * (int64_t)p], y = rec[2 * (int64_t)p + 1];
                float zz = pcov[5 * n + p];
#pragma unroll 1
                for (int j = 0; j < m; j++) {
                    p = order[j + 1 < m ? j + 1 : j];
                    const float4 nx = rec[2 * (int64_t)p], ny = rec[2 * (int64_t)p + 1];
                    const float nzz = pcov[5 * n + p];
                    const double d[3] = {x.x - mu[0], x.y - mu[1], x.z - mu[2]};
                    const double dk = d[0] * vk[0] + d[1] * vk[1] + d[2] * vk[2];
                    // T = V F = sum_{q != k} v_q f_q^T, f_q = ((d.v_q) v_k + (d.v_k) v_q) / (m (l_k - l_q))
                    double T[9];
#pragma unroll
                    for (int e = 0; e < 9; e++) T[e] = 0.0;
#pragma unroll
                    for (int q = 0; q < 3; q++) {
                        if (q == k) continue;
                        const double dq = d[0] * ev[q][0] + d[1] * ev[q][1] + d[2] * ev[q][2];
                        const double inv = 1.0 / (m * (lk - l[q]));
#pragma unroll
                        for (int r = 0; r < 3; r++)
#pragma unroll
                            for (int c = 0; c < 3; c++) T[r * 3 + c] += ev[q][r] * ((dq * vk[c] + dk * ev[q][c]) * inv);
                    }
                    const double S[9] = {x.w, y.x, y.y, y.x, y.z, y.w, y.y, y.w, zz};
                    // J = [T; I/m] (6 x 3), G += J S J^T
                    double J[6][3], JS[6][3];
#pragma unroll
                    for (int r = 0; r < 3; r++)
#pragma unroll
                        for (int c = 0; c < 3; c++) J[r][c] = T[r * 3 + c], J[3 + r][c] = r == c ? 1.0 / m : 0.0;
#pragma unroll
                    for (int r = 0; r < 6; r++)
#pragma unroll
                        for (int c = 0; c < 3; c++) JS[r][c] = J[r][0] * S[c] + J[r][1] * S[3 + c] + J[r][2] * S[6 + c];
#pragma unroll
                    for (int r = 0; r < 6; r++)
#pragma unroll
                        for (int c = r; c < 6; c++)
                            G[r * 6 - r * (r - 1) / 2 + (c - r)] += JS[r][0] * J[c][0] + JS[r][1] * J[c][1] + JS[r][2] * J[c][2];
                    x = nx, y = ny, zz = nzz;
                }
                tr = G[0] + G[6] + G[11];  // (0,0), (1,1), (2,2) of the upper triangle
            }
            if (sg)
#pragma unroll
                for (int e = 0; e < 21; e++) sg[(int64_t)e * n + v] = (float)G[e];
        }
        const int64_t N = n;
        for (int c = 0; c < 3; c++) {
            V.mu[c * N + v] = (float)mu[c];
            V.evals[c * N + v] = (float)l[c];
            V.s_pca[c * N + v] = (float)(0.5 * log(fmax(l[2 - c], kLamFloor)));
        }
        for (int k = 0; k < 9; k++) V.R[k * N + v] = (float)R[k];
        V.trace[v] = (float)tr;
        V.cls[v] = cls;
        V.reliable[v] = (cls != 2 && tr < kRelTrace) ? 1 : 0;
    }
}

}  // namespace gsr

using namespace gsr;

extern "C" gsr_status gsr_exclusive_scan_small_launch(uint32_t *, int, uint32_t *, hipStream_t);
extern "C" size_t gsr_sort_pairs_ws_bytes(int64_t n);
extern "C" gsr_status gsr_sort_pairs_launch(uint32_t *, uint32_t *, uint32_t *, uint32_t *, uint32_t, int, void *,
                                            hipStream_t);
extern "C" gsr_status gsr_sort_positions_launch(uint32_t *k[2], uint32_t *v[2], uint32_t *w[2], uint32_t n, int bits,
                                                void *ws, hipStream_t st);
extern "C" gsr_status gsr_fill_u32_launch(void *, uint32_t, int64_t, hipStream_t);

namespace {
// rec takes the place of the sort's arrays once the points are in order
struct VoxWs {
    float4 *rec;  // [2 n]
    uint32_t *k[2], *h[2], *i[2], *bsum;
    void *sort_ws;
    size_t bytes;
};
size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }
// points per numbering block: 1,024 fill the chip sooner (a block of 4,096 took 29 us at 100k points, a
// quarter of that 12), 4,096 keep the block sums few enough to be added up by their readers
int64_t vox_tile(int64_t n) { return n <= (1 << 20) ? 1024 : 4096; }
VoxWs vox_layout(void *base, int64_t n) {
    VoxWs w{};
    char *p = static_cast<char *>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        void *r = p ? p + off : nullptr;
        off += al256(bytes);
        return r;
    };
    const size_t nb = (size_t)(n > 0 ? n : 1) * 4;
    for (int q = 0; q < 2; q++) {
        w.k[q] = (uint32_t *)take(nb);
        w.h[q] = (uint32_t *)take(nb);
        w.i[q] = (uint32_t *)take(nb);
    }
    w.rec = (float4 *)w.k[0];
    if (off < 8 * nb) take(8 * nb - off);
    w.sort_ws = take(gsr_sort_pairs_ws_bytes(n));
    // (1,024 block sums at least above 2^20 points, where the blocks grow: the workspace never shrinks)
    const int64_t blocks = ceil_div(n > 0 ? n : 1, vox_tile(n));
    w.bsum = (uint32_t *)take((size_t)(n > (1 << 20) && blocks < 1024 ? 1024 : blocks) * 4);
    w.bytes = off;
    return w;
}
int grid(int64_t n) { return (int)(ceil_div(n > 0 ? n : 1, 256) < 16384 ? ceil_div(n > 0 ? n : 1, 256) : 16384); }
}  // namespace

extern "C" size_t gsr_voxel_pca_ws_bytes(int64_t n) { return vox_layout(nullptr, n).bytes; }

static gsr_status voxel_pca_run(const float *pts, int64_t n, uint64_t seed, const gsr_voxels *out, void *ws,
                                hipStream_t st, const float *pcov, float *sg) {
    if (n == 0) {
        gsr_status s = gsr_fill_u32_launch(out->n_outside, 0u, 1, st);
        return s != GSR_OK ? s : gsr_fill_u32_launch(out->n_voxels, 0u, 1, st);
    }
    VoxWs w = vox_layout(ws, n);
    const int g = grid(n);
    // Leading hash bits sorted on: with 16, points of one voxel that agree in them are rare (1 in 130
    // voxels of 32 points holds two), and a run of them averages n / 2^16 points even if all points lie in
    // one voxel; beyond 2^24 points that bound asks for 24.  Two passes and the key's four instead of
    // twelve (the whole hash, then the key).  All in one voxel, 4M and 16.7M points take 659 and 2,842 us (764 and
    // 3,024 in twelve passes; 17,500 and 435,000 with one lane ordering a run).
    const int hash_bits = n <= (1 << 24) ? 16 : 24;
    k_vox_prep<<<g, 256, 0, st>>>(pts, n, seed, hash_bits, w.k[0], w.h[0], out->n_outside);
    gsr_status s = gsr_sort_positions_launch(w.h, w.k, w.i, (uint32_t)n, hash_bits, w.sort_ws, st);
    if (s != GSR_OK) return s;
    // four passes: the result lands back in (k[0], i[0])
    s = gsr_sort_pairs_launch(w.k[0], w.i[0], w.k[1], w.i[1], (uint32_t)n, 32, w.sort_ws, st);
    if (s != GSR_OK) return s;
    const int nb = (int)ceil_div(n, vox_tile(n));
    const bool scanned = nb > 2048, few = vox_tile(n) == 1024;
    if (few) k_vox_heads<4><<<nb, 256, 0, st>>>(w.k[0], n, w.bsum);
    else k_vox_heads<16><<<nb, 256, 0, st>>>(w.k[0], n, w.bsum);
    if (scanned) {
        s = gsr_exclusive_scan_small_launch(w.bsum, nb, out->n_voxels, st);
        if (s != GSR_OK) return s;
    }
    if (few) k_vox_assign<4><<<nb, 256, 0, st>>>(w.k[0], w.i[0], n, seed, hash_bits, w.bsum, scanned, *out);
    else k_vox_assign<16><<<nb, 256, 0, st>>>(w.k[0], w.i[0], n, seed, hash_bits, w.bsum, scanned, *out);
    const int64_t fits = ceil_div(n, 64);
    const int gf = (int)(fits < 16384 ? fits : 16384);
    if (pcov) {
        k_vox_records<true><<<g, 256, 0, st>>>(pts, pcov, n, w.rec);
        k_vox_pca<true><<<gf, 64, 0, st>>>(w.rec, n, *out, pcov, sg);
    } else {
        k_vox_records<false><<<g, 256, 0, st>>>(pts, nullptr, n, w.rec);
        k_vox_pca<false><<<gf, 64, 0, st>>>(w.rec, n, *out, nullptr, nullptr);
    }
    return last_launch();
}

extern "C" gsr_status gsr_voxel_pca_launch(const float *pts, int64_t n, uint64_t seed, const gsr_voxels *out,
                                           void *ws, hipStream_t st) {
    return voxel_pca_run(pts, n, seed, out, ws, st, nullptr, nullptr);
}

extern "C" gsr_status gsr_voxel_pca_cov_launch(const float *pts, const float *pcov, int64_t n, uint64_t seed,
                                               const gsr_voxels *out, float *sg, void *ws, hipStream_t st) {
    return voxel_pca_run(pts, n, seed, out, ws, st, pcov, sg);
}

// ---- cascaded initialisation (Eq. 3, 5, 6) ------------------------------------------------------
namespace gsr {

constexpr float kOpacityConst = 0.1f;
constexpr float kY00 = 0.28209479177387814f;

// Eq. 3's valid model prediction: finite outputs, non-zero quaternion, log-scales in
// [log 2 mm, log 0.5 m].  pred [8][stride] = (s[3], q[4], omega) per voxel.
__device__ __forceinline__ bool pred_valid(const float *pred, int64_t stride, uint32_t v) {
    if (!pred) return false;
    float q2 = 0.f;
    for (int k = 0; k < 8; k++) {
        const float x = pred[k * stride + v];
        if (!isfinite(x)) return false;
        if (k >= 3 && k < 7) q2 += x * x;
    }
    if (!(q2 > 0.f)) return false;
    for (int k = 0; k < 3; k++) {
        const float s = pred[k * stride + v];
        if (s < -6.2146080984221914f || s > -0.69314718055994531f) return false;  // log 0.002, log 0.5
    }
    return true;
}

// rotation matrix (row-major) -> unit quaternion (w, x, y, z), w >= 0, largest-pivot method
__device__ void rot_to_quat(const double r[9], double q[4]) {
    const double tr = r[0] + r[4] + r[8];
    if (tr > 0) {
        const double s = 2.0 * sqrt(1.0 + tr);
        q[0] = 0.25 * s, q[1] = (r[7] - r[5]) / s, q[2] = (r[2] - r[6]) / s, q[3] = (r[3] - r[1]) / s;
    } else if (r[0] > r[4] && r[0] > r[8]) {
        const double s = 2.0 * sqrt(1.0 + r[0] - r[4] - r[8]);
        q[0] = (r[7] - r[5]) / s, q[1] = 0.25 * s, q[2] = (r[1] + r[3]) / s, q[3] = (r[2] + r[6]) / s;
    } else if (r[4] > r[8]) {
        const double s = 2.0 * sqrt(1.0 + r[4] - r[0] - r[8]);
        q[0] = (r[2] - r[6]) / s, q[1] = (r[1] + r[3]) / s, q[2] = 0.25 * s, q[3] = (r[5] + r[7]) / s;
    } else {
        const double s = 2.0 * sqrt(1.0 + r[8] - r[0] - r[4]);
        q[0] = (r[3] - r[1]) / s, q[1] = (r[2] + r[6]) / s, q[2] = (r[5] + r[7]) / s, q[3] = 0.25 * s;
    }
    const double nq = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const double sg = q[0] < 0 ? -1.0 : 1.0;
    for (int k = 0; k < 4; k++) q[k] = sg * q[k] / nq;
}

// What Eq. 3 takes from a voxel, the same for all its points: the branch (0 model, 1 PCA, 2 heuristic)
// and for the first two the log-scales before their per-point or per-segment shift (Eq. 4's axis
// ratios when anchored), the quaternion and the model's opacity logit.
struct VoxInit {
    float ls[3], lo, q[4];
};

__device__ __forceinline__ uint8_t voxel_init(const gsr_voxels &V, const float *__restrict__ pred, int64_t n, uint32_t v,
                                              int anchored, VoxInit &o) {
    if (pred_valid(pred, n, v)) {
        float nq = 0.f;
        for (int k = 0; k < 4; k++) nq += pred[(3 + k) * n + v] * pred[(3 + k) * n + v];
        nq = sqrtf(nq);
        for (int k = 0; k < 3; k++) o.ls[k] = pred[k * n + v];
        if (anchored) {
            const float mx = fmaxf(o.ls[0], fmaxf(o.ls[1], o.ls[2]));
            for (int k = 0; k < 3; k++) o.ls[k] -= mx;
        }
        for (int k = 0; k < 4; k++) o.q[k] = pred[(3 + k) * n + v] / nq;
        o.lo = pred[7 * n + v];
        return 0;
    }
    if (V.reliable[v]) {
        for (int k = 0; k < 3; k++) o.ls[k] = V.s_pca[k * n + v];
        double r[9], qd[4];
        for (int k = 0; k < 9; k++) r[k] = V.R[k * n + v];
        rot_to_quat(r, qd);
        for (int k = 0; k < 4; k++) o.q[k] = (float)qd[k];
        o.lo = 0.f;
        return 1;
    }
    return 2;
}

// Every voxel's VoxInit, computed once instead of once per point, in the sh output (written last, by
// k_cascade_sh): records, then branch bytes.  There is room unless the voxels hold very few points
// (sh holds 3 K floats per point); `rows` decides on the device, where the voxel count is.  A point
// then gathers one byte and one 32-byte record where it gathered some twenty values and formed a
// quaternion in FP64: 6.4M points of 200k voxels in random order, 162 us and 34 for the table and the sh output (827 before), and
// the segment counts 39 (228).
// The count only says how many voxels the table holds: a point of a voxel past it takes the per-point form,
// so the results do not depend on it.
// Its two launches take 5 us, so small clouds go without: the whole call takes 40 us without and 43 with it at
// 100k points with a model's predictions, 56 and 52 at 200k, and without predictions 61 either way at 200k and 82 and 78 at 500k.
constexpr int64_t kTableFrom = 1 << 17;  // points, twice as many without predictions
struct CascadeTable {
    VoxInit *rec;  // null: no table (no count, or the sh output overlaps an input or is not 16-byte aligned)
    int64_t floats;  // of the sh output
    __device__ __forceinline__ uint32_t rows(const gsr_voxels &V, int64_t n) const {
        const uint32_t nv = rec ? *V.n_voxels : 0u;
        return (int64_t)nv <= n && (int64_t)nv * 8 + (nv + 3) / 4 <= floats ? nv : 0u;
    }
    __device__ __forceinline__ uint8_t *branch(uint32_t nv) const { return reinterpret_cast<uint8_t *>(rec + nv); }
};

__global__ __launch_bounds__(256) void k_cascade_voxels(gsr_voxels V, const float *__restrict__ pred, int64_t n,
                                                        int anchored, CascadeTable T) {
    const uint32_t nv = T.rows(V, n);
    for (uint32_t v = blockIdx.x * 256 + threadIdx.x; v < nv; v += gridDim.x * 256) {
        VoxInit o;
        const uint8_t br = voxel_init(V, pred, n, v, anchored, o);
        T.branch(nv)[v] = br;
        if (br == 2) continue;
        float4 *r = reinterpret_cast<float4 *>(T.rec + v);
        r[0] = make_float4(o.ls[0], o.ls[1], o.ls[2], o.lo);
        r[1] = make_float4(o.q[0], o.q[1], o.q[2], o.q[3]);
    }
}

// Per-segment point counts for beta.  Points of one segment arrive together, so per-point global
// atomics would all hit one address; each workgroup counts in LDS (up to kSegLds segments), a wave
// whose points share a segment in one add, and adds its totals once.
constexpr int kSegLds = 1024;

__global__ __launch_bounds__(256) void k_seg_counts(const uint32_t *__restrict__ pvox, gsr_voxels V,
                                                    const float *__restrict__ pred, int64_t n,
                                                    const int32_t *__restrict__ seg, int nseg, CascadeTable T,
                                                    uint32_t *__restrict__ cnt, uint32_t *__restrict__ fb) {
    __shared__ uint32_t s_cnt[kSegLds], s_fb[kSegLds];
    const bool lds = nseg <= kSegLds;
    if (lds)
        for (int e = threadIdx.x; e < nseg; e += 256) s_cnt[e] = s_fb[e] = 0u;
    __syncthreads();
    const uint32_t nv = T.rows(V, n);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t v = pvox[i];
        const int s = seg ? seg[i] : 0;
        if (v == kOutside || s < 0 || s >= nseg) continue;
        const bool f = v < nv ? T.branch(nv)[v] == 1 : V.reliable[v] && !pred_valid(pred, n, v);
        uint32_t *c = lds ? s_cnt : cnt, *b = lds ? s_fb : fb;
        const uint64_t here = __ballot(true), fall = __ballot(f);
        if (__ballot(s == __builtin_amdgcn_readfirstlane(s)) == here) {
            if (__lane_id() == __builtin_ctzll(here)) {
                atomicAdd(&c[s], (uint32_t)__popcll(here));
                if (fall) atomicAdd(&b[s], (uint32_t)__popcll(fall));
            }
        } else {
            atomicAdd(&c[s], 1u);
            if (f) atomicAdd(&b[s], 1u);
        }
    }
    __syncthreads();
    if (lds)
        for (int e = threadIdx.x; e < nseg; e += 256) {
            if (s_cnt[e]) atomicAdd(&cnt[e], s_cnt[e]);
            if (s_fb[e]) atomicAdd(&fb[e], s_fb[e]);
        }
}

__device__ __forceinline__ void write_sh(const float *__restrict__ col, int64_t n, int64_t i, int K, float *__restrict__ sh) {
    for (int c = 0; c < 3; c++) sh[c * n + i] = (col[c * n + i] - 0.5f) / kY00;
    for (int k = 3; k < 3 * K; k++) sh[k * n + i] = 0.f;
}

__global__ void k_cascade(const float *__restrict__ pts, const float *__restrict__ col, const float *__restrict__ depth,
                          const int32_t *__restrict__ seg, int nseg, int64_t n, gsr_voxels V,
                          const float *__restrict__ pred, float focal, float beta_fixed,
                          const uint32_t *__restrict__ cnt, const uint32_t *__restrict__ fb, int K, CascadeTable T,
                          gsr_params out, uint8_t *__restrict__ branch, int anchored) {
    const uint32_t nv = T.rows(V, n);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t v = V.point_voxel[i];
        for (int c = 0; c < 3; c++) out.means[c * n + i] = pts[c * n + i];
        if (!nv) write_sh(col, n, i, K, out.sh);
        VoxInit o;
        uint8_t br = 2;
        if (v != kOutside) {
            if (v >= nv) {
                br = voxel_init(V, pred, n, v, anchored, o);
            } else {
                br = T.branch(nv)[v];
                if (br != 2) {
                    const float4 *r = reinterpret_cast<const float4 *>(T.rec + v);
                    const float4 a = r[0], q = r[1];
                    o = VoxInit{{a.x, a.y, a.z}, a.w, {q.x, q.y, q.z, q.w}};
                }
            }
        }
        branch[i] = br;
        float ls[3], q[4] = {1.f, 0.f, 0.f, 0.f}, lo = logf(kOpacityConst / (1.f - kOpacityConst));
        if (br == 0) {
            for (int k = 0; k < 3; k++) ls[k] = o.ls[k];
            if (anchored) {
                // Eq. 4: keep the axis ratios a = exp(s - max s) and anchor the size at d / f
                const float a0 = logf(depth[i] / focal);
                for (int k = 0; k < 3; k++) ls[k] = a0 + o.ls[k];
            }
            for (int k = 0; k < 4; k++) q[k] = o.q[k];
            lo = o.lo;
        } else if (br == 1) {
            float beta = beta_fixed;
            if (!(beta > 0.f)) {
                const int s = seg ? seg[i] : 0;
                const uint32_t c = (s >= 0 && s < nseg) ? cnt[s] : 0u;
                const float rho = c ? (float)fb[s] / (float)c : 0.f;
                beta = fminf(fmaxf(1.f - rho, 0.5f), 1.f);
            }
            const float lb = logf(beta);
            for (int k = 0; k < 3; k++) ls[k] = o.ls[k] + lb;
            for (int k = 0; k < 4; k++) q[k] = o.q[k];
        } else {
            const float s = logf(depth[i] / focal);
            ls[0] = ls[1] = ls[2] = s;
        }
        for (int k = 0; k < 3; k++) out.log_scales[k * n + i] = ls[k];
        for (int k = 0; k < 4; k++) out.quats[k * n + i] = q[k];
        out.opacity_logits[i] = lo;
    }
}

__global__ void k_cascade_sh(const float *__restrict__ col, int64_t n, gsr_voxels V, int K, CascadeTable T,
                             float *__restrict__ sh) {
    if (!T.rows(V, n)) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        write_sh(col, n, i, K, sh);
}

// Training targets of the point network (Sec. III-B): for every voxel, the mean covariance
// R(q/|q|) diag(exp(2 s)) R^T (xx, xy, xz, yy, yz, zz) and the mean opacity sigmoid(logit) of the
// Gaussians seeded one per point, over all the voxel's points.  One thread per voxel sums in float64
// in the voxel's point order (fixed, so the targets repeat exactly); rows at or past the voxel count
// are zero with has = 0.
__global__ void k_voxel_targets(const float *__restrict__ ls, const float *__restrict__ qs,
                                const float *__restrict__ lo, int64_t n, gsr_voxels V, float *__restrict__ cov,
                                float *__restrict__ ot, uint8_t *__restrict__ has) {
    const uint32_t nv = *V.n_voxels;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, op = 0.0;
        const uint32_t c = v < nv ? V.count[v] : 0u;
        const uint32_t s0 = c ? V.start[v] : 0u;
        for (uint32_t k = 0; k < c; k++) {
            const int64_t i = V.point_order[s0 + k];
            double w = qs[i], x = qs[n + i], y = qs[2 * n + i], z = qs[3 * n + i];
            const double nq = sqrt(w * w + x * x + y * y + z * z);
            w /= nq, x /= nq, y /= nq, z /= nq;
            const double R[3][3] = {{1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)},
                                    {2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)},
                                    {2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)}};
            const double e[3] = {exp(2.0 * (double)ls[i]), exp(2.0 * (double)ls[n + i]), exp(2.0 * (double)ls[2 * n + i])};
            int q = 0;
            for (int a = 0; a < 3; a++)
                for (int b = a; b < 3; b++, q++)
                    acc[q] += R[a][0] * e[0] * R[b][0] + R[a][1] * e[1] * R[b][1] + R[a][2] * e[2] * R[b][2];
            op += 1.0 / (1.0 + exp(-(double)lo[i]));
        }
        const double inv = c ? 1.0 / (double)c : 0.0;
        for (int q = 0; q < 6; q++) cov[q * n + v] = (float)(acc[q] * inv);
        ot[v] = (float)(op * inv);
        has[v] = c ? 1 : 0;
    }
}


}  // namespace gsr

extern "C" size_t gsr_cascade_ws_bytes(int nseg) { return (size_t)(2 * (nseg > 0 ? nseg : 1) * 4 + 512); }

extern "C" gsr_status gsr_cascade_launch(const float *pts, const float *col, const float *depth, const int32_t *seg,
                                         int nseg, int64_t n, const gsr_voxels *vox, const float *pred, float focal,
                                         float beta, int sh_degree, const gsr_params *out, uint8_t *branch, void *ws,
                                         hipStream_t st, int anchored) {
    if (n == 0) return GSR_OK;
    uint32_t *cnt = static_cast<uint32_t *>(ws);
    uint32_t *fb = cnt + (nseg > 0 ? nseg : 1);
    gsr_status s = gsr_fill_u32_launch(cnt, 0u, 2 * (int64_t)(nseg > 0 ? nseg : 1), st);
    if (s != GSR_OK) return s;
    const int g = grid(n), K = (sh_degree + 1) * (sh_degree + 1);
    // the sh output holds the voxel table until it is written, unless it shares memory with something
    // read or written before that (a caller may convert colours in place), the cloud is small, or the caller
    // gives no voxel count
    CascadeTable T{reinterpret_cast<VoxInit *>(out->sh), 3 * (int64_t)K * n};
    const uintptr_t lo = reinterpret_cast<uintptr_t>(out->sh), hi = lo + (uintptr_t)T.floats * 4;
    auto clash = [&](const void *p, int64_t bytes) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(p);
        return p && a < hi && a + (uintptr_t)bytes > lo;
    };
    if (n < (pred ? kTableFrom : 2 * kTableFrom) || !vox->n_voxels || (lo & 15) || clash(pts, 12 * n) || clash(col, 12 * n) || clash(depth, 4 * n) || clash(seg, 4 * n) ||
        clash(pred, 32 * n) || clash(vox->point_voxel, 4 * n) || clash(vox->reliable, n) || clash(vox->s_pca, 12 * n) ||
        clash(vox->R, 36 * n) || clash(vox->n_voxels, 4) || clash(out->means, 12 * n) || clash(out->log_scales, 12 * n) ||
        clash(out->quats, 16 * n) || clash(out->opacity_logits, 4 * n) || clash(branch, n) || clash(ws, gsr_cascade_ws_bytes(nseg)))
        T.rec = nullptr;
    // colours are read last, so with the table no other output may take their place before that
    const uintptr_t c0 = reinterpret_cast<uintptr_t>(col), c1 = c0 + (uintptr_t)(12 * n);
    auto over_colours = [&](const void *p, int64_t bytes) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(p);
        return a < c1 && a + (uintptr_t)bytes > c0;
    };
    if (over_colours(out->means, 12 * n) || over_colours(out->log_scales, 12 * n) || over_colours(out->quats, 16 * n) ||
        over_colours(out->opacity_logits, 4 * n) || over_colours(branch, n))
        T.rec = nullptr;
    if (T.rec) k_cascade_voxels<<<g < 1024 ? g : 1024, 256, 0, st>>>(*vox, pred, n, anchored, T);
    k_seg_counts<<<g < 1024 ? g : 1024, 256, 0, st>>>(vox->point_voxel, *vox, pred, n, seg, nseg, T, cnt, fb);
    k_cascade<<<g, 256, 0, st>>>(pts, col, depth, seg, nseg, n, *vox, pred, focal, beta, cnt, fb, K, T, *out, branch,
                                 anchored);
    if (T.rec) k_cascade_sh<<<g, 256, 0, st>>>(col, n, *vox, K, T, out->sh);
    return last_launch();
}

extern "C" gsr_status gsr_voxel_targets_launch(const gsr_params *g, int64_t n, const gsr_voxels *vox, float *cov,
                                              float *ot, uint8_t *has, hipStream_t st) {
    if (n == 0) return GSR_OK;
    const int64_t nb = ceil_div(n, 256);
    k_voxel_targets<<<(int)(nb < 4096 ? nb : 4096), 256, 0, st>>>(g->log_scales, g->quats, g->opacity_logits, n,
                                                                   *vox, cov, ot, has);
    return last_launch();
}
