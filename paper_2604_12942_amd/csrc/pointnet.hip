// Per-voxel point network of the model branch of the cascaded initialisation (Sec. III-B,
// Eq. 3): a shared MLP 3 -> 64 -> 64 -> 64 (ReLU) over each voxel's 32 input rows, max-pool, the
// 12 voxel-PCA features appended, 76 -> 64 (ReLU) -> 8 = (log-scales, quaternion, opacity logit).
//
// The shared layers run on the matrix cores (v_mfma_f32_32x32x16_bf16, BF16 inputs, FP32
// accumulate), a voxel's 32 rows per product.  BF16 rounding points (round to nearest even):
// weights and every GEMM input, upstream gradients included; bias, ReLU and accumulation in FP32.
//
// The backward (one training step's gradient) is persistent: each wave recomputes the forward of
// its voxels, forms the loss gradient per voxel (KL(N(0, Sigma_pred) || N(0, Sigma_tgt)) +
// 0.1 |sigmoid(omega) - o_tgt|, mean over voxels with a target), back-propagates (max-pool to the
// argmax row, lowest row on ties) and keeps its weight-gradient sums in registers; workgroups add
// their waves' in order, and a fixed-order reduction over workgroups follows.
#include "gsr_internal.h"

namespace gsr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kRows = 32, kWidth = 64, kFeat = 12, kOut = 8;
// flat weight layout (floats): W1[3][64] b1 W2[64][64] b2 W3[64][64] b3 W4[76][64] b4 W5[64][8] b5
constexpr int oW1 = 0, oB1 = 192, oW2 = 256, oB2 = 4352, oW3 = 4416, oB3 = 8512, oW4 = 8576, oB4 = 13440,
              oW5 = 13504, oB5 = 14016, kNW = 14024;

__device__ __forceinline__ __bf16 tobf(float x) { return (__bf16)x; }
__device__ __forceinline__ float fbf(__bf16 x) { return (float)x; }

// ---- forward (inference) ------------------------------------------------------------------------
// Persistent, wave-independent: each wave takes an equal contiguous range of voxels (its share of
// the whole batch, so that no wave runs a group more than another) in groups of 32.  Per voxel the
// wave runs the
// three shared layers on the matrix cores with the activations kept in registers:
//   layers 1 and 2 transposed, out^T = W^T h^T (M = 64 output features in two row tiles, N = the
//   voxel's 32 rows), so the accumulators hold, per lane, one row and 16 features of each tile;
//   those 32 values, bias + ReLU + BF16, are directly the next layer's K-operand once K is taken in
//   the order phi below (the weights are loaded in the same order; the contraction does not care);
//   layer 3 the other way round, out = h2 W3 (M = the 32 rows), so that each lane holds one output
//   column over 16 rows and the max-pool is 15 maxima and one cross-half exchange.
// Biases enter as the accumulators' initial value.  The pooled features of the group's 32 voxels
// and their 12 PCA features gather in the wave's LDS block; the head 76 -> 64 -> 8 then runs
// transposed on the matrix cores for all 32 voxels at once (N = 32 voxels, the output's 8 rows
// padded to 32).  Rounding points as everywhere: BF16 weights and layer inputs, FP32 bias, ReLU
// and accumulation.
//
// K order of a 64-wide chained operand: position (kb, half, j) of k-block kb (16 wide), lane half
// and element j (0..7) holds feature phi = 32 (kb / 2) + 16 (kb % 2) + 8 (j / 4) + 4 half + j % 4,
// which is where the 32 x 32 accumulator layout keeps it (register 8 (kb % 2) + j of tile kb / 2).
__device__ __forceinline__ int phi_k(int kb, int half, int j) {
    return 32 * (kb >> 1) + 16 * (kb & 1) + 8 * (j >> 2) + 4 * half + (j & 3);
}

constexpr int kGrp = 32;   // voxels per wave group (the head's N)
constexpr int kStage = 16; // voxels whose input rows are staged at once
constexpr int kZld = 80;   // LDS row of the head input (76 used), bf16

struct PnFwdShared {
    bf16x8 a4[2][5][64];  // layer-4 A fragments (W4^T, K padded to 80)
    bf16x8 a5[4][64];     // layer-5 A fragments (W5^T, M padded to 32, K in phi order)
    float b1[kWidth], b2[kWidth], b4[kWidth], b5[kOut];
    __attribute__((aligned(16))) __bf16 z[4][kGrp][kZld];            // per wave: head inputs
    __attribute__((aligned(8))) __bf16 xs[4][kStage][kRows][4];      // per wave: staged input rows
};

__device__ __forceinline__ f32x16 bias_tile(const float *b, int rt, int half) {
    // accumulator register r of row tile rt holds feature 32 rt + 8 (r / 4) + 4 half + r % 4
    f32x16 c;
    const float4 *p = reinterpret_cast<const float4 *>(b + 32 * rt + 4 * half);
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const float4 v = p[2 * q];
        c[4 * q] = v.x;
        c[4 * q + 1] = v.y;
        c[4 * q + 2] = v.z;
        c[4 * q + 3] = v.w;
    }
    return c;
}

// bias already in the accumulators: h = bf16(relu(acc)), as the four k-blocks of the next layer.
// The ReLU is taken after the rounding, on the BF16 bit patterns as signed 16-bit integers
// (negative values and -0 have the sign bit set): rounding keeps the sign, so this equals
// rounding the ReLU.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void relu_operands(const f32x16 d[2], bf16x8 h[4]) {
#pragma unroll
    for (int kb = 0; kb < 4; kb++) {
        u32x4 u;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int r = 8 * (kb & 1) + 2 * i;
            const f32x2 f = {d[kb >> 1][r], d[kb >> 1][r + 1]};
            const bf16x2 b = __builtin_convertvector(f, bf16x2);  // round to nearest even
            const i16x2 m = __builtin_elementwise_max(__builtin_bit_cast(i16x2, b), i16x2{});
            u[i] = __builtin_bit_cast(uint32_t, m);
        }
        h[kb] = __builtin_bit_cast(bf16x8, u);
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_pn_fwd(const float *__restrict__ pts, int64_t n, gsr_voxels V,
                                                const float *__restrict__ W, float *__restrict__ y) {
    __shared__ PnFwdShared S;
    const uint32_t nv = *V.n_voxels;
    const int t = threadIdx.x, lane = __lane_id(), w = t >> 6, half = lane >> 5, l32 = lane & 31;
    const uint32_t nwaves = gridDim.x * 4, gw = blockIdx.x * 4 + w;
    const uint32_t vbeg = (uint32_t)((uint64_t)gw * nv / nwaves), vend = (uint32_t)((uint64_t)(gw + 1) * nv / nwaves);
    // head fragments and biases
    for (int q = t; q < 2 * 5 * 64; q += 256) {
        const int rt = q / 320, kb = (q / 64) % 5, ln = q % 64, h = ln >> 5, o = 32 * rt + (ln & 31);
        bf16x8 f;
        for (int j = 0; j < 8; j++) {
            const int k = 16 * kb + 8 * h + j;
            f[j] = tobf(k < kWidth + kFeat ? W[oW4 + k * kWidth + o] : 0.f);
        }
        S.a4[rt][kb][ln] = f;
    }
    for (int q = t; q < 4 * 64; q += 256) {
        const int kb = q / 64, ln = q % 64, h = ln >> 5, o = ln & 31;
        bf16x8 f;
        for (int j = 0; j < 8; j++) f[j] = tobf(o < kOut ? W[oW5 + phi_k(kb, h, j) * kOut + o] : 0.f);
        S.a5[kb][ln] = f;
    }
    if (t < kWidth) {
        S.b1[t] = W[oB1 + t];
        S.b2[t] = W[oB2 + t];
        S.b4[t] = W[oB4 + t];
    }
    if (t < kOut) S.b5[t] = W[oB5 + t];
    for (int q = lane; q < kGrp * (kZld - kWidth - kFeat); q += 64)
        S.z[w][q / (kZld - kWidth - kFeat)][kWidth + kFeat + q % (kZld - kWidth - kFeat)] = tobf(0.f);
    // shared-layer fragments in registers: W1^T (K = 3 padded to 16), W2^T and W3 in phi order
    bf16x8 a1[2], a2[2][4], b3[2][4];
    for (int rt = 0; rt < 2; rt++) {
        for (int j = 0; j < 8; j++) a1[rt][j] = tobf(half == 0 && j < 3 ? W[oW1 + j * kWidth + 32 * rt + l32] : 0.f);
        for (int kb = 0; kb < 4; kb++)
            for (int j = 0; j < 8; j++) {
                const int k = phi_k(kb, half, j);
                a2[rt][kb][j] = tobf(W[oW2 + k * kWidth + 32 * rt + l32]);
                b3[rt][kb][j] = tobf(W[oW3 + k * kWidth + 32 * rt + l32]);
            }
    }
    const float bb3[2] = {W[oB3 + l32], W[oB3 + 32 + l32]};
    float *const y4 = y + 4 * n;  // outputs 4..7
    __syncthreads();
    __bf16(*Z)[kZld] = S.z[w];
    for (uint32_t vg = vbeg; vg < vend; vg += kGrp) {
        const int ng = (int)min((uint32_t)kGrp, vend - vg);  // voxels of this group
        for (int s0 = 0; s0 < ng; s0 += kStage) {
            // stage the input rows of kStage voxels: lane -> voxel lane / 4, rows 8 (lane % 4) ..
            {
                const int sv = lane >> 2, r0 = 8 * (lane & 3);
                const uint32_t v = vg + s0 + sv;
                float x[8][3];
                if (s0 + sv < ng) {
                    const uint32_t cnt = V.count[v], st = V.start[v];
                    const uint32_t m = cnt < (uint32_t)kRows ? cnt : (uint32_t)kRows;
                    const float m0 = V.mu[v], m1 = V.mu[n + v], m2 = V.mu[2 * n + v];
                    uint32_t p[8];
#pragma unroll
                    for (int i = 0; i < 8; i++) p[i] = V.point_order[st + (uint32_t)(r0 + i) % m];
#pragma unroll
                    for (int i = 0; i < 8; i++) {
                        x[i][0] = (pts[p[i]] - m0) / 0.5f;
                        x[i][1] = (pts[n + p[i]] - m1) / 0.5f;
                        x[i][2] = (pts[2 * n + p[i]] - m2) / 0.5f;
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; i++) x[i][0] = x[i][1] = x[i][2] = 0.f;
                }
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    __bf16 *d = S.xs[w][sv][r0 + i];
                    d[0] = tobf(x[i][0]);
                    d[1] = tobf(x[i][1]);
                    d[2] = tobf(x[i][2]);
                    d[3] = tobf(0.f);
                }
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
            __builtin_amdgcn_wave_barrier();
            const int s1 = min(s0 + kStage, ng);
            for (int s = s0; s < s1; s++) {
                // layer 1: B = the voxel's rows (K = 3 of 16, first half-wave)
                bf16x8 bx = bf16x8{};
                if (half == 0) {
                    // the staged row: three BF16 coordinates and a zero
                    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
                    const bf16x4 xr = *reinterpret_cast<const bf16x4 *>(S.xs[w][s - s0][l32]);
                    bx[0] = xr[0];
                    bx[1] = xr[1];
                    bx[2] = xr[2];
                }
                f32x16 d[2];
#pragma unroll
                for (int rt = 0; rt < 2; rt++)
                    d[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[rt], bx, bias_tile(S.b1, rt, half), 0, 0, 0);
                bf16x8 h[4];
                relu_operands(d, h);
                // layer 2
#pragma unroll
                for (int rt = 0; rt < 2; rt++) {
                    f32x16 acc = bias_tile(S.b2, rt, half);
#pragma unroll
                    for (int kb = 0; kb < 4; kb++)
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2[rt][kb], h[kb], acc, 0, 0, 0);
                    d[rt] = acc;
                }
                relu_operands(d, h);
                // layer 3 (rows = the voxel's points) and the max-pool: relu(max_r acc + b) equals
                // max_r relu(acc + b), rounding included (both maps are monotone)
#pragma unroll
                for (int ct = 0; ct < 2; ct++) {
                    f32x16 acc = f32x16{};
#pragma unroll
                    for (int kb = 0; kb < 4; kb++)
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h[kb], b3[ct][kb], acc, 0, 0, 0);
                    float best = acc[0];
#pragma unroll
                    for (int r = 1; r < 16; r++) best = fmaxf(best, acc[r]);
                    best = fmaxf(best, __shfl_xor(best, 32));
                    if (half == 0) Z[s][32 * ct + l32] = tobf(fmaxf(best + bb3[ct], 0.f));
                }
            }
            __builtin_amdgcn_wave_barrier();  // the next stage overwrites the rows just read
        }
        // the 12 voxel features: log(max(lambda, floor) / 0.25) ascending, then v_min, v_mid, v_max
        if (half == 0) {
            const uint32_t v = vg + l32;
            float f[kFeat];
            for (int q = 0; q < kFeat; q++) f[q] = 0.f;
            if (l32 < ng) {
                for (int q = 0; q < 3; q++) f[q] = logf(fmaxf(V.evals[q * n + v], 0.005f * 0.005f) / 0.25f);
                for (int q = 3; q < kFeat; q++) {
                    const int col = 2 - (q - 3) / 3, row = (q - 3) % 3;  // R_pca columns: v_max, v_mid, v_min
                    f[q] = V.R[(row * 3 + col) * n + v];
                }
            }
            for (int q = 0; q < kFeat; q++) Z[l32][kWidth + q] = tobf(f[q]);
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_wave_barrier();
        // layer 4 (76 -> 64), transposed over the 32 voxels
        f32x16 d[2];
#pragma unroll
        for (int rt = 0; rt < 2; rt++) {
            f32x16 acc = bias_tile(S.b4, rt, half);
#pragma unroll
            for (int kb = 0; kb < 5; kb++) {
                const bf16x8 bz = *reinterpret_cast<const bf16x8 *>(&Z[l32][16 * kb + 8 * half]);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(S.a4[rt][kb][lane], bz, acc, 0, 0, 0);
            }
            d[rt] = acc;
        }
        bf16x8 h[4];
        relu_operands(d, h);
        // layer 5 (64 -> 8; rows 8..31 are padding): lane holds outputs 4 half .. 4 half + 3 of voxel l32
        f32x16 acc = f32x16{};
#pragma unroll
        for (int r = 0; r < 4; r++) acc[r] = S.b5[4 * half + r];
#pragma unroll
        for (int kb = 0; kb < 4; kb++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(S.a5[kb][lane], h[kb], acc, 0, 0, 0);
        const uint32_t v = vg + l32;
        // (one store path per half-wave, each from a uniform base)
        if (l32 < ng && half == 0) {
#pragma unroll
            for (int r = 0; r < 4; r++) y[(int64_t)r * n + v] = acc[r];
        }
        if (l32 < ng && half == 1) {
#pragma unroll
            for (int r = 0; r < 4; r++) y4[(int64_t)r * n + v] = acc[r];
        }
        __builtin_amdgcn_wave_barrier();  // the next group overwrites the head inputs
    }
}

// ---- backward ----------------------------------------------------------------------------------
// One 512-lane workgroup per CU, eight waves, each with eight voxels per turn and its own share of
// the network in registers:
//   A  per voxel, layers 1-3 and the max-pool (one pooled value and row per lane);
//   B  the head 76 -> 64 -> 8, the loss gradient (FP64) and the head's backward, a lane per feature,
//      all eight voxels side by side; the layer-4 weight gradient contracts the block's 64 voxels
//      on the matrix cores (operands gathered transposed in LDS);
//   C  per voxel, layers 1 and 2 again (cheaper than keeping 32 rows of them), the data gradients
//      and the weight gradients of the shared layers.
// A product of 32 rows leaves the matrix cores with one column per lane and 16 rows in its
// registers.  That is an operand of the weight gradients as it stands (they contract rows, in the
// order phi_k on both sides).  The next layer wants one row per lane instead: the same product with
// its operands exchanged gives that, and an exchange between the wave's halves restores the natural
// K order, so every activation and data gradient is the same bits as with row-major staging.
// Neither needs LDS for the activations, and no wave waits for another within A and C.
//
// Bound: latency, at two waves per SIMD (256 registers, 128 of them the two 64 x 64 accumulators):
// per voxel about 2,300 VALU instructions, the chain MFMA -> round -> MFMA and some 150 LDS reads.
// 13.8k voxels take 182 us (the matrix cores' floor is 12 us).  Staging 256 rows of activations in
// LDS held one workgroup of four waves per CU, with about twenty barriers per eight voxels and the
// weight gradients on the VALU: 665 us.
constexpr int kBW = 8;                 // waves per workgroup
constexpr int kBV = 8;                 // voxels per wave and turn
constexpr int kZT = kBW * kBV + 8;     // padded LDS row of the transposed head operands
constexpr int kHead = kWidth + kFeat;  // 76
constexpr int kNB = 4 * kWidth + kOut;  // biases

struct PnBwdWave {
    __attribute__((aligned(16))) float z[kBV][kHead];  // head input (rounded to BF16); da4 (rounded) afterwards
    __attribute__((aligned(16))) float h4[kBV][kWidth];
    __attribute__((aligned(16))) float dy[kBV][kOut];
    __attribute__((aligned(16))) float4 x[kRows];        // one voxel's input rows
    __attribute__((aligned(16))) uint2 xs[kBV][kRows];   // every voxel's, BF16
    __attribute__((aligned(16))) __bf16 dg[kBV][kWidth];
    __attribute__((aligned(16))) uint16_t arg[kBV][kWidth];
};

struct PnBwdShared {
    // operand fragments [tile][k block][lane]: W2, W3 (contracting inputs), and their transposes
    // (contracting outputs)
    bf16x8 w2f[2][4][64], w3f[2][4][64], w2b[2][4][64], w3b[2][4][64];
    float4 w1[kWidth];  // W1 column and b1
    float b2[kWidth], b3[kWidth], b4[kWidth], b5[kOut];
    __attribute__((aligned(16))) float w5[kWidth][kOut];
    __bf16 w4[kHead][kWidth];
    __bf16 w4t[kWidth][kWidth];  // [out][in], the 64 pooled inputs
    __attribute__((aligned(16))) __bf16 zt[96][kZT];       // head inputs of the block's 64 voxels, transposed
    __attribute__((aligned(16))) __bf16 da4t[kWidth][kZT];
    PnBwdWave wave[kBW];
};
static_assert(sizeof(PnBwdShared) <= 160 * 1024 && kBW / 2 * 38 * 64 * 16 <= 160 * 1024, "one workgroup's LDS");

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
    const f32x2 f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));  // round to nearest even
}

// 16 accumulators as two 8-element operands (order phi_k)
__device__ __forceinline__ void pack16(const float v[16], bf16x8 out[2]) {
#pragma unroll
    for (int k = 0; k < 2; k++) {
        u32x4 u;
#pragma unroll
        for (int i = 0; i < 4; i++) u[i] = pk_bf16(v[8 * k + 2 * i], v[8 * k + 2 * i + 1]);
        out[k] = __builtin_bit_cast(bf16x8, u);
    }
}

// From phi_k order to natural K order (k = 16 kb + 8 half + j): the upper half's first four elements
// change places with the lower half's last four.
__device__ __forceinline__ bf16x8 natural_k(bf16x8 v) {
    u32x4 u = __builtin_bit_cast(u32x4, v);
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const auto r = __builtin_amdgcn_permlane32_swap(u[i], u[2 + i], false, false);
        u[i] = r[0];
        u[2 + i] = r[1];
    }
    return __builtin_bit_cast(bf16x8, u);
}

// rows 8 (r / 4) + 4 half + r % 4 of the accumulators
__device__ __forceinline__ int tile_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

__device__ __forceinline__ float4 unpack_row(uint2 u) {
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), 0.f);
}

// Both 16-bit halves of w where the mask's half is not zero (zero elsewhere), and where it is zero.
__device__ __forceinline__ uint32_t keep_where(uint32_t w, uint32_t mask) {
    const u16x2 one = {1, 1};
    const u16x2 m = __builtin_elementwise_min(__builtin_bit_cast(u16x2, mask), one);
    return w & __builtin_bit_cast(uint32_t, u16x2{} - m);
}
__device__ __forceinline__ uint32_t keep_where_zero(uint32_t w, uint32_t mask) {
    const u16x2 one = {1, 1};
    const u16x2 m = __builtin_elementwise_min(__builtin_bit_cast(u16x2, mask), one);
    return w & __builtin_bit_cast(uint32_t, m - one);
}

// layer 1 of the lane's row, natural K order
__device__ __forceinline__ void layer1_rows(const float4 *w1, const float4 x, int half, bf16x8 h[4]) {
#pragma unroll
    for (int kb = 0; kb < 4; kb++) {
        u32x4 u;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            float a[2];
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const float4 c = w1[16 * kb + 8 * half + 2 * i + e];
                a[e] = __builtin_fmaf(x.z, c.z, __builtin_fmaf(x.y, c.y, __builtin_fmaf(x.x, c.x, c.w)));
                a[e] = fmaxf(a[e], 0.f);
            }
            u[i] = pk_bf16(a[0], a[1]);
        }
        h[kb] = __builtin_bit_cast(bf16x8, u);
    }
}

// a 32-row product with a 64-wide layer: column tile ct per lane column (rows in the registers), or
// with the operands exchanged row per lane
__device__ __forceinline__ f32x16 cols_of(const bf16x8 h[4], const bf16x8 (*w)[64], int lane) {
    f32x16 acc = f32x16{};
#pragma unroll
    for (int kb = 0; kb < 4; kb++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h[kb], w[kb][lane], acc, 0, 0, 0);
    return acc;
}
__device__ __forceinline__ f32x16 rows_of(const bf16x8 h[4], const bf16x8 (*w)[64], int lane) {
    f32x16 acc = f32x16{};
#pragma unroll
    for (int kb = 0; kb < 4; kb++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[kb][lane], h[kb], acc, 0, 0, 0);
    return acc;
}

// layer 2 with one row per lane: relu(h1 W2 + b2) of outputs 32 t .. 32 t + 31 in phi_k order
__device__ __forceinline__ void layer2_rows(const PnBwdShared &S, const bf16x8 h1[4], int t, int lane, int half,
                                            bf16x8 out[2]) {
    const f32x16 acc = rows_of(h1, S.w2f[t], lane);
    float v[16];
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = fmaxf(acc[r] + S.b2[32 * t + tile_row(r, half)], 0.f);
    pack16(v, out);
}

// dL/dy of one voxel: KL(N(0, Sp) || N(0, St)) + 0.1 |sigmoid(omega) - o_t|, scaled by inv_count
__device__ void loss_grad(const float y[8], const double St[6], double ot, double scale, float dy[8], double *lval) {
    double s[3] = {y[0], y[1], y[2]}, q[4] = {y[3], y[4], y[5], y[6]}, om = y[7];
    const double qn = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const double w = q[0] / qn, x = q[1] / qn, yy = q[2] / qn, z = q[3] / qn;
    const double R[9] = {1 - 2 * (yy * yy + z * z), 2 * (x * yy - w * z), 2 * (x * z + w * yy),
                         2 * (x * yy + w * z), 1 - 2 * (x * x + z * z), 2 * (yy * z - w * x),
                         2 * (x * z - w * yy), 2 * (yy * z + w * x), 1 - 2 * (x * x + yy * yy)};
    // A = St^-1 (symmetric; St = [[a, b, c], [b, d, e], [c, e, f]])
    const double a = St[0], b = St[1], c = St[2], d = St[3], e = St[4], f = St[5];
    const double c00 = d * f - e * e, c01 = c * e - b * f, c02 = b * e - c * d;
    const double c11 = a * f - c * c, c12 = b * c - a * e, c22 = a * d - b * b;
    const double det = a * c00 + b * c01 + c * c02;
    const double A[9] = {c00 / det, c01 / det, c02 / det, c01 / det, c11 / det, c12 / det, c02 / det, c12 / det,
                         c22 / det};
    double AR[9];
    for (int i = 0; i < 3; i++)
        for (int j = 0; j < 3; j++) AR[i * 3 + j] = A[i * 3] * R[j] + A[i * 3 + 1] * R[3 + j] + A[i * 3 + 2] * R[6 + j];
    double ds[3], dR[9], tr = 0.0;
    for (int j = 0; j < 3; j++) {
        const double e2 = exp(2 * s[j]);
        const double rar = R[j] * AR[j] + R[3 + j] * AR[3 + j] + R[6 + j] * AR[6 + j];
        tr += e2 * rar;
        ds[j] = e2 * rar - 1.0;
        for (int i = 0; i < 3; i++) dR[i * 3 + j] = e2 * AR[i * 3 + j];
    }
    // d R / d (w, x, y, z) of the unit quaternion, contracted with dR
    const double dqh[4] = {
        dR[1] * (-2 * z) + dR[2] * (2 * yy) + dR[3] * (2 * z) + dR[5] * (-2 * x) + dR[6] * (-2 * yy) + dR[7] * (2 * x),
        dR[1] * (2 * yy) + dR[2] * (2 * z) + dR[3] * (2 * yy) + dR[4] * (-4 * x) + dR[5] * (-2 * w) + dR[6] * (2 * z) +
            dR[7] * (2 * w) + dR[8] * (-4 * x),
        dR[0] * (-4 * yy) + dR[1] * (2 * x) + dR[2] * (2 * w) + dR[3] * (2 * x) + dR[5] * (2 * z) + dR[6] * (-2 * w) +
            dR[7] * (2 * z) + dR[8] * (-4 * yy),
        dR[0] * (-4 * z) + dR[1] * (-2 * w) + dR[2] * (2 * x) + dR[3] * (2 * w) + dR[4] * (-4 * z) + dR[5] * (2 * yy) +
            dR[6] * (2 * x) + dR[7] * (2 * yy)};
    const double qh[4] = {w, x, yy, z};
    const double pr = qh[0] * dqh[0] + qh[1] * dqh[1] + qh[2] * dqh[2] + qh[3] * dqh[3];
    const double sg = 1.0 / (1.0 + exp(-om));
    const double sgn = (sg > ot) ? 1.0 : ((sg < ot) ? -1.0 : 0.0);
    for (int j = 0; j < 3; j++) dy[j] = (float)(scale * ds[j]);
    for (int k = 0; k < 4; k++) dy[3 + k] = (float)(scale * (dqh[k] - qh[k] * pr) / qn);
    dy[7] = (float)(scale * 0.1 * sgn * sg * (1 - sg));
    *lval = scale * (0.5 * (tr - 3.0 + log(det) - 2.0 * (s[0] + s[1] + s[2])) + 0.1 * fabs(sg - ot));
}

__global__ __launch_bounds__(64 * kBW) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_pn_bwd(
    const float *__restrict__ pts, int64_t n, gsr_voxels V, const float *__restrict__ W,
    const float *__restrict__ cov_t, const float *__restrict__ o_t, const uint8_t *__restrict__ tmask, float inv_count,
    float *__restrict__ part, float *__restrict__ bias_part, double *__restrict__ loss) {
    __shared__ union {
        PnBwdShared s;
        float4 fold[kBW / 2][38 * 64];  // after the last turn: half of the waves' sums
    } U;
    PnBwdShared &S = U.s;
    const uint32_t nv = *V.n_voxels;
    const int t = threadIdx.x, lane = __lane_id(), w = t >> 6, half = lane >> 5, l32 = lane & 31;
    for (int q = t; q < 2 * 4 * 64; q += 64 * kBW) {
        const int ct = q >> 8, kb = (q >> 6) & 3, ln = q & 63;
        const int o = 32 * ct + (ln & 31), k0 = 16 * kb + 8 * (ln >> 5);
        bf16x8 f2, f3, g2, g3;
        for (int j = 0; j < 8; j++) {
            f2[j] = tobf(W[oW2 + (k0 + j) * kWidth + o]);
            f3[j] = tobf(W[oW3 + (k0 + j) * kWidth + o]);
            g2[j] = tobf(W[oW2 + o * kWidth + k0 + j]);
            g3[j] = tobf(W[oW3 + o * kWidth + k0 + j]);
        }
        S.w2f[ct][kb][ln] = f2;
        S.w3f[ct][kb][ln] = f3;
        S.w2b[ct][kb][ln] = g2;
        S.w3b[ct][kb][ln] = g3;
    }
    for (int q = t; q < kHead * kWidth; q += 64 * kBW) {
        const __bf16 v = tobf(W[oW4 + q]);
        S.w4[q / kWidth][q % kWidth] = v;
        if (q < kWidth * kWidth) S.w4t[q % kWidth][q / kWidth] = v;
    }
    if (t < kWidth) {
        S.w1[t] = make_float4(fbf(tobf(W[oW1 + t])), fbf(tobf(W[oW1 + kWidth + t])), fbf(tobf(W[oW1 + 2 * kWidth + t])),
                              W[oB1 + t]);
        S.b2[t] = W[oB2 + t];
        S.b3[t] = W[oB3 + t];
        S.b4[t] = W[oB4 + t];
    }
    if (t < kOut) S.b5[t] = W[oB5 + t];
    S.w5[t / kOut][t % kOut] = fbf(tobf(W[oW5 + t]));
    for (int q = t; q < (96 - kHead) * kZT; q += 64 * kBW) S.zt[kHead + q / kZT][q % kZT] = tobf(0.f);
    static_assert(kWidth * kOut == 64 * kBW, "one W5 entry per lane");
    __syncthreads();

    PnBwdWave &B = S.wave[w];
    f32x16 gW2[2][2], gW3[2][2], gW4 = f32x16{};
    for (int i = 0; i < 4; i++) gW2[i >> 1][i & 1] = gW3[i >> 1][i & 1] = f32x16{};
    float gW1[2][3] = {}, gb1[2] = {}, gb2[2] = {}, gb3 = 0.f, gb4 = 0.f, gb5 = 0.f, gW5[kOut] = {};
    double lsum = 0.0;
    const uint32_t turn = gridDim.x * kBW * kBV;
    for (uint32_t first = blockIdx.x * kBW * kBV; first < nv; first += turn) {
        const uint32_t v0 = first + w * kBV;  // (a wave past the last voxel runs on zeros)
        // the voxels' input rows: four independent chains of dependent loads per lane
#pragma unroll
        for (int i = 0; i < kBV * kRows / 64; i++) {
            const int v = 2 * i + half;
            float x[3] = {0.f, 0.f, 0.f};
            if (v0 + v < nv) {
                const uint32_t cnt = V.count[v0 + v], m = cnt < (uint32_t)kRows ? cnt : (uint32_t)kRows;
                const uint32_t p = V.point_order[V.start[v0 + v] + (uint32_t)l32 % m];
#pragma unroll
                for (int c = 0; c < 3; c++) x[c] = (pts[c * n + p] - V.mu[c * n + v0 + v]) / 0.5f;
            }
            B.xs[v][l32] = make_uint2(pk_bf16(x[0], x[1]), pk_bf16(x[2], 0.f));
        }
        __builtin_amdgcn_wave_barrier();
        // A: the pooled features
#pragma unroll 1
        for (int v = 0; v < kBV; v++) {
            __asm__ __volatile__("" ::: "memory");  // the operand fragments are read again, not kept in 128 registers
            const float4 x = unpack_row(B.xs[v][l32]);
            bf16x8 h1[4], h2[4];
            layer1_rows(S.w1, x, half, h1);
#pragma unroll
            for (int ot = 0; ot < 2; ot++) layer2_rows(S, h1, ot, lane, half, h2 + 2 * ot);
#pragma unroll
            for (int kb = 0; kb < 4; kb++) h2[kb] = natural_k(h2[kb]);
#pragma unroll
            for (int ct = 0; ct < 2; ct++) {
                const f32x16 acc = cols_of(h2, S.w3f[ct], lane);
                const int col = 32 * ct + l32;
                const float bb = S.b3[col];
                float best = -1.f;
                int brow = 0;
#pragma unroll
                for (int r = 0; r < 16; r++) {  // rows ascend: the first maximum is the lowest row
                    const float h = fmaxf(acc[r] + bb, 0.f);
                    if (h > best) best = h, brow = tile_row(r, half);
                }
                const float ob = __shfl_xor(best, 32);
                const int orow = __shfl_xor(brow, 32);
                if (ob > best || (ob == best && orow < brow)) best = ob, brow = orow;
                if (half == ct) {
                    B.z[v][col] = best;
                    B.arg[v][col] = (uint16_t)brow;
                }
            }
        }
        // voxel features (12): log(max(lambda, floor) / 0.25) ascending, then v_min, v_mid, v_max
        for (int q = lane; q < kBV * kFeat; q += 64) {
            const int v = q / kFeat, f = q % kFeat;
            const uint32_t vg = v0 + v;
            float val = 0.f;
            if (vg < nv) {
                const int col = 2 - (f - 3) / 3, row = (f - 3) % 3;  // R_pca columns: v_max, v_mid, v_min
                val = f < 3 ? logf(fmaxf(V.evals[f * n + vg], 0.005f * 0.005f) / 0.25f) : V.R[(row * 3 + col) * n + vg];
            }
            B.z[v][kWidth + f] = fbf(tobf(val));
        }
        __builtin_amdgcn_wave_barrier();
        // B: the head, lane = feature.  g: the pooled value, kept for its ReLU; z holds it rounded
        float g[kBV], a4[kBV];
        u32x4 zp;
#pragma unroll
        for (int v = 0; v < kBV; v++) {
            g[v] = B.z[v][lane];
            a4[v] = S.b4[lane];
        }
#pragma unroll
        for (int i = 0; i < 4; i++) zp[i] = pk_bf16(g[2 * i], g[2 * i + 1]);
        *reinterpret_cast<u32x4 *>(&S.zt[lane][kBV * w]) = zp;
#pragma unroll
        for (int v = 0; v < kBV; v++) B.z[v][lane] = fbf(tobf(g[v]));
        if (lane < kFeat) {
#pragma unroll
            for (int i = 0; i < 4; i++) zp[i] = pk_bf16(B.z[2 * i][kWidth + lane], B.z[2 * i + 1][kWidth + lane]);
            *reinterpret_cast<u32x4 *>(&S.zt[kWidth + lane][kBV * w]) = zp;
        }
        __builtin_amdgcn_wave_barrier();
        for (int k = 0; k < kHead; k += 4) {
            float wk[4];
#pragma unroll
            for (int i = 0; i < 4; i++) wk[i] = fbf(S.w4[k + i][lane]);
#pragma unroll
            for (int v = 0; v < kBV; v++) {
                const float4 z = *reinterpret_cast<const float4 *>(&B.z[v][k]);
                a4[v] = __builtin_fmaf(z.x, wk[0], a4[v]);
                a4[v] = __builtin_fmaf(z.y, wk[1], a4[v]);
                a4[v] = __builtin_fmaf(z.z, wk[2], a4[v]);
                a4[v] = __builtin_fmaf(z.w, wk[3], a4[v]);
            }
        }
        float h4[kBV];
#pragma unroll
        for (int v = 0; v < kBV; v++) {
            h4[v] = fbf(tobf(fmaxf(a4[v], 0.f)));
            B.h4[v][lane] = h4[v];
        }
        __builtin_amdgcn_wave_barrier();
        {
            const int v = lane >> 3, j = lane & 7;
            float y = S.b5[j];
            for (int k = 0; k < kWidth; k++) y = __builtin_fmaf(B.h4[v][k], S.w5[k][j], y);
            B.dy[v][j] = y;
        }
        __builtin_amdgcn_wave_barrier();
        if (lane < kBV) {  // loss gradient, one lane per voxel
            const uint32_t v = v0 + lane;
            float y[kOut], dy[kOut] = {};
            for (int j = 0; j < kOut; j++) y[j] = B.dy[lane][j];
            if (v < nv && (!tmask || tmask[v])) {
                double St[6], lv;
                for (int k = 0; k < 6; k++) St[k] = cov_t[k * n + v];
                loss_grad(y, St, o_t[v], inv_count, dy, &lv);
                lsum += lv;
            }
            for (int j = 0; j < kOut; j++) B.dy[lane][j] = dy[j];
        }
        __builtin_amdgcn_wave_barrier();
        // head backward: layer 5 (64 -> 8) and layer 4 (76 -> 64)
        if (lane < kOut)
            for (int v = 0; v < kBV; v++) gb5 += B.dy[v][lane];
        float w5[kOut], da4[kBV];
#pragma unroll
        for (int j = 0; j < kOut; j++) w5[j] = S.w5[lane][j];
#pragma unroll
        for (int v = 0; v < kBV; v++) {
            float dh = 0.f;
#pragma unroll
            for (int j = 0; j < kOut; j++) {
                const float d = fbf(tobf(B.dy[v][j]));
                gW5[j] = __builtin_fmaf(h4[v], d, gW5[j]);
                dh = __builtin_fmaf(d, w5[j], dh);
            }
            dh = a4[v] > 0.f ? dh : 0.f;
            gb4 += dh;
            da4[v] = dh;
        }
#pragma unroll
        for (int i = 0; i < 4; i++) zp[i] = pk_bf16(da4[2 * i], da4[2 * i + 1]);
        *reinterpret_cast<u32x4 *>(&S.da4t[lane][kBV * w]) = zp;
#pragma unroll
        for (int v = 0; v < kBV; v++) B.z[v][lane] = fbf(tobf(da4[v]));
        __builtin_amdgcn_wave_barrier();
        float dg[kBV] = {};
        for (int j = 0; j < kWidth; j += 4) {
            float wj[4];
#pragma unroll
            for (int i = 0; i < 4; i++) wj[i] = fbf(S.w4t[j + i][lane]);
#pragma unroll
            for (int v = 0; v < kBV; v++) {
                const float4 d = *reinterpret_cast<const float4 *>(&B.z[v][j]);
                dg[v] = __builtin_fmaf(d.x, wj[0], dg[v]);
                dg[v] = __builtin_fmaf(d.y, wj[1], dg[v]);
                dg[v] = __builtin_fmaf(d.z, wj[2], dg[v]);
                dg[v] = __builtin_fmaf(d.w, wj[3], dg[v]);
            }
        }
#pragma unroll
        for (int v = 0; v < kBV; v++) {
            dg[v] = g[v] > 0.f ? dg[v] : 0.f;  // through the ReLU at the pooled maximum
            gb3 += dg[v];
            B.dg[v][lane] = tobf(dg[v]);
        }
        // layer-4 weight gradient of the block's 64 voxels: waves 0..5 take one 32 x 32 tile each
        __syncthreads();
        if (w < 6) {
#pragma unroll
            for (int kb = 0; kb < 4; kb++) {
                const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&S.zt[32 * (w >> 1) + l32][16 * kb + 8 * half]);
                const bf16x8 b = *reinterpret_cast<const bf16x8 *>(&S.da4t[32 * (w & 1) + l32][16 * kb + 8 * half]);
                gW4 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, gW4, 0, 0, 0);
            }
        }
        __syncthreads();  // the next turn overwrites zt and da4t
        // C: the shared layers' backward
#pragma unroll 1
        for (int v = 0; v < kBV; v++) {
            __asm__ __volatile__("" ::: "memory");
            const float4 x = unpack_row(B.xs[v][l32]);
            __builtin_amdgcn_wave_barrier();
            if (half == 0) B.x[l32] = x;
            __builtin_amdgcn_wave_barrier();
            bf16x8 h1[4], h2n[2][2], h2r[2][2];
            layer1_rows(S.w1, x, half, h1);
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const f32x16 acc = cols_of(h1, S.w2f[c], lane);
                const float bb = S.b2[32 * c + l32];
                float f[16];
#pragma unroll
                for (int r = 0; r < 16; r++) f[r] = fmaxf(acc[r] + bb, 0.f);
                pack16(f, h2n[c]);
                layer2_rows(S, h1, c, lane, half, h2r[c]);
            }
            // the pooled gradient, one row per channel: as rows (natural K order) ...
            bf16x8 d3[4], d3n[2];
            const uint32_t row2 = (uint32_t)l32 * 0x10001u;
#pragma unroll
            for (int kb = 0; kb < 4; kb++) {
                const int k0 = 16 * kb + 8 * half;
                u32x4 d = *reinterpret_cast<const u32x4 *>(&B.dg[v][k0]);
                const u32x4 ar = *reinterpret_cast<const u32x4 *>(&B.arg[v][k0]);
#pragma unroll
                for (int i = 0; i < 4; i++) d[i] = keep_where_zero(d[i], ar[i] ^ row2);
                d3[kb] = __builtin_bit_cast(bf16x8, d);
            }
            // ... and as columns, for the layer-3 weight gradient
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const uint32_t d = (uint32_t)__builtin_bit_cast(uint16_t, B.dg[v][32 * c + l32]) * 0x10001u;
                const uint32_t at = (((uint32_t)B.arg[v][32 * c + l32] - 4u * half) & 0xffffu) * 0x10001u;
#pragma unroll
                for (int k = 0; k < 2; k++) {
                    u32x4 u;
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const int r = tile_row(8 * k + 2 * i, 0);
                        u[i] = keep_where_zero(d, at ^ (uint32_t)(r | (r + 1) << 16));
                    }
                    d3n[k] = __builtin_bit_cast(bf16x8, u);
                }
#pragma unroll
                for (int m = 0; m < 2; m++)
#pragma unroll
                    for (int k = 0; k < 2; k++)
                        gW3[m][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h2n[m][k], d3n[k], gW3[m][c], 0, 0, 0);
            }
            // through layer 3 and layer 2's ReLU
            bf16x8 d2[4], d2n[2][2];
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const f32x16 acc = cols_of(d3, S.w3b[c], lane);
                float f[16];
#pragma unroll
                for (int k = 0; k < 2; k++) {
                    const u32x4 h = __builtin_bit_cast(u32x4, h2n[c][k]);  // (activations are not negative)
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const int r = 8 * k + 2 * i;
                        f[r] = (uint16_t)h[i] != 0 ? acc[r] : 0.f;
                        f[r + 1] = h[i] > 0xffffu ? acc[r + 1] : 0.f;
                        gb2[c] += f[r] + f[r + 1];
                    }
                }
                pack16(f, d2n[c]);
                const f32x16 row = rows_of(d3, S.w3b[c], lane);
#pragma unroll
                for (int k = 0; k < 2; k++) {
                    const u32x4 h = __builtin_bit_cast(u32x4, h2r[c][k]);
                    u32x4 u;
#pragma unroll
                    for (int i = 0; i < 4; i++) u[i] = keep_where(pk_bf16(row[8 * k + 2 * i], row[8 * k + 2 * i + 1]), h[i]);
                    d2[2 * c + k] = __builtin_bit_cast(bf16x8, u);
                }
            }
#pragma unroll
            for (int kb = 0; kb < 4; kb++) d2[kb] = natural_k(d2[kb]);
            // through layer 2 and layer 1's ReLU; layer 1's output again, one column per lane
#pragma unroll
            for (int m = 0; m < 2; m++) {
                const float4 c = S.w1[32 * m + l32];
                const f32x16 acc = cols_of(d2, S.w2b[m], lane);
                float f[16];
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const float4 xr = B.x[tile_row(r, half)];
                    f[r] = fmaxf(__builtin_fmaf(xr.z, c.z, __builtin_fmaf(xr.y, c.y, __builtin_fmaf(xr.x, c.x, c.w))), 0.f);
                    const float da = fbf(tobf(f[r])) > 0.f ? acc[r] : 0.f;
                    gb1[m] += da;
                    const float db = fbf(tobf(da));
                    gW1[m][0] = __builtin_fmaf(xr.x, db, gW1[m][0]);
                    gW1[m][1] = __builtin_fmaf(xr.y, db, gW1[m][1]);
                    gW1[m][2] = __builtin_fmaf(xr.z, db, gW1[m][2]);
                }
                bf16x8 h1n[2];
                pack16(f, h1n);
#pragma unroll
                for (int e = 0; e < 2; e++)
#pragma unroll
                    for (int k = 0; k < 2; k++)
                        gW2[m][e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h1n[k], d2n[e][k], gW2[m][e], 0, 0, 0);
            }
        }
    }
    // the workgroup's gradient, in the flat weight layout: the waves' sums folded pairwise through LDS
    // (4 to 0, 5 to 1, ..., then 2 to 0, 3 to 1, then 1 to 0)
    lsum = wave_sum_d(lsum);
    if (lane == 0 && lsum != 0.0) atomicAdd(loss, lsum);
    for (int m = 0; m < 2; m++) {
        for (int k = 0; k < 3; k++) gW1[m][k] += __shfl_xor(gW1[m][k], 32);
        gb1[m] += __shfl_xor(gb1[m], 32);
        gb2[m] += __shfl_xor(gb2[m], 32);
    }
    if (bias_part) {  // this wave's bias sums (b1 b2 b3 b4 b5), for the ordered sum
        float *Q = bias_part + (int64_t)(blockIdx.x * kBW + w) * kNB;
        if (half == 0)
            for (int m = 0; m < 2; m++) {
                Q[32 * m + l32] = gb1[m];
                Q[kWidth + 32 * m + l32] = gb2[m];
            }
        Q[2 * kWidth + lane] = gb3;
        Q[3 * kWidth + lane] = gb4;
        if (lane < kOut) Q[4 * kWidth + lane] = gb5;
    }
    // (four sums at a time: 16-byte LDS accesses)
    auto each = [&](auto &&f) {
        int k = 0;
        auto four = [&](float &a, float &b, float &c, float &d) {
            const float4 v = f(k++, make_float4(a, b, c, d));
            a = v.x, b = v.y, c = v.z, d = v.w;
        };
        auto tile = [&](f32x16 &g) {
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                const float4 v = f(k++, make_float4(g[r], g[r + 1], g[r + 2], g[r + 3]));
                g[r] = v.x, g[r + 1] = v.y, g[r + 2] = v.z, g[r + 3] = v.w;
            }
        };
#pragma unroll
        for (int i = 0; i < 4; i++) {
            tile(gW2[i >> 1][i & 1]);
            tile(gW3[i >> 1][i & 1]);
        }
        four(gW5[0], gW5[1], gW5[2], gW5[3]);
        four(gW5[4], gW5[5], gW5[6], gW5[7]);
        four(gW1[0][0], gW1[0][1], gW1[0][2], gb1[0]);
        four(gW1[1][0], gW1[1][1], gW1[1][2], gb1[1]);
        four(gb2[0], gb2[1], gb3, gb4);
        float none = 0.f;
        four(gb5, none, none, none);
    };
    for (int fold = kBW / 2; fold > 0; fold >>= 1) {
        __syncthreads();
        float4 *F = U.fold[w & (fold - 1)];
        if (w >= fold && w < 2 * fold) each([&](int k, float4 v) { return F[k * 64 + lane] = v; });
        __syncthreads();
        if (w < fold) each([&](int k, float4 v) {
            const float4 o = F[k * 64 + lane];
            return make_float4(v.x + o.x, v.y + o.y, v.z + o.z, v.w + o.w);
        });
    }
    float *P = part + (int64_t)blockIdx.x * kNW;
    if (w < 6) {
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const int k = 32 * (w >> 1) + tile_row(r, half);
            if (k < kHead) P[oW4 + k * kWidth + 32 * (w & 1) + l32] = gW4[r];
        }
    }
    if (w != 0) return;
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int at = (32 * m + tile_row(r, half)) * kWidth + 32 * c + l32;
                P[oW2 + at] = gW2[m][c][r];
                P[oW3 + at] = gW3[m][c][r];
            }
    for (int j = 0; j < kOut; j++) P[oW5 + lane * kOut + j] = gW5[j];
    if (half == 0)
        for (int m = 0; m < 2; m++) {
            for (int k = 0; k < 3; k++) P[oW1 + k * kWidth + 32 * m + l32] = gW1[m][k];
            P[oB1 + 32 * m + l32] = gb1[m];
            P[oB2 + 32 * m + l32] = gb2[m];
        }
    P[oB3 + lane] = gb3;
    P[oB4 + lane] = gb4;
    if (lane < kOut) P[oB5 + lane] = gb5;
}

// Fixed-order sums of the partial gradients.  Blocks below kReduceBlocks: 64 weights each over the nb
// workgroups' rows, four lanes per weight so that several loads are in flight everywhere (one lane per
// weight over 512 rows took 120 us; this takes 5, 13 with the biases).  With bias_part, the blocks above take 8 biases
// each, in FP32: wave k's sum (of tiles k, k + 8 nb, ... of eight voxels, in that order) belongs to share k mod
// `blocks`, a share adds its waves in order, and the shares add up one after another.  While no wave takes a second
// tile (64 voxels a workgroup: 16,384 on 256 CUs) that is the order in which `blocks` workgroups of one tile at a
// time would have summed them: the biases enter every activation unrounded, and a training run on such a scene
// steps through the same biases whatever the number of CUs.  Beyond, the order is fixed for a number of CUs and `blocks`.
static_assert(kNB % 8 == 0, "whole blocks of biases");
constexpr int kReduceBlocks = (kNW + 63) / 64, kShares = 512, kShareCols = 8;
__global__ __launch_bounds__(256) void k_pn_reduce(const float *__restrict__ part, int nb,
                                                   const float *__restrict__ bias_part, int blocks,
                                                   float *__restrict__ grad) {
    __shared__ float s_share[kShares][kShareCols];
    __shared__ double s_sum[4][64];
    if (blockIdx.x >= kReduceBlocks) {
        const int c = threadIdx.x % kShareCols, q = (blockIdx.x - kReduceBlocks) * kShareCols + c;
        const int waves = nb * kBW, shares = blocks < waves ? blocks : waves;
        float total = 0.f;
        for (int r0 = 0; r0 < shares; r0 += kShares) {
            const int cnt = shares - r0 < kShares ? shares - r0 : kShares;
#pragma unroll 4
            for (int r = threadIdx.x / kShareCols; r < cnt; r += 256 / kShareCols) {
                float a = 0.f;
#pragma unroll 4
                for (int k = r0 + r; k < waves; k += shares) a += bias_part[(int64_t)k * kNB + q];
                s_share[r][c] = a;
            }
            __syncthreads();
            if (threadIdx.x < kShareCols) {
#pragma unroll 16
                for (int r = 0; r < cnt; r++) total += s_share[r][c];
            }
            __syncthreads();
        }
        if (threadIdx.x < kShareCols)
            grad[(q < 64 ? oB1 : (q < 128 ? oB2 - 64 : (q < 192 ? oB3 - 128 : (q < 256 ? oB4 - 192 : oB5 - 256)))) + q] = total;
        return;
    }
    const int q = blockIdx.x * 64 + (threadIdx.x & 63), g = threadIdx.x >> 6;
    const bool bias = (q >= oB1 && q < oW2) || (q >= oB2 && q < oW3) || (q >= oB3 && q < oW4) || (q >= oB4 && q < oW5) || q >= oB5;
    double s = 0.0;
    if (q < kNW) {
#pragma unroll 8
        for (int b = g; b < nb; b += 4) s += part[(int64_t)b * kNW + q];
    }
    s_sum[g][threadIdx.x & 63] = s;
    __syncthreads();
    if (g == 0 && q < kNW && !(bias && bias_part))
        grad[q] = (float)((s_sum[0][threadIdx.x] + s_sum[1][threadIdx.x]) + (s_sum[2][threadIdx.x] + s_sum[3][threadIdx.x]));
}

}  // namespace gsr

using namespace gsr;

extern "C" int gsr_pointnet_weight_count(void) { return kNW; }

extern "C" gsr_status gsr_pointnet_fwd_launch(const float *pts, int64_t n, const gsr_voxels *vox, const float *W,
                                              float *y, hipStream_t st) {
    if (n == 0) return GSR_OK;
    // persistent: three workgroups per compute unit (the LDS allows three), each wave loops over
    // groups of 32 voxels
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    const int64_t blocks = ceil_div(ceil_div(n, kGrp), 4);
    const int nb = (int)(blocks < 3 * cus ? blocks : 3 * cus);
    k_pn_fwd<<<nb, 256, 0, st>>>(pts, n, *vox, W, y);
    return last_launch();
}

extern "C" size_t gsr_pointnet_bwd_ws_bytes(int blocks) { return (size_t)blocks * kNW * sizeof(float) + 256; }

extern "C" gsr_status gsr_pointnet_bwd_launch(const float *pts, int64_t n, const gsr_voxels *vox, const float *W,
                                              const float *cov_t, const float *o_t, const uint8_t *tmask,
                                              float inv_count, int blocks, float *grad, double *loss, void *ws,
                                              hipStream_t st) {
    float *part = static_cast<float *>(ws);
    // one workgroup fills a CU's LDS: more of them would only start later
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    const int nb = blocks < cus ? blocks : cus;
    // the rows of the workgroups not launched hold the waves' bias sums (with too few of them the
    // biases are added like the weights)
    float *bias_part = (int64_t)(blocks - nb) * kNW >= (int64_t)nb * kBW * kNB ? part + (int64_t)nb * kNW : nullptr;
    k_pn_bwd<<<nb, 64 * kBW, 0, st>>>(pts, n, *vox, W, cov_t, o_t, tmask, inv_count, part, bias_part, loss);
    k_pn_reduce<<<kReduceBlocks + (bias_part ? kNB / kShareCols : 0), 256, 0, st>>>(part, nb, bias_part, blocks, grad);
    return last_launch();
}

