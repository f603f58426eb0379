// Surrogate network of the statistical regime: an ensemble of K multilayer perceptrons
// 6 -> 256 -> 256 -> 256 -> 1 (SiLU between layers) that maps the features of a bin pair
// to its log yield. Weights are kept in FP32 (master copy, Adam moments) and used in
// BF16; every product runs on the matrix cores (v_mfma_f32_16x16x32_bf16: BF16 operands,
// FP32 accumulation). Training (forward, mean-squared-error loss, backward, Adam) and
// inference run in the kernels of this file.
//
// A training step of all members is three launches: forward and backward of one 64-row tile
// of a minibatch per workgroup (k_mlp_fwd_bwd), the weight gradients (k_mlp_wgrad), and the sum
// of their slices with Adam (k_mlp_update).
//
// Rounding points, which the CPU reference reproduces: the network input, every hidden
// activation and every back-propagated pre-activation gradient are rounded to BF16
// (round to nearest, ties to even) where they enter a product; bias additions, the
// activation and its derivative, the loss and Adam are FP32.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <random>
#include <vector>

#include "tril_internal.h"

namespace tril {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ float sigmoidf_(float z) { return 1.0f / (1.0f + expf(-z)); }

// Inference-only SiLU from the hardware exponential and reciprocal (about 1 ulp of FP32
// each); its result is rounded to BF16 (8 significant bits) right after.
__device__ __forceinline__ float silu_fast(float z) {
    return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z));
}

// Parameter offsets of one member in its flat FP32 vector (W row-major [out][in]).
constexpr int64_t kOffW1 = 0;
constexpr int64_t kOffB1 = kOffW1 + (int64_t)kMlpHidden * kMlpIn;
constexpr int64_t kOffW2 = kOffB1 + kMlpHidden;
constexpr int64_t kOffB2 = kOffW2 + (int64_t)kMlpHidden * kMlpHidden;
constexpr int64_t kOffW3 = kOffB2 + kMlpHidden;
constexpr int64_t kOffB3 = kOffW3 + (int64_t)kMlpHidden * kMlpHidden;
constexpr int64_t kOffW4 = kOffB3 + kMlpHidden;
constexpr int64_t kOffB4 = kOffW4 + kMlpHidden;
static_assert(kOffB4 + 1 == kMlpParams, "parameter count");

// The BF16 hidden-layer weights are stored as the matrix cores take their A operand: 16 rows x 32
// columns per fragment, lane l holding row l & 15, columns 8 (l >> 4) .. + 7, so that a wave's
// load of a fragment is 1 KB of consecutive memory (row-major, it touches 16 half lines).
constexpr int kMlpHH = kMlpHidden * kMlpHidden;
enum : int { kFragW2 = 0, kFragW3 = 1, kFragW2T = 2, kFragW3T = 3, kFrags = 4 };
__device__ __forceinline__ int frag_at(int row, int col) {
    return (((row >> 4) * 8 + (col >> 5)) * 64 + (row & 15) + 16 * ((col & 31) >> 3)) * 8 + (col & 7);
}
__device__ __forceinline__ bf16x8 load_frag(const uint16_t *__restrict__ W, int tile, int t, int lane) {
    return *reinterpret_cast<const bf16x8 *>(W + ((tile * 8 + t) * 64 + lane) * 8);
}

constexpr int kTM = 64, kTN = 64, kTK = 32, kLdsK = kTK + 8;

struct GemmArgs {
    const uint16_t *A;
    int64_t sam, sak;   // A(m, k) = A[m sam + k sak]
    const uint16_t *B;
    int64_t sbk, sbn;   // B(k, n) = B[k sbk + n sbn]
    int M, N, K;
    float *out;         // [M x N] row-major FP32
};

// One 64 x 32 operand tile into LDS as [row][k]: element (r, k) at P[(r0 + r) sr + (k0 + k) sk],
// zero outside [0, R) x [0, K). 256 threads, 8 elements each: with the operand
// contiguous along k, one 16-byte load per thread; contiguous along rows, one 16-byte load
// of 8 rows at one k, written transposed; otherwise element by element.
__device__ __forceinline__ void load_tile(const uint16_t *__restrict__ P, int64_t sr, int64_t sk,
                                          int r0, int R, int k0, int K, uint16_t (*S)[kLdsK],
                                          int tid) {
    if (sk == 1 && (sr & 7) == 0) {
        const int r = tid >> 2, kc = (tid & 3) * 8;
        const int row = r0 + r, k = k0 + kc;
        const uint16_t *src = P + (int64_t)row * sr + k;
        if (row < R && k + 8 <= K && ((reinterpret_cast<uintptr_t>(src) & 15) == 0)) {
            *reinterpret_cast<uint4 *>(&S[r][kc]) = *reinterpret_cast<const uint4 *>(src);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                S[r][kc + e] = (row < R && k + e < K) ? P[(int64_t)row * sr + k + e] : (uint16_t)0;
        }
        return;
    }
    if (sr == 1 && (sk & 7) == 0) {
        const int kk = tid >> 3, rc = (tid & 7) * 8;
        const int k = k0 + kk, row = r0 + rc;
        const uint16_t *src = P + (int64_t)k * sk + row;
        if (k < K && row + 8 <= R && ((reinterpret_cast<uintptr_t>(src) & 15) == 0)) {
            const uint4 v = *reinterpret_cast<const uint4 *>(src);
            const uint16_t *h = reinterpret_cast<const uint16_t *>(&v);
#pragma unroll
            for (int e = 0; e < 8; ++e) S[rc + e][kk] = h[e];
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                S[rc + e][kk] = (k < K && row + e < R) ? P[(int64_t)k * sk + row + e] : (uint16_t)0;
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int idx = tid * 8 + e;
        const int r = idx >> 5, kk = idx & 31;
        const int row = r0 + r, k = k0 + kk;
        S[r][kk] = (row < R && k < K) ? P[(int64_t)row * sr + (int64_t)k * sk] : (uint16_t)0;
    }
}

// C = A B with a 64 x 64 tile per workgroup (four waves of 32 x 32, each 2 x 2 MFMA
// 16 x 16 tiles), K in steps of 32 staged in LDS (A as [m][k], B as [n][k]).
__global__ void __launch_bounds__(256) k_gemm(GemmArgs g) {
    __shared__ __align__(16) uint16_t sA[kTM][kLdsK];
    __shared__ __align__(16) uint16_t sB[kTN][kLdsK];
    const int m0 = blockIdx.y * kTM, n0 = blockIdx.x * kTN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < g.K; k0 += kTK) {
        load_tile(g.A, g.sam, g.sak, m0, g.M, k0, g.K, sA, tid);
        load_tile(g.B, g.sbn, g.sbk, n0, g.N, k0, g.K, sB, tid);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&sA[wm + i * 16 + (lane & 15)][8 * (lane >> 4)]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const bf16x8 b =
                    *reinterpret_cast<const bf16x8 *>(&sB[wn + j * 16 + (lane & 15)][8 * (lane >> 4)]);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wm + i * 16 + 4 * (lane >> 4) + r;
                const int col = n0 + wn + j * 16 + (lane & 15);
                if (row >= g.M || col >= g.N) continue;
                g.out[(int64_t)row * g.N + col] = acc[i][j][r];
            }
}

// Mean and spread over the ensemble of de-standardised outputs.
__global__ void k_mlp_reduce(const float *__restrict__ out, int64_t n, int K, float mu_y, float sd_y,
                             float *__restrict__ mean, float *__restrict__ sdev) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    float s = 0.f, s2 = 0.f;
    for (int k = 0; k < K; ++k) {
        const float v = out[(int64_t)k * n + i] * sd_y + mu_y;
        s += v;
        s2 += v * v;
    }
    const float mu = s / (float)K;
    mean[i] = mu;
    sdev[i] = K > 1 ? sqrtf(fmaxf(s2 / (float)K - mu * mu, 0.0f) * (float)K / (float)(K - 1)) : 0.0f;
}

// Inference of every member (blockIdx.y), all four layers in one kernel. A workgroup takes kFR rows
// of one member; its four waves each own 64 output features of every hidden layer. The products run on the
// matrix cores with the weights as the A operand (16 features x 32 inputs per fragment,
// read from an aligned copy of the member's BF16 weights, the next k step's fragments in
// flight while the current ones multiply) and the activations as the B operand (16 rows x
// 32 inputs from LDS); a lane's result is then 4 consecutive features of one row, which the
// epilogue (bias, SiLU from the hardware exponential and reciprocal, two-at-a-time BF16
// conversion) stores as one 8-byte LDS write. Layer 1 runs the same way with its 6 inputs
// padded with zeros to 32; layer 4 is a dot product per row on pairs of BF16 values. The
// kFR x 256 activations live in LDS as BF16 and are overwritten in place layer by layer. The
// products and the epilogue of a workgroup alternate behind barriers, so the matrix cores idle
// in its epilogues unless another workgroup is in its products: 80 rows keep three workgroups
// on a CU (49 KB of LDS, 170 registers), 128 rows only two. 1e6 rows through 4 members: 128 rows
// and a launch per member 1.49 ms (713 TFLOP/s), 80 rows and one launch for all of them 1.33 ms
// (797); 64 rows 1.39 (each weight fragment feeds fewer products), 96 rows at two workgroups
// 1.57, 64 rows at four 1.55 (registers spill).
// Same rounding points as in training (input, every hidden activation to BF16,
// FP32 accumulation); the activation uses the hardware exponential and reciprocal.
constexpr int kFR = 80;                  // rows per workgroup
constexpr int kHL = kMlpHidden + 8;      // LDS row stride of the activations (BF16), padded
constexpr int kXL = 40;                  // LDS row stride of the padded input (BF16)

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack2_bf16(float a, float b) {
    bf16x2_t v;
    v[0] = (__bf16)a;
    v[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, v);
}

__global__ void __launch_bounds__(256, 3) k_mlp_fused(const float *__restrict__ x, int64_t n,
                                                      const float *__restrict__ norm,
                                                      const uint16_t *__restrict__ wb,
                                                      const uint16_t *__restrict__ wf,
                                                      const float *__restrict__ w,
                                                      float *__restrict__ out) {
    wb += (int64_t)blockIdx.y * kMlpStride;
    wf += (int64_t)blockIdx.y * kFrags * kMlpHH;
    w += (int64_t)blockIdx.y * kMlpParams;
    out += (int64_t)blockIdx.y * n;
    __shared__ __align__(16) uint16_t sH[kFR][kHL];
    __shared__ __align__(16) uint16_t sX[kFR][kXL];
    __shared__ __align__(16) uint16_t sW4[kMlpHidden];
    const int64_t r0 = blockIdx.x * (int64_t)kFR;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // standardised input rounded to BF16, inputs 6..31 zero
    for (int i = tid; i < kFR * 32; i += 256) {
        const int r = i >> 5, c = i & 31;
        float v = 0.0f;
        if (c < kMlpIn && r0 + r < n) v = (x[(r0 + r) * kMlpIn + c] - norm[c]) / norm[kMlpIn + c];
        sX[r][c] = __builtin_bit_cast(uint16_t, (__bf16)v);
    }
    sW4[tid] = wb[kOffW4 + tid];
    __syncthreads();
    const int f0 = wave * 64;              // this wave's output features
    const int lr = lane & 15, lk = 8 * (lane >> 4), lf = 4 * (lane >> 4);
#pragma unroll 1
    for (int layer = 0; layer < 3; ++layer) {
        f32x4 acc[4][kFR / 16];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < kFR / 16; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (layer == 0) {
            bf16x8 a[4];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const uint16_t *wr = wb + kOffW1 + (int64_t)(f0 + mt * 16 + lr) * kMlpIn;
                uint16_t e[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) e[c] = (lk == 0 && c < kMlpIn) ? wr[c] : (uint16_t)0;
                a[mt] = __builtin_bit_cast(bf16x8, e);
            }
#pragma unroll
            for (int nt = 0; nt < kFR / 16; ++nt) {
                const bf16x8 bv = *reinterpret_cast<const bf16x8 *>(&sX[nt * 16 + lr][lk]);
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], bv, acc[mt][nt], 0, 0, 0);
            }
        } else {
            const uint16_t *W = wf + (layer == 1 ? kFragW2 : kFragW3) * kMlpHH;
            bf16x8 a[4], an[4];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                a[mt] = load_frag(W, wave * 4 + mt, 0, lane);
#pragma unroll
            for (int k0 = 0; k0 < kMlpHidden; k0 += 32) {
                if (k0 + 32 < kMlpHidden) {
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt)
                        an[mt] = load_frag(W, wave * 4 + mt, (k0 >> 5) + 1, lane);
                }
#pragma unroll
                for (int nt = 0; nt < kFR / 16; ++nt) {
                    const bf16x8 bv = *reinterpret_cast<const bf16x8 *>(&sH[nt * 16 + lr][k0 + lk]);
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], bv, acc[mt][nt], 0, 0, 0);
                }
                if (k0 + 32 < kMlpHidden) {
#pragma unroll
                    for (int mt = 0; mt < 4; ++mt) a[mt] = an[mt];
                }
            }
        }
        __syncthreads();  // every wave has read the previous activations
        const float *bias = w + (layer == 0 ? kOffB1 : (layer == 1 ? kOffB2 : kOffB3));
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const int f = f0 + mt * 16 + lf;
            const float b0 = bias[f], b1 = bias[f + 1], b2 = bias[f + 2], b3 = bias[f + 3];
#pragma unroll
            for (int nt = 0; nt < kFR / 16; ++nt) {
                const f32x4 z = acc[mt][nt];
                uint2 pk;
                pk.x = pack2_bf16(silu_fast(z[0] + b0), silu_fast(z[1] + b1));
                pk.y = pack2_bf16(silu_fast(z[2] + b2), silu_fast(z[3] + b3));
                *reinterpret_cast<uint2 *>(&sH[nt * 16 + lr][f]) = pk;
            }
        }
        __syncthreads();
    }
    if (tid < 2 * kFR) {  // layer 4: two threads per row, 64 pairs of BF16 products each
        const int row = tid >> 1, half = tid & 1;
        const uint32_t *hrow = reinterpret_cast<const uint32_t *>(&sH[row][half * 128]);
        const uint32_t *wrow = reinterpret_cast<const uint32_t *>(&sW4[half * 128]);
        float s = 0.0f;
#pragma unroll 8
        for (int c = 0; c < 64; ++c)
            s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, hrow[c]),
                                                __builtin_bit_cast(bf16x2_t, wrow[c]), s, false);
        s += __shfl_xor(s, 1);
        if (half == 0 && r0 + row < n) out[r0 + row] = s + w[kOffB4];
    }
}

// ------------------------------------------------------------------------------ training

// What the three launches of a training step share. Transposed activations and gradients of a
// member (act, one row of ld batch rows each): silu(z) of the three hidden layers, d loss / d z of
// the three, the input and d loss / d output, so that the products over the batch (the weight
// gradients) read both operands along k.
constexpr int kActH = 0, kActDz = 3 * kMlpHidden, kActX = 6 * kMlpHidden, kActDy = kActX + 8;
constexpr int64_t kActRows = kActDy + 8;
constexpr int kBiasCols = 3 * kMlpHidden + 1;
struct TrainArgs {
    const float *x, *y;
    int64_t n, batch, ld, tiles, kc;
    int ns, k0, group, hashed, add_loss;
    uint64_t seed;
    int64_t step;
    const float *norm;
    float mu_y, sd_y;
    const float *w;
    const uint16_t *wb, *wf;
    uint16_t *act;
    float *part, *bpart, *loss;
};

// Minibatch row i of member k at a training step: a counter-based hash of (seed, k, step, i)
// reduced to [0, n) (rows drawn with replacement).
__device__ __forceinline__ int32_t batch_row(uint64_t seed, int k, int64_t step, int64_t n, int64_t i) {
    uint64_t h = seed ^ ((uint64_t)(k + 1) * 0x9E3779B97F4A7C15ull) ^ ((uint64_t)step << 24) ^ (uint64_t)i;
    h ^= h >> 33;
    h *= 0xff51afd7ed558ccdull;
    h ^= h >> 33;
    h *= 0xc4ceb9fe1a85ec53ull;
    h ^= h >> 33;
    return (int32_t)(h % (uint64_t)n);
}

// Workgroup barrier for data that passes through LDS: unlike __syncthreads() it does not wait
// for the global loads and stores in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A layer's weights as the product's A operand, k in eight steps of 32. The fragments of the
// first kAhead steps are loaded before the tile of the layer in front is stored: loads and
// stores complete in order, and a load behind the transposed stores waits for them. 4 steps
// ahead: 68.7 us per launch at batch 8192 x 4 members; 2: 69.8; 6 and 8 spill: 73.9 and 78.8.
constexpr int kAhead = 4;
struct Weights {
    bf16x8 a[8][2];
};
__device__ __forceinline__ void load_weights(Weights &w, const uint16_t *__restrict__ W, int wave,
                                             int lane) {
#pragma unroll
    for (int t = 0; t < kAhead; ++t)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) w.a[t][mt] = load_frag(W, wave * 2 + mt, t, lane);
}

// acc[mt][nt] = W[f0 + 16 mt ..][k] H[16 nt ..][k], summed over k = 0 .. 255; H in LDS.
__device__ __forceinline__ void train_product(Weights &w, const uint16_t *__restrict__ W,
                                              const uint16_t (*sH)[kHL], int wave, int lane,
                                              f32x4 (&acc)[2][4]) {
    const int lr = lane & 15, lk = 8 * (lane >> 4);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        if (t + kAhead < 8) {
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                w.a[t + kAhead][mt] = load_frag(W, wave * 2 + mt, t + kAhead, lane);
        }
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const bf16x8 b = *reinterpret_cast<const bf16x8 *>(&sH[nt * 16 + lr][32 * t + lk]);
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.a[t][mt], b, acc[mt][nt], 0, 0, 0);
        }
    }
}

// Forward and backward of 64 batch rows of one member; workgroup (tile, member). Eight waves of
// 32 features each hold every layer's product and silu'(z) in registers (three layers of 32
// values a lane), so that neither pre-activations nor gradients are stored and read back
// between layers; the BF16 activations and gradients pass through one LDS tile from layer to
// layer and leave it once, transposed, for the weight gradients. The products run as in
// k_mlp_fused (weights the A operand, k in ascending steps of 32). Bias gradients: each feature
// summed over the tile's rows in order (k_mlp_update adds the tiles in order).
// Four members at batch 8192: 69 us (17 GFLOP: 15 us at the rate of a large product). A third of
// it is issue of the epilogues' exponentials and IEEE divisions, a sixth matrix products; the
// rest is latency between the barriers that two waves per SIMD leave uncovered (without the
// products 55 us, without the exponentials 72 of 89, without the stores 77 of 89 at the time).
__global__ void __launch_bounds__(512, 2) k_mlp_fwd_bwd(TrainArgs g) {
    __shared__ __align__(16) uint16_t sH[64][kHL];
    __shared__ __align__(16) float sD[64][kMlpHidden + 4];
    __shared__ __align__(16) uint16_t sX[64][kXL];
    __shared__ int32_t sRow[64];
    __shared__ __align__(16) float sBias[3 * kMlpHidden];
    __shared__ __align__(16) uint16_t sW4[kMlpHidden];
    __shared__ float sT[64], sDy[64], sL[64];
    __shared__ uint16_t sDyb[64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    const int k = g.k0 + (int)blockIdx.y;
    const float *w = g.w + (int64_t)k * kMlpParams;
    const uint16_t *wb = g.wb + (int64_t)k * kMlpStride;
    const uint16_t *wfr = g.wf + (int64_t)k * kFrags * kMlpHH;
    uint16_t *act = g.act + (int64_t)blockIdx.y * kActRows * g.ld + r0;
    float *bpart = g.bpart + ((int64_t)blockIdx.y * g.tiles + blockIdx.x) * kBiasCols;
    const int f0 = wave * 32, lr = lane & 15, lk = 8 * (lane >> 4), lf = 4 * (lane >> 4);
    if (tid < 64)
        sRow[tid] = r0 + tid < g.batch
                        ? (g.hashed ? batch_row(g.seed, k, g.step, g.n, r0 + tid) : (int32_t)(r0 + tid))
                        : -1;
    for (int e = tid; e < 3 * kMlpHidden; e += 512)
        sBias[e] = w[(e < kMlpHidden ? kOffB1 : (e < 2 * kMlpHidden ? kOffB2 : kOffB3)) + (e & (kMlpHidden - 1))];
    if (tid < kMlpHidden) sW4[tid] = wb[kOffW4 + tid];
    const float b4 = w[kOffB4];
    lds_barrier();
    if (tid < 64) sT[tid] = sRow[tid] >= 0 ? (g.y[sRow[tid]] - g.mu_y) / g.sd_y : 0.0f;
    for (int e = tid; e < 64 * 32; e += 512) {  // standardised input in BF16, inputs 6..31 zero
        const int r = e >> 5, c = e & 31;
        const int64_t row = sRow[r];
        sX[r][c] = c < kMlpIn && row >= 0 ? to_bf16((g.x[row * kMlpIn + c] - g.norm[c]) / g.norm[kMlpIn + c])
                                          : (uint16_t)0;
    }
    lds_barrier();
    if (tid < 8 * 64) act[(int64_t)(kActX + wave) * g.ld + lane] = sX[lane][wave];

    // the tile in sH to the rows at `to` of act, transposed: eight rows of two features at a time,
    // eight lanes to a feature's 64 rows, so that a store writes whole 128-B lines
    auto store_transposed = [&](int to) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int id = tid + 512 * u;
            const int fp = (id & 7) | (id >> 6) << 3, rg = (id >> 3) & 7;
            uint32_t v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = *reinterpret_cast<const uint32_t *>(&sH[rg * 8 + e][fp * 2]);
            uint4 lo, hi;
            lo.x = (v[0] & 0xffffu) | v[1] << 16; hi.x = (v[0] >> 16) | (v[1] & 0xffff0000u);
            lo.y = (v[2] & 0xffffu) | v[3] << 16; hi.y = (v[2] >> 16) | (v[3] & 0xffff0000u);
            lo.z = (v[4] & 0xffffu) | v[5] << 16; hi.z = (v[4] >> 16) | (v[5] & 0xffff0000u);
            lo.w = (v[6] & 0xffffu) | v[7] << 16; hi.w = (v[6] >> 16) | (v[7] & 0xffff0000u);
            uint16_t *o = act + (int64_t)(to + fp * 2) * g.ld + rg * 8;
            *reinterpret_cast<uint4 *>(o) = lo;
            *reinterpret_cast<uint4 *>(o + g.ld) = hi;
        }
    };
    // bias and SiLU of a layer's product: BF16 activation into sH, silu'(z) kept
    auto activate = [&](const f32x4 (&acc)[2][4], const float *bias, f32x4 (&sp)[2][4]) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            const int f = f0 + mt * 16 + lf;
            float b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] = bias[f + e];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                float h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float z = acc[mt][nt][e] + b[e];
                    const float sg = sigmoidf_(z);
                    h[e] = z * sg;
                    sp[mt][nt][e] = sg * (1.0f + z * (1.0f - sg));
                }
                *reinterpret_cast<uint2 *>(&sH[nt * 16 + lr][f]) =
                    uint2{pack2_bf16(h[0], h[1]), pack2_bf16(h[2], h[3])};
            }
        }
    };
    // d loss / d z of a layer, v silu'(z): FP32 into sD for the bias gradient, BF16 into sH
    auto gradient = [&](const f32x4 (&v)[2][4], const f32x4 (&sp)[2][4]) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const int f = f0 + mt * 16 + lf;
                f32x4 d;
#pragma unroll
                for (int e = 0; e < 4; ++e) d[e] = v[mt][nt][e] * sp[mt][nt][e];
                *reinterpret_cast<f32x4 *>(&sD[nt * 16 + lr][f]) = d;
                *reinterpret_cast<uint2 *>(&sH[nt * 16 + lr][f]) =
                    uint2{pack2_bf16(d[0], d[1]), pack2_bf16(d[2], d[3])};
            }
    };
    auto bias_sums = [&](int col0) {
        if (tid < kMlpHidden) {
            float s = 0.f;
#pragma unroll 16
            for (int r = 0; r < 64; ++r) s += sD[r][tid];
            bpart[col0 + tid] = s;
        }
    };

    f32x4 acc[2][4], sp1[2][4], sp2[2][4], sp3[2][4];
    Weights wf;
    {   // layer 1: 6 inputs padded with zeros to 32
        bf16x8 a[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            const uint16_t *wr = wb + kOffW1 + (f0 + mt * 16 + lr) * kMlpIn;
            uint16_t e[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) e[c] = (lk == 0 && c < kMlpIn) ? wr[c] : (uint16_t)0;
            a[mt] = __builtin_bit_cast(bf16x8, e);
        }
        load_weights(wf, wfr + kFragW2 * kMlpHH, wave, lane);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const bf16x8 b = *reinterpret_cast<const bf16x8 *>(&sX[nt * 16 + lr][lk]);
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], b, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
    }
    activate(acc, sBias, sp1);
    lds_barrier();
    store_transposed(kActH);
    train_product(wf, wfr + kFragW2 * kMlpHH, sH, wave, lane, acc);
    load_weights(wf, wfr + kFragW3 * kMlpHH, wave, lane);
    lds_barrier();
    activate(acc, sBias + kMlpHidden, sp2);
    lds_barrier();
    store_transposed(kActH + kMlpHidden);
    train_product(wf, wfr + kFragW3 * kMlpHH, sH, wave, lane, acc);
    load_weights(wf, wfr + kFragW3T * kMlpHH, wave, lane);
    lds_barrier();
    activate(acc, sBias + 2 * kMlpHidden, sp3);
    lds_barrier();
    store_transposed(kActH + 2 * kMlpHidden);
    if (wave < 4) {  // output layer and loss: 16 rows per wave
        f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k0 = 0; k0 < kMlpHidden; k0 += 32) {
            bf16x8 a = *reinterpret_cast<const bf16x8 *>(&sW4[k0 + lk]);
            if (lr != 0) a = bf16x8{};
            const bf16x8 b = *reinterpret_cast<const bf16x8 *>(&sH[wave * 16 + lr][k0 + lk]);
            o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, o, 0, 0, 0);
        }
        if (lane < 16) {
            const int r = wave * 16 + lane;
            float l = 0.f, dy = 0.f;
            if (sRow[r] >= 0) {
                const float d = (o[0] + b4) - sT[r];
                l = d * d;
                dy = 2.0f * d / (float)g.batch;
            }
            sL[r] = l;
            sDy[r] = dy;
            sDyb[r] = to_bf16(dy);
        }
    }
    lds_barrier();
    if (wave == 0) {
        float l = sL[lane];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) l += __shfl_xor(l, off);
        if (lane == 0 && l != 0.f && g.add_loss) atomicAdd(g.loss + k, l);
        act[(int64_t)kActDy * g.ld + lane] = sDyb[lane];
    } else if (tid == 64) {
        float s = 0.f;
        for (int r = 0; r < 64; ++r) s += sDy[r];
        bpart[3 * kMlpHidden] = s;
    }
    // d loss / d z3 = (dy w4) silu'(z3)
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[mt][nt][e] = from_bf16(sW4[f0 + mt * 16 + lf + e]) * from_bf16(sDyb[nt * 16 + lr]);
    gradient(acc, sp3);
    lds_barrier();
    store_transposed(kActDz + 2 * kMlpHidden);
    bias_sums(2 * kMlpHidden);
    train_product(wf, wfr + kFragW3T * kMlpHH, sH, wave, lane, acc);
    load_weights(wf, wfr + kFragW2T * kMlpHH, wave, lane);
    lds_barrier();
    gradient(acc, sp2);
    lds_barrier();
    store_transposed(kActDz + kMlpHidden);
    bias_sums(kMlpHidden);
    train_product(wf, wfr + kFragW2T * kMlpHH, sH, wave, lane, acc);
    lds_barrier();
    gradient(acc, sp1);
    lds_barrier();
    store_transposed(kActDz);
    bias_sums(0);
}

// Weight gradients of one slice of the batch (kc rows), k in ascending steps of 32: jobs 0..3 and
// 4..7 take the 128 x 128 quarters of dW3 = dZ3^T H2 and dW2 = dZ2^T H1 (operands staged in LDS
// 64 rows ahead), 8 takes dW1 = dZ1^T X, 9 dW4 = H3^T dy. Partial products to part. 31 us for
// four members at batch 8192; 76 us with the staged rows spilled and the jobs of a slice on
// different XCDs, each reading the slice's 1.6 MB from beyond its L2.
constexpr int kGradJobs = 10;
__global__ void __launch_bounds__(256, 2) k_mlp_wgrad(TrainArgs g) {
    constexpr int kC = 64, kS = kC + 8;  // rows of the batch per stage, LDS stride
    __shared__ __align__(16) uint16_t sA[2][128][kS], sB[2][128][kS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lk = 8 * (lane >> 4), lf = 4 * (lane >> 4);
    // the ten jobs of a slice read the same rows: workgroups go to the eight XCDs in turn, so
    // slice s of all members' takes the workgroups with the same remainder by eight
    const int job = (int)(blockIdx.x / 8 % kGradJobs);
    const int sl = (int)(blockIdx.x / (8 * kGradJobs)) * 8 + (int)(blockIdx.x % 8);
    if (sl >= g.ns * g.group) return;
    const int z = sl % g.ns, member = sl / g.ns;
    const int64_t kb = z * g.kc, ke = min(g.batch, kb + g.kc);
    const uint16_t *act = g.act + (int64_t)member * kActRows * g.ld;
    float *part = g.part + (int64_t)sl * kMlpParams;
    if (job >= 8) {
        const uint16_t *A = act + (int64_t)((job == 8 ? kActDz : kActH + 2 * kMlpHidden) + wave * 64 + lr) * g.ld;
        const uint16_t *B = act + (int64_t)(job == 8 ? kActX + min(lr, kMlpIn - 1) : kActDy) * g.ld;
        const bool col = job == 8 ? lr < kMlpIn : lr == 0;
        f32x4 acc[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int64_t k0 = kb; k0 < ke; k0 += 32) {
            bf16x8 b = *reinterpret_cast<const bf16x8 *>(B + k0 + lk);
            if (!col) b = bf16x8{};
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const bf16x8 a = *reinterpret_cast<const bf16x8 *>(A + mt * 16 * g.ld + k0 + lk);
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[mt], 0, 0, 0);
            }
        }
        if (!col) return;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = wave * 64 + mt * 16 + lf + e;
                if (job == 8) part[kOffW1 + j * kMlpIn + lr] = acc[mt][e];
                else part[kOffW4 + j] = acc[mt][e];
            }
        return;
    }
    const int layer = job < 4 ? 1 : 0;  // 1: W3, 0: W2
    const int m0 = (job & 1) * 128, n0 = ((job >> 1) & 1) * 128;
    const uint16_t *A = act + (int64_t)(kActDz + (layer + 1) * kMlpHidden + m0) * g.ld;
    const uint16_t *B = act + (int64_t)(kActH + layer * kMlpHidden + n0) * g.ld;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 ra[4], rb[4];
    auto load = [&](int64_t k0) {  // 128 rows x 64 of each operand, 16 bytes a piece
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int id = tid + 256 * u, row = id >> 3, c = (id & 7) * 8;
            ra[u] = *reinterpret_cast<const u32x4 *>(A + (int64_t)row * g.ld + k0 + c);
            rb[u] = *reinterpret_cast<const u32x4 *>(B + (int64_t)row * g.ld + k0 + c);
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int id = tid + 256 * u, row = id >> 3, c = (id & 7) * 8;
            *reinterpret_cast<u32x4 *>(&sA[buf][row][c]) = ra[u];
            *reinterpret_cast<u32x4 *>(&sB[buf][row][c]) = rb[u];
        }
    };
    int buf = 0;
    auto multiply = [&](int h) {
        bf16x8 a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = *reinterpret_cast<const bf16x8 *>(&sA[buf][wm + i * 16 + lr][h + lk]);
            b[i] = *reinterpret_cast<const bf16x8 *>(&sB[buf][wn + i * 16 + lr][h + lk]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    };
    load(kb);
    store(0);
    lds_barrier();
    for (int64_t k0 = kb; k0 < ke; k0 += kC) {
        const bool more = k0 + kC < ke;
        if (more) load(k0 + kC);
        multiply(0);
        if (k0 + 32 < ke) multiply(32);
        buf ^= 1;
        if (more) store(buf);
        lds_barrier();
    }
    float *out = part + (layer ? kOffW3 : kOffW2);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                out[(m0 + wm + i * 16 + lf + e) * kMlpHidden + n0 + wn + j * 16 + lr] = acc[i][j][e];
}

// Gradients (slices, and tiles of the biases, added in order) into g, or, where g is null, Adam
// (Kingma & Ba 2015) on the FP32 master weights and their BF16 copies. Workgroups below
// kUpdTiles take 16 x 64 tiles of W2 and W3 (through LDS into the fragments of both products),
// the others the remaining parameters. Bound by reading the 16 slices' partials (34 MB for four
// members, 13.6 us).
constexpr int kUpdTiles = 128;
constexpr int kUpdRest = kMlpHidden * kMlpIn + 3 * kMlpHidden + kMlpHidden + 1;
struct AdamArgs {
    float *am, *av, *g;
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ uint16_t mlp_update(const TrainArgs &g, const AdamArgs &ad, int64_t k,
                                               int64_t p, float gi) {
    if (ad.g) {
        ad.g[p] = gi;
        return 0;
    }
    const int64_t i = k * kMlpParams + p;
    const float mi = ad.b1 * ad.am[i] + (1.0f - ad.b1) * gi;
    const float vi = ad.b2 * ad.av[i] + (1.0f - ad.b2) * gi * gi;
    ad.am[i] = mi;
    ad.av[i] = vi;
    float *w = const_cast<float *>(g.w) + i;
    const float wi = *w - ad.lr * (mi / ad.c1) / (sqrtf(vi / ad.c2) + ad.eps);
    *w = wi;
    const uint16_t h = to_bf16(wi);
    return h;
}

__global__ void __launch_bounds__(256) k_mlp_update(TrainArgs g, AdamArgs ad) {
    __shared__ __align__(16) uint16_t sT[64][24];
    const int tid = threadIdx.x;
    const int64_t k = g.k0 + blockIdx.y;
    const float *part = g.part + (int64_t)blockIdx.y * g.ns * kMlpParams;
    if (blockIdx.x < kUpdTiles) {
        const int layer = blockIdx.x >> 6, t = blockIdx.x & 63;  // 0: W2, 1: W3
        const int j0 = (t >> 2) * 16, i0 = (t & 3) * 64, i = tid & 63;
        const int64_t off = (layer ? kOffW3 : kOffW2) + i0 + i;
        float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int z = 0; z < g.ns; ++z)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                s[r] += part[(int64_t)z * kMlpParams + off + (int64_t)(j0 + (tid >> 6) + 4 * r) * kMlpHidden];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = (tid >> 6) + 4 * r;
            sT[i][j] = mlp_update(g, ad, k, off + (int64_t)(j0 + j) * kMlpHidden, s[r]);
        }
        if (ad.g) return;
        __syncthreads();
        uint16_t *wf = const_cast<uint16_t *>(g.wf) + k * kFrags * kMlpHH;
        const int l = tid & 127;
        if (tid < 128) {  // 16 rows j x 64 columns i: two fragments
            const int col = (l >> 6) * 32 + ((l >> 4) & 3) * 8;
            uint16_t v[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) v[c] = sT[col + c][l & 15];
            *reinterpret_cast<u32x4 *>(wf + (kFragW2 + layer) * kMlpHH + frag_at(j0 + (l & 15), i0 + col)) =
                __builtin_bit_cast(u32x4, v);
        } else {  // transposed, 64 rows i x 16 columns j: half of four fragments
            const int row = l >> 1, col = (l & 1) * 8;
            *reinterpret_cast<u32x4 *>(wf + (kFragW2T + layer) * kMlpHH + frag_at(i0 + row, j0 + col)) =
                *reinterpret_cast<const u32x4 *>(&sT[row][col]);
        }
        return;
    }
    const int e = (int)(blockIdx.x - kUpdTiles) * 256 + tid;
    if (e >= kUpdRest) return;
    constexpr int nW1 = kMlpHidden * kMlpIn;
    int64_t p;
    int col = -1;  // bias column
    if (e < nW1) p = kOffW1 + e;
    else if (e < nW1 + 3 * kMlpHidden) {
        col = e - nW1;
        p = (col < kMlpHidden ? kOffB1 : (col < 2 * kMlpHidden ? kOffB2 : kOffB3)) + (col & (kMlpHidden - 1));
    } else {
        p = kOffW4 + (e - nW1 - 3 * kMlpHidden);
        if (p == kOffB4) col = 3 * kMlpHidden;
    }
    float s = 0.f;
    if (col < 0) {
#pragma unroll 8
        for (int z = 0; z < g.ns; ++z) s += part[(int64_t)z * kMlpParams + p];
    } else {
        const float *b = g.bpart + (int64_t)blockIdx.y * g.tiles * kBiasCols + col;
        // up to 4096 partials in order; longer batches first add runs of their tiles
        const int64_t run = (g.tiles + 4095) / 4096;
        if (run == 1) {
#pragma unroll 32
            for (int64_t t = 0; t < g.tiles; ++t) s += b[t * kBiasCols];
        } else {
            for (int64_t t = 0; t < g.tiles; t += run) {
                float u = 0.f;
                for (int64_t v = t; v < min(g.tiles, t + run); ++v) u += b[v * kBiasCols];
                s += u;
            }
        }
    }
    const uint16_t h = mlp_update(g, ad, k, p, s);
    if (!ad.g) const_cast<uint16_t *>(g.wb)[k * kMlpStride + p] = h;
}

// BF16 copies of every member's parameters.
__global__ void k_mlp_cast(const float *__restrict__ w, int64_t n, uint16_t *__restrict__ wb,
                           uint16_t *__restrict__ wf) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t k = i / kMlpParams, p = i - k * kMlpParams;
    const uint16_t h = to_bf16(w[i]);
    wb[k * kMlpStride + p] = h;
    wf += k * kFrags * kMlpHH;
    for (int layer = 0; layer < 2; ++layer) {
        const int64_t q = p - (layer ? kOffW3 : kOffW2);
        if (q < 0 || q >= kMlpHH) continue;
        const int row = (int)q / kMlpHidden, col = (int)q % kMlpHidden;
        wf[(kFragW2 + layer) * kMlpHH + frag_at(row, col)] = h;
        wf[(kFragW2T + layer) * kMlpHH + frag_at(col, row)] = h;
    }
}

// Per-column sum and sum of squares (FP64) of a [n x c] row-major matrix, reduced in a fixed
// order (the same sums on every call): workgroup (slice, col) sums its strided rows per
// thread, then a tree over its 256 threads into part[(col gx + slice) 2 + {0, 1}];
// k_moments_fold adds the slices in order into out[2 col], out[2 col + 1].
__global__ void __launch_bounds__(256) k_moments(const float *__restrict__ a, int64_t n, int c,
                                                 double *__restrict__ part) {
    const int col = blockIdx.y;
    double s = 0.0, s2 = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double v = a[i * c + col];
        s += v;
        s2 += v * v;
    }
    __shared__ double r1[256], r2[256];
    r1[threadIdx.x] = s;
    r2[threadIdx.x] = s2;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) {
            r1[threadIdx.x] += r1[threadIdx.x + h];
            r2[threadIdx.x] += r2[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int64_t o = 2 * ((int64_t)col * gridDim.x + blockIdx.x);
        part[o] = r1[0];
        part[o + 1] = r2[0];
    }
}

__global__ void k_moments_fold(const double *__restrict__ part, int gx, int c,
                               double *__restrict__ out) {
    const int col = threadIdx.x;
    if (col >= c) return;
    double s = 0.0, s2 = 0.0;
#pragma unroll 16
    for (int b = 0; b < gx; ++b) {
        s += part[2 * ((int64_t)col * gx + b)];
        s2 += part[2 * ((int64_t)col * gx + b) + 1];
    }
    out[2 * col] = s;
    out[2 * col + 1] = s2;
}

inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

void mlp_fused_forward(MlpModel *m, const float *x, int64_t n, float *out) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_mlp_fused, dim3(blocks(n, kFR), m->K), dim3(256), 0, m->st, x, n, m->norm,
                       m->wb, m->wf, m->w, out);
}

void mlp_moments(const float *a, int64_t n, int c, double *out, double *part, hipStream_t st) {
    if (n <= 0) return;
    const unsigned gx = std::min<unsigned>(blocks(n, 256), kMomentSlices);
    hipLaunchKernelGGL(k_moments, dim3(gx, (unsigned)c), dim3(256), 0, st, a, n, c, part);
    hipLaunchKernelGGL(k_moments_fold, dim3(1), dim3(64), 0, st, part, (int)gx, c, out);
}

void mlp_gemm(const uint16_t *A, int64_t sam, int64_t sak, const uint16_t *B, int64_t sbk,
              int64_t sbn, int M, int N, int K, float *out, hipStream_t st) {
    if (M <= 0 || N <= 0) return;
    GemmArgs g{A, sam, sak, B, sbk, sbn, M, N, K, out};
    hipLaunchKernelGGL(k_gemm, dim3(blocks(N, kTN), blocks(M, kTM)), dim3(256), 0, st, g);
}

// ---------------------------------------------------------------------------- model

MlpModel::~MlpModel() {
    for (void *p : allocs) (void)hipFree(p);
    (void)hipFree(act);
    (void)hipFree(part);
    (void)hipFree(bpart);
    (void)hipFree(outs);
}

template <typename T>
static int mlp_alloc(MlpModel *m, T **p, size_t n) {
    *p = nullptr;
    if (hipMalloc(reinterpret_cast<void **>(p), std::max<size_t>(n, 1) * sizeof(T)) != hipSuccess) {
        *p = nullptr;
        return TRIL_E_NOMEM;
    }
    m->allocs.push_back(*p);
    return TRIL_OK;
}

int mlp_init(MlpModel *m, int K, uint64_t seed, hipStream_t st) {
    m->K = K;
    m->st = st;
    const size_t P = (size_t)K * kMlpParams;
    int r;
    if ((r = mlp_alloc(m, &m->w, P)) || (r = mlp_alloc(m, &m->wb, (size_t)K * kMlpStride)) ||
        (r = mlp_alloc(m, &m->wf, (size_t)K * kFrags * kMlpHH)) ||
        (r = mlp_alloc(m, &m->g, kMlpParams)) || (r = mlp_alloc(m, &m->am, P)) ||
        (r = mlp_alloc(m, &m->av, P)) || (r = mlp_alloc(m, &m->norm, 2 * kMlpIn)) ||
        (r = mlp_alloc(m, &m->loss, (size_t)K)))
        return r;
    // He-uniform weights scaled for SiLU, zero biases; member k from its own stream
    std::vector<float> h(P, 0.0f);
    for (int k = 0; k < K; ++k) {
        std::mt19937_64 gen(seed * 0x9E3779B97F4A7C15ull + (uint64_t)k + 1u);
        float *w = h.data() + (size_t)k * kMlpParams;
        auto fill = [&](int64_t off, int fan_in, int64_t count) {
            std::uniform_real_distribution<float> U(-1.0f, 1.0f);
            const float a = std::sqrt(6.0f / (float)fan_in);
            for (int64_t i = 0; i < count; ++i) w[off + i] = a * U(gen);
        };
        fill(kOffW1, kMlpIn, (int64_t)kMlpHidden * kMlpIn);
        fill(kOffW2, kMlpHidden, (int64_t)kMlpHidden * kMlpHidden);
        fill(kOffW3, kMlpHidden, (int64_t)kMlpHidden * kMlpHidden);
        fill(kOffW4, kMlpHidden, kMlpHidden);
        for (int64_t i = kOffW4; i < kOffB4; ++i) w[i] *= 0.1f;
    }
    if (hipMemcpy(m->w, h.data(), P * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
        return TRIL_E_HIP;
    if (hipMemset(m->am, 0, P * sizeof(float)) != hipSuccess ||
        hipMemset(m->av, 0, P * sizeof(float)) != hipSuccess)
        return TRIL_E_HIP;
    std::vector<float> nrm(2 * kMlpIn);
    for (int c = 0; c < kMlpIn; ++c) {
        nrm[c] = 0.0f;
        nrm[kMlpIn + c] = 1.0f;
    }
    if (hipMemcpy(m->norm, nrm.data(), nrm.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
        return TRIL_E_HIP;
    mlp_cast(m);
    return hipGetLastError() == hipSuccess ? TRIL_OK : TRIL_E_HIP;
}

namespace {

template <typename T>
int mlp_grow(MlpModel *m, T **p, int64_t *cap, int64_t n) {
    if (n <= *cap) return TRIL_OK;
    if (hipStreamSynchronize(m->st) != hipSuccess) return TRIL_E_HIP;
    (void)hipFree(*p);
    *p = nullptr;
    *cap = 0;
    if (hipMalloc(reinterpret_cast<void **>(p), (size_t)n * sizeof(T)) != hipSuccess) {
        *p = nullptr;
        return TRIL_E_NOMEM;
    }
    *cap = n;
    return TRIL_OK;
}

// Rows of the batch per slice of the weight gradients: kMlpSlices slices, whole k steps.
int64_t slice_rows(int64_t n) {
    return std::max<int64_t>(32, ((n + kMlpSlices - 1) / kMlpSlices + 31) / 32 * 32);
}

int64_t act_ld(int64_t n) { return (n + 63) / 64 * 64 + 64; }

}  // namespace

int mlp_outputs(MlpModel *m, int64_t n) {
    return mlp_grow(m, &m->outs, &m->outs_cap, n);
}

int mlp_train_group(const MlpModel *m, int64_t n) {
    const int64_t per = kActRows * act_ld(n) * 2 + kMlpSlices * kMlpParams * 4;
    return (int)std::max<int64_t>(1, std::min<int64_t>(m->K, kMlpScratch / per));
}

int mlp_scratch(MlpModel *m, int64_t n, int group) {
    int r;
    const int64_t tiles = (n + 63) / 64;
    if ((r = mlp_grow(m, &m->act, &m->act_cap, group * kActRows * act_ld(n))) ||
        (r = mlp_grow(m, &m->part, &m->part_cap, group * kMlpSlices * kMlpParams)) ||
        (r = mlp_grow(m, &m->bpart, &m->bpart_cap, group * tiles * kBiasCols)))
        return r;
    return TRIL_OK;
}

void mlp_step(MlpModel *m, int k0, int group, const float *x, const float *y, int64_t n,
              int64_t batch, bool hashed, uint64_t seed, int64_t step, bool add_loss, float lr) {
    const int64_t tiles = (batch + 63) / 64, kc = slice_rows(batch);
    const int ns = (int)std::max<int64_t>(1, (batch + kc - 1) / kc);
    TrainArgs a{};
    a.x = x; a.y = y; a.n = n; a.batch = batch; a.ld = act_ld(batch); a.tiles = tiles; a.kc = kc;
    a.ns = ns; a.k0 = k0; a.group = group; a.hashed = hashed ? 1 : 0; a.add_loss = add_loss ? 1 : 0;
    a.seed = seed; a.step = step; a.norm = m->norm; a.mu_y = m->mu_y; a.sd_y = m->sd_y;
    a.w = m->w; a.wb = m->wb; a.wf = m->wf; a.act = m->act; a.part = m->part; a.bpart = m->bpart;
    a.loss = m->loss;
    hipLaunchKernelGGL(k_mlp_fwd_bwd, dim3((unsigned)tiles, group), dim3(512), 0, m->st, a);
    hipLaunchKernelGGL(k_mlp_wgrad, dim3(8 * kGradJobs * blocks((int64_t)ns * group, 8)), dim3(256),
                       0, m->st, a);
    AdamArgs ad{};
    ad.am = m->am;
    ad.av = m->av;
    ad.g = hashed ? nullptr : m->g;
    ad.lr = lr;
    ad.b1 = 0.9f;
    ad.b2 = 0.999f;
    ad.eps = 1e-8f;
    const float t = (float)(step + 1);
    ad.c1 = 1.0f - std::pow(ad.b1, t);
    ad.c2 = 1.0f - std::pow(ad.b2, t);
    hipLaunchKernelGGL(k_mlp_update, dim3(kUpdTiles + blocks(kUpdRest, 256), group), dim3(256), 0,
                       m->st, a, ad);
}

void mlp_reduce(MlpModel *m, const float *out, int64_t n, float *mean, float *sdev) {
    hipLaunchKernelGGL(k_mlp_reduce, dim3(blocks(n, 256)), dim3(256), 0, m->st, out, n, m->K,
                       m->mu_y, m->sd_y, mean, sdev);
}

void mlp_cast(MlpModel *m) {
    const int64_t P = (int64_t)m->K * kMlpParams;
    hipLaunchKernelGGL(k_mlp_cast, dim3(blocks(P, 256)), dim3(256), 0, m->st, m->w, P, m->wb, m->wf);
}

}  // namespace tril
