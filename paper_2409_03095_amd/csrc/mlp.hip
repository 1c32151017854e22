// Chain-allocation network: 8 -> 64 -> 64 -> 1 ReLU MLP with BF16 weights,
// FP32 master weights and FP32 accumulation (gfx950).
//
// One wavefront handles a tile of 16 samples. Layer 1 (K = 8) runs on the VALU;
// the 64x64 layer and its two backward products run on the matrix cores with
// v_mfma_f32_16x16x16_bf16 (A: lane l holds row l%16, k = 4(l/16)..+3;
// B: column l%16, k = 4(l/16)..+3; D: column l%16, rows 4(l/16)..+3).
// Training: a workgroup's four tiles form its gradient in registers (each wave a quarter
// of dW2 over the 64 samples), one kernel adds the workgroups' partials in a fixed
// order and takes the Adam step (Kingma and Ba) on the FP32 masters, which it re-rounds
// to BF16 for the next forward. Samples of a training step are drawn with
// replacement by Philox (no host shuffling).
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "common.hpp"

namespace mcmi {
namespace {

constexpr int kIn = 8, kHid = 64;
constexpr int oW1 = 0, ob1 = 512, oW2 = 576, ob2 = 4672, ow3 = 4736, ob3 = 4800, kParams = 4801;
constexpr int kTile = 16, kWaves = 4, kWG = kWaves * 64;
constexpr uint32_t kMlpTag = 0x4D4C5000u;
constexpr int kPitch = 72;  // BF16 words per LDS row of 64 (+ 8: the 16 rows of an operand hit distinct banks)

typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

struct MlpArgs {
    const float *feat;      // n x 8
    const float *target;    // n (training)
    const int32_t *idx;     // explicit sample indices (gradient check), nullable
    int64_t n;
    int64_t count;          // samples processed by this launch
    const float *master;    // FP32 parameters
    const uint16_t *w1b, *w2b, *w3b;
    const float *norm;      // mean[8], inv_std[8]
    float *out;             // predictions (inference)
    float *partial;         // gridDim.x x (kParams + 1) gradient partials and loss
    uint64_t seed;
    uint32_t step;
    float inv_batch;
};

// Weights of a workgroup in LDS.
struct MlpLds {
    uint16_t w2[kHid * kPitch];  // [out][in]
    float w1[kHid * kIn], b1[kHid], b2[kHid], w3[kHid];
};

__device__ __forceinline__ void load_weights(const MlpArgs &a, MlpLds &m) {
    for (int p = 4 * threadIdx.x; p < kHid * kHid; p += 4 * kWG)
        *(short4v *)&m.w2[(p >> 6) * kPitch + (p & 63)] = *(const short4v *)(a.w2b + p);
    for (int p = threadIdx.x; p < kHid * kIn; p += kWG) m.w1[p] = from_bf16(a.w1b[p]);
    for (int p = threadIdx.x; p < kHid; p += kWG) {
        m.b1[p] = a.master[ob1 + p];
        m.b2[p] = a.master[ob2 + p];
        m.w3[p] = from_bf16(a.w3b[p]);
    }
}

// Forward of a tile: xb is the sample (row i) of this lane, normalized and BF16-rounded.
// A: the layer-1 activations as A operands (outs 16 kb + 4 q + r of sample i); h2[nb][r]:
// layer-2 activation 16 nb + i of sample 4 q + r; y[r]: output of sample 4 q + r.
__device__ __forceinline__ void mlp_forward(const MlpLds &m, float b3, const float (&xb)[kIn], int q, int i,
                                            short4v (&A)[4], float (&h2)[4][4], float (&y)[4]) {
    // layer 1 on the VALU, straight into the A operand of layer 2
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 16 * kb + 4 * q + r;
            const float4v wa = *(const float4v *)&m.w1[o * kIn], wb = *(const float4v *)&m.w1[o * kIn + 4];
            float z = m.b1[o];
#pragma unroll
            for (int k = 0; k < 4; ++k) z += wa[k] * xb[k];
#pragma unroll
            for (int k = 0; k < 4; ++k) z += wb[k] * xb[4 + k];
            A[kb][r] = (short)to_bf16(z > 0.f ? z : 0.f);
        }
    }
    // layer 2 on the matrix cores: Z2 (16 x 64) = H1 (16 x 64) W2^T
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        float4v D = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
            D = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                A[kb], *(const short4v *)&m.w2[(16 * nb + i) * kPitch + 16 * kb + 4 * q], D, 0, 0, 0);
        const int o = 16 * nb + i;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float z = D[r] + m.b2[o];
            h2[nb][r] = z > 0.f ? z : 0.f;
            part[r] += m.w3[o] * h2[nb][r];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) part[r] += __shfl_xor(part[r], off, 64);
        y[r] = part[r] + b3;
    }
}

__global__ void __launch_bounds__(kWG) k_mlp_predict(MlpArgs a) {
    __shared__ __align__(16) MlpLds m;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, q = l >> 4, i = l & 15;
    load_weights(a, m);
    const float b3 = a.master[ob3];
    float mean[kIn], inv[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) {
        mean[k] = a.norm[k];
        inv[k] = a.norm[kIn + k];
    }
    __syncthreads();
    const int64_t tiles = (a.count + kTile - 1) / kTile;
    for (int64_t tile = (int64_t)blockIdx.x * kWaves + w; tile < tiles; tile += (int64_t)gridDim.x * kWaves) {
        const int64_t sa = tile * kTile + i;
        const bool valid = sa < a.count;
        float xb[kIn];
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            const float x = valid ? a.feat[sa * kIn + k] : 0.f;
            xb[k] = from_bf16(to_bf16((x - mean[k]) * inv[k]));
        }
        short4v A[4];
        float h2[4][4], y[4];
        mlp_forward(m, b3, xb, q, i, A, h2, y);
        if (i == 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (tile * kTile + 4 * q + r < a.count) a.out[tile * kTile + 4 * q + r] = y[r];
        }
    }
}

// Gradient of a step: four tiles (64 samples) per workgroup and round, all gradient
// sums in registers: dW2 as a 64 x 64 x 64-sample product, wave w rows 16 w .. 16 w + 15;
// the others per lane over its own samples, the lanes' shares added at the end. A
// parameter's sum is that of its tiles' (or lanes') shares, then of the workgroups', each
// in index order; the shares of db3 and of the loss are a tile's (for the loss those of its
// samples q, 4 + q, 8 + q, 12 + q, one q after the other). That is one of the orders in
// which LDS atomics of four waves add, those on one address taken together in a wave: a
// step whose workgroups hold one tile each has the bits of a kernel of such atomics. With LDS float atomics for every share (110 per tile, the four waves
// on the same addresses) a 4096-sample step's kernel took 50 us, the sum of its partials
// 16 us and Adam 5 us: a step 68.8 us, now 17.4 (of 262144 samples 907 -> 107 us). Adding
// the shares and partials as trees took 15.7 us, but 200 steps then ended 0.014 from the
// sequential sums' parameters, against 0.003 between two orders of sequential sums.
// What is left is one tile's serial chain: code fetch, weights, the three products.
__global__ void __launch_bounds__(kWG) k_mlp_train(MlpArgs a) {
    __shared__ __align__(16) MlpLds m;
    __shared__ __align__(16) uint16_t operands[3 * kHid * kPitch];
    uint16_t *w2t = operands;              // [in][out]
    uint16_t *h1t = w2t + kHid * kPitch;   // [in][sample], 64 samples
    uint16_t *dzt = h1t + kHid * kPitch;   // [out][sample], 64 samples
    __shared__ __align__(16) uint16_t dzs[kWaves][kTile * kPitch];  // [sample][out] of a wave's tile
    __shared__ __align__(16) float xt[kWaves][kTile * kIn];
    __shared__ float red_out[4 * kWaves];
    __shared__ __align__(16) float squares[4 * kTile];  // [wave][sample mod 4][sample / 4]
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, q = l >> 4, i = l & 15;
    const int64_t tiles = (a.count + kTile - 1) / kTile;
    const int64_t rounds = (tiles + kWaves - 1) / kWaves;
    // a round's samples are drawn and gathered ahead: the first while the weights load,
    // each next one during the products of the round before
    float x[kIn], tgt = 0.f;
    auto fetch = [&](int64_t round) {
        const int64_t slot = (round * kWaves + w) * kTile + i;
        const bool valid = round < rounds && slot < a.count;
        int64_t sa = 0;
        if (valid) {
            if (a.idx) {
                sa = a.idx[slot];
            } else {
                const u32x4 rnd = philox4x32_10(a.step, (uint32_t)slot, kMlpTag, 0u, (uint32_t)a.seed,
                                                (uint32_t)(a.seed >> 32));
                sa = (int64_t)(((uint64_t)rnd.x * (uint64_t)a.n) >> 32);
            }
        }
        tgt = valid ? a.target[sa] : 0.f;
#pragma unroll
        for (int k = 0; k < kIn; ++k) x[k] = valid ? a.feat[sa * kIn + k] : 0.f;
    };
    fetch(blockIdx.x);
    load_weights(a, m);
    for (int p = tid; p < kHid * kHid; p += kWG) w2t[(p & 63) * kPitch + (p >> 6)] = a.w2b[p];
    const float b3 = a.master[ob3];
    float4v G[4];
    float gw1[4][kIn], gb1[4], gw3[4], gb2[4], gb3 = 0.f, sq[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        G[nb] = (float4v){0.f, 0.f, 0.f, 0.f};
        gb1[nb] = gw3[nb] = gb2[nb] = 0.f;
#pragma unroll
        for (int k = 0; k < kIn; ++k) gw1[nb][k] = 0.f;
    }
    __syncthreads();
    for (int64_t round = blockIdx.x; round < rounds; round += gridDim.x) {
        const int64_t tile = round * kWaves + w;
        const float tgt_now = tgt;
        float xb[kIn];
#pragma unroll
        for (int k = 0; k < kIn; ++k) xb[k] = from_bf16(to_bf16((x[k] - a.norm[k]) * a.norm[kIn + k]));
        short4v A[4];
        float h2[4][4], y[4], dy[4];
        mlp_forward(m, b3, xb, q, i, A, h2, y);
        if (q == 0) {
            *(float4v *)&xt[w][i * kIn] = (float4v){xb[0], xb[1], xb[2], xb[3]};
            *(float4v *)&xt[w][i * kIn + 4] = (float4v){xb[4], xb[5], xb[6], xb[7]};
        }
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) h1t[(16 * kb + 4 * q + r) * kPitch + 16 * w + i] = (uint16_t)A[kb][r];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float t = __shfl(tgt_now, 4 * q + r, 64);
            const float diff = tile * kTile + 4 * q + r < a.count ? y[r] - t : 0.f;
            dy[r] = 2.f * diff * a.inv_batch;
            gb3 += dy[r];
            sq[r] += diff * diff;
        }
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            const int o = 16 * nb + i;
            short4v d4;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                gw3[nb] += dy[r] * h2[nb][r];
                const float d = h2[nb][r] > 0.f ? dy[r] * m.w3[o] : 0.f;
                gb2[nb] += d;
                d4[r] = (short)to_bf16(d);
                dzs[w][(4 * q + r) * kPitch + o] = (uint16_t)d4[r];
            }
            *(short4v *)&dzt[o * kPitch + 16 * w + 4 * q] = d4;
        }
        __syncthreads();
        fetch(round + gridDim.x);
        // dW2 (64 x 64) = dZ2^T H1 over the workgroup's 64 samples
#pragma unroll
        for (int t = 0; t < kWaves; ++t) {
            const short4v Av = *(const short4v *)&dzt[(16 * w + i) * kPitch + 16 * t + 4 * q];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
                G[kb] += __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                    Av, *(const short4v *)&h1t[(16 * kb + i) * kPitch + 16 * t + 4 * q],
                    (float4v){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
        // dH1 (16 x 64) = dZ2 (16 x 64) W2, masked by the stored H1; dW1, db1
        short4v Ad[4];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) Ad[kb] = *(const short4v *)&dzs[w][i * kPitch + 16 * kb + 4 * q];
        float4v xa[4], xc[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            xa[r] = *(const float4v *)&xt[w][(4 * q + r) * kIn];
            xc[r] = *(const float4v *)&xt[w][(4 * q + r) * kIn + 4];
        }
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            float4v E = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
                E = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                    Ad[kb], *(const short4v *)&w2t[(16 * nb + i) * kPitch + 16 * kb + 4 * q], E, 0, 0, 0);
            const short4v h = *(const short4v *)&h1t[(16 * nb + i) * kPitch + 16 * w + 4 * q];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float d = from_bf16((uint16_t)h[r]) > 0.f ? E[r] : 0.f;
                gb1[nb] += d;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    gw1[nb][k] += d * xa[r][k];
                    gw1[nb][4 + k] += d * xc[r][k];
                }
            }
        }
        __syncthreads();
    }
    float *dst = a.partial + (size_t)blockIdx.x * (kParams + 1);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[oW2 + (16 * w + 4 * q + r) * kHid + 16 * kb + i] = G[kb][r];
    // the other sums: the 16 lanes (four waves' rows) that hold a parameter's share, added
    // one after the other, 32 outs at a time
    float *red = (float *)operands;  // [share][out][11]
    constexpr int kHalf = kHid / 2 * 11;
    static_assert(4 * kWaves * kHalf * sizeof(float) <= sizeof(operands), "shares");
    if (i == 0) {
        red_out[4 * w + q] = gb3;
#pragma unroll
        for (int r = 0; r < 4; ++r) squares[kTile * w + 4 * r + q] = sq[r];
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            float *to = red + (4 * w + q) * kHalf + (16 * b + i) * 11;
            const int nb = 2 * half + b;
#pragma unroll
            for (int k = 0; k < kIn; ++k) to[k] = gw1[nb][k];
            to[8] = gb1[nb];
            to[9] = gw3[nb];
            to[10] = gb2[nb];
        }
        __syncthreads();
        for (int p = tid; p < kHalf; p += kWG) {
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < 4 * kWaves; ++j) s += red[j * kHalf + p];
            const int o = 32 * half + p / 11, k = p % 11;
            dst[k < kIn ? oW1 + o * kIn + k : k == 8 ? ob1 + o : k == 9 ? ow3 + o : ob2 + o] = s;
        }
    }
    // db3 and the loss: the four lanes of a tile first
    if (tid == 0) {
        float s = 0.f;
        for (int j = 0; j < 4 * kWaves; j += 4) s += ((red_out[j] + red_out[j + 1]) + red_out[j + 2]) + red_out[j + 3];
        dst[ob3] = s;
    }
    if (tid == 3 * 64) {  // (a wave with no share left to add above)
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < kWaves * kTile; j += 4)
            s += ((squares[j] + squares[j + 1]) + squares[j + 2]) + squares[j + 3];
        dst[kParams] = s;
    }
}

struct AdamArgs {
    float *master, *m, *v;
    uint16_t *w1b, *w2b, *w3b;
    float lr, beta1, beta2, eps, bc1, bc2;
};

__device__ __forceinline__ void adam_param(const AdamArgs &a, int p, float g) {
    const float mm = a.beta1 * a.m[p] + (1.f - a.beta1) * g;
    const float vv = a.beta2 * a.v[p] + (1.f - a.beta2) * g * g;
    a.m[p] = mm;
    a.v[p] = vv;
    const float th = a.master[p] - a.lr * (mm / a.bc1) / (sqrtf(vv / a.bc2) + a.eps);
    a.master[p] = th;
    if (p < ob1) a.w1b[p - oW1] = to_bf16(th);
    else if (p >= oW2 && p < ob2) a.w2b[p - oW2] = to_bf16(th);
    else if (p >= ow3 && p < ob3) a.w3b[p - ow3] = to_bf16(th);
}

// The workgroups' partials added in index order, to grad (kParams + 1, the loss sum last)
// or straight into an Adam step.
template <bool kAdam>
__global__ void __launch_bounds__(64) k_mlp_reduce(const float *__restrict__ partial, int nwg, float *grad, AdamArgs a,
                                                   float *loss_slot, float inv_batch) {
    const int p = blockIdx.x * 64 + threadIdx.x;
    if (p > kParams) return;
    float s = 0.f;
    const float *from = partial + p;
    int r = 0;
    for (; r + 16 <= nwg; r += 16) {
        float v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = from[(size_t)(r + j) * (kParams + 1)];
#pragma unroll
        for (int j = 0; j < 16; ++j) s += v[j];
    }
    for (; r < nwg; ++r) s += from[(size_t)r * (kParams + 1)];
    if (!kAdam) {
        grad[p] = s;
    } else if (p == kParams) {
        if (loss_slot) *loss_slot = s * inv_batch;
    } else {
        adam_param(a, p, s);
    }
}

__global__ void __launch_bounds__(256) k_adam(AdamArgs a, const float *grad) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < kParams) adam_param(a, p, grad[p]);
}

__global__ void __launch_bounds__(256) k_round_weights(const float *master, uint16_t *w1b, uint16_t *w2b,
                                                       uint16_t *w3b) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < 512) w1b[p] = to_bf16(master[oW1 + p]);
    if (p < 4096) w2b[p] = to_bf16(master[oW2 + p]);
    if (p < 64) w3b[p] = to_bf16(master[ow3 + p]);
}

// mean and 1/std of each feature column (population std; 1 when the column is
// constant). Up to kStatRows rows a workgroup takes a column (k_column_stats). Beyond them,
// workgroup sums of x and x^2 of all columns, which one workgroup adds in index order: with a
// workgroup per column 7, 11, 18 and 214 us for 8000, 16000, 30000 and 200000 rows, with the
// two launches 10, 12, 14 and 16.
constexpr int kStatBlocks = 128;
constexpr int64_t kStatRows = 20000;

// column k's entries of norm from its sums over n rows
__device__ __forceinline__ void put_norm(float *norm, int k, double s, double s2, int64_t n) {
    const double mean = s / (double)n;
    const double var = s2 / (double)n - mean * mean;
    norm[k] = (float)mean;
    norm[kIn + k] = var > 1e-12 ? (float)(1.0 / sqrt(var)) : 1.f;
}

__global__ void __launch_bounds__(256) k_column_stats(const float *__restrict__ feat, int64_t n, float *norm) {
    __shared__ double red[2][256];
    const int k = blockIdx.x, t = threadIdx.x;
    double s = 0.0, s2 = 0.0;
    for (int64_t r = t; r < n; r += 256) {
        const double x = feat[r * kIn + k];
        s += x;
        s2 += x * x;
    }
    red[0][t] = s;
    red[1][t] = s2;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (t < off) {
            red[0][t] += red[0][t + off];
            red[1][t] += red[1][t + off];
        }
        __syncthreads();
    }
    if (t == 0) put_norm(norm, k, red[0][0], red[1][0], n);
}

__global__ void __launch_bounds__(256) k_feature_sums(const float *__restrict__ feat, int64_t n,
                                                      double *__restrict__ sums) {
    __shared__ double red[4][2 * kIn];
    double s[2 * kIn];
#pragma unroll
    for (int k = 0; k < 2 * kIn; ++k) s[k] = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride) {
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            const double x = feat[r * kIn + k];
            s[k] += x;
            s[kIn + k] += x * x;
        }
    }
#pragma unroll
    for (int k = 0; k < 2 * kIn; ++k) {
        const double v = wave_sum(s[k]);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][k] = v;
    }
    __syncthreads();
    const int k = threadIdx.x;
    if (k < 2 * kIn) sums[blockIdx.x * 2 * kIn + k] = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
}

__global__ void __launch_bounds__(64) k_feature_stats(const double *__restrict__ sums, int nb, int64_t n, float *norm) {
    const int k = threadIdx.x & 15;
    double v = 0.0;
    for (int b = threadIdx.x >> 4; b < nb; b += 4) v += sums[b * 2 * kIn + k];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    const double s2 = __shfl(v, (k & 7) + kIn, 64);
    if (threadIdx.x < kIn) put_norm(norm, k, v, s2, n);
}

}  // namespace
}  // namespace mcmi

using namespace mcmi;

struct mcmi_mlp {
    float *master = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr, *norm = nullptr, *partial = nullptr;
    uint16_t *w1b = nullptr, *w2b = nullptr, *w3b = nullptr;
    double *sums = nullptr;  // feature sums of k_feature_sums
    int partial_rows = 0;
    int64_t t = 0;
};

namespace {

mcmi_status mlp_alloc_partial(mcmi_mlp *net, int rows) {
    if (rows <= net->partial_rows) return MCMI_OK;
    (void)hipFree(net->partial);
    net->partial = nullptr;
    MCMI_HIP(hipMalloc(&net->partial, (size_t)rows * (kParams + 1) * sizeof(float)));
    net->partial_rows = rows;
    return MCMI_OK;
}

int mlp_grid(int64_t count) {
    const int64_t tiles = (count + kTile - 1) / kTile;
    int64_t blocks = (tiles + kWaves - 1) / kWaves;
    const int64_t cap = (int64_t)device_cus() * 4;
    if (blocks > cap) blocks = cap;
    return (int)std::max<int64_t>(blocks, 1);
}

MlpArgs mlp_args(const mcmi_mlp *net) {
    MlpArgs a;
    memset(&a, 0, sizeof(a));
    a.master = net->master;
    a.w1b = net->w1b;
    a.w2b = net->w2b;
    a.w3b = net->w3b;
    a.norm = net->norm;
    return a;
}

// Adam step number net->t
AdamArgs adam_args(const mcmi_mlp *net, float lr) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float bc1 = 1.f - powf(b1, (float)net->t), bc2 = 1.f - powf(b2, (float)net->t);
    return {net->master, net->m, net->v, net->w1b, net->w2b, net->w3b, lr, b1, b2, eps, bc1, bc2};
}

}  // namespace

extern "C" mcmi_status mcmi_mlp_create(mcmi_mlp **out) {
    if (!out) return fail(MCMI_ERR_ARG, "mcmi_mlp_create: null argument");
    *out = nullptr;
    mcmi_mlp *net = new mcmi_mlp();
    hipError_t e = hipSuccess;
    if (e == hipSuccess) e = hipMalloc(&net->master, kParams * sizeof(float));
    if (e == hipSuccess) e = hipMalloc(&net->m, kParams * sizeof(float));
    if (e == hipSuccess) e = hipMalloc(&net->v, kParams * sizeof(float));
    if (e == hipSuccess) e = hipMalloc(&net->grad, (kParams + 1) * sizeof(float));
    if (e == hipSuccess) e = hipMalloc(&net->norm, 2 * kIn * sizeof(float));
    if (e == hipSuccess) e = hipMalloc(&net->sums, kStatBlocks * 2 * kIn * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&net->w1b, 512 * sizeof(uint16_t));
    if (e == hipSuccess) e = hipMalloc(&net->w2b, 4096 * sizeof(uint16_t));
    if (e == hipSuccess) e = hipMalloc(&net->w3b, 64 * sizeof(uint16_t));
    if (e == hipSuccess) e = hipMemset(net->master, 0, kParams * sizeof(float));
    if (e == hipSuccess) e = hipMemset(net->m, 0, kParams * sizeof(float));
    if (e == hipSuccess) e = hipMemset(net->v, 0, kParams * sizeof(float));
    if (e != hipSuccess) {
        mcmi_mlp_free(net);
        return fail(MCMI_ERR_HIP, std::string("mcmi_mlp_create: ") + hipGetErrorString(e));
    }
    std::vector<float> nm(2 * kIn, 0.f);
    for (int k = 0; k < kIn; ++k) nm[kIn + k] = 1.f;
    if (hipMemcpy(net->norm, nm.data(), nm.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess) {
        mcmi_mlp_free(net);
        return fail(MCMI_ERR_HIP, "mcmi_mlp_create: copy");
    }
    *out = net;
    return MCMI_OK;
}

extern "C" void mcmi_mlp_free(mcmi_mlp *net) {
    if (!net) return;
    (void)hipFree(net->master);
    (void)hipFree(net->m);
    (void)hipFree(net->v);
    (void)hipFree(net->grad);
    (void)hipFree(net->norm);
    (void)hipFree(net->partial);
    (void)hipFree(net->sums);
    (void)hipFree(net->w1b);
    (void)hipFree(net->w2b);
    (void)hipFree(net->w3b);
    delete net;
}

extern "C" mcmi_status mcmi_mlp_set_params(mcmi_mlp *net, const float *params_host, const float *norm_host,
                                           int32_t reset_optimizer) {
    if (!net || !params_host) return fail(MCMI_ERR_ARG, "mcmi_mlp_set_params: null argument");
    MCMI_HIP(hipMemcpy(net->master, params_host, kParams * sizeof(float), hipMemcpyHostToDevice));
    if (norm_host) MCMI_HIP(hipMemcpy(net->norm, norm_host, 2 * kIn * sizeof(float), hipMemcpyHostToDevice));
    if (reset_optimizer) {
        MCMI_HIP(hipMemset(net->m, 0, kParams * sizeof(float)));
        MCMI_HIP(hipMemset(net->v, 0, kParams * sizeof(float)));
        net->t = 0;
    }
    k_round_weights<<<16, 256>>>(net->master, net->w1b, net->w2b, net->w3b);
    MCMI_HIP(hipGetLastError());
    MCMI_HIP(hipDeviceSynchronize());
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_mlp_get_params(const mcmi_mlp *net, float *params_host, float *norm_host,
                                           float *adam_m_host, float *adam_v_host, int64_t *adam_step) {
    if (!net) return fail(MCMI_ERR_ARG, "mcmi_mlp_get_params: null argument");
    MCMI_HIP(hipDeviceSynchronize());
    if (params_host) MCMI_HIP(hipMemcpy(params_host, net->master, kParams * sizeof(float), hipMemcpyDeviceToHost));
    if (norm_host) MCMI_HIP(hipMemcpy(norm_host, net->norm, 2 * kIn * sizeof(float), hipMemcpyDeviceToHost));
    if (adam_m_host) MCMI_HIP(hipMemcpy(adam_m_host, net->m, kParams * sizeof(float), hipMemcpyDeviceToHost));
    if (adam_v_host) MCMI_HIP(hipMemcpy(adam_v_host, net->v, kParams * sizeof(float), hipMemcpyDeviceToHost));
    if (adam_step) *adam_step = net->t;
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_mlp_set_adam_state(mcmi_mlp *net, const float *adam_m_host, const float *adam_v_host,
                                               int64_t adam_step) {
    if (!net || !adam_m_host || !adam_v_host || adam_step < 0)
        return fail(MCMI_ERR_ARG, "mcmi_mlp_set_adam_state: bad argument");
    MCMI_HIP(hipMemcpy(net->m, adam_m_host, kParams * sizeof(float), hipMemcpyHostToDevice));
    MCMI_HIP(hipMemcpy(net->v, adam_v_host, kParams * sizeof(float), hipMemcpyHostToDevice));
    net->t = adam_step;
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_mlp_fit_normalization(mcmi_mlp *net, const float *feat_dev, int64_t n, void *stream) {
    if (!net || !feat_dev || n < 1) return fail(MCMI_ERR_ARG, "mcmi_mlp_fit_normalization: bad argument");
    if (n <= kStatRows) {
        k_column_stats<<<kIn, 256, 0, (hipStream_t)stream>>>(feat_dev, n, net->norm);
        MCMI_HIP(hipGetLastError());
        return MCMI_OK;
    }
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, kStatBlocks);
    k_feature_sums<<<blocks, 256, 0, (hipStream_t)stream>>>(feat_dev, n, net->sums);
    MCMI_HIP(hipGetLastError());
    k_feature_stats<<<1, 64, 0, (hipStream_t)stream>>>(net->sums, blocks, n, net->norm);
    MCMI_HIP(hipGetLastError());
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_mlp_predict(const mcmi_mlp *net, const float *feat_dev, int64_t n, float *out_dev,
                                        void *stream) {
    if (!net || !feat_dev || !out_dev || n < 0) return fail(MCMI_ERR_ARG, "mcmi_mlp_predict: bad argument");
    if (n == 0) return MCMI_OK;
    MlpArgs a = mlp_args(net);
    a.feat = feat_dev;
    a.n = n;
    a.count = n;
    a.out = out_dev;
    k_mlp_predict<<<mlp_grid(n), kWG, 0, (hipStream_t)stream>>>(a);
    MCMI_HIP(hipGetLastError());
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_mlp_gradient(mcmi_mlp *net, const float *feat_dev, const float *target_dev,
                                         const int32_t *idx_dev, int64_t batch, int64_t n, float *grad_host,
                                         float *loss_host, void *stream) {
    if (!net || !feat_dev || !target_dev || !idx_dev || batch < 1 || n < 1)
        return fail(MCMI_ERR_ARG, "mcmi_mlp_gradient: bad argument");
    hipStream_t s = (hipStream_t)stream;
    const int grid = mlp_grid(batch);
    mcmi_status st = mlp_alloc_partial(net, grid);
    if (st != MCMI_OK) return st;
    MlpArgs a = mlp_args(net);
    a.feat = feat_dev;
    a.target = target_dev;
    a.idx = idx_dev;
    a.n = n;
    a.count = batch;
    a.partial = net->partial;
    a.inv_batch = 1.f / (float)batch;
    k_mlp_train<<<grid, kWG, 0, s>>>(a);
    MCMI_HIP(hipGetLastError());
    k_mlp_reduce<false><<<(kParams + 1 + 63) / 64, 64, 0, s>>>(net->partial, grid, net->grad, AdamArgs{}, nullptr, 0.f);
    MCMI_HIP(hipGetLastError());
    float tmp[kParams + 1];
    MCMI_HIP(hipMemcpyAsync(tmp, net->grad, (kParams + 1) * sizeof(float), hipMemcpyDeviceToHost, s));
    MCMI_HIP(hipStreamSynchronize(s));
    if (grad_host) memcpy(grad_host, tmp, kParams * sizeof(float));
    if (loss_host) *loss_host = tmp[kParams] / (float)batch;
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_mlp_train(mcmi_mlp *net, const float *feat_dev, const float *target_dev, int64_t n,
                                      int32_t steps, int32_t batch, float lr, uint64_t seed, float *loss_host,
                                      void *stream) {
    if (!net || !feat_dev || !target_dev || n < 1 || steps < 0 || batch < 1 || !(lr > 0.f))
        return fail(MCMI_ERR_ARG, "mcmi_mlp_train: bad argument");
    hipStream_t s = (hipStream_t)stream;
    const int grid = mlp_grid(batch);
    mcmi_status st = mlp_alloc_partial(net, grid);
    if (st != MCMI_OK) return st;
    float *losses = nullptr;
    MCMI_HIP(hipMallocAsync((void **)&losses, (size_t)std::max(steps, 1) * sizeof(float), s));
    for (int32_t k = 0; k < steps; ++k) {
        MlpArgs a = mlp_args(net);
        a.feat = feat_dev;
        a.target = target_dev;
        a.n = n;
        a.count = batch;
        a.partial = net->partial;
        a.seed = seed;
        a.step = (uint32_t)(net->t + 1);
        a.inv_batch = 1.f / (float)batch;
        k_mlp_train<<<grid, kWG, 0, s>>>(a);
        net->t += 1;
        k_mlp_reduce<true><<<(kParams + 1 + 63) / 64, 64, 0, s>>>(net->partial, grid, nullptr, adam_args(net, lr),
                                                                   losses + k, 1.f / (float)batch);
    }
    MCMI_HIP(hipGetLastError());
    if (loss_host && steps > 0)
        MCMI_HIP(hipMemcpyAsync(loss_host, losses, (size_t)steps * sizeof(float), hipMemcpyDeviceToHost, s));
    MCMI_HIP(hipFreeAsync(losses, s));
    MCMI_HIP(hipStreamSynchronize(s));
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_mlp_adam_step(mcmi_mlp *net, const float *grad_dev, float lr, void *stream) {
    if (!net || !grad_dev || !(lr > 0.f)) return fail(MCMI_ERR_ARG, "mcmi_mlp_adam_step: bad argument");
    hipStream_t s = (hipStream_t)stream;
    net->t += 1;
    k_adam<<<(kParams + 255) / 256, 256, 0, s>>>(adam_args(net, lr), grad_dev);
    MCMI_HIP(hipGetLastError());
    return MCMI_OK;
}

// ------------------------------------------------------------ allocation
// N_r = max(1, rint(lambda * exp(pred_r))) with lambda found by bisection so that
// sum_r N_r cost_r is the largest total not above the budget: hi doubles from 1
// while total(hi) <= budget (and hi < 1e30), then 100 halvings of [0, hi] keep
// total(lo) <= budget < total(hi); lambda = lo. Every total is an exact integer
// sum. A launch evaluates kCand candidates in one pass over the rows: the next
// kCand doublings, or every midpoint that the next kDepth halvings can reach; the last
// workgroup to arrive then takes the same decisions, in the same order, as a
// sequential loop would, and ends the search once a halving changes nothing. At
// 1M rows that is about 15 working passes of 17 us (26 with each candidate's sum taken by
// wave shuffles, one candidate after the other) instead of 160 passes of 15 us, each
// with a one-thread launch behind it (allocation 5.2 -> 0.35 ms). Non-finite
// predictions fall back to the uniform allocation N_r = max(1, floor(budget / sum_r cost_r)).
namespace mcmi {
namespace {

constexpr int kDepth = 4, kCand = (1 << kDepth) - 1;
constexpr int kAllocBlocks = 512;  // most workgroups of a pass
constexpr int kSumPitch = 260;     // 4 more than 256: the 16 candidates of a wave's reads hit distinct banks
constexpr int kDoublings = 101;    // hi reaches 2^100 > 1e30
constexpr int kPasses = (kDoublings + kCand - 1) / kCand + 100 / kDepth;

struct AllocState {
    double lo, hi;
    long long bad;    // non-finite predictions
    long long csum;   // sum of costs
    int32_t phase;    // 0: doubling hi, 1: halving, 2: done
    int32_t halvings;
    int32_t hi_over;  // total(hi) > budget is known
    uint32_t arrived;
};

__device__ __forceinline__ long long block_sum_ll(long long v, long long *red) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0) red[w] = v;
    __syncthreads();
    long long t = 0;
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) t += red[k];
    __syncthreads();
    return t;
}

__device__ __forceinline__ int32_t chains_of(double lam, double e) {
    return (int32_t)fmin(fmax(rint(lam * e), 1.0), 2147483647.0);  // 1 where lam e is NaN
}

__global__ void __launch_bounds__(256) k_alloc_prep(const float *pred, const int32_t *cost, int64_t n, double *e,
                                                    AllocState *st) {
    __shared__ long long red[4];
    long long bad = 0, csum = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride) {
        const float p = pred[r];
        bad += isfinite(p) ? 0 : 1;
        e[r] = exp((double)p);
        csum += cost[r];
    }
    bad = block_sum_ll(bad, red);
    csum = block_sum_ll(csum, red);
    if (threadIdx.x == 0) {
        if (bad) atomicAdd((unsigned long long *)&st->bad, (unsigned long long)bad);
        atomicAdd((unsigned long long *)&st->csum, (unsigned long long)csum);
    }
}

// One pass: the totals of this state's candidates (workgroup sums in part, kCand per
// workgroup), then the last workgroup's decisions.
__global__ void __launch_bounds__(256) k_alloc_pass(const double *__restrict__ e, const int32_t *__restrict__ cost,
                                                    int64_t n, long long budget, long long *part, AllocState *st) {
    __shared__ long long each[kCand][kSumPitch], red[16][kCand + 1], tot[kCand];
    __shared__ int last;
    const int32_t phase = st->phase;
    if (phase == 2) return;
    // candidates: hi, 2 hi, 4 hi, ..; or the midpoints as a tree (children of node i: 2 i + 1
    // after hi = mid, 2 i + 2 after lo = mid)
    double lo[kCand], hi[kCand], lam[kCand];
    lo[0] = st->lo;
    hi[0] = st->hi;
    if (phase == 0) {
        lam[0] = hi[0];
#pragma unroll
        for (int i = 1; i < kCand; ++i) lam[i] = lam[i - 1] * 2.0;
    } else {
#pragma unroll
        for (int i = 0; i < kCand; ++i) {
            if (i > 0) {
                const int up = (i - 1) / 2;
                lo[i] = (i & 1) ? lo[up] : lam[up];
                hi[i] = (i & 1) ? lam[up] : hi[up];
            }
            lam[i] = 0.5 * (lo[i] + hi[i]);
        }
    }
    long long sum[kCand];
#pragma unroll
    for (int i = 0; i < kCand; ++i) sum[i] = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride) {
        const double er = e[r];
        const int32_t c = cost[r];
#pragma unroll
        for (int i = 0; i < kCand; ++i) sum[i] += (long long)chains_of(lam[i], er) * (long long)c;
    }
    // 16 threads to a candidate: of a workgroup's 256 shares each adds every 16th, and of
    // the workgroups' sums likewise
    const int t = threadIdx.x, ci = t & 15, cg = t >> 4;
#pragma unroll
    for (int i = 0; i < kCand; ++i) each[i][t] = sum[i];
    __syncthreads();
    if (ci < kCand) {
        long long v = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) v += each[ci][16 * k + cg];
        red[cg][ci] = v;
    }
    __syncthreads();
    if (t < kCand) {
        long long v = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) v += red[k][t];
        __hip_atomic_store(part + (size_t)blockIdx.x * kCand + t, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (t == 0)
        last = __hip_atomic_fetch_add(&st->arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1u;
    __syncthreads();
    if (!last) return;
    if (ci < kCand) {
        long long v = 0;
#pragma unroll 8
        for (int b = cg; b < (int)gridDim.x; b += 16)
            v += __hip_atomic_load(part + (size_t)b * kCand + ci, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        red[cg][ci] = v;
    }
    __syncthreads();
    if (t < kCand) {
        long long v = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) v += red[k][t];
        tot[t] = v;
    }
    __syncthreads();
    if (t != 0) return;
    st->arrived = 0u;
    if (phase == 0) {
        double h = st->hi;
        for (int i = 0; i < kCand; ++i) {
            const bool fits = tot[i] <= budget;
            if (fits && h < 1e30) {
                h *= 2.0;
            } else {
                st->hi_over = !fits;
                st->phase = 1;
                break;
            }
        }
        st->hi = h;
        return;
    }
    double l = st->lo, h = st->hi;
    int32_t over = st->hi_over, done = st->halvings, node = 0;
    bool settled = false;
    for (int d = 0; d < kDepth && done < 100 && !settled; ++d, ++done) {
        const double mid = 0.5 * (l + h);
        // a midpoint that equals an end whose side is known changes nothing from here on
        settled = (mid == l && l > 0.0) || (mid == h && over);
        if (tot[node] <= budget) {
            l = mid;
            node = 2 * node + 2;
        } else {
            h = mid;
            over = 1;
            node = 2 * node + 1;
        }
    }
    st->lo = l;
    st->hi = h;
    st->hi_over = over;
    st->halvings = done;
    if (done == 100 || settled) st->phase = 2;
}

__global__ void __launch_bounds__(256) k_alloc_write(const double *e, int64_t n, long long budget,
                                                     const AllocState *st, int32_t *chains, double *lam_out,
                                                     int32_t *fallback_out) {
    const bool fb0 = st->bad > 0 || st->csum <= 0;
    const double lam = fb0 ? 0.0 : st->lo;
    const bool fb = fb0 || !(lam > 0.0);
    const long long csum = st->csum;
    const long long uni = csum > 0 ? (budget / csum > 1 ? budget / csum : 1) : 1;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride)
        chains[r] = fb ? (int32_t)(uni < 2147483647LL ? uni : 2147483647LL) : (int32_t)chains_of(lam, e[r]);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *lam_out = lam;
        *fallback_out = fb ? 1 : 0;
    }
}

// the bisection's starting state, written on the device (the no-allocation
// variant clears its static workspace with this instead of a host copy)
__global__ void k_alloc_init(AllocState *st) {
    if (threadIdx.x == 0) {
        st->lo = 0.0;
        st->hi = 1.0;
        st->bad = 0;
        st->csum = 0;
        st->phase = 0;
        st->halvings = 0;
        st->hi_over = 0;
        st->arrived = 0u;
    }
}

// Workspace of mcmi_allocate_noalloc: the bisection state, the lambda and
// fallback slots, a pass's workgroup sums, then exp(pred_r) for up to kNoAllocMaxRows rows.
constexpr int64_t kNoAllocMaxRows = int64_t(1) << 22;
constexpr size_t kNoAllocPart = 256;
constexpr size_t kNoAllocHead = 65536;
static_assert(kNoAllocPart + (size_t)kAllocBlocks * kCand * sizeof(long long) <= kNoAllocHead, "workgroup sums");
constexpr size_t kNoAllocBytes = kNoAllocHead + (size_t)kNoAllocMaxRows * sizeof(double);
static_assert(sizeof(AllocState) <= 64, "state slot");

unsigned alloc_grid(int64_t n) { return (unsigned)std::min<int64_t>((n + 255) / 256, kAllocBlocks); }

// The whole search on `s`: st, part (kAllocBlocks x kCand), e (n) and the outputs on the device.
hipError_t launch_allocation(const float *pred, const int32_t *cost, int64_t n, int64_t budget, AllocState *st,
                             long long *part, double *e, int32_t *chains, double *lam, int32_t *fbk, hipStream_t s) {
    const unsigned blocks = alloc_grid(n);
    k_alloc_init<<<1, 64, 0, s>>>(st);
    k_alloc_prep<<<blocks, 256, 0, s>>>(pred, cost, n, e, st);
    for (int it = 0; it < kPasses; ++it)  // passes after the search has ended return at once
        k_alloc_pass<<<blocks, 256, 0, s>>>(e, cost, n, (long long)budget, part, st);
    k_alloc_write<<<blocks, 256, 0, s>>>(e, n, (long long)budget, st, chains, lam, fbk);
    return hipGetLastError();
}

}  // namespace
}  // namespace mcmi

// Static workspace (one copy per GPU, alive until the process ends). Host code
// never passes this name to a kernel: it uses the device address that
// hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[mcmi::kNoAllocBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device.
hipError_t scratch_address(void **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}
}  // namespace

extern "C" mcmi_status mcmi_allocate(const float *pred_dev, const int32_t *cost_dev, int64_t n, int64_t budget,
                                     int32_t *chains_dev, double *lambda_host, int32_t *fallback_host,
                                     void *stream) {
    if (!pred_dev || !cost_dev || !chains_dev || n < 1 || budget < 1)
        return fail(MCMI_ERR_ARG, "mcmi_allocate: bad argument");
    hipStream_t s = (hipStream_t)stream;
    // exp(pred), then the state, lambda, fallback flag and workgroup sums
    double *e = nullptr;
    unsigned char *head = nullptr;
    MCMI_HIP(dev_alloc((void **)&e, (size_t)n * sizeof(double), s));
    hipError_t err = dev_alloc((void **)&head, kNoAllocHead, s);
    if (err != hipSuccess) {
        dev_release(e, s);
        return fail(MCMI_ERR_HIP, std::string("mcmi_allocate: ") + hipGetErrorString(err));
    }
    double *lam = (double *)(head + 64);
    int32_t *fbk = (int32_t *)(head + 72);
    err = launch_allocation(pred_dev, cost_dev, n, budget, (AllocState *)head, (long long *)(head + kNoAllocPart), e,
                            chains_dev, lam, fbk, s);
    double hl = 0.0;
    int32_t hf = 0;
    if (err == hipSuccess) err = hipMemcpyAsync(&hl, lam, sizeof(double), hipMemcpyDeviceToHost, s);
    if (err == hipSuccess) err = hipMemcpyAsync(&hf, fbk, sizeof(int32_t), hipMemcpyDeviceToHost, s);
    if (err == hipSuccess) err = hipStreamSynchronize(s);
    dev_release(e, s);
    dev_release(head, s);
    if (err != hipSuccess) return fail(MCMI_ERR_HIP, std::string("mcmi_allocate: ") + hipGetErrorString(err));
    if (lambda_host) *lambda_host = hl;
    if (fallback_host) *fallback_host = hf;
    return MCMI_OK;
}

extern "C" mcmi_status mcmi_allocate_noalloc(const float *pred_dev, const int32_t *cost_dev, int64_t n,
                                             int64_t budget, int32_t *chains_dev, double *lambda_dev,
                                             int32_t *fallback_dev, void *stream) {
    using namespace mcmi;
    if (!pred_dev || !cost_dev || !chains_dev || n < 1 || budget < 1)
        return fail(MCMI_ERR_ARG, "mcmi_allocate_noalloc: bad argument");
    if (n > kNoAllocMaxRows)
        return fail(MCMI_ERR_ARG, "mcmi_allocate_noalloc: n = " + std::to_string(n) +
                                      " rows exceeds the static workspace (" + std::to_string(kNoAllocMaxRows) +
                                      " rows); use mcmi_allocate");
    void *base = nullptr;
    hipError_t err = scratch_address(&base);
    if (err != hipSuccess)
        return fail(MCMI_ERR_HIP, std::string("mcmi_allocate_noalloc: workspace address: ") + hipGetErrorString(err));
    hipStream_t s = (hipStream_t)stream;
    unsigned char *head = (unsigned char *)base;
    err = launch_allocation(pred_dev, cost_dev, n, budget, (AllocState *)head, (long long *)(head + kNoAllocPart),
                            (double *)(head + kNoAllocHead), chains_dev,
                            lambda_dev ? lambda_dev : (double *)(head + 64),
                            fallback_dev ? fallback_dev : (int32_t *)(head + 72), s);
    if (err != hipSuccess) return fail(MCMI_ERR_HIP, std::string("mcmi_allocate_noalloc: ") + hipGetErrorString(err));
    return MCMI_OK;
}
