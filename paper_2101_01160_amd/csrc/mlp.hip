// Surrogate network for the MDLG equilibrium distribution on gfx950:
// 6 -> 256 -> 256 -> 256 -> 49, SiLU, softmax, trained with the Kullback-
// Leibler divergence (Eq.(kullback_leibler)) against measured f_eq.
//
// Matrix products run on the BF16 matrix cores (v_mfma_f32_16x16x32_bf16):
// bf16 operands, fp32 accumulation, fp32 master weights and Adam state.  A
// training step is three launches: forward and backward of a few samples per
// block, all weight gradients, and their sum with the Adam update.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "mdlg_internal.h"

namespace mdlg {
namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kIn = 6, kHid = 256, kOut = 49, kOutP = 64;
constexpr long kW1 = 0, kB1 = 1536, kW2 = 1792, kB2 = 67328, kW3 = 67584, kB3 = 133120, kW4 = 133376, kB4 = 145920;
constexpr long kParams = 145969;
constexpr int kMaxSplit = 32, kMidSplit = 16;  // splits of the batch for gradients: layers 1 and 4, layers 2 and 3
// Fixed input map of x = (phi, kT, dt_cg/dx, |u|, cos, sin): phi / 0.4,
// ln kT / ln 20, (ln(dt_cg/dx) + 6) / 1.5, and the drift as the vector
// 5 |u| (cos, sin) with its length 5 |u|; fp32, every operation rounded once.
__device__ __forceinline__ float encode_in(const float* __restrict__ xr, int k) {
#pragma clang fp contract(off)
    const float inv_ln20 = (float)(1.0 / 2.995732273553991);
    switch (k) {
        case 0: return xr[0] * 2.5f;
        case 1: return logf(fmaxf(xr[1], 1e-30f)) * inv_ln20;
        case 2: return (logf(fmaxf(xr[2], 1e-30f)) + 6.0f) * (float)(1.0 / 1.5);
        case 3: return (xr[3] * xr[4]) * 5.0f;
        case 4: return (xr[3] * xr[5]) * 5.0f;
        default: return xr[3] * 5.0f;
    }
}

// Logistic function and SiLU in fp32, the reciprocal from the hardware
// estimate (about one ulp); every consumer rounds the result to bf16 (8
// significant bits) first.  Training and inference share them.
__device__ __forceinline__ float sigmoid_f(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_f(float z) { return z * sigmoid_f(z); }

__device__ __forceinline__ float wave_max_f(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_sum_f(float v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// bf16 copies of the weights in the order in which the products read them: a
// product with K rows (k) and N columns (n) takes, per 16 columns and 32 rows,
// one 16-byte vector per lane, and these 1 KB fragments lie one after the other
// (k fastest), so that a wave's load is one contiguous run.  Forward products
// have k = a layer's inputs, backward ones k = its outputs; K and N are padded
// to whole fragments with zeros.  Read as 64-byte pieces of 16 rows instead,
// the training kernel below took 27 us for 2048 samples (16.7 so) and inference
// 59 us for 65,536 (41 so).
constexpr long kFrag = 512;
constexpr long kF1 = 0, kF2 = kF1 + 16 * kFrag, kF3 = kF2 + 128 * kFrag, kF4 = kF3 + 128 * kFrag,
               kR4 = kF4 + 32 * kFrag, kR3 = kR4 + 32 * kFrag, kR2 = kR3 + 128 * kFrag, kCopies = kR2 + 128 * kFrag;
__device__ __forceinline__ long frag_pos(long k, long n, long ksteps) {
    return ((n >> 4) * ksteps + (k >> 5)) * kFrag + (((k >> 3) & 3) * 16 + (n & 15)) * 8 + (k & 7);
}
// A lane's vector of fragment (16-column tile, k step) of the copy at `at`; cl: the copies at the lane's offset (8 values).
__device__ __forceinline__ bf16x8 frag(const bf16* __restrict__ cl, long at, int tile, int ks, int ksteps) {
    return *reinterpret_cast<const bf16x8*>(cl + at + ((long)tile * ksteps + ks) * kFrag);
}

__device__ __forceinline__ void store_copies(long i, float wi, bf16* __restrict__ c) {
    const bf16 v = (bf16)wi;
    if (i < kB1) {
        c[kF1 + frag_pos(i / kHid, i % kHid, 1)] = v;
    } else if (i >= kW2 && i < kB2) {
        const long k = (i - kW2) / kHid, n = (i - kW2) % kHid;
        c[kF2 + frag_pos(k, n, 8)] = v;
        c[kR2 + frag_pos(n, k, 8)] = v;
    } else if (i >= kW3 && i < kB3) {
        const long k = (i - kW3) / kHid, n = (i - kW3) % kHid;
        c[kF3 + frag_pos(k, n, 8)] = v;
        c[kR3 + frag_pos(n, k, 8)] = v;
    } else if (i >= kW4 && i < kB4) {
        const long k = (i - kW4) / kOut, n = (i - kW4) % kOut;
        c[kF4 + frag_pos(k, n, 8)] = v;
        c[kR4 + frag_pos(n, k, 2)] = v;
    }
}

__global__ void k_to_bf16(const float* __restrict__ w, long n, bf16* __restrict__ c) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) store_copies(i, w[i], c);
}

__global__ void k_zero_bf16(bf16* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = (bf16)0.0f;
}

// What a training step's launches hand over: inputs (16 rows), activations,
// their gradients (kHid rows) and logit gradients (kOutP rows) of the batch
// padded to `steps` k steps of 32 samples (zero gradients past it), in fragments
// of 16 rows by 32 samples like the weights' copies.
struct TrainBufs {
    bf16 *x, *h[3], *g[3], *g4;
    long steps;
};

// Forward and backward of kTB samples per block.
//
// One launch per product and layer, 17 of them with the reductions, took 8 to
// 13 us each for short sums (k = 256 or less) over 128 blocks: 130 us per step
// of 2048 samples.  A block here keeps its samples through all layers, forward
// and back: activations and gradients go from layer to layer through LDS,
// pre-activations stay in the accumulator registers of the wave that made them
// (the backward product of a layer gives a wave the same samples and columns),
// and the weights come from L2 straight into operand registers, a whole layer's
// share of a wave (16 vectors of 16 bytes per lane) in flight during the
// products and the epilogue of the layer before.  The bound is what a compute
// unit reads from L2, 0.6 MB of weights per block, and the chain of layers: 16.7
// us for 2048 samples (13.5 us for 32; 17.5 us in a long training run).
//
// Wave w owns columns 32 w .. 32 w + 31 (two 16 x 16 tiles) of a hidden layer.
// MFMA 16x16x32 lane layout: lane l holds A(row l%16, k 8*(l/16) .. +7),
// B(k 8*(l/16) .. +7, col l%16) and D(rows 4*(l/16) .. +3, col l%16).
constexpr int kTB = 16;            // samples per block
constexpr int kTrainBS = 512;      // 8 waves
constexpr int kTLD = kHid + 8;     // LDS row strides (bf16): 16-byte aligned, rows spread over the banks
constexpr int kTLDO = kOutP + 8;

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kTrainBS) __attribute__((amdgpu_waves_per_eu(2))) void k_train_fb(
    const float* __restrict__ x, const float* __restrict__ R, int B, const float* __restrict__ w,
    const bf16* __restrict__ wc, TrainBufs t, float* __restrict__ loss_b) {
    constexpr int KS = kHid / 32;  // k steps of a hidden layer
    __shared__ __attribute__((aligned(16))) bf16 Ha[kTB][kTLD], Hb[kTB][kTLD];
    __shared__ __attribute__((aligned(16))) bf16 X[kTB][40], G4[kTB][kTLDO];
    __shared__ float z4[kTB][kOutP + 1];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int lr = lane & 15, lq = lane >> 4, lk = lq * 8;
    const long row0 = (long)blockIdx.x * kTB;
    const bf16 zero = (bf16)0.0f;
    const bf16* __restrict__ cl = wc + lane * 8;

    bf16x8 wa[KS][2], wn[KS][2];
    auto load = [&](long at, bf16x8 (&f)[KS][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < 2; ++j) f[ks][j] = frag(cl, at, 2 * wv + j, ks, KS);
    };
    auto product = [&](bf16 (*S)[kTLD], const bf16x8 (&f)[KS][2], f32x4 (&acc)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(&S[lr][32 * ks + lk]);
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, f[ks][j], acc[j], 0, 0, 0);
        }
    };
    // a wave's tiles to LDS (for the next product) and to the transposed copy
    auto put = [&](const float (&v)[2][4], bf16 (*S)[kTLD], bf16* __restrict__ T) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = 32 * wv + 16 * j + lr;
            bf16x4 q;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                q[r] = (bf16)v[j][r];
                if (S) S[4 * lq + r][col] = q[r];
            }
            *reinterpret_cast<bf16x4*>(T + frag_pos(row0 + 4 * lq, col, t.steps)) = q;
        }
    };
    auto forward = [&](f32x4 (&acc)[2], const float* __restrict__ bias, f32x4 (&z)[2], bf16 (*S)[kTLD],
                       bf16* __restrict__ T) __attribute__((always_inline)) {
        float h[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float bj = bias[32 * wv + 16 * j + lr];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                z[j][r] = acc[j][r] + bj;
                h[j][r] = silu_f(z[j][r]);
            }
        }
        put(h, S, T);
    };
    auto backward = [&](f32x4 (&acc)[2], const f32x4 (&z)[2], bf16 (*S)[kTLD], bf16* __restrict__ T)
                        __attribute__((always_inline)) {
        float g[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float zz = z[j][r], sg = sigmoid_f(zz);
                g[j][r] = acc[j][r] * sg * (1.0f + zz * (1.0f - sg));
            }
        put(g, S, T);
    };

    load(kF2, wa);
    {
        const int r = tid >> 5, k = tid & 31;
        float v = 0.f;
        if (k < kIn && row0 + r < B) v = encode_in(x + (row0 + r) * kIn, k);
        X[r][k] = (bf16)v;
        if (k < 16) t.x[frag_pos(row0 + r, k, t.steps)] = (bf16)v;
    }
    __syncthreads();
    f32x4 acc[2], z1[2], z2[2], z3[2];
    {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&X[lr][lk]);
#pragma unroll
        for (int j = 0; j < 2; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, frag(cl, kF1, 2 * wv + j, 0, 1), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    load(kF3, wn);
    forward(acc, w + kB1, z1, Ha, t.h[0]);
    __syncthreads();
    product(Ha, wa, acc);
    // layer 4: waves 0 .. 3 take 16 of the 64 (padded) outputs each
    bf16x8 w4[KS];
    if (wv < 4) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) w4[ks] = frag(cl, kF4, wv, ks, KS);
    }
    bf16x8 wp[2][2];  // W4 for the way back
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 2; ++j) wp[ks][j] = frag(cl, kR4, 2 * wv + j, ks, 2);
    forward(acc, w + kB2, z2, Hb, t.h[1]);
    __syncthreads();
    product(Hb, wn, acc);
    load(kR3, wa);
    forward(acc, w + kB3, z3, Ha, t.h[2]);
    __syncthreads();
    if (wv < 4) {
        f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(&Ha[lr][32 * ks + lk]);
            o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w4[ks], o, 0, 0, 0);
        }
        const int col = 16 * wv + lr;
        const float bj = col < kOut ? w[kB4 + col] : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) z4[4 * lq + r][col] = o[r] + bj;
    }
    load(kR2, wn);
    __syncthreads();
    // Softmax, loss and logit gradient: a wave takes two samples, lane i < 49
    // logit i: q = softmax(z); with the target R the loss sum_i R_i (log R_i -
    // log q_i) and the gradient (q sum_i R_i - R) / B.
#pragma unroll
    for (int m = 0; m < kTB / 8; ++m) {
        const int r = kTB / 8 * wv + m;
        const long b = row0 + r;
        const bool on = b < B && lane < kOut;
        const float zi = on ? z4[r][lane] : -INFINITY;
        const float ri = on ? R[b * kOut + lane] : 0.f;
        const float mx = wave_max_f(zi);
        const float ei = on ? __expf(zi - mx) : 0.f;
        const float ls = __logf(wave_sum_f(ei));
        const float logq = zi - mx - ls;
        const float qi = on ? __expf(logq) : 0.f;
        const float rs = wave_sum_f(ri);
        const float li = wave_sum_f(on && ri > 0.f ? ri * (__logf(ri) - logq) : 0.f);
        G4[r][lane] = on ? (bf16)((qi * rs - ri) / (float)B) : zero;
        if (lane == 0 && b < B) loss_b[b] = li;
    }
    __syncthreads();
    if (tid < kOutP * 4) {
        const int n = tid >> 2, q = tid & 3;
        bf16x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = G4[4 * q + r][n];
        *reinterpret_cast<bf16x4*>(t.g4 + frag_pos(row0 + 4 * q, n, t.steps)) = v;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&G4[lr][32 * ks + lk]);
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, wp[ks][j], acc[j], 0, 0, 0);
    }
    backward(acc, z3, Hb, t.g[2]);
    __syncthreads();
    product(Hb, wa, acc);
    backward(acc, z2, Ha, t.g[1]);
    __syncthreads();
    product(Ha, wn, acc);
    backward(acc, z1, nullptr, t.g[0]);
}

// Weight and bias gradients of all layers: dW = prev^T G, db = the column sums
// of G, as products over the samples (k): both operands lie in fragments and go
// from L2 straight into operand registers.  Block (tile,
// split): 64 x 64 outputs of one layer (4 waves of 2 x 2 MFMA tiles) over one
// chunk of the samples, into the partials part[split][parameter]; the blocks of
// a layer's first row of tiles also take the column sums, as the products of a
// row of ones.  Launch latency and operand latency bound it at these sizes:
// 8.2 us for 2048 samples in 8 splits (11.8 us with 64-byte pieces of rows for
// operands); the sums and the update after it 4.9 us (7.6 and 4.8 us in a long
// training run).
constexpr int kTK = 32;            // k step, and the padding of the samples
constexpr int kWgTiles = 4 + 16 + 16 + 4;

// Splits of a training batch: k steps of a split and how many there are, for
// layers 1 and 4 and for layers 2 and 3.
struct Splits {
    int chunk, n, chunk_mid, n_mid;
};

__global__ __launch_bounds__(256) void k_train_wgrad(TrainBufs t, Splits sp, float* __restrict__ part) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int lr = lane & 15, lq = lane >> 4;
    // the tile's layer: inputs A [M rows], gradients G [N rows], output W [M][N] and bias [N]
    int tile = blockIdx.x, M = kHid, N = kHid, last = kHid / 16 - 1;
    const bool mid = tile >= 4 && tile < 36;
    if (mid && (int)blockIdx.y >= sp.n_mid) return;
    const int chunk = mid ? sp.chunk_mid : sp.chunk;
    const bf16 *A, *G;
    long ow, ob;
    if (tile < 4) {
        A = t.x, G = t.g[0], ow = kW1, ob = kB1, M = kIn, last = 0;
    } else if (tile < 20) {
        tile -= 4;
        A = t.h[0], G = t.g[1], ow = kW2, ob = kB2;
    } else if (tile < 36) {
        tile -= 20;
        A = t.h[1], G = t.g[2], ow = kW3, ob = kB3;
    } else {
        tile -= 36;
        A = t.h[2], G = t.g4, ow = kW4, ob = kB4, N = kOut;
    }
    const int tn = (N + 63) / 64;
    const int m0 = tile / tn * 64 + (wv >> 1) * 32, n0 = tile % tn * 64 + (wv & 1) * 32;
    const bool sums = m0 == 0;
    const long k0 = (long)blockIdx.y * chunk, k1 = min(k0 + chunk, t.steps);
    float* __restrict__ out = part + blockIdx.y * kParams;
    f32x4 acc[2][2], cs[2];
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = lr == 0 ? (bf16)1.0f : (bf16)0.0f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        cs[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const bf16* __restrict__ pa[2];
    const bf16* __restrict__ pb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        pa[i] = A + (min(m0 / 16 + i, last) * t.steps) * kFrag + lane * 8;  // rows past M are not stored
        pb[i] = G + ((n0 / 16 + i) * t.steps) * kFrag + lane * 8;
    }
#pragma unroll 4
    for (long k = k0; k < k1; ++k) {
        bf16x8 a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[i] = *reinterpret_cast<const bf16x8*>(pa[i] + k * kFrag);
            b[i] = *reinterpret_cast<const bf16x8*>(pb[i] + k * kFrag);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            if (sums) cs[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, b[j], cs[j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int n = n0 + 16 * j + lr;
        if (n >= N) continue;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + 16 * i + 4 * lq + r;
                if (m < M) out[ow + (long)m * N + n] = acc[i][j][r];
            }
        if (sums && lq == 0) out[ob + n] = cs[j][0];
    }
}

// The gradient of each parameter, its partials added in order, and with ADAM
// the update of the fp32 master weights and their bf16 copies; without, the
// gradient itself.  The last block adds the samples' losses up (fixed order).
template <bool ADAM>
__global__ __launch_bounds__(256) void k_train_sum(const float* __restrict__ part, Splits sp,
                                                   const float* __restrict__ loss_b, int B, float* __restrict__ loss,
                                                   float* __restrict__ grad, float* __restrict__ w, float* __restrict__ m,
                                                   float* __restrict__ v, float lr, float b1, float b2, float eps,
                                                   float bc1, float bc2, bf16* __restrict__ wc) {
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ float red[4];
        float s = 0.f;
        for (int i = threadIdx.x; i < B; i += 256) s += loss_b[i];
        s = wave_sum_f(s);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0 && loss) *loss = ((red[0] + red[1]) + (red[2] + red[3])) * (1.0f / B);
        return;
    }
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= kParams) return;
    const int splits = i >= kW2 && i < kW4 ? sp.n_mid : sp.n;  // the same for a whole block
    float gi = 0.f;
    for (int z0 = 0; z0 < splits; z0 += 8) {
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = z0 + e < splits ? part[(z0 + e) * kParams + i] : 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) gi += p[e];
    }
    if (!ADAM) {
        if (grad) grad[i] = gi;
        return;
    }
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    w[i] = wi;
    store_copies(i, wi, wc);
}

// Whole-network inference for 64 samples per block.  The activations stay
// in LDS from layer to layer; the weights come from their bf16 copies, from L2,
// straight into MFMA operand registers (loading a k step ahead by hand cost
// registers and 1.5 us; 128 samples per block gained 1 us here and cost small
// batches 4).
// Wave w computes output columns 64 w .. 64 w + 63 of a hidden layer (4 x 4
// tiles of 16 x 16, accumulators in registers), then every wave's results
// replace the layer input in LDS; the last layer (49 outputs, padded to 64)
// gives wave w the 16 rows 16 w .. 16 w + 15, whose softmax is reduced across
// the 16 lanes that hold a row.  Same roundings as the layer-wise products:
// scaled inputs, weights and hidden activations in bf16, fp32 accumulation,
// fp32 biases.
constexpr int kFB = 64;            // samples per block
constexpr int kHLD = kHid + 8;     // LDS row stride of the activations (bf16)

__device__ __forceinline__ void hidden_epilogue(const f32x4 (&acc)[4][4], const float* __restrict__ bias,
                                                bf16 (*H)[kHLD], int wv, int lane) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int col = 64 * wv + 16 * j + (lane & 15);
        const float bj = bias[col];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float z = acc[i][j][r] + bj;
                H[16 * i + 4 * (lane >> 4) + r][col] = (bf16)silu_f(z);
            }
    }
}

// At most 128 registers per lane: four waves per SIMD, so that one block's
// epilogue overlaps another's products.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_mlp_infer(const float* __restrict__ x, int B, const bf16* __restrict__ wc,
                                                   const float* __restrict__ w, float* __restrict__ g) {
    __shared__ __attribute__((aligned(16))) bf16 H[kFB][kHLD];
    __shared__ __attribute__((aligned(16))) bf16 X[kFB][40];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int row0 = blockIdx.x * kFB;
    for (int i = tid; i < kFB * 32; i += 256) {
        const int r = i >> 5, k = i & 31;
        float v = 0.f;
        if (k < kIn && row0 + r < B) v = encode_in(x + (long)(row0 + r) * kIn, k);
        X[r][k] = (bf16)v;
    }
    __syncthreads();
    const int lr = lane & 15, lk = (lane >> 4) * 8;
    const bf16* __restrict__ cl = wc + lane * 8;
    f32x4 acc[4][4];
    // layer 1: k = 6, one MFMA step over k padded to 32
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    {
        bf16x8 a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const bf16x8*>(&X[16 * i + lr][lk]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bf16x8 b = frag(cl, kF1, 4 * wv + j, 0, 1);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b, acc[i][j], 0, 0, 0);
        }
    }
    // layers 2 and 3: k = 256; the first weight fragments of a layer are loaded
    // before the previous layer's epilogue
    const long wo[2] = {kF2, kF3}, bo[2] = {kB2, kB3};
    bf16x8 b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        b[j] = frag(cl, kF2, 4 * wv + j, 0, kHid / 32);
    hidden_epilogue(acc, w + kB1, H, wv, lane);
    __syncthreads();
#pragma unroll
    for (int l = 0; l < 2; ++l) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int ks = 0; ks < kHid / 32; ++ks) {
            bf16x8 a[4];
            if (ks > 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) b[j] = frag(cl, wo[l], 4 * wv + j, ks, kHid / 32);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const bf16x8*>(&H[16 * i + lr][32 * ks + lk]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (l == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                b[j] = frag(cl, kF3, 4 * wv + j, 0, kHid / 32);
        }
        __syncthreads();  // every wave has read this layer's input
        hidden_epilogue(acc, w + bo[l], H, wv, lane);
        __syncthreads();
    }
    // layer 4: 49 outputs; wave wv takes rows 16 wv .. 16 wv + 15
    f32x4 o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int ks = 0; ks < kHid / 32; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&H[16 * wv + lr][32 * ks + lk]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bf16x8 b = frag(cl, kF4, j, ks, kHid / 32);
            o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, o[j], 0, 0, 0);
        }
    }
    // softmax of each row over the 16 lanes (x 4 tiles) that hold it
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = row0 + 16 * wv + 4 * (lane >> 4) + r;
        float z[4], mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = 16 * j + lr;
            z[j] = col < kOut ? o[j][r] + w[kB4 + col] : -INFINITY;
            mx = fmaxf(mx, z[j]);
        }
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
        float e[4], sum = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            e[j] = 16 * j + lr < kOut ? __expf(z[j] - mx) : 0.f;
            sum += e[j];
        }
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) sum += __shfl_xor(sum, d, 64);
        if (row < B) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int col = 16 * j + lr;
                if (col < kOut) g[(long)row * kOut + col] = e[j] / sum;
            }
        }
    }
}

}  // namespace
}  // namespace mdlg

using namespace mdlg;

struct mdlg_mlp {
    int max_batch = 0;
    long step = 0;
    float* w = nullptr;   // fp32 master parameters
    float* m = nullptr;   // Adam moments
    float* v = nullptr;
    bf16* wc = nullptr;   // bf16 copies of the weights [kCopies]
    bf16* hand = nullptr; // what the launches of a training step hand over (see TrainBufs)
    float* loss_b = nullptr;
    float* part = nullptr;  // partials of the gradients [kMaxSplit][kParams]
    float* x1 = nullptr;  // one-sample staging for the surrogate call
    float* g1 = nullptr;
};

namespace {

unsigned nblk(long n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

// Rows of the buffers between the launches of a training step: inputs, three
// layers of activations and gradients, logit gradients.
constexpr size_t kHandRows = 16 + 6 * kHid + kOutP;
size_t padded(size_t B) { return (B + kTK - 1) / kTK * kTK; }

TrainBufs train_bufs(const mdlg_mlp* m, int B) {
    TrainBufs t{};
    t.steps = (long)padded(B) / kTK;
    bf16* p = m->hand;
    auto take = [&](size_t rows) {
        bf16* q = p;
        p += rows * t.steps * kTK;
        return q;
    };
    t.x = take(16);
    for (int l = 0; l < 3; ++l) t.h[l] = take(kHid);
    for (int l = 0; l < 3; ++l) t.g[l] = take(kHid);
    t.g4 = take(kOutP);
    return t;
}

// Forward, backward and the gradient's partials; *sp receives their splits.
hipError_t gradient_partials(mdlg_mlp* m, const float* x, const float* R, int B, Splits* sp, hipStream_t st) {
    const TrainBufs t = train_bufs(m, B);
    hipLaunchKernelGGL(k_train_fb, dim3((unsigned)(t.steps * kTK / kTB)), dim3(kTrainBS), 0, st, x, R, B, (const float*)m->w,
                       (const bf16*)m->wc, t, m->loss_b);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // at least eight k steps in each of a power of two of splits: shorter FP32
    // chains, and enough blocks.  Up to 16 for layers 2 and 3, whose 32 tiles
    // then are two blocks per compute unit (40 tiles x 8 splits for 2048 samples:
    // 16 made the products and the sums 0.6 and 0.9 us longer), up to 32 for the
    // eight tiles of layers 1 and 4.
    auto split = [&](int most, int* n) {
        int want = 1;
        while (2 * want <= most && B >= 16 * want * kTK) want *= 2;
        const int chunk = ((int)t.steps + want - 1) / want;
        *n = ((int)t.steps + chunk - 1) / chunk;
        return chunk;
    };
    sp->chunk = split(kMaxSplit, &sp->n);
    sp->chunk_mid = split(kMidSplit, &sp->n_mid);
    hipLaunchKernelGGL(k_train_wgrad, dim3(kWgTiles, (unsigned)sp->n), dim3(256), 0, st, t, *sp, m->part);
    return hipGetLastError();
}

template <typename T>
hipError_t dalloc(T** p, size_t n) {
    return hipMalloc((void**)p, sizeof(T) * (n > 0 ? n : 1));
}

mdlg_status check_batch(const mdlg_mlp* m, int B, const char* who) {
    if (!m) return fail(MDLG_EINVAL, std::string(who) + ": NULL handle");
    if (B < 1 || B > m->max_batch)
        return fail(MDLG_EINVAL, std::string(who) + ": batch must be in [1, max_batch]");
    return MDLG_OK;
}

}  // namespace

extern "C" void mdlg_mlp_destroy(mdlg_mlp* m) {
    if (!m) return;
    void* p[] = {m->w, m->m, m->v, m->wc, m->hand, m->loss_b, m->part, m->x1, m->g1};
    for (void* q : p)
        if (q) (void)hipFree(q);
    delete m;
}

extern "C" mdlg_status mdlg_mlp_create(mdlg_mlp** out, const float* params, int32_t max_batch, void* stream) {
    if (!out || !params) return fail(MDLG_EINVAL, "mdlg_mlp_create: NULL argument");
    *out = nullptr;
    if (max_batch < 1 || max_batch > (1 << 20)) return fail(MDLG_EINVAL, "mdlg_mlp_create: max_batch in [1, 2^20]");
    for (long i = 0; i < kParams; ++i)
        if (!std::isfinite(params[i])) return fail(MDLG_EINVAL, "mdlg_mlp_create: non-finite parameter");
    hipStream_t st = (hipStream_t)stream;
    mdlg_mlp* m = new mdlg_mlp();
    m->max_batch = max_batch;
    const size_t B = max_batch;
    hipError_t ae = hipSuccess;
    auto take = [&](hipError_t r) {
        if (ae == hipSuccess) ae = r;
    };
    take(dalloc(&m->w, kParams));
    take(dalloc(&m->m, kParams));
    take(dalloc(&m->v, kParams));
    take(dalloc(&m->wc, kCopies));
    take(dalloc(&m->hand, kHandRows * padded(B)));
    take(dalloc(&m->loss_b, B));
    take(dalloc(&m->part, (size_t)kMaxSplit * kParams));
    take(dalloc(&m->x1, kIn));
    take(dalloc(&m->g1, kOut));
    if (ae != hipSuccess) {
        mdlg_mlp_destroy(m);
        return fail(MDLG_ENOMEM, std::string("mdlg_mlp_create: device allocation failed: ") + hipGetErrorString(ae));
    }
    hipError_t e = hipMemcpyAsync(m->w, params, sizeof(float) * kParams, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemsetAsync(m->m, 0, sizeof(float) * kParams, st);
    if (e == hipSuccess) e = hipMemsetAsync(m->v, 0, sizeof(float) * kParams, st);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_zero_bf16, dim3(nblk(kCopies)), dim3(256), 0, st, m->wc, (int)kCopies);
        hipLaunchKernelGGL(k_to_bf16, dim3(nblk(kParams)), dim3(256), 0, st, (const float*)m->w, kParams, m->wc);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        mdlg_mlp_destroy(m);
        return fail(MDLG_EHIP, std::string("mdlg_mlp_create: ") + hipGetErrorString(e));
    }
    *out = m;
    return MDLG_OK;
}

extern "C" mdlg_status mdlg_mlp_params(const mdlg_mlp* m, float* host_out, void* stream) {
    if (!m || !host_out) return fail(MDLG_EINVAL, "mdlg_mlp_params: NULL argument");
    MDLG_HIP(hipStreamSynchronize((hipStream_t)stream));
    MDLG_HIP(hipMemcpy(host_out, m->w, sizeof(float) * kParams, hipMemcpyDeviceToHost));
    return MDLG_OK;
}

extern "C" mdlg_status mdlg_mlp_forward(mdlg_mlp* m, const float* x, int32_t B, float* g_out, void* stream) {
    mdlg_status s = check_batch(m, B, "mdlg_mlp_forward");
    if (s != MDLG_OK) return s;
    if (!x || !g_out) return fail(MDLG_EINVAL, "mdlg_mlp_forward: NULL argument");
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_mlp_infer, dim3((unsigned)((B + kFB - 1) / kFB)), dim3(256), 0, st, x, B,
                       (const bf16*)m->wc, (const float*)m->w, g_out);
    MDLG_HIP(hipGetLastError());
    return MDLG_OK;
}

extern "C" mdlg_status mdlg_mlp_gradient(mdlg_mlp* m, const float* x, const float* target, int32_t B, float* loss,
                                         float* grad, void* stream) {
    mdlg_status s = check_batch(m, B, "mdlg_mlp_gradient");
    if (s != MDLG_OK) return s;
    if (!x || !target) return fail(MDLG_EINVAL, "mdlg_mlp_gradient: NULL argument");
    hipStream_t st = (hipStream_t)stream;
    Splits sp{};
    MDLG_HIP(gradient_partials(m, x, target, B, &sp, st));
    hipLaunchKernelGGL(k_train_sum<false>, dim3(nblk(kParams) + 1), dim3(256), 0, st, (const float*)m->part, sp,
                       (const float*)m->loss_b, B, loss, grad, m->w, m->m, m->v, 0.f, 0.f, 0.f, 0.f, 1.f, 1.f, m->wc);
    MDLG_HIP(hipGetLastError());
    return MDLG_OK;
}

extern "C" mdlg_status mdlg_mlp_train_step(mdlg_mlp* m, const float* x, const float* target, int32_t B, float lr,
                                           float* loss, void* stream) {
    mdlg_status s = check_batch(m, B, "mdlg_mlp_train_step");
    if (s != MDLG_OK) return s;
    if (!x || !target) return fail(MDLG_EINVAL, "mdlg_mlp_train_step: NULL argument");
    if (!(lr > 0.f) || !std::isfinite(lr)) return fail(MDLG_EINVAL, "mdlg_mlp_train_step: lr must be > 0");
    hipStream_t st = (hipStream_t)stream;
    Splits sp{};
    MDLG_HIP(gradient_partials(m, x, target, B, &sp, st));
    m->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float bc1 = 1.0f - std::pow(b1, (float)m->step), bc2 = 1.0f - std::pow(b2, (float)m->step);
    hipLaunchKernelGGL(k_train_sum<true>, dim3(nblk(kParams) + 1), dim3(256), 0, st, (const float*)m->part, sp,
                       (const float*)m->loss_b, B, loss, (float*)nullptr, m->w, m->m, m->v, lr, b1, b2, 1e-8f, bc1, bc2,
                       m->wc);
    MDLG_HIP(hipGetLastError());
    return MDLG_OK;
}

extern "C" mdlg_status mdlg_feq_surrogate(mdlg_mlp* m, const double* x, double a2, double lambda, double tol,
                                          double* g_out, int32_t* used_fallback, double* err, void* stream) {
    if (!m || !x || !g_out) return fail(MDLG_EINVAL, "mdlg_feq_surrogate: NULL argument");
    hipStream_t st = (hipStream_t)stream;
    float xf[kIn];
    for (int i = 0; i < kIn; ++i) xf[i] = (float)x[i];
    MDLG_HIP(hipMemcpyAsync(m->x1, xf, sizeof(xf), hipMemcpyHostToDevice, st));
    mdlg_status s = mdlg_mlp_forward(m, m->x1, 1, m->g1, stream);
    if (s != MDLG_OK) return s;
    float gf[kOut];
    MDLG_HIP(hipMemcpyAsync(gf, m->g1, sizeof(gf), hipMemcpyDeviceToHost, st));
    MDLG_HIP(hipStreamSynchronize(st));
    // the guard: the Poisson-WSG closed form at the drift (|u| cos, |u| sin)
    const double u[2] = {x[3] * x[4], x[3] * x[5]};
    double gw[MDLG_NQ];
    s = mdlg_feq_wsg(a2, lambda, u, gw);
    if (s != MDLG_OK) return s;
    double e = 0.0;
    for (int i = 0; i < kOut; ++i) e = std::fmax(e, std::fabs((double)gf[i] - gw[i]));
    const bool fallback = !(e <= tol);
    for (int i = 0; i < kOut; ++i) g_out[i] = fallback ? gw[i] : (double)gf[i];
    if (used_fallback) *used_fallback = fallback ? 1 : 0;
    if (err) *err = e;
    return MDLG_OK;
}

extern "C" mdlg_status mdlg_feq_surrogate_table(mdlg_mlp* m, const mdlg_moment_table* table, const double* x,
                                                double tol, double* g_out, int32_t* used_fallback, double* err,
                                                double* a2_out, double* lambda_out, void* stream) {
    if (!m || !table || !x || !g_out) return fail(MDLG_EINVAL, "mdlg_feq_surrogate_table: NULL argument");
    double a2 = 0.0, lambda = 0.0;
    mdlg_status s = mdlg_moment_table_eval(table, x, &a2, &lambda, nullptr);
    if (s != MDLG_OK) return s;
    if (a2_out) *a2_out = a2;
    if (lambda_out) *lambda_out = lambda;
    return mdlg_feq_surrogate(m, x, a2, lambda, tol, g_out, used_fallback, err, stream);
}
