// Surrogate network for D(t)/D_b: 6 -> 256 -> 256 -> 256 -> 1, SiLU, trained
// and evaluated on the GPU with BF16 MFMA (32x32x16, FP32 accumulation),
// FP32 master weights and Adam.
//
// The input and output layers are padded to 32 columns and rows with zero
// weights, so that one MFMA shape serves every layer:
//   forward   Z_l = A_{l-1} W_l^T + b_l,  A_l = silu(Z_l)
//   backward  dA_{l-1} = dZ_l W_l,  dZ_{l-1} = dA_{l-1} * silu'(Z_{l-1})
//             dW_l = dZ_l^T A_{l-1}
// A training step is three launches: k_train_rows takes a block of rows
// through the forward and the backward pass, k_train_grads forms the
// parameter gradients over splits of the batch, k_train_update adds the
// splits and applies Adam. Every product accumulates in increasing K.
#include <cmath>
#include <vector>

#include "lbmp_internal.hpp"

namespace lbmp {
namespace mlp {

using bf16x8 = __bf16 __attribute__((ext_vector_type(8)));
using bf16x4 = __bf16 __attribute__((ext_vector_type(4)));
using f32x16 = float __attribute__((ext_vector_type(16)));

constexpr int NLAYER = 4;
constexpr int WIDTH = 256;
constexpr int PAD_IN = 32;   // 6 features padded
constexpr int PAD_OUT = 32;  // 1 output padded
constexpr int NFEAT = 6;

__host__ __device__ constexpr int lin(int l) { return l == 0 ? PAD_IN : WIDTH; }
__host__ __device__ constexpr int lout(int l) { return l == NLAYER - 1 ? PAD_OUT : WIDTH; }
__host__ __device__ constexpr int tin(int l) { return l == 0 ? NFEAT : WIDTH; }   // true fan-in
__host__ __device__ constexpr int tout(int l) { return l == NLAYER - 1 ? 1 : WIDTH; }

// Parameters packed layer by layer: W_l [out][in], then b_l.
__host__ __device__ constexpr int woff(int l) {
    int k = 0;
    for (int i = 0; i < l; ++i) k += tout(i) * tin(i) + tout(i);
    return k;
}
__host__ __device__ constexpr int boff(int l) { return woff(l) + tout(l) * tin(l); }
constexpr int NPAR = woff(NLAYER);
static_assert(boff(0) % 4 == 0 && boff(1) % 4 == 0 && boff(2) % 4 == 0, "hidden biases are read four at a time");

// The logistic function through the hardware reciprocal (v_rcp_f32, 1 ulp):
// an IEEE division would cost ten instructions per value, and the epilogues
// are rounded to bf16 anyway.
__device__ __forceinline__ float sigm(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }
__device__ __forceinline__ float silu_grad(float z) {
    const float s = sigm(z);
    return s * (1.0f + z * (1.0f - s));
}

// Fused inference: one block (8 waves) per FS samples runs all four layers
// with the activations in LDS (one buffer: a layer's products read it, and
// after a barrier its epilogue overwrites it) and the weights read as MFMA
// operands straight from global memory, where all blocks share them in L2;
// each weight fragment a wave loads serves the block's 128 samples. The
// arithmetic is that of the training pass (bf16 operands, fp32 accumulation in
// increasing K, bias and SiLU in fp32, activations rounded to bf16).
constexpr int FS = 128;              // samples per block
constexpr int FWAVES = 8;            // waves per block
constexpr int APITCH = WIDTH + 8;    // bf16 per activation row (padded against bank conflicts)

__global__ void __launch_bounds__(64 * FWAVES) __attribute__((amdgpu_waves_per_eu(4)))
k_mlp_forward(const float* __restrict__ x, int64_t n, const float* __restrict__ norm,
              const __bf16* __restrict__ W0, const float* __restrict__ b0, const __bf16* __restrict__ W1,
              const float* __restrict__ b1, const __bf16* __restrict__ W2, const float* __restrict__ b2,
              const __bf16* __restrict__ W3, const float* __restrict__ b3, float* __restrict__ y) {
    __shared__ __align__(16) __bf16 act[FS * APITCH];
    const int64_t s0 = (int64_t)blockIdx.x * FS;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int r = lane & 31, kh = (lane >> 5) * 8;
    // normalised features, zero padded to PAD_IN columns
    for (int i = t; i < FS * PAD_IN; i += 64 * FWAVES) {
        const int row = i / PAD_IN, c = i % PAD_IN;
        const int64_t si = s0 + row;
        float v = 0.0f;
        if (c < NFEAT && si < n) v = (x[si * NFEAT + c] - norm[c]) / norm[6 + c];
        act[row * APITCH + c] = (__bf16)v;
    }
    __syncthreads();
    // hidden layer: wave w computes output features 32 w .. 32 w + 31 of all
    // FS samples as the transposed product (weights as the MFMA's first
    // operand), so each lane holds runs of 4 consecutive features of one
    // sample and writes them to LDS as one 8-byte store
    constexpr int ST = FS / 32;  // sample tiles
    auto hidden = [&](const __bf16* __restrict__ W, const float* __restrict__ bias, int K) {
        const int n0 = 32 * wave;
        f32x16 acc[ST] = {};
#pragma unroll 2
        for (int k0 = 0; k0 < K; k0 += 16) {
            const bf16x8 w = *reinterpret_cast<const bf16x8*>(W + (size_t)(n0 + r) * K + k0 + kh);
            bf16x8 a[ST];
#pragma unroll
            for (int j = 0; j < ST; ++j) a[j] = *reinterpret_cast<const bf16x8*>(act + (32 * j + r) * APITCH + k0 + kh);
#pragma unroll
            for (int j = 0; j < ST; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, a[j], acc[j], 0, 0, 0);
        }
        __syncthreads();  // every wave has read the layer's input
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int nf = n0 + 8 * g + 4 * (lane >> 5);  // features nf .. nf + 3
            const float4 bc = *reinterpret_cast<const float4*>(bias + nf);
#pragma unroll
            for (int j = 0; j < ST; ++j) {
                bf16x4 o;
                o[0] = (__bf16)silu(acc[j][4 * g + 0] + bc.x);
                o[1] = (__bf16)silu(acc[j][4 * g + 1] + bc.y);
                o[2] = (__bf16)silu(acc[j][4 * g + 2] + bc.z);
                o[3] = (__bf16)silu(acc[j][4 * g + 3] + bc.w);
                *reinterpret_cast<bf16x4*>(act + (32 * j + r) * APITCH + nf) = o;
            }
        }
    };
    hidden(W0, b0, PAD_IN);
    __syncthreads();
    hidden(W1, b1, WIDTH);
    __syncthreads();
    hidden(W2, b2, WIDTH);
    __syncthreads();
    // output layer (PAD_OUT features, feature 0 is the network's output), also
    // transposed: waves 0 .. ST - 1 take samples 32 w .. 32 w + 31; feature 0
    // of sample 32 w + r sits in element 0 of lane r
    if (wave < ST) {
        f32x16 acc = {};
#pragma unroll 4
        for (int k0 = 0; k0 < WIDTH; k0 += 16) {
            const bf16x8 w = *reinterpret_cast<const bf16x8*>(W3 + (size_t)r * WIDTH + k0 + kh);
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(act + (32 * wave + r) * APITCH + k0 + kh);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, a, acc, 0, 0, 0);
        }
        const int64_t si = s0 + 32 * wave + r;
        if (lane < 32 && si < n) y[si] = norm[12] + norm[13] * (acc[0] + b3[0]);
    }
}

// ------------------------------------------------------------------ training
constexpr int GSPLIT_MAX = 32;
// a split's weight-gradient partials: W_1 [256][32], W_2, W_3 [256][256], W_4 [256]; bias partials
constexpr int GP1 = WIDTH * PAD_IN, GP2 = GP1 + WIDTH * WIDTH, GP3 = GP2 + WIDTH * WIDTH, GP = GP3 + WIDTH;
constexpr int GPB = 3 * WIDTH + 1;

struct TrainBufs {
    const float* norm;                    // [6] mean, [6] std, y_mean, y_std
    const float* P;                       // packed parameters
    const __bf16 *W0, *W1, *W2, *W3;      // [out][in], padded
    const __bf16 *WT1, *WT2;              // [in][out]
    // batch-major rows [feature][B]: inputs, activations, gradients by pre-activation
    __bf16 *xT, *AT[3], *dZT[3], *dYT;
    float* sq;                            // [B] squared errors
};

// Forward and backward pass of 32 ST rows (x[idx], y[idx]; idx null: in order)
// in one block of 8 waves: wave w owns features 32 w .. 32 w + 31 of every
// layer, as the transposed product (weights first), so its pre-activations
// stay in the accumulators' registers from the forward to the backward pass.
// Activations and gradients pass between the waves through LDS and leave,
// batch-major, as the operands of the weight gradients. The weight fragments
// of a layer are loaded while the layer before computes. Bound by the chain
// of six 256-wide layers (an MFMA chain, an epilogue and a barrier each);
// as 12 launches (gather, GEMMs, loss) it took 75 us at batch 1,024.
template <int ST>
__global__ void __launch_bounds__(512) k_train_rows(const float* __restrict__ x, const float* __restrict__ y,
                                                    const int32_t* __restrict__ idx, int B, TrainBufs T) {
    constexpr int RB = 32 * ST, KS = WIDTH / 16;
    __shared__ __align__(16) __bf16 act[2][RB * APITCH];
    __shared__ __align__(16) __bf16 w3[WIDTH];
    __shared__ float ty[RB], dy[RB];
    const int r0 = blockIdx.x * RB;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 31, hi = lane >> 5, kh = hi * 8, n0 = 32 * wave;
    auto load_w = [&](const __bf16* __restrict__ W, bf16x8 (&w)[KS]) {
#pragma unroll
        for (int k = 0; k < KS; ++k) w[k] = *reinterpret_cast<const bf16x8*>(W + (n0 + r) * WIDTH + 16 * k + kh);
    };
    bf16x8 wa[KS], wb[KS], w0[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) w0[k] = *reinterpret_cast<const bf16x8*>(T.W0 + (n0 + r) * PAD_IN + 16 * k + kh);
    load_w(T.W1, wa);
    for (int i = t; i < RB * PAD_IN; i += 512) {
        const int row = i / PAD_IN, c = i % PAD_IN;
        __bf16 v = (__bf16)0.0f;
        if (c < NFEAT) {
            const int64_t s = idx ? idx[r0 + row] : r0 + row;
            v = (__bf16)((x[s * NFEAT + c] - T.norm[c]) / T.norm[6 + c]);
            T.xT[(size_t)c * B + r0 + row] = v;
        }
        act[0][row * APITCH + c] = v;
    }
    if (t < RB) {
        const int64_t s = idx ? idx[r0 + t] : r0 + t;
        ty[t] = (y[s] - T.norm[12]) / T.norm[13];
    }
    if (t < WIDTH) w3[t] = T.W3[t];
    __syncthreads();
    float Z[3][ST][16];
    f32x16 acc[ST];
    auto product = [&](const bf16x8* w, int ks, const __bf16* in) {
#pragma unroll
        for (int j = 0; j < ST; ++j) acc[j] = f32x16{};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            if (k >= ks) break;
            if (k % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // at most 4 steps' operands in flight: registers
#pragma unroll
            for (int j = 0; j < ST; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    w[k], *reinterpret_cast<const bf16x8*>(in + (32 * j + r) * APITCH + 16 * k + kh), acc[j], 0, 0, 0);
        }
    };
    // element v of a lane's tile: feature n0 + 8 (v / 4) + 4 hi + v % 4, row 32 j + r
    auto put = [&](int j, int g, const bf16x4& o, __bf16* lds, __bf16* __restrict__ out) {
        const int fw = 8 * g + 4 * hi;  // feature within the wave's 32
        *reinterpret_cast<bf16x4*>(lds + (32 * j + r) * APITCH + n0 + fw) = o;
        // a scalar base per wave and 32-bit byte offsets from it (B up to 2^26)
        char* const base = reinterpret_cast<char*>(out + (size_t)n0 * B + r0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            *reinterpret_cast<__bf16*>(base + 2u * ((uint32_t)(fw + e) * (uint32_t)B + (uint32_t)(32 * j + r))) = o[e];
    };
    auto hidden = [&](auto lc, __bf16* lds) {
        constexpr int l = decltype(lc)::value;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            __builtin_amdgcn_sched_barrier(0);
            const float4 bc = *reinterpret_cast<const float4*>(T.P + boff(l) + n0 + 8 * g + 4 * hi);
            const float b4[4] = {bc.x, bc.y, bc.z, bc.w};
#pragma unroll
            for (int j = 0; j < ST; ++j) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float z = acc[j][4 * g + e] + b4[e];
                    Z[l][j][4 * g + e] = z;
                    o[e] = (__bf16)silu(z);
                }
                put(j, g, o, lds, T.AT[l]);
            }
        }
    };
    auto dhidden = [&](auto lc, __bf16* lds) {
        constexpr int l = decltype(lc)::value;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < ST; ++j) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // the output layer's gradient has one nonzero column
                    const float c = l == 2 ? dy[32 * j + r] * (float)w3[n0 + 8 * g + 4 * hi + e] : acc[j][4 * g + e];
                    float z = Z[l][j][4 * g + e];
                    asm volatile("" : "+v"(z));  // its logistic is formed again, not kept since the forward pass
                    o[e] = (__bf16)(c * silu_grad(z));
                }
                put(j, g, o, lds, T.dZT[l]);
            }
        }
    };
    // the next layer's fragments: into the other set while this layer's
    // epilogue runs, or (ST = 2, whose pre-activations leave registers for one
    // set) into the same one after it
    auto ahead = [&](const __bf16* __restrict__ W, bf16x8 (&w)[KS]) { if constexpr (ST == 1) load_w(W, w); };
    auto after = [&](const __bf16* __restrict__ W) { if constexpr (ST > 1) load_w(W, wa); };
    bf16x8(&wc)[KS] = ST == 1 ? wb : wa;
    product(w0, 2, act[0]);
    ahead(T.W2, wb);
    hidden(std::integral_constant<int, 0>(), act[1]);
    __syncthreads();
    product(wa, KS, act[1]);
    hidden(std::integral_constant<int, 1>(), act[0]);
    after(T.W2);
    __syncthreads();
    product(wc, KS, act[0]);
    hidden(std::integral_constant<int, 2>(), act[1]);
    __syncthreads();
    load_w(T.WT2, wa);
    // output layer and loss: wave w the rows 32 w .. 32 w + 31, feature 0 in element 0 of lanes 0 .. 31
    if (wave < ST) {
        f32x16 o = {};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            if (k % 4 == 0) __builtin_amdgcn_sched_barrier(0);
            bf16x8 w{};
            if (r == 0) w = *reinterpret_cast<const bf16x8*>(w3 + 16 * k + kh);
            o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                w, *reinterpret_cast<const bf16x8*>(act[1] + (32 * wave + r) * APITCH + 16 * k + kh), o, 0, 0, 0);
        }
        if (lane < 32) {
            const int b = 32 * wave + r;
            const float e = (o[0] + T.P[boff(3)]) - ty[b];
            const __bf16 d = (__bf16)(2.0f * e / (float)B);
            dy[b] = (float)d;
            T.dYT[r0 + b] = d;
            T.sq[r0 + b] = e * e;
        }
    }
    __syncthreads();
    ahead(T.WT1, wb);
    dhidden(std::integral_constant<int, 2>(), act[0]);
    __syncthreads();
    product(wa, KS, act[0]);
    dhidden(std::integral_constant<int, 1>(), act[1]);
    after(T.WT1);
    __syncthreads();
    product(wc, KS, act[1]);
    dhidden(std::integral_constant<int, 0>(), act[0]);
}

// Parameter gradients over batch splits of kc rows. Wave job (split, tile):
// one 32 x 32 tile of dW_l = dZ_l^T A_{l-1} over the split's rows, its partial
// in P[split]; both operands are batch-major, so a lane's 8 rows are one
// 16-byte load. The blocks behind them sum dZ for the biases, one thread per
// (split, output): eight interleaved partial sums, then their sum in order.
// Splitting K keeps the whole GPU busy where a 256 x 256 gradient has only 64
// tiles; the partials are added in split order, so the result does not depend
// on scheduling.
constexpr int GTILES = 2 * (WIDTH / 32) * (WIDTH / 32) + 2 * (WIDTH / 32);

__global__ void __launch_bounds__(256) k_train_grads(TrainBufs T, int B, int kc, int splits, float* __restrict__ P,
                                                     float* __restrict__ Pb) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wblocks = GTILES / 4 * splits;
    static_assert(GTILES % 4 == 0, "four wave jobs per block");
    if ((int)blockIdx.x < wblocks) {
        constexpr int TN = WIDTH / 32;
        const int job = blockIdx.x * 4 + wv, split = job / GTILES;
        int t = job % GTILES;
        const __bf16 *dz, *a;
        int m0, n0, po, ld, na = WIDTH, nb = WIDTH;  // valid rows of the operands
        if (t < 2 * TN * TN) {
            const int l = t < TN * TN ? 1 : 2;
            t -= (l - 1) * TN * TN;
            dz = T.dZT[l];
            a = T.AT[l - 1];
            m0 = t / TN * 32;
            n0 = t % TN * 32;
            po = l == 1 ? GP1 : GP2;
            ld = WIDTH;
        } else if ((t -= 2 * TN * TN) < TN) {
            dz = T.dZT[0];
            a = T.xT;
            m0 = 32 * t;
            n0 = 0;
            po = 0;
            ld = PAD_IN;
            nb = NFEAT;
        } else {
            dz = T.dYT;
            a = T.AT[2];
            m0 = 0;
            n0 = 32 * (t - TN);
            po = GP3;
            ld = WIDTH;
            na = 1;
        }
        const int r = lane & 31, kh = (lane >> 5) * 8;
        const bool va = m0 + r < na, vb = n0 + r < nb;
        const __bf16* pa = dz + (size_t)(va ? m0 + r : 0) * B + split * kc + kh;
        const __bf16* pb = a + (size_t)(vb ? n0 + r : 0) * B + split * kc + kh;
        f32x16 acc = {};
#pragma unroll 8
        for (int k0 = 0; k0 < kc; k0 += 16) {
            bf16x8 fa = *reinterpret_cast<const bf16x8*>(pa + k0), fb = *reinterpret_cast<const bf16x8*>(pb + k0);
            if (!va) fa = bf16x8{};
            if (!vb) fb = bf16x8{};
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc, 0, 0, 0);
        }
        float* const out = P + (size_t)split * GP + po;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = m0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            if (row < na) out[row * ld + n0 + r] = acc[v];
        }
        return;
    }
    const int id = ((int)blockIdx.x - wblocks) * 256 + (int)threadIdx.x;
    if (id >= GPB * splits) return;
    const int split = id / GPB, o = id % GPB;
    const __bf16* p = (o < 3 * WIDTH ? T.dZT[o / WIDTH] + (size_t)(o % WIDTH) * B : T.dYT) + split * kc;
    float s[8] = {};
#pragma unroll 4
    for (int b = 0; b < kc; b += 8) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(p + b);
#pragma unroll
        for (int g = 0; g < 8; ++g) s[g] += (float)v[g];
    }
    float a = 0.0f;
#pragma unroll
    for (int g = 0; g < 8; ++g) a += s[g];
    Pb[split * GPB + o] = a;
}

// Layer, row and column (-1: bias) of packed parameter i.
__device__ __forceinline__ void locate(int i, int& l, int& o, int& c) {
    l = i < woff(1) ? 0 : i < woff(2) ? 1 : i < woff(3) ? 2 : 3;
    const int k = i - (l == 0 ? 0 : l == 1 ? woff(1) : l == 2 ? woff(2) : woff(3));
    const int in = l == 0 ? NFEAT : WIDTH, nw = (l == 3 ? 1 : WIDTH) * in;
    o = k < nw ? k / in : k - nw;
    c = k < nw ? k % in : -1;
}

struct Copies {  // bf16 copies of the weights
    __bf16 *W[NLAYER], *WT[NLAYER];  // WT of the two square layers
};
__device__ __forceinline__ void copy_bf16(const Copies& K, int l, int o, int c, float w) {
    if (c < 0) return;
    K.W[l][o * (l == 0 ? PAD_IN : WIDTH) + c] = (__bf16)w;
    if (l == 1 || l == 2) K.WT[l][c * WIDTH + o] = (__bf16)w;
}
__global__ void k_copies(const float* __restrict__ P, Copies K) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NPAR) return;
    int l, o, c;
    locate(i, l, o, c);
    copy_bf16(K, l, o, c, P[i]);
}

// The gradient of a parameter from its partials in split order, then Adam on
// the fp32 master copy and the bf16 copies; or (G not null) the gradient alone.
__global__ void __launch_bounds__(256) k_train_update(const float* __restrict__ Pw, const float* __restrict__ Pb,
                                                      int splits, float* __restrict__ W, float* __restrict__ m,
                                                      float* __restrict__ v, float lr, float c1, float c2, float b1,
                                                      float b2, float eps, Copies K, float* __restrict__ G) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NPAR) return;
    int l, o, c;
    locate(i, l, o, c);
    const float* p;
    int stride;
    if (c < 0) {
        p = Pb + (l < 3 ? l * WIDTH + o : 3 * WIDTH);
        stride = GPB;
    } else {
        p = Pw + (l == 0 ? o * PAD_IN + c : l == 1 ? GP1 + o * WIDTH + c : l == 2 ? GP2 + o * WIDTH + c : GP3 + c);
        stride = GP;
    }
    float gi = 0.0f;
#pragma unroll 4
    for (int sp = 0; sp < splits; ++sp) gi += p[(size_t)sp * stride];
    if (G) {
        G[i] = gi;
        return;
    }
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    float w = W[i];
    w -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    W[i] = w;
    copy_bf16(K, l, o, c, w);
}

__global__ void k_sum(const float* __restrict__ v, int n, float* __restrict__ out) {
    __shared__ float s[256];
    float a = 0.0f;
    for (int i = threadIdx.x; i < n; i += 256) a += v[i];
    s[threadIdx.x] = a;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) s[threadIdx.x] += s[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = s[0] / (float)n;
}

}  // namespace mlp
}  // namespace lbmp

// ------------------------------------------------------------------ host side
namespace lbmp {
namespace mlp {
constexpr uint32_t SG_MAGIC = 0x4c425347u;  // "LBSG"
}  // namespace mlp
}  // namespace lbmp

struct lbmp_sg {
    uint32_t magic;
    int bmax;
    int64_t step;
    hipStream_t stream;
    float *P, *m, *v, *G;       // packed parameters, Adam moments, gradients (sg_gradients)
    float* norm;                // [6] mean, [6] std, y_mean, y_std
    lbmp::mlp::Copies K;        // bf16 weights
    __bf16 *xT, *AT[3], *dZT[3], *dYT;  // a batch's rows, batch-major
    float* sq;                  // per-row squared errors [bmax]
    float* loss;                // [1]
    float* gsplit;              // [GSPLIT_MAX][GP] weight-gradient partials over batch splits
    float* bsplit;              // [GSPLIT_MAX][GPB] bias-gradient partials
};

namespace lbmp {
namespace mlp {

static void carve_sg(lbmp_sg* h, Carver& c) {
    h->P = c.take<float>(NPAR);
    h->m = c.take<float>(NPAR);
    h->v = c.take<float>(NPAR);
    h->G = c.take<float>(NPAR);
    for (int l = 0; l < NLAYER; ++l) {
        h->K.W[l] = c.take<__bf16>((size_t)lout(l) * lin(l));
        h->K.WT[l] = l == 1 || l == 2 ? c.take<__bf16>((size_t)lout(l) * lin(l)) : nullptr;
    }
    h->norm = c.take<float>(16);
    const size_t B = (size_t)h->bmax;
    h->xT = c.take<__bf16>(B * NFEAT);
    for (int l = 0; l < 3; ++l) {
        h->AT[l] = c.take<__bf16>(B * WIDTH);
        h->dZT[l] = c.take<__bf16>(B * WIDTH);
    }
    h->dYT = c.take<__bf16>(B);
    h->sq = c.take<float>(B);
    h->loss = c.take<float>(4);
    h->gsplit = c.take<float>((size_t)GSPLIT_MAX * GP);
    h->bsplit = c.take<float>((size_t)GSPLIT_MAX * GPB);
}

constexpr float ADAM_B1 = 0.9f, ADAM_B2 = 0.999f, ADAM_EPS = 1e-8f;

// Batch splits of the parameter gradients: of 256 rows at least (B a multiple
// of 32: fewer, longer splits when B / 256 is small).
static int grad_splits(int B) {
    int splits = 1;
    while (splits * 2 <= GSPLIT_MAX && B % (splits * 2 * 16) == 0 && B / (splits * 2) >= 256) splits *= 2;
    return splits;
}

// Partial gradients of a batch: 32 rows per block while the blocks leave CUs
// free, 64 (which halve the weight fragments read per row) from 512 blocks on.
static void gradients(lbmp_sg* h, const float* x, const float* y, const int32_t* idx, int B) {
    hipStream_t s = h->stream;
    const TrainBufs T{h->norm, h->P, h->K.W[0], h->K.W[1], h->K.W[2], h->K.W[3], h->K.WT[1], h->K.WT[2], h->xT,
                      {h->AT[0], h->AT[1], h->AT[2]}, {h->dZT[0], h->dZT[1], h->dZT[2]}, h->dYT, h->sq};
    if (B % 64 == 0 && B >= 512 * 32) k_train_rows<2><<<(unsigned)(B / 64), 512, 0, s>>>(x, y, idx, B, T);
    else k_train_rows<1><<<(unsigned)(B / 32), 512, 0, s>>>(x, y, idx, B, T);
    const int splits = grad_splits(B);
    const unsigned nb = (unsigned)(GTILES / 4 * splits + (GPB * splits + 255) / 256);
    k_train_grads<<<nb, 256, 0, s>>>(T, B, B / splits, splits, h->gsplit, h->bsplit);
}

static lbmp_status check(const lbmp_sg* h) {
    if (!h || h->magic != SG_MAGIC) return fail(LBMP_ESTATE, "invalid surrogate handle");
    return LBMP_OK;
}

// splitmix64: the published 64-bit mixing generator (Steele, Lea, Flood 2014)
static uint64_t splitmix(uint64_t& x) {
    uint64_t z = (x += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

}  // namespace mlp
}  // namespace lbmp

using namespace lbmp;
using namespace lbmp::mlp;

extern "C" lbmp_status sg_param_count(int64_t* n) {
    if (!n) return fail(LBMP_EINVAL, "n is NULL");
    *n = NPAR;
    return LBMP_OK;
}

extern "C" lbmp_status sg_workspace_bytes(int batch_max, size_t* bytes) {
    if (batch_max < 32 || batch_max % 32 != 0) return fail(LBMP_EINVAL, "batch_max must be a positive multiple of 32");
    if (!bytes) return fail(LBMP_EINVAL, "bytes is NULL");
    lbmp_sg tmp{};
    tmp.bmax = batch_max;
    Carver c(nullptr, ~size_t(0));
    carve_sg(&tmp, c);
    *bytes = c.off;
    return LBMP_OK;
}

extern "C" lbmp_status sg_set_params(lbmp_sg* h, const float* p);

extern "C" lbmp_status sg_create(int batch_max, uint64_t seed, void* dev_ws, size_t ws_bytes, void* hip_stream,
                                 lbmp_sg** out) {
    if (!out) return fail(LBMP_EINVAL, "out is NULL");
    *out = nullptr;
    size_t need = 0;
    lbmp_status st = sg_workspace_bytes(batch_max, &need);
    if (st != LBMP_OK) return st;
    if (!dev_ws || ws_bytes < need) return fail(LBMP_ENOMEM, "workspace %zu bytes, need %zu", ws_bytes, need);
    auto* h = new lbmp_sg();
    h->magic = SG_MAGIC;
    h->bmax = batch_max;
    h->step = 0;
    h->stream = static_cast<hipStream_t>(hip_stream);
    Carver c(dev_ws, ws_bytes);
    carve_sg(h, c);
    hipStream_t s = h->stream;
    // zero everything once (padding rows/columns stay zero for good)
    if (hipMemsetAsync(dev_ws, 0, c.off, s) != hipSuccess) {
        delete h;
        return fail(LBMP_EDEVICE, "memset failed");
    }
    // default initialisation: U(-1/sqrt(fan_in), 1/sqrt(fan_in)) from splitmix64(seed)
    std::vector<float> p((size_t)NPAR);
    uint64_t x = seed;
    size_t k = 0;
    for (int l = 0; l < NLAYER; ++l) {
        const double bound = 1.0 / std::sqrt((double)tin(l));
        const int n = tout(l) * tin(l) + tout(l);
        for (int i = 0; i < n; ++i) {
            const double u = (double)(splitmix(x) >> 11) * (1.0 / 9007199254740992.0);
            p[k++] = (float)((2.0 * u - 1.0) * bound);
        }
    }
    const float norm[16] = {0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 0, 1, 0, 0};
    if (hipMemcpyAsync(h->norm, norm, sizeof norm, hipMemcpyHostToDevice, s) != hipSuccess) {
        delete h;
        return fail(LBMP_EDEVICE, "copy failed");
    }
    st = sg_set_params(h, p.data());
    if (st != LBMP_OK) {
        delete h;
        return st;
    }
    *out = h;
    return LBMP_OK;
}

// Parameters packed as the FP64 reference orders them: W_1 [256][6], b_1,
// W_2 [256][256], b_2, W_3, b_3, W_4 [1][256], b_4 (fp32).
extern "C" lbmp_status sg_set_params(lbmp_sg* h, const float* p) {
    lbmp_status st = check(h);
    if (st != LBMP_OK) return st;
    if (!p) return fail(LBMP_EINVAL, "params is NULL");
    hipStream_t s = h->stream;
    LBMP_HIP(hipMemcpyAsync(h->P, p, NPAR * 4, hipMemcpyHostToDevice, s));
    LBMP_HIP(hipMemsetAsync(h->m, 0, NPAR * 4, s));
    LBMP_HIP(hipMemsetAsync(h->v, 0, NPAR * 4, s));
    k_copies<<<(NPAR + 255) / 256, 256, 0, s>>>(h->P, h->K);
    LBMP_HIP(hipGetLastError());
    LBMP_HIP(hipStreamSynchronize(s));
    h->step = 0;
    return LBMP_OK;
}

extern "C" lbmp_status sg_get_params(lbmp_sg* h, float* p) {
    lbmp_status st = check(h);
    if (st != LBMP_OK) return st;
    if (!p) return fail(LBMP_EINVAL, "params is NULL");
    LBMP_HIP(hipMemcpyAsync(p, h->P, NPAR * 4, hipMemcpyDeviceToHost, h->stream));
    LBMP_HIP(hipStreamSynchronize(h->stream));
    return LBMP_OK;
}

extern "C" lbmp_status sg_set_normalization(lbmp_sg* h, const float* x_mean, const float* x_std, float y_mean,
                                            float y_std) {
    lbmp_status st = check(h);
    if (st != LBMP_OK) return st;
    if (!x_mean || !x_std) return fail(LBMP_EINVAL, "normalisation arrays are NULL");
    float v[16] = {0};
    for (int c = 0; c < NFEAT; ++c) {
        if (!(x_std[c] > 0.0f)) return fail(LBMP_EINVAL, "x_std[%d] must be > 0", c);
        v[c] = x_mean[c];
        v[6 + c] = x_std[c];
    }
    if (!(y_std > 0.0f)) return fail(LBMP_EINVAL, "y_std must be > 0");
    v[12] = y_mean;
    v[13] = y_std;
    LBMP_HIP(hipMemcpyAsync(h->norm, v, sizeof v, hipMemcpyHostToDevice, h->stream));
    LBMP_HIP(hipStreamSynchronize(h->stream));
    return LBMP_OK;
}

extern "C" lbmp_status sg_train_step(lbmp_sg* h, const float* x_dev, const float* y_dev, const int32_t* idx_dev,
                                     int B, float lr, float* loss_host) {
    lbmp_status st = check(h);
    if (st != LBMP_OK) return st;
    if (B < 32 || B > h->bmax || B % 32 != 0) return fail(LBMP_EINVAL, "batch must be a multiple of 32 <= batch_max");
    if (!x_dev || !y_dev) return fail(LBMP_EINVAL, "data pointers are NULL");
    hipStream_t s = h->stream;
    gradients(h, x_dev, y_dev, idx_dev, B);
    h->step += 1;
    const float c1 = 1.0f - powf(ADAM_B1, (float)h->step), c2 = 1.0f - powf(ADAM_B2, (float)h->step);
    k_train_update<<<(NPAR + 255) / 256, 256, 0, s>>>(h->gsplit, h->bsplit, grad_splits(B), h->P, h->m, h->v, lr, c1,
                                                     c2, ADAM_B1, ADAM_B2, ADAM_EPS, h->K, nullptr);
    LBMP_HIP(hipGetLastError());
    if (loss_host) {
        k_sum<<<1, 256, 0, s>>>(h->sq, B, h->loss);
        LBMP_HIP(hipMemcpyAsync(loss_host, h->loss, 4, hipMemcpyDeviceToHost, s));
        LBMP_HIP(hipStreamSynchronize(s));
    }
    return LBMP_OK;
}

extern "C" lbmp_status sg_gradients(lbmp_sg* h, const float* x_dev, const float* y_dev, int B, float* grads_host,
                                    float* loss_host) {
    lbmp_status st = check(h);
    if (st != LBMP_OK) return st;
    if (B < 32 || B > h->bmax || B % 32 != 0) return fail(LBMP_EINVAL, "batch must be a multiple of 32 <= batch_max");
    hipStream_t s = h->stream;
    gradients(h, x_dev, y_dev, nullptr, B);
    k_train_update<<<(NPAR + 255) / 256, 256, 0, s>>>(h->gsplit, h->bsplit, grad_splits(B), h->P, h->m, h->v, 0.0f,
                                                     1.0f, 1.0f, ADAM_B1, ADAM_B2, ADAM_EPS, h->K, h->G);
    k_sum<<<1, 256, 0, s>>>(h->sq, B, h->loss);
    LBMP_HIP(hipGetLastError());
    if (grads_host) LBMP_HIP(hipMemcpyAsync(grads_host, h->G, NPAR * 4, hipMemcpyDeviceToHost, s));
    if (loss_host) LBMP_HIP(hipMemcpyAsync(loss_host, h->loss, 4, hipMemcpyDeviceToHost, s));
    LBMP_HIP(hipStreamSynchronize(s));
    return LBMP_OK;
}

extern "C" lbmp_status sg_predict(lbmp_sg* h, const float* x_dev, int64_t n, float* y_dev) {
    lbmp_status st = check(h);
    if (st != LBMP_OK) return st;
    if (n < 0 || (n > 0 && (!x_dev || !y_dev))) return fail(LBMP_EINVAL, "bad arguments");
    hipStream_t s = h->stream;
    if (n > 0) {
        k_mlp_forward<<<(unsigned)((n + FS - 1) / FS), 64 * FWAVES, 0, s>>>(
            x_dev, n, h->norm, h->K.W[0], h->P + boff(0), h->K.W[1], h->P + boff(1), h->K.W[2], h->P + boff(2),
            h->K.W[3], h->P + boff(3), y_dev);
    }
    LBMP_HIP(hipGetLastError());
    return LBMP_OK;
}

extern "C" lbmp_status sg_sync(lbmp_sg* h) {
    lbmp_status st = check(h);
    if (st != LBMP_OK) return st;
    LBMP_HIP(hipStreamSynchronize(h->stream));
    return LBMP_OK;
}

extern "C" void sg_free(lbmp_sg* h) {
    if (!h || h->magic != SG_MAGIC) return;
    (void)hipStreamSynchronize(h->stream);
    h->magic = 0;
    delete h;
}
