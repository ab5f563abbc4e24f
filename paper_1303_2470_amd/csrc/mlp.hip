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
constexpr int SQ = WIDTH * WIDTH;
static_assert(boff(0) % 4 == 0 && boff(1) % 4 == 0 && boff(2) % 4 == 0, "hidden biases are read four at a time");
static_assert(boff(2) - boff(1) == boff(1) - boff(0), "hidden biases at one stride");

// MFMA operands are stored fragment by fragment: a 32 x 16 piece (32 rows, 16
// consecutive k) is 64 runs of 8 values, run (k / 8) 32 + row, so a wave's
// operand load is one contiguous kilobyte. (Row-major, a load touches 32
// lines for 32 bytes each, four loads share a line, and between them the
// block's other loads have evicted it: a layer's weights crossed from the L2
// four times, 3.4 us of a CU's bandwidth.)
// Offset of element (row, k) of a matrix with ks fragments of k per row tile.
__host__ __device__ constexpr int frag(int row, int k, int ks) {
    return ((row / 32 * ks + k / 16) * 64 + k % 16 / 8 * 32 + row % 32) * 8 + k % 8;
}

// The logistic function through the hardware reciprocal (v_rcp_f32, 1 ulp):
// an IEEE division would cost ten instructions per value, and the epilogues
// are rounded to bf16 anyway.
__device__ __forceinline__ float sigm(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }

constexpr int APITCH = WIDTH + 8;    // bf16 per activation row (padded against bank conflicts)
constexpr int XPITCH = PAD_IN + 8;
constexpr int FBLOCKS = 256;         // one per CU

// Barrier for data passed through LDS: waits for this wave's LDS operations
// only. __syncthreads() also waits for every global store and load in flight,
// which nothing in the block depends on.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt at their maxima
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Fused inference. A block of 8 waves takes groups of 32 ST samples through
// all four layers, wave w computing features 32 w .. 32 w + 31 of every layer
// as the transposed product (weights first), so each lane holds runs of 4
// consecutive features of one sample and writes them to LDS as one 8-byte
// store. The weights of the three hidden layers stay in the wave's registers
// for all groups (136 VGPRs); activations alternate between two LDS buffers,
// one barrier per layer; the output layer runs on ST waves, by turns, while the
// others start the next group. Within a layer the products of one 32-sample
// tile are issued between the activations of the tile before, so that MFMA and
// VALU overlap inside a wave. Bound by the SiLU: 768 per sample, an
// exponential, a reciprocal and 5 more VALU operations each.
// 2^20 rows: 421 us with weights read from the L2 for every group and the
// epilogue after the products, 354 us now (0.31 of the 2.5 PFLOP/s peak); 256
// rows: 19.6 -> 7.7 us.
// The arithmetic is that of the training pass (bf16 operands, fp32
// accumulation in increasing K, bias and SiLU in fp32, activations rounded to
// bf16).
template <int ST>
__global__ void __launch_bounds__(512) k_mlp_forward(const float* __restrict__ x, int64_t n,
                                                     const float* __restrict__ norm, const __bf16* __restrict__ W0,
                                                     const __bf16* __restrict__ Wsq, const __bf16* __restrict__ W3,
                                                     const float* __restrict__ P, float* __restrict__ y) {
    constexpr int RS = 32 * ST, KS = WIDTH / 16, NX = (RS * NFEAT + 511) / 512;
    __shared__ __align__(16) __bf16 act[2][RS * APITCH];
    __shared__ __align__(16) __bf16 xs[RS * XPITCH];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 31, hi = lane >> 5, kh = hi * 8, n0 = 32 * wave;
    bf16x8 w0[2], w1[KS], w2[KS];
#pragma unroll
    for (int k = 0; k < 2; ++k) w0[k] = *reinterpret_cast<const bf16x8*>(W0 + frag(n0, 16 * k, 2) + lane * 8);
#pragma unroll
    for (int k = 0; k < KS; ++k) w1[k] = *reinterpret_cast<const bf16x8*>(Wsq + frag(n0, 16 * k, KS) + lane * 8);
#pragma unroll
    for (int k = 0; k < KS; ++k) w2[k] = *reinterpret_cast<const bf16x8*>(Wsq + SQ + frag(n0, 16 * k, KS) + lane * 8);
    // normalised features of the group that starts at sample s0, through
    // registers so that their loads run ahead of the group
    const int64_t groups = (n + RS - 1) / RS;
    float xv[NX];
    auto fetch = [&](int64_t s0) {
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int e = t + 512 * i;
            const int64_t at = s0 * NFEAT + e;
            xv[i] = e < RS * NFEAT && at < n * NFEAT ? x[at] : 0.0f;
        }
    };
    auto stage = [&](int64_t s0) {
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int e = t + 512 * i;
            if (e < RS * NFEAT) {
                const int row = e / NFEAT, c = e % NFEAT;
                xs[row * XPITCH + c] = s0 + row < n ? (__bf16)((xv[i] - norm[c]) / norm[6 + c]) : (__bf16)0.0f;
            }
        }
    };
    for (int i = t; i < RS * (PAD_IN - NFEAT); i += 512)
        xs[i / (PAD_IN - NFEAT) * XPITCH + NFEAT + i % (PAD_IN - NFEAT)] = (__bf16)0.0f;
    if ((int64_t)blockIdx.x < groups) {
        fetch((int64_t)blockIdx.x * RS);
        stage((int64_t)blockIdx.x * RS);
    }
    lds_barrier();
    // one hidden layer: in (pitch ip) -> out
    auto hidden = [&](const bf16x8* w, auto ksc, const __bf16* in, int ip, const float* __restrict__ bias, __bf16* out) {
        constexpr int ks = decltype(ksc)::value;
        auto product = [&](int j) {
            f32x16 acc = {};
#pragma unroll
            for (int k = 0; k < ks; ++k)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    w[k], *reinterpret_cast<const bf16x8*>(in + (32 * j + r) * ip + 16 * k + kh), acc, 0, 0, 0);
            return acc;
        };
        float4 bc[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) bc[g] = *reinterpret_cast<const float4*>(bias + n0 + 8 * g + 4 * hi);
        f32x16 acc = product(0);
#pragma unroll
        for (int j = 0; j < ST; ++j) {
            f32x16 nxt = {};
            if (j + 1 < ST) nxt = product(j + 1);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bf16x4 o;
                o[0] = (__bf16)silu(acc[4 * g + 0] + bc[g].x);
                o[1] = (__bf16)silu(acc[4 * g + 1] + bc[g].y);
                o[2] = (__bf16)silu(acc[4 * g + 2] + bc[g].z);
                o[3] = (__bf16)silu(acc[4 * g + 3] + bc[g].w);
                *reinterpret_cast<bf16x4*>(out + (32 * j + r) * APITCH + n0 + 8 * g + 4 * hi) = o;
            }
            acc = nxt;
        }
    };
    int turn = 0;
    for (int64_t grp = blockIdx.x; grp < groups; grp += gridDim.x, turn ^= 1) {
        const int64_t s0 = grp * RS, s1 = s0 + (int64_t)gridDim.x * RS;
        // a group's buffers are the last one's, swapped: its output layer may
        // still be reading act[turn ^ 1] while this one fills act[turn]
        __bf16 *const A = act[turn], *const B = act[turn ^ 1];
        fetch(s1);
        hidden(w0, std::integral_constant<int, 2>(), xs, XPITCH, P + boff(0), A);
        lds_barrier();
        stage(s1);
        hidden(w1, std::integral_constant<int, KS>(), A, APITCH, P + boff(1), B);
        lds_barrier();
        hidden(w2, std::integral_constant<int, KS>(), B, APITCH, P + boff(2), A);
        lds_barrier();
        // output layer (PAD_OUT features, feature 0 is the network's output), also
        // transposed: feature 0 of sample 32 j + r sits in element 0 of lane r
        const int j = (wave + (turn ? ST : 0)) & 7;
        if (j < ST) {
            f32x16 acc = {};
#pragma unroll 4
            for (int k = 0; k < KS; ++k)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    *reinterpret_cast<const bf16x8*>(W3 + frag(0, 16 * k, KS) + lane * 8),
                    *reinterpret_cast<const bf16x8*>(A + (32 * j + r) * APITCH + 16 * k + kh), acc, 0, 0, 0);
            const int64_t si = s0 + 32 * j + r;
            if (lane < 32 && si < n) y[si] = norm[12] + norm[13] * (acc[0] + P[boff(3)]);
        }
    }
}

// ------------------------------------------------------------------ training
constexpr int GSPLIT_MAX = 32;
// a split's weight-gradient partials: W_1 [256][32], W_2, W_3 [256][256], W_4 [256]; bias partials
constexpr int GP1 = WIDTH * PAD_IN, GP2 = GP1 + WIDTH * WIDTH, GP3 = GP2 + WIDTH * WIDTH, GP = GP3 + WIDTH;
constexpr int GPB = 3 * WIDTH + 1;

struct TrainBufs {
    const float* norm;      // [6] mean, [6] std, y_mean, y_std
    const float* P;         // packed parameters
    const __bf16 *W0, *W3;  // fragments of [out][in], padded
    const __bf16* Wsq;      // the square layers: W_2, W_3 [out][in], then W_3, W_2 [in][out]
    // fragments of [feature][B]: inputs (padded), activations and gradients by
    // pre-activation of the hidden layers (lstride apart); output gradient [B]
    __bf16 *xT, *AT, *dZT, *dYT;
    size_t lstride;
    float* sq;              // [B] squared errors
};

// Forward and backward pass of 32 rows (x[idx], y[idx]; idx null: in order) in
// one block of 8 waves: wave w owns features 32 w .. 32 w + 31 of every layer,
// as the transposed product (weights first). Activations, gradients and
// silu'(Z) pass through LDS; activations and gradients also leave,
// batch-major, as the operands of the weight gradients.
// At batch 1,024 the 32 blocks run once, and a quarter of the rows a block
// takes as long: bound by the chain of six layers, each of them 128 KB of
// weights through the CU's load path (0.85 us), 16 MFMA in a row, epilogue,
// barrier. So nothing in the chain waits for a load just issued: the rows, the
// biases and the output layer's weights go out before any weights, and two
// layers' weights are held, loaded a layer ahead. With biases from memory in
// each epilogue, one layer's weights and rolled loops 19.1 us, now 15.8; a training
// step 30.1 -> 27.2 us.
constexpr int RB = 32;           // rows per block
constexpr int ZP = WIDTH + 4;    // floats per row of silu'(Z)

__global__ void __launch_bounds__(512) k_train_rows(const float* __restrict__ x, const float* __restrict__ y,
                                                    const int32_t* __restrict__ idx, int B, TrainBufs T) {
    constexpr int KS = WIDTH / 16;
    __shared__ __align__(16) __bf16 act[2][RB * APITCH];
    __shared__ __align__(16) float G[3][RB * ZP];  // silu'(Z) of the hidden layers
    __shared__ __align__(16) __bf16 w3[WIDTH];
    __shared__ __align__(16) float bias[3][WIDTH];
    __shared__ float ty[RB], dy[RB];
    const int r0 = blockIdx.x * RB;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 31, hi = lane >> 5, kh = hi * 8, n0 = 32 * wave;
    bf16x8 wa[KS], wb[KS], w0[2];
    auto load_w = [&](int m, bf16x8 (&w)[KS]) {  // square matrix m
        const __bf16* const W = T.Wsq + (size_t)m * SQ + frag(n0, 0, KS) + lane * 8;
#pragma unroll
        for (int k = 0; k < KS; ++k) w[k] = *reinterpret_cast<const bf16x8*>(W + 512 * k);
    };
    // the small operands go out before the weights, which fill the load path
    // for most of a microsecond
    constexpr int NX = (RB * PAD_IN + 511) / 512;
    float xv[NX] = {}, mean[NX] = {}, sd[NX];
    float yv = 0.0f;
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        const int i = t + 512 * j, row = i / PAD_IN, c = i % PAD_IN;
        sd[j] = 1.0f;
        if (row < RB && c < NFEAT) {
            const int64_t s = idx ? idx[r0 + row] : r0 + row;
            xv[j] = x[s * NFEAT + c];
            mean[j] = T.norm[c];
            sd[j] = T.norm[6 + c];
        }
    }
    if (t < RB) yv = y[idx ? idx[r0 + t] : r0 + t];
    const float ym = T.norm[12], ys = T.norm[13], bout = T.P[boff(3)];
    float4 bv{};
    if (t < 3 * WIDTH / 4) bv = *reinterpret_cast<const float4*>(T.P + boff(0) + t / 64 * (boff(1) - boff(0)) + t % 64 * 4);
    __bf16 w3v{};
    if (t < WIDTH) w3v = T.W3[frag(0, t, KS)];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < 2; ++k) w0[k] = *reinterpret_cast<const bf16x8*>(T.W0 + frag(n0, 16 * k, 2) + lane * 8);
    load_w(0, wa);
    load_w(1, wb);
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        const int i = t + 512 * j, row = i / PAD_IN, c = i % PAD_IN;
        if (row >= RB) break;
        const __bf16 v = c < NFEAT ? (__bf16)((xv[j] - mean[j]) / sd[j]) : (__bf16)0.0f;
        if (c < NFEAT) T.xT[frag(c, r0 + row, 0)] = v;  // one row tile
        act[0][row * APITCH + c] = v;
    }
    if (t < RB) ty[t] = (yv - ym) / ys;
    if (t < 3 * WIDTH / 4) *reinterpret_cast<float4*>(&bias[0][0] + 4 * t) = bv;
    if (t < WIDTH) w3[t] = w3v;
    lds_barrier();
    f32x16 acc = {};
    auto product = [&](const __bf16* in, const bf16x8 (&w)[KS]) {
        acc = f32x16{};
#pragma unroll
        for (int k = 0; k < KS; ++k)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                w[k], *reinterpret_cast<const bf16x8*>(in + r * APITCH + 16 * k + kh), acc, 0, 0, 0);
    };
    // element v of a lane's tile: feature n0 + 8 (v / 4) + 4 hi + v % 4, row r.
    // Group g = v / 4 of the four is moved to elements 0 .. 3.
    auto rotate = [&]() {
#pragma unroll
        for (int v = 0; v < 12; ++v) acc[v] = acc[v + 4];
    };
    auto put = [&](int fw, const bf16x4& o, __bf16* lds, __bf16* __restrict__ out) {
        *reinterpret_cast<bf16x4*>(lds + r * APITCH + n0 + fw) = o;
        // the wave's row tile, the block's two fragments of it
        __bf16* const base = out + ((size_t)wave * (B / 16) + r0 / 16) * 512 + frag(fw, r, 2);
#pragma unroll
        for (int e = 0; e < 4; ++e) base[8 * e] = o[e];
    };
#pragma unroll
    for (int k = 0; k < 2; ++k)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            w0[k], *reinterpret_cast<const bf16x8*>(act[0] + r * APITCH + 16 * k + kh), acc, 0, 0, 0);
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        __bf16* const to = act[(l & 1) ^ 1];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 bc = *reinterpret_cast<const float4*>(&bias[l][n0 + 8 * g + 4 * hi]);
            const float b4[4] = {bc.x, bc.y, bc.z, bc.w};
            bf16x4 o;
            float4 d;
            float* const dp = reinterpret_cast<float*>(&d);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float z = acc[e] + b4[e], s = sigm(z);
                o[e] = (__bf16)(z * s);
                dp[e] = s * (1.0f + z * (1.0f - s));
            }
            *reinterpret_cast<float4*>(&G[l][r * ZP + n0 + 8 * g + 4 * hi]) = d;
            put(8 * g + 4 * hi, o, to, T.AT + l * T.lstride);
            rotate();
        }
        lds_barrier();
        if (l < 2) {
            if (l == 0) {
                product(to, wa);
                load_w(2, wa);  // W_3 [in][out]
            } else {
                product(to, wb);
                load_w(3, wb);  // W_2 [in][out]
            }
        }
    }
    // output layer and loss: feature 0 in element 0 of wave 0's lanes 0 .. 31
    if (wave == 0) {
        f32x16 o = {};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            bf16x8 f{};
            if (r == 0) f = *reinterpret_cast<const bf16x8*>(w3 + 16 * k + kh);
            o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                f, *reinterpret_cast<const bf16x8*>(act[1] + r * APITCH + 16 * k + kh), o, 0, 0, 0);
        }
        if (lane < 32) {
            const float e = (o[0] + bout) - ty[r];
            const __bf16 d = (__bf16)(2.0f * e / (float)B);
            dy[r] = (float)d;
            T.dYT[r0 + r] = d;
            T.sq[r0 + r] = e * e;
        }
    }
    lds_barrier();
    // the output layer's gradient has one nonzero column: dA_3 = dy w3
    {
        const float d = dy[r];
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = d * (float)w3[n0 + 8 * (v >> 2) + 4 * hi + (v & 3)];
    }
#pragma unroll
    for (int l = 2; l >= 0; --l) {
        __bf16* const to = act[l & 1];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 d = *reinterpret_cast<const float4*>(&G[l][r * ZP + n0 + 8 * g + 4 * hi]);
            bf16x4 o;
            o[0] = (__bf16)(acc[0] * d.x);
            o[1] = (__bf16)(acc[1] * d.y);
            o[2] = (__bf16)(acc[2] * d.z);
            o[3] = (__bf16)(acc[3] * d.w);
            put(8 * g + 4 * hi, o, to, T.dZT + l * T.lstride);
            rotate();
        }
        if (l == 0) break;
        lds_barrier();
        if (l == 2) product(to, wa);
        else product(to, wb);
    }
}

// Parameter gradients over batch splits of kc rows. Wave job (split, tile):
// one 32 x 32 tile of dW_l = dZ_l^T A_{l-1} over the split's rows, its partial
// in P[split]; both operands are batch-major, so a lane's 8 rows are one
// 16-byte load, a wave's a contiguous kilobyte. The blocks behind them sum dZ for the biases, one thread per
// (split, output): eight interleaved partial sums, then their sum in order.
// Splitting K keeps the whole GPU busy where a 256 x 256 gradient has only 64
// tiles; the partials are added in split order, so the result does not depend
// on scheduling.
// NP products and NR runs of 8 rows are loaded at a time: the kernel waits for
// memory (the operands come from the caches of other XCDs), and the compiler
// left to itself asks for a few and waits. 16 and 16 while the jobs leave room
// for the registers, 4 and 8 where several waves of a SIMD hide each other's
// loads: a training step of 512, 1,024, 1,536, 8,192 rows 25.2, 27.3, 30.3,
// 38.6 us before. With 16 and 16 against 4 and 8: 512 rows 22.1 and 23.4, 1,024
// 24.1 and 25.3, 2,048 (8 splits) 28.6 and 29.2, 4,096 (16) 32.2 and 32.2, 6,144
// 34.4 and 34.0, 8,192 (32) 38.9 and 38.0, 16,384 60.5 and 60.5; from 32,768 rows
// on, long splits, 2 % the other way (65,536: 203 and 208).
constexpr int GTILES = 2 * (WIDTH / 32) * (WIDTH / 32) + 2 * (WIDTH / 32);

template <int NP, int NR>
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
        int m0, n0, po, ld;
        const int nk = B / 16;  // fragments per row tile
        bool one = false;       // a single output row (the output layer)
        if (t < 2 * TN * TN) {
            const int l = t < TN * TN ? 1 : 2;
            t -= (l - 1) * TN * TN;
            m0 = t / TN * 32;
            n0 = t % TN * 32;
            dz = T.dZT + l * T.lstride;
            a = T.AT + (l - 1) * T.lstride;
            po = l == 1 ? GP1 : GP2;
            ld = WIDTH;
        } else if ((t -= 2 * TN * TN) < TN) {
            m0 = 32 * t;
            n0 = 0;
            dz = T.dZT;
            a = T.xT;
            po = 0;
            ld = PAD_IN;
        } else {
            m0 = 0;
            n0 = 32 * (t - TN);
            dz = T.dYT;
            a = T.AT + 2 * T.lstride;
            po = GP3;
            ld = WIDTH;
            one = true;
        }
        const int r = lane & 31, kh = (lane >> 5) * 8;
        const __bf16* pb = a + ((size_t)(n0 / 32) * nk + split * kc / 16) * 512 + lane * 8;
        const __bf16* pa = one ? dz + split * kc + kh : dz + ((size_t)(m0 / 32) * nk + split * kc / 16) * 512 + lane * 8;
        f32x16 acc = {};
        // N products, every operand asked for before the first is waited for
        const int sa = one ? 16 : 512;
        const bool has = !one || r == 0;
        auto products = [&](auto nc, int k) {
            constexpr int N = decltype(nc)::value;
            bf16x8 fa[N], fb[N];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                fa[j] = bf16x8{};
                if (has) fa[j] = *reinterpret_cast<const bf16x8*>(pa + sa * (k + j));
                fb[j] = *reinterpret_cast<const bf16x8*>(pb + 512 * (k + j));
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int j = 0; j < N; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[j], fb[j], acc, 0, 0, 0);
        };
        int k = 0;
        for (; k + NP <= kc / 16; k += NP) products(std::integral_constant<int, NP>(), k);
        if constexpr (NP > 4)
            for (; k + 4 <= kc / 16; k += 4) products(std::integral_constant<int, 4>(), k);
        for (; k < kc / 16; ++k) products(std::integral_constant<int, 1>(), k);
        float* const out = P + (size_t)split * GP + po;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = m0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            if (!one || row == 0) out[row * ld + n0 + r] = acc[v];
        }
        return;
    }
    const int id = ((int)blockIdx.x - wblocks) * 256 + (int)threadIdx.x;
    if (id >= GPB * splits) return;
    const int split = id / GPB, o = id % GPB;
    const __bf16* p = T.dYT + split * kc;
    int half = 8, step = 16;  // from a run of 8 rows to the next, from a fragment to the next
    if (o < 3 * WIDTH) {
        p = T.dZT + o / WIDTH * T.lstride + ((size_t)(o % WIDTH / 32) * (B / 16) + split * kc / 16) * 512 + o % 32 * 8;
        half = 256;
        step = 512;
    }
    float s[8] = {};
    auto runs = [&](auto nc, int b) {
        constexpr int N = decltype(nc)::value;
        bf16x8 v[N];
#pragma unroll
        for (int j = 0; j < N; ++j)
            v[j] = *reinterpret_cast<const bf16x8*>(p + ((b + j) >> 1) * step + ((b + j) & 1) * half);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int g = 0; g < 8; ++g) s[g] += (float)v[j][g];
    };
    int b = 0;
    for (; b + NR <= kc / 8; b += NR) runs(std::integral_constant<int, NR>(), b);
    for (; b + 4 <= kc / 8; b += 4) runs(std::integral_constant<int, 4>(), b);
    for (; b < kc / 8; ++b) runs(std::integral_constant<int, 1>(), b);
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

struct Copies {  // bf16 copies of the weights, as TrainBufs holds them
    __bf16 *W0, *W3, *Wsq;
};
__device__ __forceinline__ void copy_bf16(const Copies& K, int l, int o, int c, float w) {
    if (c < 0) return;
    const __bf16 b = (__bf16)w;
    if (l == 0) K.W0[frag(o, c, 2)] = b;
    else if (l == 3) K.W3[frag(0, c, WIDTH / 16)] = b;
    else {
        K.Wsq[(l - 1) * SQ + frag(o, c, WIDTH / 16)] = b;
        K.Wsq[(4 - l) * SQ + frag(c, o, WIDTH / 16)] = b;
    }
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
    __bf16 *xT, *AT, *dZT, *dYT;  // a batch's rows, batch-major
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
    h->K.W0 = c.take<__bf16>(WIDTH * PAD_IN);
    h->K.W3 = c.take<__bf16>(PAD_OUT * WIDTH);
    h->K.Wsq = c.take<__bf16>(4 * SQ);
    h->norm = c.take<float>(16);
    const size_t B = (size_t)h->bmax;
    h->xT = c.take<__bf16>(B * PAD_IN);  // columns past the features stay zero
    h->AT = c.take<__bf16>(3 * B * WIDTH);
    h->dZT = c.take<__bf16>(3 * B * WIDTH);
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

// Partial gradients of a batch.
static void gradients(lbmp_sg* h, const float* x, const float* y, const int32_t* idx, int B) {
    hipStream_t s = h->stream;
    const TrainBufs T{h->norm, h->P, h->K.W0, h->K.W3, h->K.Wsq, h->xT, h->AT, h->dZT, h->dYT,
                      (size_t)h->bmax * WIDTH, h->sq};
    k_train_rows<<<(unsigned)(B / RB), 512, 0, s>>>(x, y, idx, B, T);
    const int splits = grad_splits(B);
    const unsigned nb = (unsigned)(GTILES / 4 * splits + (GPB * splits + 255) / 256);
    // up to 8 splits: at most about one block per CU
    if (splits <= 8) k_train_grads<16, 16><<<nb, 256, 0, s>>>(T, B, B / splits, splits, h->gsplit, h->bsplit);
    else k_train_grads<4, 8><<<nb, 256, 0, s>>>(T, B, B / splits, splits, h->gsplit, h->bsplit);
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
        // samples per group: 32 until every CU has one (least latency), then 64,
        // then 128 (fewest barriers per sample), a block per CU and group by group
        auto go = [&](auto stc) {
            constexpr int ST = decltype(stc)::value;
            const int64_t groups = (n + 32 * ST - 1) / (32 * ST);
            k_mlp_forward<ST><<<(unsigned)std::min<int64_t>(groups, FBLOCKS), 512, 0, s>>>(x_dev, n, h->norm, h->K.W0, h->K.Wsq,
                                                                                    h->K.W3, h->P, y_dev);
        };
        if (n <= 32 * FBLOCKS) go(std::integral_constant<int, 1>());
        else if (n <= 64 * FBLOCKS) go(std::integral_constant<int, 2>());
        else go(std::integral_constant<int, 4>());
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
