// MLP device code shared by the surrogate's training kernels and P2G:
// BF16/FP32 MFMA fragments, the network staged in LDS, and the forward pass
// of a 16-sample tile (layers in transposed form Z^T = W A^T, so the
// output fragment of one layer is the B fragment of the next).
#pragma once

#include "mpm_internal.h"
#include "mpm_surrogate.h"

namespace mpm {
namespace mlp {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// tanh(x) = 1 - 2 / (1 + exp(2x)): one exponential and one division, exact
// to ~1e-7 absolute, well inside the BF16 operands it feeds (and -> +-1 for
// large |x| without overflow trouble: exp -> inf gives 1, exp -> 0 gives -1).
// exp(2x) as 2^(x 2 log2 e): the doubling goes into the constant, exactly.
__device__ __forceinline__ float act_tanh(float x) {
    return 1.0f - 2.0f / (1.0f + __builtin_amdgcn_exp2f(x * (2.0f * 1.44269504f)));
}

// FP32 operands (gradient checks): v_mfma_f32_16x16x4_f32 over the K rows
// {4g + r}, four of them for a K = 16 step, on the fragments a K = 16 BF16
// MFMA would take.  The weights of one layer as the A operand, staged in LDS
// row-major [rows][ld].  acc += W_tile(mt, kt) * B.
__device__ __forceinline__ f32x4 mma_w(f32x4 acc, const float* W, int ld, int mt, int kt, const float b[4]) {
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const float* row = W + (16 * mt + i) * ld + 16 * kt + 4 * g;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(row[r], b[r], acc, 0, 0, 0);
    return acc;
}

// acc += A * B where both operands come from LDS: A[i][k] = a[(16*mt + i) * lda + 16*kt + k]
// and B[k][j] = bmat[(16*kt + k) * ldb + 16*nt + j] (row-major K x N).
__device__ __forceinline__ f32x4 mma_ll(f32x4 acc, const float* a, int lda, int mt, int kt, const float* bm, int ldb,
                                        int nt) {
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[(16 * mt + i) * lda + 16 * kt + 4 * g + r],
                                                   bm[(16 * kt + 4 * g + r) * ldb + 16 * nt + i], acc, 0, 0, 0);
    return acc;
}

// The network staged in LDS for the forward pass (FP32, zero padded):
// W1 [64][16], W2 [64][64], W3 [16][64], biases and the normalisation.
struct NetLds {
    float W1[64 * 16], b1[64], W2[64 * 64], b2[64], W3[16 * 64], b3[16];
    float imu[16], isd[16], omu[16], osd[16];
};

// Transposed weights for backpropagation: W2T [64][64], W3T [64][16].
struct NetLdsT {
    float W2T[64 * 64], W3T[64 * 16];
};

__device__ inline void load_net(NetLds& L, const float* __restrict__ th, const float* __restrict__ norm) {
    for (int t = threadIdx.x; t < 64 * 16; t += blockDim.x) {
        const int o = t >> 4, i = t & 15;
        L.W1[t] = i < SUR_IN ? th[SUR_W1 + o * SUR_IN + i] : 0.0f;
        const int o3 = t >> 6, i3 = t & 63;  // W3 padded to 16 outputs
        L.W3[t] = o3 < SUR_OUT ? th[SUR_W3 + o3 * SUR_H + i3] : 0.0f;
    }
    for (int t = threadIdx.x; t < 64 * 64; t += blockDim.x) L.W2[t] = th[SUR_W2 + t];
    for (int t = threadIdx.x; t < 64; t += blockDim.x) {
        L.b1[t] = th[SUR_B1 + t];
        L.b2[t] = th[SUR_B2 + t];
    }
    for (int t = threadIdx.x; t < 16; t += blockDim.x) {
        L.b3[t] = t < SUR_OUT ? th[SUR_B3 + t] : 0.0f;
        L.imu[t] = t < SUR_IN ? norm[t] : 0.0f;
        L.isd[t] = t < SUR_IN ? norm[SUR_IN + t] : 1.0f;
        L.omu[t] = t < SUR_OUT ? norm[2 * SUR_IN + t] : 0.0f;
        L.osd[t] = t < SUR_OUT ? norm[2 * SUR_IN + SUR_OUT + t] : 1.0f;
    }
}

__device__ inline void load_net_t(NetLdsT& L, const float* __restrict__ th) {
    for (int t = threadIdx.x; t < 64 * 16; t += blockDim.x) {
        const int o3 = t >> 6, i3 = t & 63;
        L.W3T[i3 * 16 + o3] = o3 < SUR_OUT ? th[SUR_W3 + o3 * SUR_H + i3] : 0.0f;
    }
    for (int t = threadIdx.x; t < 64 * 64; t += blockDim.x) L.W2T[(t & 63) * 64 + (t >> 6)] = th[SUR_W2 + t];
}

// Forward pass of one 16-sample tile held by a wave.  xin: the tile's
// normalised inputs in LDS [16 samples][16].  Outputs h1, h2 (tanh
// activations, D layout: per hidden tile mt, lane holds units 16mt+4g+r of
// sample l%16) and y (normalised outputs, D layout over 16 output rows).
__device__ __forceinline__ void forward_tile(const NetLds& L, const float* xin, float h1[4][4], float h2[4][4],
                                             float y[4]) {
    const int lane = threadIdx.x & 63, g = lane >> 4, s = lane & 15;
    float xb[4];  // B fragment of X^T: features 4g..4g+3 of sample s
#pragma unroll
    for (int j = 0; j < 4; ++j) xb[j] = xin[s * 16 + 4 * g + j];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mma_w(acc, L.W1, 16, mt, 0, xb);
#pragma unroll
        for (int r = 0; r < 4; ++r) h1[mt][r] = act_tanh(acc[r] + L.b1[16 * mt + 4 * g + r]);
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) acc = mma_w(acc, L.W2, 64, mt, kt, h1[kt]);
#pragma unroll
        for (int r = 0; r < 4; ++r) h2[mt][r] = act_tanh(acc[r] + L.b2[16 * mt + 4 * g + r]);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) acc = mma_w(acc, L.W3, 64, 0, kt, h2[kt]);
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = acc[r] + L.b3[4 * g + r];
}

// Normalised input row of sample `row` into LDS (zero padded to 16).
__device__ __forceinline__ void stage_input(const NetLds& L, const float* __restrict__ X, int64_t row, bool valid,
                                            float* xin, int s) {
    // 4 lanes per sample: lane group g writes features 4g..4g+3
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int f = 4 * g + j;
        float v = 0.0f;
        if (valid && f < SUR_IN) v = (X[row * SUR_IN + f] - L.imu[f]) / L.isd[f];
        xin[s * 16 + f] = v;
    }
}

// Inference copy of the network for P2G: the weights rounded to BF16 once
// as they are staged, biases and normalisation FP32.  The hidden layers run
// on gfx950's 16x16x32 BF16 MFMA: a K = 32 fragment of lane (i, g) holds the
// eight k' = 8g..8g+7, and k' is a permutation of the 32 hidden units of the
// block chosen so that the B fragment is the D output of the previous layer
// as it lies in the registers (units 4g..4g+3 of two consecutive 16-unit
// tiles); the weight rows are stored in that k' order, so an A fragment is
// one 16-byte LDS read.  Rows are padded to W16_LD so the 16 rows one read
// instruction touches start in different banks.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4h __attribute__((ext_vector_type(4)));
constexpr int W16_LD = 72;

struct __attribute__((aligned(16))) NetLds16 {
    __bf16 W1[64 * 16];      // [unit][feature], the K = 16 first layer
    __bf16 W2[64 * W16_LD];  // [unit][k'] of the two K = 32 blocks
    __bf16 W3[16 * W16_LD];  // [output][k'] (outputs padded to 16)
    float b1[64], b2[64], b3[16];
    float imu[16], isd[16], omu[16], osd[16];  // (in this order: load_net16)
};

// Position k' of hidden unit u in its K = 32 block: unit 32 kb + 16 h + 4 g + r
// sits at 32 kb + 8 g + 4 h + r.
__device__ __forceinline__ int kperm(int u) {
    const int w = u & 31;
    return (u & 32) + 8 * ((w & 15) >> 2) + 4 * (w >> 4) + (w & 3);
}

// Stage the network with the NT threads of the workgroup.  The parameters
// are loaded coalesced, every load of a thread in flight at once, and then
// written where they belong (a loop that loads and stores element by element
// waits for memory some forty times; it took most of a training step).
// TRAIN: hidden units in their own order (K = 16 steps), and the transposed
// copies that backpropagation reads: W2T [hidden 1][hidden 2], W3T [hidden 2]
// [output].
constexpr int W3T_LD = 20;
struct __attribute__((aligned(16))) NetLdsT16 {
    __bf16 W2T[64 * W16_LD], W3T[64 * W3T_LD];
};

template <int NT, bool TRAIN = false>
__device__ __forceinline__ void load_net16(NetLds16& L, const float* __restrict__ th, const float* __restrict__ norm,
                                           NetLdsT16* LT = nullptr) {
    constexpr int N2 = 64 * 64 / NT, N1 = 64 * SUR_IN / NT;  // values of W2, and of W1 and of W3, per thread
    static_assert(SUR_IN == 12 && SUR_OUT == 12 && 64 * 64 % NT == 0, "the staging loops");
    const int tid = threadIdx.x;
    auto place = [](int u) { return TRAIN ? u : kperm(u); };
    float v2[N2], v1[N1 + 1], v3[N1 + 1];
#pragma unroll
    for (int k = 0; k < N2; ++k) v2[k] = th[SUR_W2 + tid + k * NT];
#pragma unroll
    for (int k = 0; k <= N1; ++k) {
        const int e = tid + k * NT;
        v1[k] = e < 64 * SUR_IN ? th[SUR_W1 + e] : 0.0f;
        v3[k] = e < 64 * SUR_OUT ? th[SUR_W3 + e] : 0.0f;
    }
    const int c = tid & 63;
    const float b1 = th[SUR_B1 + c], b2 = th[SUR_B2 + c], b3 = c < SUR_OUT ? th[SUR_B3 + c] : 0.0f;
    const float nv = c < SUR_NORM ? norm[c] : 0.0f;
#pragma unroll
    for (int k = 0; k < N2; ++k) {
        const int e = tid + k * NT, o = e >> 6, i = e & 63;
        L.W2[o * W16_LD + place(i)] = (__bf16)v2[k];
        if constexpr (TRAIN) LT->W2T[i * W16_LD + o] = (__bf16)v2[k];
    }
#pragma unroll
    for (int k = 0; k <= N1; ++k) {
        const int e = tid + k * NT;
        if (e < 64 * SUR_IN) L.W1[e / SUR_IN * 16 + e % SUR_IN] = (__bf16)v1[k];
        if (e < 64 * SUR_OUT) {
            L.W3[(e >> 6) * W16_LD + place(e & 63)] = (__bf16)v3[k];
            if constexpr (TRAIN) LT->W3T[(e & 63) * W3T_LD + (e >> 6)] = (__bf16)v3[k];
        }
    }
    for (int e = tid; e < 4 * 64; e += NT) {  // the padding: features and outputs 12 .. 15
        L.W1[(e >> 2) * 16 + SUR_IN + (e & 3)] = (__bf16)0.0f;
        L.W3[(SUR_OUT + (e >> 6)) * W16_LD + (e & 63)] = (__bf16)0.0f;
        if constexpr (TRAIN) LT->W3T[(e >> 2) * W3T_LD + SUR_OUT + (e & 3)] = (__bf16)0.0f;
    }
    if (tid < 64) {
        L.b1[tid] = b1;
        L.b2[tid] = b2;
        // the normalisation, [12] input means, input sds, output means, output sds, each padded to 16
        if (tid < SUR_NORM) (&L.imu[0])[tid / 12 * 16 + tid % 12] = nv;
        if (tid < 16) {
            L.b3[tid] = b3;
            if (tid >= 12) {
                L.imu[tid] = L.omu[tid] = 0.0f;
                L.isd[tid] = L.osd[tid] = 1.0f;
            }
        }
    }
}

// tanh of the four accumulators and their BF16 B-fragment halves
__device__ __forceinline__ void act_pack(f32x4 a0, f32x4 a1, bf16x8& b) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        b[r] = (__bf16)act_tanh(a0[r]);
        b[4 + r] = (__bf16)act_tanh(a1[r]);
    }
}

// Forward pass of a 16-sample tile: xb the B fragment of the first layer
// (normalised features 4g .. 4g+3 of sample lane % 16, in BF16), returns the
// normalised outputs 4g .. 4g+3 of that sample (g = 3: the padding outputs).
__device__ __forceinline__ f32x4 forward_tile16(const NetLds16& L, const bf16x4h xb) {
    const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
    f32x4 h[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        const bf16x4h a = *reinterpret_cast<const bf16x4h*>(L.W1 + (16 * mt + i) * 16 + 4 * g);
        h[mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, a), __builtin_bit_cast(bf16x4, xb),
                                                           *reinterpret_cast<const f32x4*>(L.b1 + 16 * mt + 4 * g), 0, 0, 0);
    }
    bf16x8 hb[2];
    act_pack(h[0], h[1], hb[0]);
    act_pack(h[2], h[3], hb[1]);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        f32x4 acc = *reinterpret_cast<const f32x4*>(L.b2 + 16 * mt + 4 * g);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(L.W2 + (16 * mt + i) * W16_LD + 32 * kb + 8 * g);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, hb[kb], acc, 0, 0, 0);
        }
        h[mt] = acc;
    }
    act_pack(h[0], h[1], hb[0]);
    act_pack(h[2], h[3], hb[1]);
    f32x4 acc = *reinterpret_cast<const f32x4*>(L.b3 + 4 * g);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(L.W3 + i * W16_LD + 32 * kb + 8 * g);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, hb[kb], acc, 0, 0, 0);
    }
    return acc;
}

// Forward pass of the wave's 64 samples, one per lane: xn the lane's
// normalised inputs, yn its normalised outputs.  stage: FWD_STAGE floats of
// LDS owned by the wave, 16-byte aligned (the rows move as 16-byte vectors),
// the inputs as BF16 rows [64][16] in the first 512
// and the outputs [64][12] after them.  The four 16-sample tiles run one
// after the other with no barrier between them (the four output tiles of a
// layer are independent MFMA chains).
constexpr int FWD_STAGE = 512 + 64 * SUR_OUT;

__device__ __forceinline__ void forward_wave16(const NetLds16& L, float* stage, const float xn[SUR_IN],
                                               float yn[SUR_OUT]) {
    static_assert(SUR_OUT == 12, "the output rows are three float4");
    const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
    __bf16* xs = reinterpret_cast<__bf16*>(stage);
    float* ys = stage + 512;
    {
        bf16x8 r0, r1;
#pragma unroll
        for (int j = 0; j < 8; ++j) r0[j] = (__bf16)xn[j];
#pragma unroll
        for (int j = 0; j < 8; ++j) r1[j] = (__bf16)(8 + j < SUR_IN ? xn[8 + j] : 0.0f);
        *reinterpret_cast<bf16x8*>(xs + lane * 16) = r0;
        *reinterpret_cast<bf16x8*>(xs + lane * 16 + 8) = r1;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll 1
    for (int t = 0; t < 4; ++t) {
        // the weights are read again for every tile rather than held in registers
        // across the four (they would take some 80 VGPRs from the caller)
        asm volatile("" ::: "memory");
        // B fragment of the first layer: features 4g..4g+3 of sample 16t + i
        const f32x4 acc = forward_tile16(L, *reinterpret_cast<const bf16x4h*>(xs + (16 * t + i) * 16 + 4 * g));
        // outputs 4g..4g+3 of sample 16t + i (g = 3 holds the padding outputs)
        if (g < 3) *reinterpret_cast<f32x4*>(ys + (16 * t + i) * SUR_OUT + 4 * g) = acc;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int o = 0; o < SUR_OUT; ++o) yn[o] = ys[lane * SUR_OUT + o];
    __builtin_amdgcn_wave_barrier();
}

// Columns 4g .. 4g+3 of a 12-wide row; VEC: the array is 16-byte aligned.
template <bool VEC>
__device__ __forceinline__ void load_row4(const float* __restrict__ A, int64_t row, int g, float v[4]) {
    const float* p = A + row * 12 + 4 * g;
    if constexpr (VEC) {
        const f32x4 q = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = q[j];
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = p[j];
    }
}

}  // namespace mlp
}  // namespace mpm
