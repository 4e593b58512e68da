// Learned constitutive surrogate on gfx950: an MLP 12 -> 64 -> 64 -> 12
// (tanh hidden layers, linear output) that maps the trial elastic singular
// values, the plastic volume and the hardening state of a snow particle to
// the projected singular values and principal Kirchhoff stress.  This file
// holds the network's forward pass, its loss gradient by backpropagation,
// Adam, the normalisation statistics and the generation of training pairs
// from a running simulation with the exact return map.
//
// MI355X design:
//  * Every layer runs on MFMA in transposed form, Z^T = W A^T: the weight
//    tile is the A operand and the activations the B operand.  The 16x16
//    output fragment of v_mfma_f32_16x16x16_bf16 (lane l: rows 4(l/16)+r,
//    column l%16) is then exactly the B fragment the next layer needs, so
//    hidden activations never leave registers in the forward pass.
//  * Precision: BF16 operands with FP32 accumulation (the product path), or
//    FP32 operands on v_mfma_f32_16x16x4_f32 for checking gradients.  The
//    FP32 form splits each K=16 step into four K=4 steps over the K rows
//    {4g + r}, g = 0..3, so it consumes the same register fragments.
//  * Training (BF16): a wave takes 16 samples at a time; activations and
//    deltas are staged in LDS in BF16, sample-contiguous, so that the weight
//    gradients (samples as the K dimension) read MFMA operands in one 8-byte
//    LDS read each.  The gradients accumulate in MFMA accumulators; a
//    workgroup sums its four waves in LDS and stores one partial gradient,
//    and the Adam kernel sums the partials as it reads them.  No atomics, no
//    clearing and no index array: two launches per step.
#include "mpm_mlp.h"

namespace mpm {

namespace {

constexpr int SW = 256;  // threads per workgroup (4 waves)
using namespace mlp;

__global__ __launch_bounds__(SW) void k_sur_forward(const float* __restrict__ th, const float* __restrict__ norm,
                                                    const float* __restrict__ X, int64_t count,
                                                    float* __restrict__ Y) {
    __shared__ NetLds L;
    __shared__ float xin[SW / 64][16 * 16];
    load_net(L, th, norm);
    __syncthreads();
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, s = lane & 15;
    const int64_t tiles = (count + 15) / 16;
    for (int64_t t = (int64_t)blockIdx.x * (SW / 64) + w; t < tiles; t += (int64_t)gridDim.x * (SW / 64)) {
        const int64_t row = 16 * t + s;
        const bool valid = row < count;
        stage_input(L, X, row, valid, xin[w], s);
        __builtin_amdgcn_wave_barrier();
        float h1[4][4], h2[4][4], y[4];
        forward_tile(L, xin[w], h1, h2, y);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 4 * g + r;
            if (valid && o < SUR_OUT) Y[row * SUR_OUT + o] = y[r] * L.osd[o] + L.omu[o];
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Y = network(X) with the BF16 inference copy of the network: the weights
// rounded to BF16 once as they are staged (NetLds16) and the tile pass P2G
// runs (forward_tile16), with P2G's input normalisation.  A lane loads four
// columns of a row straight into the first layer's fragment and stores four
// outputs straight from the last one's, and a wave keeps the weights in
// registers over its tiles.  Instruction issue binds: 64 exponentials and
// reciprocals at a quarter of the rate and 200 other VALU instructions per
// tile and wave, 59 us for 1.28M rows (81 us with rows staged in LDS and the
// network staged by twice the workgroups).  VEC: X and Y are 16-byte aligned.
template <bool VEC>
__global__ __launch_bounds__(SW, 4) void k_sur_forward16(const float* __restrict__ th, const float* __restrict__ norm,
                                                         const float* __restrict__ X, int64_t count,
                                                         float* __restrict__ Y) {
    __shared__ NetLds16 L;
    const int lane = threadIdx.x & 63, g = lane >> 4, s = lane & 15;
    const int64_t tiles = (count + 15) / 16, stride = (int64_t)gridDim.x * (SW / 64);
    int64_t t = (int64_t)blockIdx.x * (SW / 64) + (threadIdx.x >> 6);
    float xv[4] = {0.f, 0.f, 0.f, 0.f};
    if (16 * t + s < count && g < 3) load_row4<VEC>(X, 16 * t + s, g, xv);
    load_net16<SW>(L, th, norm);
    __syncthreads();
    for (; t < tiles; t += stride) {
        const int64_t row = 16 * t + s, next = 16 * (t + stride) + s;
        bf16x4h xb;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            xb[j] = (__bf16)(row < count && g < 3 ? (xv[j] - L.imu[4 * g + j]) / L.isd[4 * g + j] : 0.0f);
        if (next < count && g < 3) load_row4<VEC>(X, next, g, xv);
        const f32x4 y = forward_tile16(L, xb);
        if (row < count && g < 3) {
            f32x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = y[j] * L.osd[4 * g + j] + L.omu[4 * g + j];
            float* p = Y + row * SUR_OUT + 4 * g;
            if constexpr (VEC) {
                *reinterpret_cast<f32x4*>(p) = o;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) p[j] = o[j];
            }
        }
    }
}

// Loss 1/2 |y~ - t~|^2 averaged over `count` samples (normalised space) and
// its gradient in FP32 (for checking gradients), accumulated into
// grad[SUR_PARAMS] and *loss (both zeroed by the caller).
__global__ __launch_bounds__(SW) void k_sur_grad(const float* __restrict__ th, const float* __restrict__ norm,
                                                 const float* __restrict__ X, const float* __restrict__ T,
                                                 int64_t count, float* __restrict__ grad, float* __restrict__ loss) {
    __shared__ NetLds L;
    __shared__ NetLdsT LT;
    // per wave: inputs [16][16], a1 [16][64], a2 [16][64] (sample-major), deltas d3^T [16][16],
    // d2^T [64][16], d1^T [64][16] (unit-major)
    __shared__ float st_x[SW / 64][16 * 16], st_a1[SW / 64][16 * 64], st_a2[SW / 64][16 * 64];
    __shared__ float st_d3[SW / 64][16 * 16], st_d2[SW / 64][64 * 16], st_d1[SW / 64][64 * 16];
    load_net(L, th, norm);
    load_net_t(LT, th);
    __syncthreads();
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, s = lane & 15;
    const float inv_n = 1.0f / (float)count;
    // gradient accumulators (D layout): gW1 4 tiles [64x16], gW2 16 tiles, gW3 4 tiles [16x64]
    f32x4 gW1[4], gW2[4][4], gW3[4];
    float gb1[4][4], gb2[4][4], gb3[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        gW1[a] = f32x4{0.f, 0.f, 0.f, 0.f};
        gW3[a] = f32x4{0.f, 0.f, 0.f, 0.f};
        gb3[a] = 0.0f;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            gW2[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
            gb1[a][b] = gb2[a][b] = 0.0f;
        }
    }
    float lsum = 0.0f;
    const int64_t tiles = (count + 15) / 16;
    float* xs = st_x[w];
    float* a1 = st_a1[w];
    float* a2 = st_a2[w];
    float* d3 = st_d3[w];
    float* d2 = st_d2[w];
    float* d1 = st_d1[w];
    for (int64_t t = (int64_t)blockIdx.x * (SW / 64) + w; t < tiles; t += (int64_t)gridDim.x * (SW / 64)) {
        const int64_t pos = 16 * t + s;
        const bool valid = pos < count;
        const int64_t row = valid ? pos : 0;
        stage_input(L, X, row, valid, xs, s);
        __builtin_amdgcn_wave_barrier();
        float h1[4][4], h2[4][4], y[4];
        forward_tile(L, xs, h1, h2, y);
        // output delta (normalised targets), D layout rows 4g+r of sample s
        float dy[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 4 * g + r;
            float e = 0.0f;
            if (valid && o < SUR_OUT) {
                e = y[r] - (T[row * SUR_OUT + o] - L.omu[o]) / L.osd[o];
                lsum += 0.5f * e * e;
            }
            dy[r] = e * inv_n;
            d3[o * 16 + s] = dy[r];  // [out][sample]: the gW3 A operand
        }
        // activations staged [sample][unit] for the weight-gradient B operands
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                a1[s * 64 + 16 * mt + 4 * g + r] = h1[mt][r];
                a2[s * 64 + 16 * mt + 4 * g + r] = h2[mt][r];
            }
        // delta2^T = (W3^T dy^T) * (1 - a2^2): A = W3T tile (hidden x out), B = dy^T fragment
        float e2[4][4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            acc = mma_w(acc, LT.W3T, 16, mt, 0, dy);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                e2[mt][r] = acc[r] * (1.0f - h2[mt][r] * h2[mt][r]);
                d2[(16 * mt + 4 * g + r) * 16 + s] = e2[mt][r];  // [unit][sample]
            }
        }
        // delta1^T = (W2^T delta2^T) * (1 - a1^2)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) acc = mma_w(acc, LT.W2T, 64, mt, kt, e2[kt]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float e1 = acc[r] * (1.0f - h1[mt][r] * h1[mt][r]);
                d1[(16 * mt + 4 * g + r) * 16 + s] = e1;
                gb1[mt][r] += e1;
            }
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) gb2[mt][r] += e2[mt][r];
#pragma unroll
        for (int r = 0; r < 4; ++r) gb3[r] += dy[r];
        __builtin_amdgcn_wave_barrier();
        // weight gradients, samples as K: gW3 (16 x 64) += d3^T (16 x 16s) * a2 (16s x 64)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) gW3[nt] = mma_ll(gW3[nt], d3, 16, 0, 0, a2, 64, nt);
        // gW2 (64 x 64) += d2^T (64 x 16s) * a1 (16s x 64)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) gW2[mt][nt] = mma_ll(gW2[mt][nt], d2, 16, mt, 0, a1, 64, nt);
        // gW1 (64 x 16) += d1^T (64 x 16s) * x (16s x 16)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) gW1[mt] = mma_ll(gW1[mt], d1, 16, mt, 0, xs, 16, 0);
        __builtin_amdgcn_wave_barrier();
    }
    // one atomic per parameter per wave (D layout: lane holds rows 4g+r, column s)
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 16 * mt + 4 * g + r;
            if (s < SUR_IN) atomicAdd(&grad[SUR_W1 + o * SUR_IN + s], gW1[mt][r]);
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) atomicAdd(&grad[SUR_W2 + o * SUR_H + 16 * nt + s], gW2[mt][nt][r]);
        }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 4 * g + r;
            if (o < SUR_OUT) atomicAdd(&grad[SUR_W3 + o * SUR_H + 16 * nt + s], gW3[nt][r]);
        }
    // bias gradients: sums over the wave's samples (lanes with equal g hold the same units)
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float v1 = gb1[mt][r], v2 = gb2[mt][r];
#pragma unroll
            for (int d = 1; d < 16; d <<= 1) {
                v1 += __shfl_xor(v1, d, 64);
                v2 += __shfl_xor(v2, d, 64);
            }
            if (s == 0) {
                atomicAdd(&grad[SUR_B1 + 16 * mt + 4 * g + r], v1);
                atomicAdd(&grad[SUR_B2 + 16 * mt + 4 * g + r], v2);
            }
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float v3 = gb3[r];
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) v3 += __shfl_xor(v3, d, 64);
        if (s == 0 && 4 * g + r < SUR_OUT) atomicAdd(&grad[SUR_B3 + 4 * g + r], v3);
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) lsum += __shfl_xor(lsum, d, 64);
    if (lane == 0) atomicAdd(loss, lsum * inv_n);
}

// ---------------------------------------------------- BF16 training step
// Sum over a 16-lane row of the wave (every lane of the row gets it).
__device__ __forceinline__ float row_sum(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));  // row_ror:8
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));  // row_ror:4
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false));  // row_ror:2
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false));  // row_ror:1
    return v;
}

// Minibatch row i of Adam step `step`: splitmix64(seed + (step * 2^32 + i) * golden) mod count
// (splitmix64 as published by Steele, Lea and Flood: add the golden gamma,
// then two xor-shift-multiply rounds and a final xor-shift).
__device__ __forceinline__ int64_t batch_row(uint64_t seed, int step, int64_t i, int64_t count) {
    uint64_t z = seed + (((uint64_t)step << 32) + (uint64_t)i) * 0x9E3779B97F4A7C15ull + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (int64_t)(z % (uint64_t)count);
}

// A wave's 16 samples, [unit][sample]: one 8-byte read is an operand fragment
// of K = 16 samples (rows of 40 bytes, so 16 rows start in different banks).
constexpr int TS_LD = 20;
struct __attribute__((aligned(16))) TrainStage {
    __bf16 x[16 * TS_LD], a1[64 * TS_LD], a2[64 * TS_LD], d1[64 * TS_LD], d2[64 * TS_LD], d3[16 * TS_LD];
};

// The partial gradient of one workgroup: SUR_PARAMS gradients, then the loss.
constexpr int PART_LD = SUR_PARAMS + 4;

// Loss 1/2 |y~ - t~|^2 averaged over `batch` samples (normalised space) and
// its gradient, BF16 operands with FP32 accumulation, as one partial sum per
// workgroup in part[blockIdx.x][PART_LD].  step >= 0: the samples are rows
// batch_row(seed, step, i, count) of X and T; step < 0: rows 0 .. batch-1.
// A wave's chain of dependent MFMAs, exponentials and LDS round trips binds
// this kernel (a batch of 16,384 is one 16-sample tile per wave on every
// SIMD), so the operands are rounded to BF16 once and the rows are loaded
// straight into fragments: 14 us, and 4 us for the sum over the partials, where
// one global atomic per parameter and wave took 145 us.
template <bool VEC>
__global__ __launch_bounds__(SW) void k_sur_grad16(const float* __restrict__ th, const float* __restrict__ norm,
                                                   const float* __restrict__ X, const float* __restrict__ T,
                                                   int64_t batch, int64_t count, uint64_t seed, int step,
                                                   float* __restrict__ part) {
    __shared__ NetLds16 L;
    __shared__ NetLdsT16 LT;
    __shared__ union {
        TrainStage stage[SW / 64];
        float red[SW / 64][PART_LD];
    } u;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, s = lane & 15;
    const int64_t tiles = (batch + 15) / 16, t0 = (int64_t)blockIdx.x * (SW / 64) + w;
    const int64_t stride = (int64_t)gridDim.x * (SW / 64);
    // a tile's inputs and targets (columns 4g .. 4g+3 of sample s); the first tile's load while the
    // network is staged
    float xv[4] = {0.f, 0.f, 0.f, 0.f}, tv[4] = {0.f, 0.f, 0.f, 0.f};
    auto load_tile = [&](int64_t t) {
        const int64_t pos = 16 * t + s;
        if (pos < batch && g < 3) {
            const int64_t row = step >= 0 ? batch_row(seed, step, pos, count) : pos;
            load_row4<VEC>(X, row, g, xv);
            load_row4<VEC>(T, row, g, tv);
        }
    };
    if (t0 < tiles) load_tile(t0);
    load_net16<SW, true>(L, th, norm, &LT);
    __syncthreads();
    const float inv_n = 1.0f / (float)batch;
    TrainStage& st = u.stage[w];
    f32x4 gW1[4], gW2[4][4], gW3[4];  // gradient accumulators (D layout)
    float gb1[4][4], gb2[4][4], gb3[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        gW1[a] = f32x4{0.f, 0.f, 0.f, 0.f};
        gW3[a] = f32x4{0.f, 0.f, 0.f, 0.f};
        gb3[a] = 0.0f;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            gW2[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
            gb1[a][b] = gb2[a][b] = 0.0f;
        }
    }
    float lsum = 0.0f;
    for (int64_t t = t0; t < tiles; t += stride) {
        const bool mine = 16 * t + s < batch && g < 3;  // this lane's four columns hold data
        bf16x4h xb;
        float tt[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int f = 4 * g + j;
            xb[j] = (__bf16)(mine ? (xv[j] - L.imu[f]) / L.isd[f] : 0.0f);
            tt[j] = tv[j];
            st.x[f * TS_LD + s] = xb[j];
        }
        if (t + stride < tiles) load_tile(t + stride);
        // Every layer in K = 16 steps: a fragment of the next one is the four values that the lane holds
        // of one output tile (units 4g .. 4g+3).
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        f32x4 z[4];
        float h1[4][4], h2[4][4];
        bf16x4 hb[4];
        auto step16 = [&](const __bf16* W, int ld, int mt, int kt, const bf16x4 b, const f32x4 acc) {
            const bf16x4h a = *reinterpret_cast<const bf16x4h*>(W + (16 * mt + s) * ld + 16 * kt + 4 * g);
            return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4, a), b, acc, 0, 0, 0);
        };
        auto activate = [&](const float* bias, float h[4][4], __bf16* at) {  // tanh, staged, the next fragments
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const f32x4 b = *reinterpret_cast<const f32x4*>(bias + 16 * mt + 4 * g);
                bf16x4h hr;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    h[mt][r] = act_tanh(z[mt][r] + b[r]);
                    hr[r] = (__bf16)h[mt][r];
                    at[(16 * mt + 4 * g + r) * TS_LD + s] = hr[r];
                }
                hb[mt] = __builtin_bit_cast(bf16x4, hr);
            }
        };
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) z[mt] = step16(L.W1, 16, mt, 0, __builtin_bit_cast(bf16x4, xb), zero);
        activate(L.b1, h1, st.a1);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) z[mt] = zero;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) z[mt] = step16(L.W2, W16_LD, mt, kt, hb[kt], z[mt]);
        activate(L.b2, h2, st.a2);
        f32x4 y = zero;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) y = step16(L.W3, W16_LD, 0, kt, hb[kt], y);
        bf16x4h db;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float yr = y[r] + L.b3[4 * g + r];
            const float e = mine ? yr - (tt[r] - L.omu[4 * g + r]) / L.osd[4 * g + r] : 0.0f;
            lsum += 0.5f * e * e;
            const float d = e * inv_n;
            gb3[r] += d;
            db[r] = (__bf16)d;
            st.d3[(4 * g + r) * TS_LD + s] = db[r];
        }
        auto backward = [&](const float h[4][4], float gb[4][4], __bf16* at) {  // through tanh: (1 - h^2) z
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                bf16x4h dr;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float d = z[mt][r] * (1.0f - h[mt][r] * h[mt][r]);
                    gb[mt][r] += d;
                    dr[r] = (__bf16)d;
                    at[(16 * mt + 4 * g + r) * TS_LD + s] = dr[r];
                }
                hb[mt] = __builtin_bit_cast(bf16x4, dr);
            }
        };
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) z[mt] = step16(LT.W3T, W3T_LD, mt, 0, __builtin_bit_cast(bf16x4, db), zero);
        backward(h2, gb2, st.d2);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) z[mt] = zero;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) z[mt] = step16(LT.W2T, W16_LD, mt, kt, hb[kt], z[mt]);
        backward(h1, gb1, st.d1);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // weight gradients, samples as K: row tile of a delta times column tile of an activation
        auto frag = [&](const __bf16* a, int tile) {
            return __builtin_bit_cast(bf16x4, *reinterpret_cast<const bf16x4h*>(a + (16 * tile + s) * TS_LD + 4 * g));
        };
        const bf16x4 fx = frag(st.x, 0), fd3 = frag(st.d3, 0);
        bf16x4 fa1[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            fa1[nt] = frag(st.a1, nt);
            gW3[nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fd3, frag(st.a2, nt), gW3[nt], 0, 0, 0);
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const bf16x4 fd2 = frag(st.d2, mt);
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                gW2[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fd2, fa1[nt], gW2[mt][nt], 0, 0, 0);
            gW1[mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(frag(st.d1, mt), fx, gW1[mt], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    // the waves' sums side by side in LDS (D layout: lane holds rows 4g+r, column s), then their sum
    __syncthreads();
    float* red = u.red[w];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 16 * mt + 4 * g + r;
            if (s < SUR_IN) red[SUR_W1 + o * SUR_IN + s] = gW1[mt][r];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) red[SUR_W2 + o * SUR_H + 16 * nt + s] = gW2[mt][nt][r];
            const float v1 = row_sum(gb1[mt][r]), v2 = row_sum(gb2[mt][r]);
            if (s == 0) {
                red[SUR_B1 + o] = v1;
                red[SUR_B2 + o] = v2;
            }
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = 4 * g + r;
        const float v3 = row_sum(gb3[r]);
        if (g < 3) {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) red[SUR_W3 + o * SUR_H + 16 * nt + s] = gW3[nt][r];
            if (s == 0) red[SUR_B3 + o] = v3;
        }
    }
    lsum = row_sum(lsum);
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
    if (lane == 0) red[SUR_PARAMS] = lsum * inv_n;
    __syncthreads();
    for (int i = threadIdx.x; i <= SUR_PARAMS; i += SW) {
        float v = u.red[0][i];
#pragma unroll
        for (int k = 1; k < SW / 64; ++k) v += u.red[k][i];
        part[(int64_t)blockIdx.x * PART_LD + i] = v;
    }
}

// Sums the workgroups' partial gradients (lanes along the parameters, the 16
// waves of a workgroup along the partials) and stores the loss; ADAM: then
// steps the 64 parameters (bias-corrected moments), else stores the gradient.
constexpr int RED_WAVES = 16;
template <bool ADAM>
__global__ __launch_bounds__(64 * RED_WAVES) void k_sur_reduce(const float* __restrict__ part, int n,
                                                               float* __restrict__ th, float* __restrict__ grad,
                                                               float* __restrict__ m, float* __restrict__ v, int step,
                                                               float lr, float b1, float b2, float eps,
                                                               float* __restrict__ loss) {
    __shared__ float acc[RED_WAVES][64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int i = blockIdx.x * 64 + lane;
    float a = 0.0f;
    if (i <= SUR_PARAMS) {
#pragma unroll 8
        for (int k = w; k < n; k += RED_WAVES) a += part[(int64_t)k * PART_LD + i];
    }
    acc[w][lane] = a;
    __syncthreads();
    if (w != 0 || i > SUR_PARAMS) return;
    float gi = 0.0f;
#pragma unroll
    for (int k = 0; k < RED_WAVES; ++k) gi += acc[k][lane];
    if (i == SUR_PARAMS) {
        *loss = gi;
        return;
    }
    if constexpr (ADAM) {
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float mh = mi / (1.0f - powf(b1, (float)step));
        const float vh = vi / (1.0f - powf(b2, (float)step));
        th[i] -= lr * mh / (sqrtf(vh) + eps);
    } else {
        grad[i] = gi;
    }
}

__global__ __launch_bounds__(SW) void k_sur_zero(float* __restrict__ p, int n) {
    const int i = blockIdx.x * SW + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// Column sums of X and T [count][12] and of their squares in FP64, one
// partial per workgroup (blockIdx.y: X or T).  A thread reads groups of V
// consecutive values (V = 4 where the array is 16-byte aligned) at a stride of
// a whole number of rows, so its V columns stay the same: the arrays are read
// once, coalesced, which HBM binds (10.9M rows: 0.19 ms, 5.6 TB/s; 24
// workgroups of one column each, 48 bytes apart, took 19.4 ms).
constexpr int NORM_MAX_WG = 1536;  // workgroups per array, a multiple of 3 (threads: a multiple of 12)
template <int V>
__global__ __launch_bounds__(SW) void k_sur_norm_sums(const float* __restrict__ X, const float* __restrict__ T,
                                                      int64_t count, double* __restrict__ part) {
    static_assert(SUR_IN == 12 && SUR_OUT == 12 && (3 * SW) % 12 == 0, "rows of 12 values");
    constexpr int PER = 12 / V;  // groups per row
    typedef float vec __attribute__((ext_vector_type(V)));
    const float* A = blockIdx.y == 0 ? X : T;
    const int64_t groups = count * PER, stride = (int64_t)gridDim.x * SW;
    const int64_t first = (int64_t)blockIdx.x * SW + threadIdx.x;
    double s1[V] = {}, s2[V] = {};
    auto take = [&](const vec q) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const double a = (double)q[j];
            s1[j] += a;
            s2[j] += a * a;
        }
    };
    int64_t i = first;
    for (; i + 3 * stride < groups; i += 4 * stride) {  // four loads in flight
        vec q[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = *reinterpret_cast<const vec*>(A + (i + k * stride) * V);
#pragma unroll
        for (int k = 0; k < 4; ++k) take(q[k]);
    }
    for (; i < groups; i += stride) take(*reinterpret_cast<const vec*>(A + i * V));
    __shared__ double r1[SW][V], r2[SW][V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        r1[threadIdx.x][j] = s1[j];
        r2[threadIdx.x][j] = s2[j];
    }
    __syncthreads();
    // column c is held by the threads k with (first + k) mod PER = c / V: eight threads add a share of
    // them each (c + 12: the squares), then one the eight shares
    __shared__ double share[8][24];
    const int c24 = threadIdx.x % 24, c = c24 % 12, p = threadIdx.x / 24;
    if (p < 8) {
        const int base = (int)(((int64_t)blockIdx.x * SW) % PER);
        double sum = 0.0;
        for (int k = (c / V - base + PER) % PER + PER * p; k < SW; k += 8 * PER) sum += (c24 < 12 ? r1 : r2)[k][c % V];
        share[p][c24] = sum;
    }
    __syncthreads();
    if (threadIdx.x < 24) {
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += share[k][threadIdx.x];
        part[((int64_t)blockIdx.y * NORM_MAX_WG + blockIdx.x) * 24 + threadIdx.x] = sum;
    }
}

// Means and standard deviations (floored), one workgroup per column: from the
// n partial sums, or (ROWS) straight from the rows of X and T.  Up to NORM_ROWS
// rows that one launch is the faster way: a call takes 15.4 us against 18.4 at
// 1,000 rows, 16.8 against 18.5 at 8,000, 18.5 against 18.7 at 16,000.
constexpr int64_t NORM_ROWS = 16384;
template <bool ROWS>
__global__ __launch_bounds__(SW) void k_sur_norm(const float* __restrict__ X, const float* __restrict__ T,
                                                 const double* __restrict__ part, int n, int64_t count, float floor_sd,
                                                 float* __restrict__ norm) {
    const int y = blockIdx.x / 12, c = blockIdx.x % 12;  // inputs, then outputs
    double s1 = 0.0, s2 = 0.0;
    if constexpr (ROWS) {
        const float* A = (y == 0 ? X : T) + c;
#pragma unroll 4
        for (int k = threadIdx.x; k < (int)count; k += SW) {
            const double a = (double)A[12 * k];
            s1 += a;
            s2 += a * a;
        }
    } else {
        for (int k = threadIdx.x; k < n; k += SW) {
            const double* p = part + ((int64_t)y * NORM_MAX_WG + k) * 24 + c;
            s1 += p[0];
            s2 += p[12];
        }
    }
    __shared__ double r1[SW], r2[SW];
    r1[threadIdx.x] = s1;
    r2[threadIdx.x] = s2;
    __syncthreads();
    for (int d = SW / 2; d > 0; d >>= 1) {
        if ((int)threadIdx.x < d) {
            r1[threadIdx.x] += r1[threadIdx.x + d];
            r2[threadIdx.x] += r2[threadIdx.x + d];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double mean = r1[0] / (double)count;
        double var = r2[0] / (double)count - mean * mean;
        if (var < 0.0) var = 0.0;
        norm[24 * y + c] = (float)mean;
        norm[24 * y + 12 + c] = fmaxf((float)sqrt(var), floor_sd);
    }
}

// Training pairs: the trial state of each particle of `scene` (the deferred
// update applied when `pending`) through the exact snow return map, written
// as feature and target rows (compacted with a counter, one atomic add per
// wave for the wave's rows; rows of inverted particles are skipped).
__global__ __launch_bounds__(SW) void k_sur_sample(const float* __restrict__ S, int64_t cap, int N, Scenes T,
                                                   int scene, int pending, float E, float dt_ref, int64_t max_rows,
                                                   float* __restrict__ X, float* __restrict__ Y,
                                                   unsigned long long* __restrict__ counter) {
    const int j0 = blockIdx.x * SW + threadIdx.x;
    bool ok = j0 < N && fsid_scene(S[sidx(FSID, j0 < N ? j0 : 0, cap)]) == scene;
    const int j = ok ? j0 : 0;
    const Scene& sc = T.scene[scene];
    const Mat& M = sc.M;
    float C[9], F[9], Fh[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        C[k] = S[sidx(FC + k, j, cap)];
        F[k] = S[sidx(FF + k, j, cap)];
    }
    const float Jp = S[sidx(FS, j, cap)];
    if (pending)
        advance_gradient(C, sc.P.dt, F, Fh);
    else
#pragma unroll
        for (int k = 0; k < 9; ++k) Fh[k] = F[k];
    float U[9], sig[3], J;
    left_svd(Fh, U, sig, J);
    // descending order
    float a = sig[0], b = sig[1], c = sig[2], t;
    if (a < b) { t = a; a = b; b = t; }
    if (b < c) { t = b; b = c; c = t; }
    if (a < b) { t = a; a = b; b = t; }
    ok = ok && c > 0.0f && Jp > 0.0f;
    // the wave's rows take consecutive slots from one add to the counter
    const unsigned long long m = __ballot(ok);
    if (m == 0ull) return;
    const int lane = threadIdx.x & 63, first = __ffsll((long long)m) - 1;
    unsigned long long base = 0;
    if (lane == first) base = atomicAdd(counter, (unsigned long long)__popcll(m));
    base = ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(base >> 32), first) << 32) |
           (unsigned)__builtin_amdgcn_readlane((int)(unsigned)base, first);
    if (!ok) return;
    const float s[3] = {a, b, c};
    float sn[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) sn[k] = fminf(fmaxf(s[k], M.lo), M.hi);
    const float Js = s[0] * s[1] * s[2], Jn = sn[0] * sn[1] * sn[2];
    const float Jpn = Jp * Js / Jn;
    const float hn = expf(M.xi * (1.0f - Jpn));
    const unsigned long long r = base + (unsigned long long)__popcll(m & ((1ull << lane) - 1ull));
    if ((int64_t)r >= max_rows) return;
    float* x = X + r * SUR_IN;
    float* y = Y + r * SUR_OUT;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        x[k] = s[k];
        x[3 + k] = logf(s[k]);
        y[k] = sn[k];
        y[3 + k] = logf(sn[k] / s[k]);
        y[6 + k] = (2.0f * M.mu * hn * (sn[k] - 1.0f) * sn[k] + M.la * hn * (Jn - 1.0f) * Jn) / E;
    }
    x[6] = Jp;
    x[7] = logf(Jp);
    x[8] = expf(M.xi * (1.0f - Jp));
    x[9] = div_refined(sc.P.dt, dt_ref);  // as P2G computes it (exactly 1 at dt_ref)
    x[10] = Js;
    x[11] = 1.0f;
    y[9] = Jpn / Jp;
    y[10] = hn;
    y[11] = Jn;
}

}  // namespace

void sur_sample(hipStream_t st, const float* S, int64_t cap, int N, const Scenes& T, int scene, int pending, float E,
                float dt_ref, int64_t max_rows, float* X, float* Y, unsigned long long* counter) {
    if (N <= 0) return;
    hipLaunchKernelGGL(k_sur_sample, dim3((N + SW - 1) / SW), dim3(SW), 0, st, S, cap, N, T, scene, pending, E, dt_ref,
                       max_rows, X, Y, counter);
}

namespace {
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
}  // namespace

void sur_forward(hipStream_t st, int bf16, const float* th, const float* norm, const float* X, int64_t count,
                 float* Y) {
    if (count <= 0) return;
    const int64_t tiles = (count + 15) / 16;
    const int grid = (int)((tiles + 3) / 4 < 4096 ? (tiles + 3) / 4 : 4096);
    if (bf16) {  // the inference path P2G runs; at most the workgroups that are resident at once
        const int g16 = (int)((tiles + 3) / 4 < 2048 ? (tiles + 3) / 4 : 2048);
        if (aligned16(X) && aligned16(Y))
            hipLaunchKernelGGL(k_sur_forward16<true>, dim3(g16), dim3(SW), 0, st, th, norm, X, count, Y);
        else
            hipLaunchKernelGGL(k_sur_forward16<false>, dim3(g16), dim3(SW), 0, st, th, norm, X, count, Y);
    } else {
        hipLaunchKernelGGL(k_sur_forward, dim3(grid), dim3(SW), 0, st, th, norm, X, count, Y);
    }
}

void sur_grad_fp32(hipStream_t st, const float* th, const float* norm, const float* X, const float* T, int64_t count,
                   float* grad, float* loss) {
    hipLaunchKernelGGL(k_sur_zero, dim3((SUR_PARAMS + SW - 1) / SW), dim3(SW), 0, st, grad, SUR_PARAMS);
    hipLaunchKernelGGL(k_sur_zero, dim3(1), dim3(SW), 0, st, loss, 1);
    const int64_t tiles = (count + 15) / 16;
    const int grid = (int)((tiles + 3) / 4 < 1024 ? (tiles + 3) / 4 : 1024);
    hipLaunchKernelGGL(k_sur_grad, dim3(grid), dim3(SW), 0, st, th, norm, X, T, count, grad, loss);
}

namespace {

// One workgroup per CU at most: a wave keeps its gradient over all its tiles,
// and every further workgroup is 23 KB more for the sum over the partials.
int launch_grad16(hipStream_t st, const float* th, const float* norm, const float* X, const float* T, int64_t batch,
                  int64_t count, uint64_t seed, int step, float* part) {
    const int64_t wgs = (batch + 16 * (SW / 64) - 1) / (16 * (SW / 64));
    const int grid = (int)(wgs < SUR_MAX_PARTS ? wgs : SUR_MAX_PARTS);
    if (aligned16(X) && aligned16(T))
        hipLaunchKernelGGL(k_sur_grad16<true>, dim3(grid), dim3(SW), 0, st, th, norm, X, T, batch, count, seed, step, part);
    else
        hipLaunchKernelGGL(k_sur_grad16<false>, dim3(grid), dim3(SW), 0, st, th, norm, X, T, batch, count, seed, step, part);
    return grid;
}

constexpr int RED_GRID = (SUR_PARAMS + 64) / 64;  // the parameters and the loss, 64 per workgroup

}  // namespace

int64_t sur_workspace_bytes() {
    const int64_t parts = sizeof(float) * (int64_t)SUR_MAX_PARTS * PART_LD;
    const int64_t sums = sizeof(double) * 2 * (int64_t)NORM_MAX_WG * 24;
    return parts > sums ? parts : sums;
}

void sur_grad16(hipStream_t st, const float* th, const float* norm, const float* X, const float* T, int64_t count,
                float* grad, float* loss, void* work) {
    float* part = static_cast<float*>(work);
    const int n = launch_grad16(st, th, norm, X, T, count, count, 0, -1, part);
    hipLaunchKernelGGL(k_sur_reduce<false>, dim3(RED_GRID), dim3(64 * RED_WAVES), 0, st, part, n, nullptr, grad, nullptr,
                       nullptr, 0, 0.0f, 0.0f, 0.0f, 0.0f, loss);
}

void sur_train_step(hipStream_t st, float* th, const float* norm, const float* X, const float* T, int64_t count,
                    int batch, uint64_t seed, int step, float* m, float* v, float lr, float* loss, void* work) {
    float* part = static_cast<float*>(work);
    const int n = launch_grad16(st, th, norm, X, T, batch, count, seed, step, part);
    hipLaunchKernelGGL(k_sur_reduce<true>, dim3(RED_GRID), dim3(64 * RED_WAVES), 0, st, part, n, th, nullptr, m, v,
                       step + 1, lr, 0.9f, 0.999f, 1e-8f, loss);
}

void sur_zero(hipStream_t st, float* p, int n) {
    if (n > 0) hipLaunchKernelGGL(k_sur_zero, dim3((n + SW - 1) / SW), dim3(SW), 0, st, p, n);
}

void sur_norm(hipStream_t st, const float* X, const float* T, int64_t count, float* norm, void* work) {
    double* part = static_cast<double*>(work);
    if (count <= NORM_ROWS) {
        hipLaunchKernelGGL(k_sur_norm<true>, dim3(SUR_IN + SUR_OUT), dim3(SW), 0, st, X, T, part, 0, count, 1e-6f, norm);
        return;
    }
    const bool vec = aligned16(X) && aligned16(T);
    const int64_t groups = count * (vec ? 3 : 12), wgs = (groups + 3 * SW - 1) / (3 * SW) * 3;
    const int grid = (int)(wgs < NORM_MAX_WG ? wgs : NORM_MAX_WG);
    if (vec)
        hipLaunchKernelGGL(k_sur_norm_sums<4>, dim3(grid, 2), dim3(SW), 0, st, X, T, count, part);
    else
        hipLaunchKernelGGL(k_sur_norm_sums<1>, dim3(grid, 2), dim3(SW), 0, st, X, T, count, part);
    hipLaunchKernelGGL(k_sur_norm<false>, dim3(SUR_IN + SUR_OUT), dim3(SW), 0, st, X, T, part, grid, count, 1e-6f, norm);
}

}  // namespace mpm
