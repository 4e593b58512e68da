// Layout of the constitutive surrogate's parameters and normalisation, and
// the launchers of its kernels (mpm_surrogate.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mpm {

// MLP 12 -> 64 -> 64 -> 12.  Flat FP32 parameters, weights row-major
// (output, input): W1 [64][12], b1 [64], W2 [64][64], b2 [64], W3 [12][64], b3 [12].
constexpr int SUR_IN = 12, SUR_H = 64, SUR_OUT = 12;
constexpr int SUR_W1 = 0;
constexpr int SUR_B1 = SUR_W1 + SUR_H * SUR_IN;
constexpr int SUR_W2 = SUR_B1 + SUR_H;
constexpr int SUR_B2 = SUR_W2 + SUR_H * SUR_H;
constexpr int SUR_W3 = SUR_B2 + SUR_H;
constexpr int SUR_B3 = SUR_W3 + SUR_OUT * SUR_H;
constexpr int SUR_PARAMS = SUR_B3 + SUR_OUT;  // 5772
// Normalisation: input means [12], input sds [12], output means [12], output sds [12].
constexpr int SUR_NORM = 2 * (SUR_IN + SUR_OUT);

// Features of a trial state (descending singular values s, plastic volume
// J_P): [s1..s3, ln s1..s3, J_P, ln J_P, exp(xi (1 - J_P)), dt/dt_ref, s1 s2 s3, 1].
// Targets: [s'1..s'3, ln(s'/s)1..3, tau1..3 / E, J_P'/J_P, exp(xi (1 - J_P')), s'1 s'2 s'3].

void sur_forward(hipStream_t st, int bf16, const float* th, const float* norm, const float* X, int64_t count,
                 float* Y);
// Loss and gradient over the rows of X and T: FP32 operands, or BF16 operands.  `work`:
// sur_workspace_bytes() of device memory, owned by the caller, free again when the call's work has run.
constexpr int SUR_MAX_PARTS = 256;  // workgroups of the BF16 gradient
int64_t sur_workspace_bytes();
void sur_grad_fp32(hipStream_t st, const float* th, const float* norm, const float* X, const float* T, int64_t count,
                   float* grad, float* loss);
void sur_grad16(hipStream_t st, const float* th, const float* norm, const float* X, const float* T, int64_t count,
                float* grad, float* loss, void* work);
// Adam step `step` (from 0) on a minibatch of `batch` rows drawn by (seed, step); the batch's loss into *loss.
void sur_train_step(hipStream_t st, float* th, const float* norm, const float* X, const float* T, int64_t count,
                    int batch, uint64_t seed, int step, float* m, float* v, float lr, float* loss, void* work);
void sur_zero(hipStream_t st, float* p, int n);
void sur_norm(hipStream_t st, const float* X, const float* T, int64_t count, float* norm, void* work);
struct Scenes;
void sur_sample(hipStream_t st, const float* S, int64_t cap, int N, const Scenes& T, int scene, int pending, float E,
                float dt_ref, int64_t max_rows, float* X, float* Y, unsigned long long* counter);

}  // namespace mpm
