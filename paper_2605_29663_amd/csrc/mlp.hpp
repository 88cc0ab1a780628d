// Internal interface of the learned-proposal kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace emppi {

constexpr int FEAT_BINS = 64;  // polar range histogram bins

// Feature / output scaling of one proposal.
struct FeatArgs {
    int T, nu, in_dim;
    float r_max;             // histogram range clip (m); also scales the goal
    float goal[2];
    float umin[3], umax[3];  // control box: features and outputs use (u - mid) / half
    float res_scale;         // > 0: the output is a residual on the previous sequence
};

enum { EPI_STORE = 0, EPI_BIAS = 1, EPI_BIAS_GELU = 2, EPI_GELU_GRAD = 3, JOB_COLSUM = 4, JOB_TRANSPOSE = 5 };

// One product of a launch (or a column sum, or a transposed copy): C[M x N] = A[M x K] B[N x K]^T,
// both operands bf16 with k contiguous, rows of lda / ldb elements (multiples
// of 32) that are zero from K to the next multiple of 32.
struct MlpJob {
    int kind;                // EPI_* (product and its epilogue) or JOB_*
    int M, N, K;
    const uint16_t* A;
    const float* A32;        // not null: A is this fp32 matrix [M][K], rounded on the way in
    uint16_t* xb;            // A32: bf16 copy [M][lda] to store
    const uint16_t* B;
    int lda, ldb;
    float* C;                // fp32 output, [M][N]
    float* C2;               // EPI_BIAS: second copy, or nullptr
    uint16_t* Cb;            // bf16 output [M][ldcb], or nullptr
    uint16_t* Ct;            // bf16 output transposed [N][ldt], zero up to the next multiple of 32 of M, or nullptr
    int ldcb, ldt;
    const float* bias;       // EPI_BIAS, EPI_BIAS_GELU
    const float* aux;        // EPI_GELU_GRAD: pre-activation; JOB_*: the matrix [M][N] to sum or copy
    const float* tgt;        // EPI_BIAS, not null: dout = 2 (C - tgt) / (M N) goes to dout, Cb and Ct
    float* dout;
    float* U;                // EPI_BIAS, not null: the output as a control sequence (feat: the features)
    const float* feat;
    FeatArgs F;
    int W, tiles_m, tiles_n, block0;  // set by launch_mlp: 16 W x 16 W results a wave
};
constexpr int MLP_JOBS = 4;
struct MlpJobs {
    MlpJob job[MLP_JOBS];
    int n;
};

struct AdamArgs {
    // decay rates b1, b2 and their complements ob1 = 1 - b1, ob2 = 1 - b2 (formed in
    // double, so that at t = 1 the moment scale and the bias correction cancel exactly);
    // c1 = 1 - b1^t, c2 = 1 - b2^t
    float lr, b1, b2, ob1, ob2, eps, c1, c2;
};

hipError_t launch_features(const float* px, const float* py, const int* n_valid, const float* q0s,
                           const float* U_prev, const FeatArgs& F, int n_states, float* feat,
                           hipStream_t s);
hipError_t launch_mlp(MlpJobs& jobs, hipStream_t s);
hipError_t launch_loss(const float* out, const float* tgt, int M, int n_out, float* row_sq, float* loss,
                       hipStream_t s);
// The parameter vector's matrices as the products read them: bf16,
// transposed ([n][k]) for the forward pass and as they are for the backward
// pass, rows padded to multiples of 32.
struct MlpWeights {
    int in, H, out;
    long off[6];
    uint16_t *w1t, *w2t, *w3t, *w2, *w3;
    int ld_in, ld_h, ld_out;
};
hipError_t launch_adam(float* w, const float* grad, float* m, float* v, long n, const AdamArgs& a,
                       const MlpWeights& mw, hipStream_t s);
hipError_t launch_weights(const float* w, long n, const MlpWeights& mw, hipStream_t s);
hipError_t launch_normalize(const float* U, const float* feat, int M, int T, int nu, const FeatArgs& F, float* y,
                            hipStream_t s);
}  // namespace emppi
