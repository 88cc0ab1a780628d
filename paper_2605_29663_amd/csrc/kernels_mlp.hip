// Learned sampling proposal: feature extraction, bf16 matrix-core GEMMs with
// fused epilogues, loss, bias gradients, Adam and weight conversion.
//
// Network: features (64-bin polar range histogram, goal in the robot frame,
// previous control sequence) -> Linear -> GELU -> Linear -> GELU -> Linear ->
// mean control sequence (normalised units).  bf16 operands on the gfx950
// matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulation, fp32 master
// weights and Adam moments.
#include "devmath.hpp"
#include "mlp.hpp"

namespace emppi {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t to_bf16(float x) {
    const uint32_t u = __float_as_uint(x);
    return static_cast<uint16_t>((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// GELU with the exact error function and its derivative.
__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float x) {
    return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) +
           x * 0.39894228040143268f * expf(-0.5f * x * x);
}

// Normalised network output y at (state m, sequence entry k) -> control in
// the actuator box: u = clamp(mid + half y, u_min, u_max) of its channel.  In
// residual mode (res_scale > 0) the output is added to the previous
// sequence's scaled value carried in the features: ys = feat_U + res_scale y.
__device__ __forceinline__ float control_of(float y, const float* __restrict__ feat, int m, int k,
                                            const FeatArgs& F) {
    const int ch = k % F.nu;
    const float ys = F.res_scale > 0.0f
                         ? __builtin_fmaf(F.res_scale, y, feat[static_cast<size_t>(m) * F.in_dim + FEAT_BINS + 2 + k])
                         : y;
    const float mid = (F.umax[ch] + F.umin[ch]) * 0.5f;
    const float half = (F.umax[ch] - F.umin[ch]) * 0.5f;
    return fminf(fmaxf(mid + half * ys, F.umin[ch]), F.umax[ch]);
}

// ---------------------------------------------------------------- features
// One workgroup per state.  Points go to the robot frame at q0 (rotation by
// the single-precision sin/cos sequence), the bin is a pseudo-angle built from
// correctly rounded divisions only (quadrant q, t in [0,1], bin = 16 q +
// min(15, floor(16 t))), the range is the correctly rounded square root; the
// per-bin minimum is an LDS atomicMin on the bits of the non-negative float.
__global__ __launch_bounds__(1024) void k_features(const float* __restrict__ px,
                                                   const float* __restrict__ py,
                                                   const int* __restrict__ n_valid,
                                                   const float* __restrict__ q0s,
                                                   const float* __restrict__ U_prev, FeatArgs F,
                                                   float* __restrict__ feat) {
    __shared__ unsigned int hist[FEAT_BINS];
    const int state = blockIdx.x;
    const float* q0 = q0s + 3 * state;
    const float* Up = U_prev + static_cast<size_t>(state) * F.T * F.nu;
    float* out = feat + static_cast<size_t>(state) * F.in_dim;
    for (int b = threadIdx.x; b < FEAT_BINS; b += blockDim.x) hist[b] = __float_as_uint(F.r_max);
    __syncthreads();
    float s, c;
    seq_sincos(q0[2], s, c);
    const int nv = *n_valid;
    for (int i = threadIdx.x; i < nv; i += blockDim.x) {
        const float dx = px[i] - q0[0], dy = py[i] - q0[1];
        const float x = c * dx + s * dy;
        const float y = c * dy - s * dx;
        int q;
        float t;
        if (y >= 0.0f) {
            if (x >= 0.0f) {
                q = 0;
                t = (x == 0.0f && y == 0.0f) ? 0.0f : y / (x + y);
            } else {
                q = 1;
                t = -x / (y - x);
            }
        } else {
            if (x < 0.0f) {
                q = 2;
                t = -y / (-x - y);
            } else {
                q = 3;
                t = x / (x - y);
            }
        }
        const int bin = q * 16 + min(15, static_cast<int>(t * 16.0f));
        const float r = seq_sqrt(x * x + y * y);
        // neighbouring points share bins (the set is in spatial order), so a
        // read first spares most of the atomics: a bin's minimum only falls
        const unsigned int rb = __float_as_uint(fminf(r, F.r_max));
        if (rb < *static_cast<volatile unsigned int*>(&hist[bin])) atomicMin(&hist[bin], rb);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < FEAT_BINS; b += blockDim.x) out[b] = __uint_as_float(hist[b]) / F.r_max;
    if (threadIdx.x == 0) {
        const float gx = F.goal[0] - q0[0], gy = F.goal[1] - q0[1];
        out[FEAT_BINS] = (c * gx + s * gy) / F.r_max;
        out[FEAT_BINS + 1] = (c * gy - s * gx) / F.r_max;
    }
    for (int k = threadIdx.x; k < F.T * F.nu; k += blockDim.x) {
        const int ch = k % F.nu;
        const float mid = (F.umax[ch] + F.umin[ch]) * 0.5f;
        const float half = (F.umax[ch] - F.umin[ch]) * 0.5f;
        out[FEAT_BINS + 2 + k] = half > 0.0f ? (Up[k] - mid) / half : 0.0f;
    }
}

// ---------------------------------------------------------------- products
// C[M x N] = A[M x K] B[N x K]^T by waves of W x W blocks of
// v_mfma_f32_16x16x32_bf16, each wave on its own: both operands are stored
// k-contiguous (the producers write transposed copies where a product sums
// over the batch), so a lane's 8 consecutive k values are one 16-byte load
// from the L1 / L2 and no LDS staging, barrier or index arithmetic stands in
// the loop.  The products of this network are small (1024 x 256 x 256 is 0.13
// GFLOP) and bound by latency: what counts is one round of loads in flight
// and a short chain of launches.  A training step of 1024 rows (in 146,
// hidden 256, out 80) takes 7 launches; with 64 x 64 tiles staged element by
// element and one launch per product it took 18 and 480 us.  Lane l of the
// instruction holds A rows l % 16, k = 8 (l / 16) .. +7, B rows l % 16 with the
// same k, and D rows 4 (l / 16) .. +3 of column l % 16; k ascends in steps of
// 32, so every sum has one order whatever the tiles.
template <int W>
__device__ __forceinline__ void product_wave(const MlpJob& g, int tm, int tn) {
    const int l = threadIdx.x & (WAVE - 1), r = l & 15, kq = (l >> 4) * 8;
    const int m0 = tm * 16 * W, n0 = tn * 16 * W;
    f32x4 acc[W][W];
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // rows past the end read the last row (their results are not stored)
    const uint16_t* pb[W];
#pragma unroll
    for (int j = 0; j < W; ++j) pb[j] = g.B + static_cast<size_t>(min(n0 + 16 * j + r, g.N - 1)) * g.ldb + kq;
    // what the epilogue reads, on its way before the operands
    float ext[W][W][4], bias[W];
    const float* side = g.kind == EPI_GELU_GRAD ? g.aux : g.tgt;
#pragma unroll
    for (int j = 0; j < W; ++j) {
        const int n = min(n0 + 16 * j + r, g.N - 1);
        bias[j] = g.bias ? g.bias[n] : 0.f;
        if (side)
#pragma unroll
            for (int i = 0; i < W; ++i)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int m = min(m0 + 16 * i + 4 * (l >> 4) + t, g.M - 1);
                    ext[i][j][t] = side[static_cast<size_t>(m) * g.N + n];
                }
    }
    // S steps are loaded as one round and consumed while the next round is on
    // its way; steps past K load the last one and are skipped
    constexpr int S = 8 / W;
    bf16x8 a[2][S][W], b[2][S][W];
    const int kend = (g.K + 31) & ~31;
    auto consume = [&](int buf, int k0) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (k0 + 32 * s >= kend) break;
#pragma unroll
            for (int i = 0; i < W; ++i)
#pragma unroll
                for (int j = 0; j < W; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[buf][s][i], b[buf][s][j], acc[i][j], 0, 0, 0);
        }
    };
    if (g.A32) {
        const bool store = tn == 0;
        for (int k0 = 0; k0 < kend; k0 += 32 * S) {
            float x[S][W][8];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int k = min(k0 + 32 * s, kend - 32);
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    const float* pa = g.A32 + static_cast<size_t>(min(m0 + 16 * i + r, g.M - 1)) * g.K;
                    if (k + 32 <= g.K) {
                        __builtin_memcpy(x[s][i], pa + k + kq, 32);  // two 16-byte loads, 4-byte aligned
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) x[s][i][e] = pa[min(k + kq + e, g.K - 1)];
                    }
                }
#pragma unroll
                for (int j = 0; j < W; ++j) b[0][s][j] = *reinterpret_cast<const bf16x8*>(pb[j] + k);
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int k = k0 + 32 * s + kq;
                if (k0 + 32 * s >= kend) break;
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    const int m = m0 + 16 * i + r;
                    union {
                        uint16_t h[8];
                        bf16x8 v;
                        uint4 q;
                    } u;
#pragma unroll
                    for (int e = 0; e < 8; ++e) u.h[e] = k + e < g.K ? to_bf16(x[s][i][e]) : 0;
                    a[0][s][i] = u.v;
                    if (store && m < g.M) *reinterpret_cast<uint4*>(g.xb + static_cast<size_t>(m) * g.lda + k) = u.q;
                }
            }
            consume(0, k0);
        }
    } else {
        const uint16_t* pa[W];
#pragma unroll
        for (int i = 0; i < W; ++i) pa[i] = g.A + static_cast<size_t>(min(m0 + 16 * i + r, g.M - 1)) * g.lda + kq;
        auto fetch = [&](int buf, int k0) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int k = min(k0 + 32 * s, kend - 32);
#pragma unroll
                for (int i = 0; i < W; ++i) a[buf][s][i] = *reinterpret_cast<const bf16x8*>(pa[i] + k);
#pragma unroll
                for (int j = 0; j < W; ++j) b[buf][s][j] = *reinterpret_cast<const bf16x8*>(pb[j] + k);
            }
        };
        fetch(0, 0);
        for (int k0 = 0; k0 < kend; k0 += 64 * S) {
            if (k0 + 32 * S < kend) fetch(1, k0 + 32 * S);
            consume(0, k0);
            if (k0 + 32 * S >= kend) break;
            if (k0 + 64 * S < kend) fetch(0, k0 + 64 * S);
            consume(1, k0 + 32 * S);
        }
    }
    const float scale = 2.0f / (static_cast<float>(g.M) * static_cast<float>(g.N));
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const int n = n0 + 16 * j + r, mq = m0 + 16 * i + 4 * (l >> 4);
            if (n >= g.N) continue;
            uint16_t h[4] = {0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int m = mq + t;
                if (m >= g.M) continue;
                const size_t o = static_cast<size_t>(m) * g.N + n;
                const float v = acc[i][j][t];
                switch (g.kind) {
                case EPI_STORE:
                    g.C[o] = v;
                    break;
                case EPI_BIAS: {
                    const float y = v + bias[j];
                    g.C[o] = y;
                    if (g.C2) g.C2[o] = y;
                    if (g.tgt) {
                        const float d = scale * (y - ext[i][j][t]);
                        g.dout[o] = d;
                        h[t] = to_bf16(d);
                    }
                    if (g.U) g.U[o] = control_of(y, g.feat, m, n, g.F);
                    break;
                }
                case EPI_BIAS_GELU: {
                    const float pre = v + bias[j];
                    g.C[o] = pre;
                    h[t] = to_bf16(gelu(pre));
                    break;
                }
                default: {  // EPI_GELU_GRAD
                    const float d = v * gelu_grad(ext[i][j][t]);
                    g.C[o] = d;
                    h[t] = to_bf16(d);
                    break;
                }
                }
                if (g.Cb) g.Cb[static_cast<size_t>(m) * g.ldcb + n] = h[t];
            }
            // rows past M up to the transposed copy's padding are zero
            if (g.Ct && mq < ((g.M + 31) & ~31)) {
                const uint2 q = make_uint2(h[0] | (static_cast<unsigned>(h[1]) << 16),
                                           h[2] | (static_cast<unsigned>(h[3]) << 16));
                *reinterpret_cast<uint2*>(g.Ct + static_cast<size_t>(n) * g.ldt + mq) = q;
            }
        }
}

// Column sums over the batch (bias gradients), fixed order: COLSUM_GROUPS row
// groups; group g adds rows g, g + COLSUM_GROUPS, ... in turn, and the group
// partials are added in group order.  A workgroup holds 16 columns x 16
// groups.
constexpr int COLSUM_GROUPS = 16;

__device__ __forceinline__ void colsum_block(const MlpJob& g, int block) {
    __shared__ float sh[COLSUM_GROUPS][16];
    const int c = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int n = block * 16 + c;
    float s = 0.f;
    if (n < g.N) {
        constexpr int R = 32;  // loads in flight
        int m = grp;
        for (; m + (R - 1) * COLSUM_GROUPS < g.M; m += R * COLSUM_GROUPS) {
            float x[R];
#pragma unroll
            for (int t = 0; t < R; ++t) x[t] = g.aux[static_cast<size_t>(m + t * COLSUM_GROUPS) * g.N + n];
#pragma unroll
            for (int t = 0; t < R; ++t) s += x[t];
        }
        for (; m < g.M; m += COLSUM_GROUPS) s += g.aux[static_cast<size_t>(m) * g.N + n];
    }
    sh[grp][c] = s;
    __syncthreads();
    if (grp == 0 && n < g.N) {
        float t = sh[0][c];
#pragma unroll
        for (int k = 1; k < COLSUM_GROUPS; ++k) t += sh[k][c];
        g.C[n] = t;
    }
}

// Ct[N][ldt] = bf16(aux[M][N])^T, 32 x 32 a workgroup through the LDS.
__device__ __forceinline__ void transpose_block(const MlpJob& g, int block) {
    __shared__ uint16_t sh[32][33];
    const int tm = block / g.tiles_n, m0 = tm * 32, n0 = (block - tm * g.tiles_n) * 32;
    const int c = threadIdx.x & 31, r = threadIdx.x >> 5;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + r + 8 * i, n = n0 + c;
        sh[r + 8 * i][c] = m < g.M && n < g.N ? to_bf16(g.aux[static_cast<size_t>(m) * g.N + n]) : 0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int n = n0 + r + 8 * i;
        if (n < g.N) g.Ct[static_cast<size_t>(n) * g.ldt + m0 + c] = sh[c][r + 8 * i];
    }
}

// The jobs of one launch side by side, each with a range of workgroups.
__global__ __launch_bounds__(256) void k_mlp(MlpJobs jobs) {
    int j = 0;
    while (j + 1 < jobs.n && static_cast<int>(blockIdx.x) >= jobs.job[j + 1].block0) ++j;
    const MlpJob& g = jobs.job[j];
    const int block = static_cast<int>(blockIdx.x) - g.block0;
    if (g.kind == JOB_COLSUM) {
        colsum_block(g, block);
        return;
    }
    if (g.kind == JOB_TRANSPOSE) {
        transpose_block(g, block);
        return;
    }
    const int t = block * 4 + static_cast<int>(threadIdx.x) / WAVE;
    const int tm = t / g.tiles_n;
    if (tm >= g.tiles_m) return;
    if (g.W == 2)
        product_wave<2>(g, tm, t - tm * g.tiles_n);
    else
        product_wave<1>(g, tm, t - tm * g.tiles_n);
}

// ---------------------------------------------------------------- loss
// Squared error of each row of the output.
__global__ void k_row_sq(const float* __restrict__ out, const float* __restrict__ tgt, int n_out,
                         float* __restrict__ row_sq) {
    const int m = blockIdx.x;
    float acc = 0.f;
    for (int j = threadIdx.x; j < n_out; j += blockDim.x) {
        const size_t o = static_cast<size_t>(m) * n_out + j;
        const float e = out[o] - tgt[o];
        acc += e * e;
    }
    // fixed-order block sum (binary tree; blockDim.x is 256)
    __shared__ float sh[256];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) row_sq[m] = sh[0];
}

// Loss = sum of the row sums / (M n_out), fixed order: thread t adds rows
// t, t + 1024, ... in turn, then a fixed binary tree over the 1024 partials.
constexpr int LOSS_THREADS = 1024;

__global__ __launch_bounds__(LOSS_THREADS) void k_loss_sum(const float* __restrict__ row_sq, int M,
                                                           int n_out, float* __restrict__ loss) {
    __shared__ float sh[LOSS_THREADS];
    float s = 0.f;
    for (int m = threadIdx.x; m < M; m += LOSS_THREADS) s += row_sq[m];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = LOSS_THREADS / 2; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = sh[0] / (static_cast<float>(M) * static_cast<float>(n_out));
}

// ---------------------------------------------------------------- Adam
// The bf16 copies of parameter i (matrices only; MlpWeights).
__device__ __forceinline__ void store_weight(const MlpWeights& mw, long i, float w) {
    const uint16_t h = to_bf16(w);
    if (i < mw.off[1]) {
        const int k = static_cast<int>(i) / mw.H, n = static_cast<int>(i) % mw.H;
        mw.w1t[static_cast<size_t>(n) * mw.ld_in + k] = h;
    } else if (i >= mw.off[2] && i < mw.off[3]) {
        const int j = static_cast<int>(i - mw.off[2]), k = j / mw.H, n = j % mw.H;
        mw.w2t[static_cast<size_t>(n) * mw.ld_h + k] = h;
        mw.w2[static_cast<size_t>(k) * mw.ld_h + n] = h;
    } else if (i >= mw.off[4] && i < mw.off[5]) {
        const int j = static_cast<int>(i - mw.off[4]), k = j / mw.out, n = j % mw.out;
        mw.w3t[static_cast<size_t>(n) * mw.ld_h + k] = h;
        mw.w3[static_cast<size_t>(k) * mw.ld_out + n] = h;
    }
}

// w -= lr * mhat / (sqrt(vhat) + eps), mhat = m / (1 - b1^t), vhat = v / (1 - b2^t).
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ grad, float* __restrict__ m,
                       float* __restrict__ v, long n, AdamArgs a, MlpWeights mw) {
    const long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = grad[i];
    const float mi = a.b1 * m[i] + a.ob1 * g;
    const float vi = a.b2 * v[i] + a.ob2 * (g * g);
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / a.c1, vh = vi / a.c2;
    const float wi = w[i] - a.lr * mh / (sqrtf(vh) + a.eps);
    w[i] = wi;
    store_weight(mw, i, wi);
}

__global__ void k_weights(const float* __restrict__ w, long n, MlpWeights mw) {
    const long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) store_weight(mw, i, w[i]);
}

// Control sequences -> normalised training targets: y = (u - mid) / half.
// (residual mode: y = (ys - feat_U) / res_scale)
__global__ void k_normalize(const float* __restrict__ U, const float* __restrict__ feat, int M,
                            int T, int nu, FeatArgs F, float* __restrict__ y) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M * T * nu) return;
    const int ch = i % nu;
    const int m = i / (T * nu), k = i % (T * nu);
    const float mid = (F.umax[ch] + F.umin[ch]) * 0.5f;
    const float half = (F.umax[ch] - F.umin[ch]) * 0.5f;
    const float ys = half > 0.0f ? (U[i] - mid) / half : 0.0f;
    y[i] = F.res_scale > 0.0f
               ? (ys - feat[static_cast<size_t>(m) * F.in_dim + FEAT_BINS + 2 + k]) / F.res_scale
               : ys;
}

}  // namespace

hipError_t launch_normalize(const float* U, const float* feat, int M, int T, int nu,
                            const FeatArgs& F, float* y, hipStream_t s) {
    const int n = M * T * nu;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_normalize, dim3((n + 255) / 256), dim3(256), 0, s, U, feat, M, T, nu, F, y);
    return hipGetLastError();
}

hipError_t launch_features(const float* px, const float* py, const int* n_valid, const float* q0s,
                           const float* U_prev, const FeatArgs& F, int n_states, float* feat,
                           hipStream_t s) {
    if (n_states <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_features, dim3(n_states), dim3(1024), 0, s, px, py, n_valid, q0s, U_prev, F,
                       feat);
    return hipGetLastError();
}

hipError_t launch_mlp(MlpJobs& jobs, hipStream_t s) {
    int blocks = 0;
    for (int j = 0; j < jobs.n; ++j) {
        MlpJob& g = jobs.job[j];
        g.block0 = blocks;
        if (g.kind == JOB_COLSUM) {
            blocks += (g.N + 15) / 16;
            continue;
        }
        if (g.kind == JOB_TRANSPOSE) {
            g.tiles_n = (g.N + 31) / 32;
            blocks += (g.M + 31) / 32 * g.tiles_n;
            continue;
        }
        // 32 x 32 per wave (half the operand traffic) once that gives every
        // SIMD of the chip a wave, 16 x 16 below (four times the waves).  The
        // forward pass of 32768 rows (hidden 256) takes 148 us with the one and
        // 224 with the other, of 4096 rows 38 and 42, of 2048 rows 43 and 32.
        g.W = static_cast<long>((g.M + 31) / 32) * ((g.N + 31) / 32) >= 1024 ? 2 : 1;
        // whole steps of 32 rows: the transposed copies are zero up to there
        g.tiles_m = (g.M + 31) / 32 * 2 / g.W;
        g.tiles_n = (g.N + 16 * g.W - 1) / (16 * g.W);
        const long t = static_cast<long>(g.tiles_m) * g.tiles_n;
        blocks += static_cast<int>((t + 3) / 4);
    }
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp, dim3(blocks), dim3(256), 0, s, jobs);
    return hipGetLastError();
}

hipError_t launch_loss(const float* out, const float* tgt, int M, int n_out, float* row_sq, float* loss,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_row_sq, dim3(M), dim3(256), 0, s, out, tgt, n_out, row_sq);
    hipLaunchKernelGGL(k_loss_sum, dim3(1), dim3(LOSS_THREADS), 0, s, row_sq, M, n_out, loss);
    return hipGetLastError();
}

hipError_t launch_adam(float* w, const float* grad, float* m, float* v, long n, const AdamArgs& a,
                       const MlpWeights& mw, hipStream_t s) {
    hipLaunchKernelGGL(k_adam, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, w,
                       grad, m, v, n, a, mw);
    return hipGetLastError();
}

hipError_t launch_weights(const float* w, long n, const MlpWeights& mw, hipStream_t s) {
    hipLaunchKernelGGL(k_weights, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, w, n, mw);
    return hipGetLastError();
}

}  // namespace emppi
