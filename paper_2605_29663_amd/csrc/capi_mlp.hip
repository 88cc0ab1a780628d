// C ABI of the learned sampling proposal (declared in include/exact_mppi.h):
// parameters, features, forward pass, training step (hand-written forward and
// backward GEMMs on the matrix cores, Adam), save / load.
#include <cstdio>

#include "ctx.hpp"
#include "mlp.hpp"

using namespace emppi;
using namespace emppi_host;

struct mppi_proposal_s {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string err;
    int T = 0, nu = 0, in = 0, H = 0, out = 0, max_batch = 0;
    long long n_params = 0;
    long long off[6] = {0};  // W1, b1, W2, b2, W3, b3 in the flat parameter vector
    DevBuf w, g, m, v;       // fp32 master parameters, gradients, Adam moments
    DevBuf w1t, w2t, w3t, w2b, w3b;    // bf16 weight copies (MlpWeights)
    int ld_in = 0, ld_h = 0, ld_out = 0, ld_m = 0;  // padded rows of the bf16 matrices
    DevBuf xt, a1t, a2t, doutt, dh2t, dh1t;  // bf16, transposed over the batch: [cols][ld_m]
    DevBuf xb, pre1, a1b, pre2, a2b, outb, dout, doutb, dh2, dh2b, dh1, dh1b, rowsq, loss;
    float* h_loss = nullptr;  // pinned
    long long t = 0;          // Adam step
    FeatArgs F{};
};

namespace {

int pfail(mppi_proposal p, int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (p)
        p->err = buf;
    else
        g_create_error = buf;
    return code;
}

#define PHIP(p, expr)                                                                         \
    do {                                                                                      \
        hipError_t _e = (expr);                                                               \
        if (_e != hipSuccess)                                                                 \
            return pfail((p), MPPI_E_HIP, "%s failed: %s", #expr, hipGetErrorString(_e));     \
    } while (0)

float* W(mppi_proposal p, DevBuf& b, int k) { return b.as<float>() + p->off[k]; }

MlpWeights weights(mppi_proposal p) {
    MlpWeights mw{};
    mw.in = p->in;
    mw.H = p->H;
    mw.out = p->out;
    for (int k = 0; k < 6; ++k) mw.off[k] = static_cast<long>(p->off[k]);
    mw.w1t = p->w1t.as<uint16_t>();
    mw.w2t = p->w2t.as<uint16_t>();
    mw.w3t = p->w3t.as<uint16_t>();
    mw.w2 = p->w2b.as<uint16_t>();
    mw.w3 = p->w3b.as<uint16_t>();
    mw.ld_in = p->ld_in;
    mw.ld_h = p->ld_h;
    mw.ld_out = p->ld_out;
    return mw;
}

int refresh_bf16(mppi_proposal p) {
    PHIP(p, launch_weights(p->w.as<float>(), static_cast<long>(p->n_params), weights(p), p->stream));
    return MPPI_OK;
}

// C = A B^T of bf16 matrices with padded rows; the epilogue's fields are the
// caller's.
MlpJob product(int kind, int M, int N, int K, const DevBuf& A, int lda, const DevBuf& B, int ldb, float* C) {
    MlpJob g{};
    g.kind = kind;
    g.M = M;
    g.N = N;
    g.K = K;
    g.A = A.as<uint16_t>();
    g.lda = lda;
    g.B = B.as<uint16_t>();
    g.ldb = ldb;
    g.C = C;
    return g;
}

MlpJob colsum(int M, int N, const float* d, float* out) {
    MlpJob g{};
    g.kind = JOB_COLSUM;
    g.M = M;
    g.N = N;
    g.aux = d;
    g.C = out;
    return g;
}

int run_jobs(mppi_proposal p, std::initializer_list<MlpJob> list) {
    MlpJobs j{};
    for (const MlpJob& g : list) j.job[j.n++] = g;
    PHIP(p, launch_mlp(j, p->stream));
    return MPPI_OK;
}

// Forward pass of M feature rows (device fp32, M x in) into p->outb (M x out),
// and where asked for a copy of the output, the output as control sequences,
// or (training) the transposed activations and the gradient of the loss.
int forward(mppi_proposal p, const float* dfeat, int M, float* copy, float* dU, const float* dtarget) {
    const int in = p->in, H = p->H, O = p->out;
    const bool train = dtarget != nullptr;
    MlpJob g = product(EPI_BIAS_GELU, M, H, in, p->xb, p->ld_in, p->w1t, p->ld_in, p->pre1.as<float>());
    g.A32 = dfeat;
    g.xb = p->xb.as<uint16_t>();
    g.bias = W(p, p->w, 1);
    g.Cb = p->a1b.as<uint16_t>();
    g.ldcb = p->ld_h;
    g.Ct = train ? p->a1t.as<uint16_t>() : nullptr;
    g.ldt = p->ld_m;
    if (int rc = run_jobs(p, {g})) return rc;
    g = product(EPI_BIAS_GELU, M, H, H, p->a1b, p->ld_h, p->w2t, p->ld_h, p->pre2.as<float>());
    g.bias = W(p, p->w, 3);
    g.Cb = p->a2b.as<uint16_t>();
    g.ldcb = p->ld_h;
    g.Ct = train ? p->a2t.as<uint16_t>() : nullptr;
    g.ldt = p->ld_m;
    MlpJob xt{};
    xt.kind = JOB_TRANSPOSE;
    xt.M = M;
    xt.N = in;
    xt.aux = dfeat;
    xt.Ct = p->xt.as<uint16_t>();
    xt.ldt = p->ld_m;
    if (int rc = train ? run_jobs(p, {g, xt}) : run_jobs(p, {g})) return rc;
    g = product(EPI_BIAS, M, O, H, p->a2b, p->ld_h, p->w3t, p->ld_h, p->outb.as<float>());
    g.bias = W(p, p->w, 5);
    g.C2 = copy;
    g.U = dU;
    g.feat = dfeat;
    g.F = p->F;
    if (train) {
        g.tgt = dtarget;
        g.dout = p->dout.as<float>();
        g.Cb = p->doutb.as<uint16_t>();
        g.ldcb = p->ld_out;
        g.Ct = p->doutt.as<uint16_t>();
        g.ldt = p->ld_m;
    }
    return run_jobs(p, {g});
}

int check_batch(mppi_proposal p, int M) {
    if (M < 1 || M > p->max_batch) return pfail(p, MPPI_E_CAPACITY, "batch %d outside [1, %d]", M, p->max_batch);
    return MPPI_OK;
}

}  // namespace

extern "C" {

int proposal_create(mppi_proposal* out, int device, void* hip_stream, int T, int nu, int hidden,
                    int max_batch) {
    if (!out) return pfail(nullptr, MPPI_E_ARG, "out is NULL");
    *out = nullptr;
    if (T < 1 || T > MPPI_MAX_T || nu < 1 || nu > 3 || hidden < 1 || hidden > 4096 || max_batch < 1 ||
        max_batch > (1 << 20))
        return pfail(nullptr, MPPI_E_CAPACITY, "bad proposal shape");
    mppi_proposal p = new mppi_proposal_s;
    p->device = device;
    p->stream = static_cast<hipStream_t>(hip_stream);
    p->T = T;
    p->nu = nu;
    p->in = FEAT_BINS + 2 + T * nu;
    p->H = hidden;
    p->out = T * nu;
    p->max_batch = max_batch;
    const long long sizes[6] = {(long long)p->in * hidden, hidden, (long long)hidden * hidden, hidden,
                                (long long)hidden * p->out, p->out};
    long long acc = 0;
    for (int k = 0; k < 6; ++k) {
        p->off[k] = acc;
        acc += sizes[k];
    }
    p->n_params = acc;
    p->F.T = T;
    p->F.nu = nu;
    p->F.in_dim = p->in;
    p->F.r_max = 8.0f;
    for (int c = 0; c < 3; ++c) {
        p->F.umin[c] = -1.0f;
        p->F.umax[c] = 1.0f;
    }
    DeviceGuard g(device);
    const size_t P = sizeof(float) * acc, MB = max_batch;
    hipError_t e = hipSuccess;
    DevBuf* f32[] = {&p->w, &p->g, &p->m, &p->v};
    for (DevBuf* b : f32)
        if (e == hipSuccess) e = b->ensure(P);
    // odd multiples of 64 bytes: rows a power of two apart share few L2 channels
    auto pad = [](int v) { return (((v + 31) / 32) | 1) * 32; };
    p->ld_in = pad(p->in);
    p->ld_h = pad(hidden);
    p->ld_out = pad(p->out);
    p->ld_m = pad(max_batch);
    // bf16 matrices, padding and all zero
    const size_t LI = p->ld_in, LH = p->ld_h, LO = p->ld_out, LM = p->ld_m;
    const std::pair<DevBuf*, size_t> b16[] = {
        {&p->w1t, hidden * LI}, {&p->w2t, hidden * LH}, {&p->w3t, p->out * LH}, {&p->w2b, hidden * LH},
        {&p->w3b, hidden * LO}, {&p->xb, MB * LI}, {&p->a1b, MB * LH}, {&p->a2b, MB * LH},
        {&p->doutb, MB * LO}, {&p->dh2b, MB * LH}, {&p->dh1b, MB * LH}, {&p->xt, p->in * LM},
        {&p->a1t, hidden * LM}, {&p->a2t, hidden * LM}, {&p->doutt, p->out * LM}, {&p->dh2t, hidden * LM},
        {&p->dh1t, hidden * LM}};
    for (const auto& x : b16) {
        if (e == hipSuccess) e = x.first->ensure(2 * x.second);
        if (e == hipSuccess) e = hipMemsetAsync(x.first->p, 0, 2 * x.second, p->stream);
    }
    if (e == hipSuccess) e = p->pre1.ensure(4 * MB * hidden);
    if (e == hipSuccess) e = p->pre2.ensure(4 * MB * hidden);
    if (e == hipSuccess) e = p->outb.ensure(4 * MB * p->out);
    if (e == hipSuccess) e = p->dout.ensure(4 * MB * p->out);
    if (e == hipSuccess) e = p->dh2.ensure(4 * MB * hidden);
    if (e == hipSuccess) e = p->dh1.ensure(4 * MB * hidden);
    if (e == hipSuccess) e = p->rowsq.ensure(4 * MB);
    if (e == hipSuccess) e = p->loss.ensure(4);
    if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void**>(&p->h_loss), sizeof(float), 0);
    if (e == hipSuccess) e = hipMemsetAsync(p->w.p, 0, P, p->stream);
    if (e == hipSuccess) e = hipMemsetAsync(p->m.p, 0, P, p->stream);
    if (e == hipSuccess) e = hipMemsetAsync(p->v.p, 0, P, p->stream);
    // the matrix-core copies of the (zero) weights must be valid before any forward pass
    if (e == hipSuccess && refresh_bf16(p) != MPPI_OK) e = hipErrorLaunchFailure;
    if (e == hipSuccess) e = hipStreamSynchronize(p->stream);
    if (e != hipSuccess) {
        proposal_destroy(p);
        return pfail(nullptr, MPPI_E_HIP, "proposal setup: %s", hipGetErrorString(e));
    }
    *out = p;
    return MPPI_OK;
}

int proposal_destroy(mppi_proposal p) {
    if (!p) return MPPI_OK;
    {
        DeviceGuard g(p->device);
        (void)hipStreamSynchronize(p->stream);
        DevBuf* bufs[] = {&p->w, &p->g, &p->m, &p->v, &p->w1t, &p->w2t, &p->w3t, &p->w2b, &p->w3b, &p->xb,
                          &p->xt, &p->a1t, &p->a2t, &p->doutt, &p->dh2t, &p->dh1t, &p->pre1,
                          &p->a1b, &p->pre2, &p->a2b, &p->outb, &p->dout, &p->doutb, &p->dh2,
                          &p->dh2b, &p->dh1, &p->dh1b, &p->rowsq, &p->loss};
        for (DevBuf* b : bufs) b->release();
        if (p->h_loss) (void)hipHostFree(p->h_loss);
    }
    delete p;
    return MPPI_OK;
}

const char* proposal_last_error(mppi_proposal p) { return p ? p->err.c_str() : g_create_error.c_str(); }

long long proposal_num_params(mppi_proposal p) { return p ? p->n_params : -1; }

int proposal_shape(mppi_proposal p, int* in_dim, int* hidden, int* out_dim) {
    if (!p) return MPPI_E_ARG;
    if (in_dim) *in_dim = p->in;
    if (hidden) *hidden = p->H;
    if (out_dim) *out_dim = p->out;
    return MPPI_OK;
}

int proposal_set_params(mppi_proposal p, const float* host, long long n) {
    if (!p || !host) return MPPI_E_ARG;
    if (n != p->n_params) return pfail(p, MPPI_E_ARG, "expected %lld parameters", p->n_params);
    DeviceGuard g(p->device);
    PHIP(p, hipMemcpyAsync(p->w.p, host, sizeof(float) * n, hipMemcpyHostToDevice, p->stream));
    PHIP(p, hipMemsetAsync(p->m.p, 0, sizeof(float) * n, p->stream));
    PHIP(p, hipMemsetAsync(p->v.p, 0, sizeof(float) * n, p->stream));
    p->t = 0;
    if (int rc = refresh_bf16(p)) return rc;
    PHIP(p, hipStreamSynchronize(p->stream));
    return MPPI_OK;
}

int proposal_get_params(mppi_proposal p, float* host, long long n) {
    if (!p || !host) return MPPI_E_ARG;
    if (n != p->n_params) return pfail(p, MPPI_E_ARG, "expected %lld parameters", p->n_params);
    DeviceGuard g(p->device);
    PHIP(p, hipMemcpyAsync(host, p->w.p, sizeof(float) * n, hipMemcpyDeviceToHost, p->stream));
    PHIP(p, hipStreamSynchronize(p->stream));
    return MPPI_OK;
}

int proposal_set_scaling(mppi_proposal p, const mppi_params* prm, float r_max) {
    if (!p || !prm) return MPPI_E_ARG;
    if (prm->T != p->T || prm->nu != p->nu) return pfail(p, MPPI_E_ARG, "T / nu differ from the proposal's");
    if (!(r_max > 0)) return pfail(p, MPPI_E_ARG, "r_max must be positive");
    p->F.r_max = r_max;
    p->F.goal[0] = prm->goal[0];
    p->F.goal[1] = prm->goal[1];
    for (int c = 0; c < 3; ++c) {
        p->F.umin[c] = c < prm->nu ? prm->u_min[c] : -1.0f;
        p->F.umax[c] = c < prm->nu ? prm->u_max[c] : 1.0f;
    }
    return MPPI_OK;
}

int proposal_features(mppi_proposal p, mppi_ctx ctx, const float* dq0, const float* dU_prev, int M,
                      float* dfeat) {
    if (!p || !ctx || !dq0 || !dU_prev || !dfeat) return MPPI_E_ARG;
    if (M < 1) return pfail(p, MPPI_E_ARG, "M < 1");
    DeviceGuard g(p->device);
    PHIP(p, launch_features(ctx->px.as<float>(), ctx->py.as<float>(), ctx->n_valid.as<int>(), dq0,
                            dU_prev, p->F, M, dfeat, p->stream));
    return MPPI_OK;
}

int proposal_forward(mppi_proposal p, const float* dfeat, int M, float* dout) {
    if (!p || !dfeat || !dout) return MPPI_E_ARG;
    if (int rc = check_batch(p, M)) return rc;
    DeviceGuard g(p->device);
    return forward(p, dfeat, M, dout, nullptr, nullptr);
}

int proposal_mean(mppi_proposal p, const float* dfeat, int M, float* dU) {
    if (!p || !dfeat || !dU) return MPPI_E_ARG;
    if (int rc = check_batch(p, M)) return rc;
    DeviceGuard g(p->device);
    return forward(p, dfeat, M, nullptr, dU, nullptr);
}

int proposal_normalize(mppi_proposal p, const float* dU, const float* dfeat, int M, float* dtarget) {
    if (!p || !dU || !dtarget) return MPPI_E_ARG;
    if (M < 1) return pfail(p, MPPI_E_ARG, "M < 1");
    if (p->F.res_scale > 0.0f && !dfeat) return pfail(p, MPPI_E_ARG, "residual targets need the features");
    DeviceGuard g(p->device);
    PHIP(p, launch_normalize(dU, dfeat, M, p->T, p->nu, p->F, dtarget, p->stream));
    return MPPI_OK;
}

int proposal_set_residual(mppi_proposal p, float scale) {
    if (!p) return MPPI_E_ARG;
    if (!(scale >= 0.0f) || !std::isfinite(scale)) return pfail(p, MPPI_E_ARG, "scale must be >= 0");
    p->F.res_scale = scale;
    return MPPI_OK;
}

int proposal_train_step(mppi_proposal p, const float* dfeat, const float* dtarget, int M, float lr,
                        float* loss_out) {
    if (!p || !dfeat || !dtarget) return MPPI_E_ARG;
    if (int rc = check_batch(p, M)) return rc;
    if (!(lr >= 0)) return pfail(p, MPPI_E_ARG, "lr must be >= 0");
    DeviceGuard g(p->device);
    const int in = p->in, H = p->H, O = p->out;
    if (int rc = forward(p, dfeat, M, nullptr, nullptr, dtarget)) return rc;
    if (loss_out)
        PHIP(p, launch_loss(p->outb.as<float>(), dtarget, M, O, p->rowsq.as<float>(), p->loss.as<float>(), p->stream));
    // Gradients: dH2 = (dOut W3^T) * gelu'(pre2), dH1 = (dH2 W2^T) * gelu'(pre1),
    // dW = A^T dY, db = sum dY.  Three launches: the chain dOut -> dH2 -> dH1 ->
    // dW1 is three products long, and everything else runs beside its last two.
    auto grad_h = [&](const DevBuf& dy, const DevBuf& w, int K, int ld, const DevBuf& pre, const DevBuf& d,
                      const DevBuf& db, const DevBuf& dt) {
        MlpJob g = product(EPI_GELU_GRAD, M, H, K, dy, ld, w, ld, d.as<float>());
        g.aux = pre.as<float>();
        g.Cb = db.as<uint16_t>();
        g.ldcb = p->ld_h;
        g.Ct = dt.as<uint16_t>();
        g.ldt = p->ld_m;
        return g;
    };
    auto grad_w = [&](int rows, int cols, const DevBuf& at, const DevBuf& dyt, int k) {
        return product(EPI_STORE, rows, cols, M, at, p->ld_m, dyt, p->ld_m, W(p, p->g, k));
    };
    if (int rc = run_jobs(p, {grad_h(p->doutb, p->w3b, O, p->ld_out, p->pre2, p->dh2, p->dh2b, p->dh2t)})) return rc;
    if (int rc = run_jobs(p, {grad_w(H, H, p->a1t, p->dh2t, 2), grad_w(H, O, p->a2t, p->doutt, 4),
                              grad_h(p->dh2b, p->w2b, H, p->ld_h, p->pre1, p->dh1, p->dh1b, p->dh1t)}))
        return rc;
    if (int rc = run_jobs(p, {grad_w(in, H, p->xt, p->dh1t, 0), colsum(M, H, p->dh1.as<float>(), W(p, p->g, 1)),
                              colsum(M, H, p->dh2.as<float>(), W(p, p->g, 3)),
                              colsum(M, O, p->dout.as<float>(), W(p, p->g, 5))}))
        return rc;
    // Adam
    p->t += 1;
    AdamArgs a;
    a.lr = lr;
    a.b1 = 0.9f;
    a.b2 = 0.999f;
    a.ob1 = static_cast<float>(1.0 - 0.9);
    a.ob2 = static_cast<float>(1.0 - 0.999);
    a.eps = 1e-8f;
    a.c1 = static_cast<float>(1.0 - std::pow(0.9, static_cast<double>(p->t)));
    a.c2 = static_cast<float>(1.0 - std::pow(0.999, static_cast<double>(p->t)));
    PHIP(p, launch_adam(p->w.as<float>(), p->g.as<float>(), p->m.as<float>(), p->v.as<float>(), p->n_params,
                        a, weights(p), p->stream));
    if (loss_out) {
        PHIP(p, hipMemcpyAsync(p->h_loss, p->loss.p, sizeof(float), hipMemcpyDeviceToHost, p->stream));
        PHIP(p, hipStreamSynchronize(p->stream));
        *loss_out = *p->h_loss;
    }
    return MPPI_OK;
}

int proposal_get_buffer(mppi_proposal p, int which, float* host, long long n) {
    if (!p || !host) return MPPI_E_ARG;
    DeviceGuard g(p->device);
    DevBuf* f32[] = {&p->pre1, &p->pre2, &p->outb, &p->dout, &p->dh2, &p->dh1, &p->g};
    DevBuf* b16[] = {&p->xb, &p->a1b, &p->a2b, &p->doutb, &p->dh2b, &p->dh1b};
    if (which >= 0 && which < 7) {
        if (static_cast<size_t>(n) * 4 > f32[which]->cap) return pfail(p, MPPI_E_ARG, "n too large");
        PHIP(p, hipMemcpyAsync(host, f32[which]->p, sizeof(float) * n, hipMemcpyDeviceToHost, p->stream));
        PHIP(p, hipStreamSynchronize(p->stream));
        return MPPI_OK;
    }
    if (which >= 10 && which < 16) {
        DevBuf* b = b16[which - 10];
        // stored with padded rows, returned without the padding
        const int cols = which == 10 ? p->in : which == 13 ? p->out : p->H;
        const int ld = which == 10 ? p->ld_in : which == 13 ? p->ld_out : p->ld_h;
        if (n < 0 || n > static_cast<long long>(p->max_batch) * cols) return pfail(p, MPPI_E_ARG, "n too large");
        const long long rows = (n + cols - 1) / cols;
        std::vector<uint16_t> tmp(static_cast<size_t>(rows) * cols);
        if (rows > 0)
            PHIP(p, hipMemcpy2DAsync(tmp.data(), 2 * static_cast<size_t>(cols), b->p, 2 * static_cast<size_t>(ld),
                                     2 * static_cast<size_t>(cols), rows, hipMemcpyDeviceToHost, p->stream));
        PHIP(p, hipStreamSynchronize(p->stream));
        for (long long i = 0; i < n; ++i) {
            const uint32_t u = static_cast<uint32_t>(tmp[i]) << 16;
            std::memcpy(&host[i], &u, 4);
        }
        return MPPI_OK;
    }
    return pfail(p, MPPI_E_ARG, "unknown buffer %d", which);
}

int proposal_save(mppi_proposal p, const char* path) {
    if (!p || !path) return MPPI_E_ARG;
    std::vector<float> w(p->n_params), m(p->n_params), v(p->n_params);
    DeviceGuard g(p->device);
    PHIP(p, hipMemcpyAsync(w.data(), p->w.p, 4 * p->n_params, hipMemcpyDeviceToHost, p->stream));
    PHIP(p, hipMemcpyAsync(m.data(), p->m.p, 4 * p->n_params, hipMemcpyDeviceToHost, p->stream));
    PHIP(p, hipMemcpyAsync(v.data(), p->v.p, 4 * p->n_params, hipMemcpyDeviceToHost, p->stream));
    PHIP(p, hipStreamSynchronize(p->stream));
    FILE* f = std::fopen(path, "wb");
    if (!f) return pfail(p, MPPI_E_ARG, "cannot open %s", path);
    const int hdr[6] = {0x50494d46, p->in, p->H, p->out, p->T, p->nu};  // "EMIP"
    bool ok = std::fwrite(hdr, sizeof hdr, 1, f) == 1 && std::fwrite(&p->t, sizeof p->t, 1, f) == 1 &&
              std::fwrite(&p->F, sizeof p->F, 1, f) == 1 &&
              std::fwrite(w.data(), 4, w.size(), f) == w.size() &&
              std::fwrite(m.data(), 4, m.size(), f) == m.size() &&
              std::fwrite(v.data(), 4, v.size(), f) == v.size();
    ok = (std::fclose(f) == 0) && ok;
    return ok ? MPPI_OK : pfail(p, MPPI_E_ARG, "write failed: %s", path);
}

int proposal_load(mppi_proposal p, const char* path) {
    if (!p || !path) return MPPI_E_ARG;
    FILE* f = std::fopen(path, "rb");
    if (!f) return pfail(p, MPPI_E_ARG, "cannot open %s", path);
    int hdr[6];
    long long t = 0;
    FeatArgs F;
    std::vector<float> w(p->n_params), m(p->n_params), v(p->n_params);
    bool ok = std::fread(hdr, sizeof hdr, 1, f) == 1 && hdr[0] == 0x50494d46 && hdr[1] == p->in &&
              hdr[2] == p->H && hdr[3] == p->out && std::fread(&t, sizeof t, 1, f) == 1 &&
              std::fread(&F, sizeof F, 1, f) == 1 && std::fread(w.data(), 4, w.size(), f) == w.size() &&
              std::fread(m.data(), 4, m.size(), f) == m.size() &&
              std::fread(v.data(), 4, v.size(), f) == v.size();
    std::fclose(f);
    if (!ok) return pfail(p, MPPI_E_ARG, "%s is not a proposal of this shape", path);
    DeviceGuard g(p->device);
    PHIP(p, hipMemcpyAsync(p->w.p, w.data(), 4 * p->n_params, hipMemcpyHostToDevice, p->stream));
    PHIP(p, hipMemcpyAsync(p->m.p, m.data(), 4 * p->n_params, hipMemcpyHostToDevice, p->stream));
    PHIP(p, hipMemcpyAsync(p->v.p, v.data(), 4 * p->n_params, hipMemcpyHostToDevice, p->stream));
    p->t = t;
    p->F = F;
    if (int rc = refresh_bf16(p)) return rc;
    PHIP(p, hipStreamSynchronize(p->stream));
    return MPPI_OK;
}

}  // extern "C"
