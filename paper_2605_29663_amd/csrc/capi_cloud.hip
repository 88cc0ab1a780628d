// C ABI of the point-cloud pre-processing pass (declared in
// include/exact_mppi.h): argument checks, the context-owned workspace and
// the launch sequence of kernels_cloud.hip.
#include <cmath>
#include <cstring>

#include "cloud.hpp"
#include "ctx.hpp"

using namespace emppi;
using namespace emppi_host;

static_assert(MPPI_MAX_CLOUD == CLOUD_MAX_POINTS, "cloud capacity of the C ABI");

extern "C" {

int cloud_downsample(mppi_ctx ctx, const float* dxyz, int m, const float center[2],
                     const mppi_cloud_params* cp, float* dx, float* dy, unsigned char* dvalid,
                     int* n_kept) {
    if (!ctx) return MPPI_E_ARG;
    if (!cp || !center) return fail(ctx, MPPI_E_ARG, "cloud: NULL parameters");
    if (m < 0 || m > MPPI_MAX_CLOUD) return fail(ctx, MPPI_E_ARG, "cloud: m=%d outside [0, %d]", m, MPPI_MAX_CLOUD);
    if (cp->n_out < 0 || cp->n_out > MPPI_MAX_CLOUD)
        return fail(ctx, MPPI_E_ARG, "cloud: n_out=%d outside [0, %d]", cp->n_out, MPPI_MAX_CLOUD);
    if (m > 0 && !dxyz) return fail(ctx, MPPI_E_ARG, "cloud: NULL input");
    if (cp->n_out > 0 && (!dx || !dy || !dvalid)) return fail(ctx, MPPI_E_ARG, "cloud: NULL output");
    const float vals[] = {cp->z_min, cp->z_max, cp->r_max, cp->voxel, center[0], center[1]};
    for (float v : vals)
        if (!std::isfinite(v)) return fail(ctx, MPPI_E_ARG, "cloud: non-finite parameter");
    if (!(cp->voxel > 0.0f) || !(cp->r_max > 0.0f) || !(cp->z_min <= cp->z_max))
        return fail(ctx, MPPI_E_ARG, "cloud: need voxel > 0, r_max > 0, z_min <= z_max");
    const double reach = std::max(std::fabs(static_cast<double>(center[0])),
                                  std::fabs(static_cast<double>(center[1]))) + cp->r_max;
    if (reach / cp->voxel >= static_cast<double>(1 << 29))
        return fail(ctx, MPPI_E_ARG, "cloud: voxel too small for the range (voxel index >= 2^29)");
    DeviceGuard g(ctx->device);
    CloudArgs a{};
    a.xyz = dxyz;
    a.m = m;
    a.cx = center[0];
    a.cy = center[1];
    a.z_min = cp->z_min;
    a.z_max = cp->z_max;
    a.rmax2 = cp->r_max * cp->r_max;
    a.voxel = cp->voxel;
    a.n_out = cp->n_out;
    CloudWork w{};
    int cap = 256;
    while (cap < 2 * m) cap <<= 1;
    // The voxels of the range as a plain grid when they are no more than the
    // hash table's slots or CLOUD_DENSE_MIN: 2^20 points take 59 us with a
    // grid of 40000 cells and 83 with one of 10^6, hashed 85 and 102; 3000
    // points with 160000 cells 39 and hashed 41, with 4 10^6 cells 54 and
    // hashed 43.  The margins cover the rounding of the range test (relative 1e-6 of r_max) and of the
    // quotient (2^-22 of its size); a squared range that overflows or loses
    // its relative precision does not bound the coordinates.
    const double vox = cp->voxel, margin = 2.0 + reach / vox * 0x1p-22;
    const double r = static_cast<double>(cp->r_max) * (1.0 + 1e-6);
    const double lx = std::floor((center[0] - r) / vox - margin), hx = std::floor((center[0] + r) / vox + margin);
    const double ly = std::floor((center[1] - r) / vox - margin), hy = std::floor((center[1] + r) / vox + margin);
    w.cells = cap;
    if ((hx - lx + 1) * (hy - ly + 1) <= std::max(cap, CLOUD_DENSE_MIN) && std::isfinite(a.rmax2) &&
        a.rmax2 >= 1e-30f) {
        w.x0 = static_cast<int>(lx);
        w.y0 = static_cast<int>(ly);
        w.nx = static_cast<int>(hx - lx) + 1;
        w.ny = static_cast<int>(hy - ly) + 1;
        w.cells = w.nx * w.ny;
    }
    const size_t C = static_cast<size_t>(w.cells), words = (static_cast<size_t>(m) + 127) / 128 * 4;
    // the hash keys are done with when the ranges are written; at most m cells
    // are occupied
    HIP_TRY(ctx, ctx->cloud_keys.ensure((w.nx == 0 ? sizeof(unsigned long long) : sizeof(uint32_t)) * C));
    HIP_TRY(ctx, ctx->cloud_first.ensure(sizeof(int) * C));
    HIP_TRY(ctx, ctx->cloud_cell.ensure(sizeof(uint2) * std::max<size_t>(std::min<size_t>(C, m), 1)));
    HIP_TRY(ctx, ctx->cloud_misc.ensure(sizeof(int) * (words + CLOUD_BINS + 8)));
    w.keys = ctx->cloud_keys.as<unsigned long long>();
    w.first = ctx->cloud_first.as<int>();
    w.cand = ctx->cloud_cell.as<uint2>();
    w.key = ctx->cloud_keys.as<uint32_t>();
    w.kept = ctx->cloud_misc.as<uint32_t>();
    w.hist = ctx->cloud_misc.as<int>() + words;
    w.state = w.hist + CLOUD_BINS;
    // the count goes straight to pinned memory
    HIP_TRY(ctx, launch_cloud(a, w, dx, dy, dvalid, n_kept ? reinterpret_cast<int*>(ctx->h_out) : nullptr, ctx->stream));
    if (n_kept) {
        HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
        std::memcpy(n_kept, ctx->h_out, sizeof(int));
    }
    return MPPI_OK;
}

}  // extern "C"
