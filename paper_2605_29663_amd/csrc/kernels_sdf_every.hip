// The distance pass over small point sets: every point against every pose, one
// lane per pose (a lane group for polygons above 16 vertices).
// The per-lane work is in sdf_device.hpp (shared with the batched kernel).
#include "sdf_device.hpp"

namespace emppi {

namespace {

// Grid: x over poses (one lane each), y over point chunks of `chunk` points.
// Each chunk's minimum is merged into the pose's key with atomicMin.
// Waves per SIMD the register budget is tuned for (512 VGPRs per lane).
template <int BP>
constexpr int poly_waves() { return BP <= 8 ? 6 : BP <= 16 ? 4 : BP <= 20 ? 3 : 2; }

template <int BP, bool MOVING, bool ARGMIN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(poly_waves<BP>())))
void k_dmin_poly(const float4* __restrict__ poses, int npose,
                                                   PoseTime pt, PointArgs pts, int chunk,
                                                   const float2* __restrict__ verts,
                                                   unsigned int* __restrict__ key,
                                                   unsigned long long* __restrict__ key64) {
    extern __shared__ __align__(16) float lds[];  // point tiles: 8- and 16-byte LDS accesses
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = g < npose;
    const float4 q = live ? poses[g] : make_float4(0.f, 0.f, 1.f, 0.f);
    const float tau = MOVING ? pose_tau(pt, g) : 0.0f;
    const int nv = *pts.n_valid;
    const int c0 = blockIdx.y * chunk;
    const int c1 = min(c0 + chunk, nv);
    float best;
    int besti;
    dmin_poly_range<BP, MOVING, ARGMIN>(q, tau, pts, c0, c1, verts, lds, best, besti);
    if (live) {
        if (ARGMIN) {
            const unsigned int idx = besti >= 0 ? static_cast<unsigned int>(pts.idx[besti]) : 0xFFFFFFFFu;
            atomicMin(&key64[g], (static_cast<unsigned long long>(dkey(best)) << 32) | idx);
        } else {
            atomicMin(&key[g], dkey(best));
        }
    }
}

// Polygons of more than 16 padded vertices: a group of L lanes per pose (a
// pair up to 32 vertices, a quad above), each lane holding HB edges
// (PolyPart); the group's first lane merges the pose's key.  Register
// budget: 4 waves per SIMD for static points (at 16 edges per lane the
// compiler then spills only in the set-up, not in the point loop), 3 for
// moving points (whose point loop would spill at 4).
template <int HB, int L, bool MOVING, bool ARGMIN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MOVING ? 3 : 4)))
void k_dmin_poly_part(const float4* __restrict__ poses, int npose, PoseTime pt, PointArgs pts,
                      int chunk, const float2* __restrict__ verts, unsigned int* __restrict__ key,
                      unsigned long long* __restrict__ key64) {
    extern __shared__ __align__(16) float lds[];  // point tiles: 8- and 16-byte LDS accesses
    const int g = static_cast<int>((blockIdx.x * blockDim.x + threadIdx.x) / L);
    const bool live = g < npose;
    const float4 q = live ? poses[g] : make_float4(0.f, 0.f, 1.f, 0.f);
    const float tau = MOVING ? pose_tau(pt, g) : 0.0f;
    const int nv = *pts.n_valid;
    const int c0 = blockIdx.y * chunk;
    const int c1 = min(c0 + chunk, nv);
    float best;
    int besti;
    dmin_poly_part_range<HB, L, MOVING, ARGMIN>(q, tau, pts, c0, c1, verts, lds, best, besti);
    if (live && (threadIdx.x & (L - 1)) == 0) {
        if (ARGMIN) {
            const unsigned int idx = besti >= 0 ? static_cast<unsigned int>(pts.idx[besti]) : 0xFFFFFFFFu;
            atomicMin(&key64[g], (static_cast<unsigned long long>(dkey(best)) << 32) | idx);
        } else {
            atomicMin(&key[g], dkey(best));
        }
    }
}

template <int RP, bool MOVING, bool ARGMIN>
__global__ __launch_bounds__(256) void k_dmin_rect(const float4* __restrict__ poses, int npose,
                                                   PoseTime pt, PointArgs pts, int chunk,
                                                   const float4* __restrict__ rects,
                                                   unsigned int* __restrict__ key,
                                                   unsigned long long* __restrict__ key64) {
    extern __shared__ __align__(16) float lds[];  // point tiles: 8- and 16-byte LDS accesses
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = g < npose;
    const float4 q = live ? poses[g] : make_float4(0.f, 0.f, 1.f, 0.f);
    const float tau = MOVING ? pose_tau(pt, g) : 0.0f;
    const int nv = *pts.n_valid;
    const int c0 = blockIdx.y * chunk;
    const int c1 = min(c0 + chunk, nv);
    float best;
    int besti;
    dmin_rect_range<RP, MOVING, ARGMIN>(q, tau, pts, c0, c1, rects, lds, best, besti);
    if (live) {
        if (ARGMIN) {
            const unsigned int idx = besti >= 0 ? static_cast<unsigned int>(pts.idx[besti]) : 0xFFFFFFFFu;
            atomicMin(&key64[g], (static_cast<unsigned long long>(dkey(best)) << 32) | idx);
        } else {
            atomicMin(&key[g], dkey(best));
        }
    }
}

template <int BP, bool MOVING, bool ARGMIN>
hipError_t launch_poly_t(const DminLaunch& L, dim3 grid, size_t lds, hipStream_t s) {
    hipLaunchKernelGGL((k_dmin_poly<BP, MOVING, ARGMIN>), grid, dim3(L.block), lds, s, L.poses,
                       L.npose, L.pt, L.pts, L.chunk, L.verts, L.key, L.key64);
    return hipGetLastError();
}

template <int RP, bool MOVING, bool ARGMIN>
hipError_t launch_rect_t(const DminLaunch& L, dim3 grid, size_t lds, hipStream_t s) {
    hipLaunchKernelGGL((k_dmin_rect<RP, MOVING, ARGMIN>), grid, dim3(L.block), lds, s, L.poses,
                       L.npose, L.pt, L.pts, L.chunk, L.rects, L.key, L.key64);
    return hipGetLastError();
}

template <int HB, int L, bool MOVING, bool ARGMIN>
hipError_t launch_part_t(const DminLaunch& D, dim3 grid, size_t lds, hipStream_t s) {
    hipLaunchKernelGGL((k_dmin_poly_part<HB, L, MOVING, ARGMIN>), grid, dim3(D.block), lds, s,
                       D.poses, D.npose, D.pt, D.pts, D.chunk, D.verts, D.key, D.key64);
    return hipGetLastError();
}

template <int HB, int L>
hipError_t launch_part(const DminLaunch& D, dim3 grid, size_t lds, hipStream_t s) {
    // L lanes per pose
    const dim3 gl((L * D.npose + D.block - 1) / D.block, grid.y);
    if (D.pts.vx) return D.argmin ? launch_part_t<HB, L, true, true>(D, gl, lds, s)
                                  : launch_part_t<HB, L, true, false>(D, gl, lds, s);
    return D.argmin ? launch_part_t<HB, L, false, true>(D, gl, lds, s)
                    : launch_part_t<HB, L, false, false>(D, gl, lds, s);
}

template <int P>
hipError_t launch_poly(const DminLaunch& L, dim3 grid, size_t lds, hipStream_t s) {
    if constexpr (P > 32) {
        return launch_part<P / 4, 4>(L, grid, lds, s);
    } else if constexpr (P > 16) {
        return launch_part<P / 2, 2>(L, grid, lds, s);
    } else {
        if (L.pts.vx) return L.argmin ? launch_poly_t<P, true, true>(L, grid, lds, s)
                                      : launch_poly_t<P, true, false>(L, grid, lds, s);
        return L.argmin ? launch_poly_t<P, false, true>(L, grid, lds, s)
                        : launch_poly_t<P, false, false>(L, grid, lds, s);
    }
}

template <int P>
hipError_t launch_rect(const DminLaunch& L, dim3 grid, size_t lds, hipStream_t s) {
    if (L.pts.vx) return L.argmin ? launch_rect_t<P, true, true>(L, grid, lds, s)
                                  : launch_rect_t<P, true, false>(L, grid, lds, s);
    return L.argmin ? launch_rect_t<P, false, true>(L, grid, lds, s)
                    : launch_rect_t<P, false, false>(L, grid, lds, s);
}

}  // namespace

hipError_t launch_dmin_every(const DminLaunch& L, hipStream_t s) {
    const dim3 grid((L.npose + L.block - 1) / L.block, L.nchunk);
    const size_t lds = static_cast<size_t>(DMIN_TILE) * (L.pts.vx ? 16 : 8);
    if (L.kind == 0) {
        switch (L.padded) {
#define EMPPI_CASE(P) \
    case P: return launch_poly<P>(L, grid, lds, s);
            EMPPI_CASE(3) EMPPI_CASE(4) EMPPI_CASE(5) EMPPI_CASE(6) EMPPI_CASE(7) EMPPI_CASE(8)
            EMPPI_CASE(9) EMPPI_CASE(10) EMPPI_CASE(11) EMPPI_CASE(12) EMPPI_CASE(13)
            EMPPI_CASE(14) EMPPI_CASE(15) EMPPI_CASE(16) EMPPI_CASE(18) EMPPI_CASE(20)
            EMPPI_CASE(22) EMPPI_CASE(24) EMPPI_CASE(26) EMPPI_CASE(28) EMPPI_CASE(30)
            EMPPI_CASE(32) EMPPI_CASE(36) EMPPI_CASE(40) EMPPI_CASE(44) EMPPI_CASE(48)
            EMPPI_CASE(52) EMPPI_CASE(56) EMPPI_CASE(60) EMPPI_CASE(64)
#undef EMPPI_CASE
        default: return hipErrorInvalidValue;
        }
    }
    switch (L.padded) {
    case 1: return launch_rect<1>(L, grid, lds, s);
    case 2: return launch_rect<2>(L, grid, lds, s);
    case 3: return launch_rect<3>(L, grid, lds, s);
    case 4: return launch_rect<4>(L, grid, lds, s);
    case 6: return launch_rect<6>(L, grid, lds, s);
    case 8: return launch_rect<8>(L, grid, lds, s);
    case 12: return launch_rect<12>(L, grid, lds, s);
    case 16: return launch_rect<16>(L, grid, lds, s);
    case 24: return launch_rect<24>(L, grid, lds, s);
    case 32: return launch_rect<32>(L, grid, lds, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace emppi
