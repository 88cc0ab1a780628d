// Single-scene kernels of the fused rollout-frame transform + exact signed
// distance + min over points stage, the footprint's bound table and the
// point-wise signed-distance kernels.  The search is in cull_device.hpp, the
// exact evaluation in sdf_device.hpp (shared with the batched kernel).
#include "cull_device.hpp"

namespace emppi {

namespace {

// Grid: x over pose tiles (P poses per wave), a workgroup taking `tiles` of
// them a grid apart, so that each has poses of several horizon steps (later
// steps, being more spread, cost more); y over ranges of `supers` super
// nodes; each range's minimum is merged into the pose's key with atomicMin.
template <typename Eval, bool MOVING, bool ARGMIN>
__global__ __launch_bounds__(CULL_WAVES * WAVE) __attribute__((amdgpu_waves_per_eu(Eval::WAVES)))
void k_dmin(CullArgs A, int P, int tiles, int supers, const float2* __restrict__ verts,
            const float4* __restrict__ rects, int nprim) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int per_tile = (blockDim.x / WAVE) * P;
    const int s0 = blockIdx.y * supers;
    cull_block<Eval, MOVING, ARGMIN>(A, verts, rects, nprim, blockIdx.x * per_tile, gridDim.x * per_tile, P, tiles, s0,
                                     s0 + supers, lds);
}

// Direction of the pseudo-angle a in [-1, 3) (far_bin).
__device__ __forceinline__ float2 far_dir(float a) {
    const float x = a <= 1.0f ? 1.0f - fabsf(a) : fabsf(a - 2.0f) - 1.0f, y = a <= 1.0f ? a : 2.0f - a;
    const float r = 1.0f / __builtin_sqrtf(x * x + y * y);
    return make_float2(x * r, y * r);
}

// FootTable::far[k] from the footprint's corners: v reaches furthest in the bin's middle; eps is the most that
// another corner reaches beyond it in the bin, widened for the rounding of
// far_bin.  w . u is a cosine of u's angle: over the bin it is largest at an
// end, or |w| if w's direction is inside.
__device__ float4 far_entry(const FootHead& F, int k, const float2* corner, int n) {
    constexpr float STEP = 4.0f / FAR_BINS;
    const float2 m = far_dir((k + 0.5f) * STEP - 1.0f), e0 = far_dir((k - 0.01f) * STEP - 1.0f),
                 e1 = far_dir((k + 1.01f) * STEP - 1.0f);
    float2 v = corner[0];
#pragma unroll 4
    for (int i = 1; i < n; ++i) {
        const float2 w = corner[i];
        if (w.x * m.x + w.y * m.y > v.x * m.x + v.y * m.y) v = w;
    }
    float eps = 0.0f;
#pragma unroll 4
    for (int i = 0; i < n; ++i) {
        float2 w = corner[i];
        w.x -= v.x;
        w.y -= v.y;
        eps = fmaxf(eps, fmaxf(w.x * e0.x + w.y * e0.y, w.x * e1.x + w.y * e1.y));
        if (e0.x * w.y - e0.y * w.x > 0.0f && w.x * e1.y - w.y * e1.x > 0.0f) eps = fmaxf(eps, __builtin_sqrtf(w.x * w.x + w.y * w.y));
    }
    return make_float4(v.x, v.y, eps + 1e-5f * F.reach, 0.0f);
}

// Cells of a footprint's bound table (FootTable), one thread each.  r: a bit
// more than half the cell's diagonal; a feature further from the centre than
// the nearest by more than 2 r is nearest nowhere in the cell.  Three kinds:
//   - the distance is linear: the nearest edge's projection stays inside the
//     edge (the nearest box's distance that of one face) and no other feature
//     is near;
//   - outside or inside by more than r, with the nearest point p, the unit
//     vector g from p to the centre and all near features on the far side of
//     the line through p across g: the way to p bounds the distance of the
//     point at h from above, sqrt((d + g h)^2 + |h|^2 - (g h)^2) <= d + g h +
//     r^2 / (2 (d - r)), and that line from below, d + g h;
//   - any other.
// The second kind takes the search from 94 to 75 us a launch on average at 8192
// corridor points and 16 vertices (the fill itself is a set-up cost).
__global__ __launch_bounds__(256) void k_foot_table(int kind, FootHead F, FootTable* __restrict__ table,
                                                    const float4* __restrict__ tab_a,
                                                    const float4* __restrict__ tab_b,
                                                    const float2* __restrict__ verts, int count) {
    // the footprint in LDS: a cell's loops are chains of its loads
    __shared__ float4 ta[FOOT_EDGES];
    __shared__ float2 tb[FOOT_EDGES], corner[4 * FOOT_BOXES];
    const int t = threadIdx.x;
    if (t < count) {
        ta[t] = tab_a[t];
        if (kind == 0) tb[t] = make_float2(tab_b[t].x, tab_b[t].y);
    }
    __syncthreads();
    if (blockIdx.x == FOOT_CELLS / 256) {
        const int n = kind == 0 ? count : 4 * count;
        if (t < n) {
            if (kind == 0) {
                corner[t] = make_float2(verts[t].x - F.cx, verts[t].y - F.cy);
            } else {
                const float4 a = ta[t >> 2];
                corner[t] = make_float2(a.x + (t & 1 ? a.z : -a.z) - F.cx, a.y + (t & 2 ? a.w : -a.w) - F.cy);
            }
        }
        __syncthreads();
        if (t == 0) *static_cast<FootHead*>(table) = F;
        if (t < FAR_BINS) table->far[t] = far_entry(F, t, corner, n);
        return;
    }
    const int c = blockIdx.x * blockDim.x + t;
    if (c >= F.nx * F.ny) return;
    const float x = (static_cast<float>(c % F.nx) + 0.5f - F.ox) * F.dx;
    const float y = (static_cast<float>(c / F.nx) + 0.5f - F.oy) * F.dy;
    const float r = F.err_cell;
    float d = INFINITY, second = INFINITY;  // nearest and next distance
    float gx = 0.0f, gy = 0.0f;             // gradient
    bool linear = false, smooth = false;
    const float tol = 1e-5f * F.reach;
    if (kind == 0) {
        float m2 = INFINITY, v = 0.0f, wx = 0.0f, wy = 0.0f;  // (wx, wy): from the nearest point
        bool odd = false, inside = false;
        EdgeEval last = edge_eval(x, y, tb[count - 1].y, ta[count - 1].x, ta[count - 1].y,
                                  ta[count - 1].z, ta[count - 1].w, tb[count - 1].x);
#pragma unroll 2
        for (int k = 0; k < count; ++k) {
            const float4 a = ta[k];
            const float len = tb[k].x;
            const EdgeEval e = edge_eval(x, y, tb[k].y, a.x, a.y, a.z, a.w, len);
            odd ^= (last.above != e.above) & last.right;
            last = e;
            if (e.d2 < m2) {
                second = m2;
                m2 = e.d2;
                const float u = __builtin_fmaf(x, a.x, __builtin_fmaf(y, a.y, a.z));
                v = __builtin_fmaf(y, a.x, __builtin_fmaf(x, -a.y, a.w));
                inside = u >= r && u <= len - r;
                gx = -a.y;
                gy = a.x;
                const float du = u - __builtin_amdgcn_fmed3f(u, 0.0f, len);
                wx = du * a.x - v * a.y;
                wy = du * a.y + v * a.x;
            } else {
                second = fminf(second, e.d2);
            }
        }
        const float dist = __builtin_sqrtf(m2);
        d = odd ? -dist : dist;
        second = __builtin_sqrtf(second);
        linear = inside && dist > 1e-4f * r && second > dist + 2.0f * r;
        if (linear) {
            if ((v < 0.0f) != odd) {
                gx = -gx;
                gy = -gy;
            }
        } else if (dist > 1.01f * r) {
            gx = wx / dist;
            gy = wy / dist;
            smooth = true;
    #pragma unroll 2
        for (int k = 0; k < count; ++k) {
                const float4 a = ta[k];
                const float len = tb[k].x;
                const EdgeEval e = edge_eval(x, y, tb[k].y, a.x, a.y, a.z, a.w, len);
                if (__builtin_sqrtf(e.d2) > dist + 2.0f * r) continue;
                // the edge's ends, (-nc e + cv n) and that + len e
                const float ax = a.w * a.y - a.z * a.x - x, ay = -a.w * a.x - a.z * a.y - y;
                const float s0 = __builtin_fmaf(ax, gx, ay * gy) + dist;
                const float s1 = s0 + len * __builtin_fmaf(a.x, gx, a.y * gy);
                smooth = smooth && s0 <= tol && s1 <= tol;
            }
            if (odd) {
                gx = -gx;
                gy = -gy;
            }
        }
    } else {
#pragma unroll 2
        for (int k = 0; k < count; ++k) {
            const float4 b = ta[k];
            const float s = signed_sqrt(box_s(x, y, b));
            if (s < d) {
                second = d;
                d = s;
                const float ex = x - b.x, ey = y - b.y;
                const float ax = fabsf(ex) - b.z, ay = fabsf(ey) - b.w;
                const bool fx = fabsf(ex) > r && ay < -r && ax > ay + 2.0f * r;
                const bool fy = fabsf(ey) > r && ax < -r && ay > ax + 2.0f * r;
                linear = fx || fy;
                gx = fx ? copysignf(1.0f, ex) : 0.0f;
                gy = fy ? copysignf(1.0f, ey) : 0.0f;
                if (!linear) {
                    gx = copysignf(fmaxf(ax, 0.0f), ex);
                    gy = copysignf(fmaxf(ay, 0.0f), ey);
                }
            } else {
                second = fminf(second, s);
            }
        }
        if (linear && !(second > d + 2.0f * r)) {
            linear = false;
            gx *= fmaxf(d, 0.0f);
            gy *= fmaxf(d, 0.0f);
        }
        if (!linear && d > 1.01f * r) {
            gx /= d;
            gy /= d;
            smooth = true;
    #pragma unroll 2
        for (int k = 0; k < count; ++k) {
                const float4 b = ta[k];
                if (signed_sqrt(box_s(x, y, b)) > d + 2.0f * r) continue;
                const float s0 = __builtin_fmaf(b.x - x, gx, (b.y - y) * gy) + d;
                smooth = smooth && s0 + b.z * fabsf(gx) + b.w * fabsf(gy) <= tol;
            }
        }
    }
    // error class: err_linear + class (err_cell - err_linear) / 7
    float cls = 7.0f;
    if (linear) {
        cls = 0.0f;
    } else if (smooth) {
        const float bend = r * r / (2.0f * (fabsf(d) - r)) * 1.0001f + tol;
        cls = fminf(ceilf(bend / ((F.err_cell - F.err_linear) * (1.0f / 7.0f))), 7.0f);
    }
    if (cls == 7.0f) gx = gy = 0.0f;
    const float v = 8.0f * fminf(fmaxf(floorf((d - F.base) / (8.0f * F.quantum)), 0.0f), 8191.0f) + cls;
    const int ix = static_cast<int>(rintf(gx * 127.0f)), iy = static_cast<int>(rintf(gy * 127.0f));
    reinterpret_cast<uint32_t*>(table + 1)[c] =
        static_cast<uint32_t>(v) | (static_cast<uint32_t>(ix & 255) << 16) | (static_cast<uint32_t>(iy & 255) << 24);
}

__global__ void k_key_init(unsigned int* __restrict__ key, unsigned long long* __restrict__ key64,
                           int n) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    if (key) key[g] = DKEY_INIT;
    if (key64) key64[g] = DKEY64_INIT;
}

// Keys -> d = sign(s) sqrt(|s|) and the argmin index.
__global__ void k_dmin_finalize(const unsigned int* __restrict__ key,
                                const unsigned long long* __restrict__ key64, int npose,
                                float* __restrict__ d_out, int* __restrict__ idx_out) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= npose) return;
    if (key64) {
        const unsigned long long k = key64[g];
        d_out[g] = signed_sqrt(dkey_value(static_cast<unsigned int>(k >> 32)));
        if (idx_out) idx_out[g] = static_cast<int>(static_cast<unsigned int>(k));
    } else {
        d_out[g] = signed_sqrt(dkey_value(key[g]));
        if (idx_out) idx_out[g] = -1;
    }
}

// ---------------------------------------------------------------- point-wise
// Body-frame query points, one lane each; the footprint table is uniform
// (scalar loads).  Polygon: tab_a[b] = (ex, ey, nc, cv) and tab_b[b] = (l,
// y_b, 0, 0) of edge b (EdgeC); rectangle cover: tab_a[j] = box j.
__global__ __launch_bounds__(256) void k_sdf_poly_points(const float* __restrict__ px,
                                                         const float* __restrict__ py, int n,
                                                         const float4* __restrict__ ta,
                                                         const float4* __restrict__ tb, int B,
                                                         float* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = px[i], y = py[i];
    float4 a = ta[0], b = tb[0];
    EdgeEval e = edge_eval(x, y, b.y, a.x, a.y, a.z, a.w, b.x);
    float m = e.d2;
    const bool above0 = e.above;
    bool above = e.above, right = e.right, odd = false;
    for (int k = 1; k < B; ++k) {
        a = ta[k];
        b = tb[k];
        e = edge_eval(x, y, b.y, a.x, a.y, a.z, a.w, b.x);
        m = fminf(m, e.d2);
        odd ^= (above != e.above) & right;
        above = e.above;
        right = e.right;
    }
    odd ^= (above != above0) & right;
    const float d = __fsqrt_rn(m);
    out[i] = odd ? -d : d;
}

__global__ __launch_bounds__(256) void k_sdf_rect_points(const float* __restrict__ px,
                                                         const float* __restrict__ py, int n,
                                                         const float4* __restrict__ ta, int R,
                                                         float* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = px[i], y = py[i];
    float s = box_s(x, y, ta[0]);
    for (int j = 1; j < R; ++j) s = fminf(s, box_s(x, y, ta[j]));
    out[i] = signed_sqrt(s);
}

template <typename Eval, bool MOVING, bool ARGMIN>
hipError_t launch_cull_t(const DminLaunch& L, hipStream_t s) {
    const int per_wg = L.waves * L.poses_per_wave * L.tiles;
    const dim3 grid((L.npose + per_wg - 1) / per_wg, L.nchunk);
    const CullArgs A{L.poses, L.npose, L.pt, L.pts, L.foot, L.key, L.key64};
    hipLaunchKernelGGL((k_dmin<Eval, MOVING, ARGMIN>), grid, dim3(L.waves * WAVE),
                       cull_lds_bytes(L.waves, MOVING, ARGMIN), s, A, L.poses_per_wave, L.tiles, L.supers,
                       L.verts, L.rects, L.padded);
    return hipGetLastError();
}

template <typename Eval>
hipError_t launch_cull(const DminLaunch& L, hipStream_t s) {
    if (L.pts.vx) return L.argmin ? launch_cull_t<Eval, true, true>(L, s) : launch_cull_t<Eval, true, false>(L, s);
    return L.argmin ? launch_cull_t<Eval, false, true>(L, s) : launch_cull_t<Eval, false, false>(L, s);
}

}  // namespace

int dmin_padded_count(int kind, int count) {
    // polygons: the exact count up to 16 vertices (one lane per pose), even
    // counts up to 32 (a lane pair per pose, half the edges each), multiples
    // of 4 above (a lane quad per pose); padding repeats vertex 0:
    // zero-length edges that change neither the minimum nor the crossing
    // parity
    if (kind == 0) {
        if (count <= 16) return count < 3 ? 3 : count;
        return count <= 32 ? ((count + 1) / 2) * 2 : ((count + 3) / 4) * 4;
    }
    static const int rb[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};
    for (int b : rb)
        if (count <= b) return b;
    return -1;
}

hipError_t launch_dmin(const DminLaunch& L, hipStream_t s) {
    if (L.every) return launch_dmin_every(L, s);
    if (L.kind == 0) {
        if (L.padded <= 16) return launch_cull<EvalPoly<1>>(L, s);
        return L.padded <= 32 ? launch_cull<EvalPoly<2>>(L, s) : launch_cull<EvalPoly<4>>(L, s);
    }
    return L.padded <= 16 ? launch_cull<EvalRect<1>>(L, s) : launch_cull<EvalRect<2>>(L, s);
}

hipError_t launch_key_init(unsigned int* key, unsigned long long* key64, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_key_init, dim3((n + 255) / 256), dim3(256), 0, s, key, key64, n);
    return hipGetLastError();
}

hipError_t launch_dmin_finalize(const unsigned int* key, const unsigned long long* key64, int npose,
                                float* d_out, int* idx_out, hipStream_t s) {
    if (npose <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_dmin_finalize, dim3((npose + 255) / 256), dim3(256), 0, s, key, key64,
                       npose, d_out, idx_out);
    return hipGetLastError();
}

hipError_t launch_sdf_points(int kind, const float* px, const float* py, int n,
                             const float4* tab_a, const float4* tab_b, int count, float* out,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const dim3 grid((n + 255) / 256);
    if (kind == 0)
        hipLaunchKernelGGL(k_sdf_poly_points, grid, dim3(256), 0, s, px, py, n, tab_a, tab_b,
                           count, out);
    else
        hipLaunchKernelGGL(k_sdf_rect_points, grid, dim3(256), 0, s, px, py, n, tab_a, count, out);
    return hipGetLastError();
}

hipError_t launch_foot_table(int kind, const FootHead& head, FootTable* table, const float4* tab_a,
                             const float4* tab_b, const float2* verts, int count, hipStream_t s) {
    hipLaunchKernelGGL(k_foot_table, dim3(FOOT_CELLS / 256 + 1), dim3(256), 0, s, kind, head, table, tab_a, tab_b,
                       verts, count);
    return hipGetLastError();
}

}  // namespace emppi
