// Obstacle-set preparation of set_points: the validity mask, a spatial order
// of the valid points, and the two-level bounding hierarchy that the
// signed-distance pass searches (LEAF_POINTS points per leaf, SUPER_LEAVES
// leaves per super node).
//
// The points are counted into the cells of a Z-order grid over the point
// set's bulk (quantiles of a 64-point sample, so that a few far outliers do
// not coarsen the grid; points outside go to the border cells), the cell
// counts are summed, and every point moves to its cell's range.  Points of
// one cell keep no particular order: the distance pass takes exact minima,
// which do not depend on it, and every point carries the caller's index.
//
// Up to POINTS_SMALL_MAX points one workgroup sorts in LDS: the point arrays
// are a few hundred KB, so the pass is a chain of memory and barrier
// latencies, and one launch is shorter than the five that a grid needs.
// Larger sets take the multi-workgroup path.
#include "kernels.hpp"
#include "wave_ops.hpp"

namespace emppi {

namespace {

constexpr int SMALL_THREADS = 1024;
constexpr int WINDOW = 8192;  // sorted points in LDS at a time (half as many moving ones)
constexpr int LARGE_CELL_BITS = 18;

// Z-order of two coordinates below 2^16 packed as y << 16 | x: the bits of x
// at the even positions, those of y at the odd ones.  Both halves are spread
// at once while they stay below 2^8.
__device__ __forceinline__ unsigned spread16(unsigned v) {
    v = (v | (v << 4)) & 0x0F0F0F0Fu;
    v = (v | (v << 2)) & 0x33333333u;
    return (v | (v << 1)) & 0x55555555u;
}
__device__ __forceinline__ unsigned z_order(unsigned x, unsigned y) {
    const unsigned lo = spread16((x & 0xFFu) | ((y & 0xFFu) << 16));
    const unsigned z = (lo & 0xFFFFu) | (lo >> 15);
    const unsigned hx = x >> 8, hy = y >> 8;
    if (__builtin_expect((hx | hy) == 0, 1)) return z;
    const unsigned hi = spread16(hx | (hy << 16));
    return z | (((hi & 0xFFFFu) | (hi >> 15)) << 16);
}

// The grid over the bulk of the points: cell coordinate = (p - lo) * scale.
struct Grid {
    float lox, loy, sx, sy;
};

// Cell of a point: Z-order of (cell_bits + 1) / 2 bits in x and cell_bits / 2
// in y; moving points of a mixed set (split) take the upper half of the
// cells, so that leaves hold points of one kind.
__device__ __forceinline__ unsigned cell_of(const Grid& G, int cell_bits, bool split, bool moves,
                                            float x, float y) {
    const int bits = split ? cell_bits - 1 : cell_bits;
    const int bx = (bits + 1) / 2, by = bits / 2;
    const float fx = __builtin_amdgcn_fmed3f((x - G.lox) * G.sx, 0.0f, static_cast<float>((1 << bx) - 1));
    const float fy = __builtin_amdgcn_fmed3f((y - G.loy) * G.sy, 0.0f, static_cast<float>((1 << by) - 1));
    const unsigned c = z_order(static_cast<unsigned>(fx), static_cast<unsigned>(fy));
    return c | (split && moves ? 1u << bits : 0u);
}

struct PointIn {
    const float *x, *y, *vx, *vy;  // vx, vy may be nullptr
    const unsigned char* valid;    // may be nullptr
    int n;
    float mid;                     // moving points are sorted and bounded by their positions at this time
};

__device__ __forceinline__ bool point_ok(const PointIn& in, int i) {
    bool ok = isfinite(in.x[i]) && isfinite(in.y[i]);
    if (in.vx) ok = ok && isfinite(in.vx[i]);
    if (in.vy) ok = ok && isfinite(in.vy[i]);
    if (in.valid) ok = ok && in.valid[i] != 0;
    return ok;
}

__device__ __forceinline__ bool point_moves(const PointIn& in, int i) {
    return (in.vx && in.vx[i] != 0.0f) || (in.vy && in.vy[i] != 0.0f);
}

// One coordinate's range from a 64-point sample (one wave, all lanes), one from
// each 1/64 of the set, at even or uneven places: the 1/16 and 15/16 quantiles of
// the valid samples (all of them where those are equal), widened by 1/4 of
// their distance on both sides; returns (lo, length).
__device__ float2 sample_range(const PointIn& in, const float* a, bool uneven) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int part = in.n / WAVE;
    const int i = static_cast<int>(static_cast<long long>(lane) * in.n / WAVE) +
                  (uneven ? static_cast<int>(((lane * 0x9E3779B1u >> 16) * static_cast<unsigned>(part)) >> 16) : 0);
    const bool ok = in.n > 0 && point_ok(in, i);
    const float v = ok ? a[i] : INFINITY;
    const int count = __popcll(__ballot(ok));
    int rank = 0;
#pragma unroll
    for (int j = 0; j < WAVE; ++j) {
        const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
        rank += (w < v || (w == v && j < lane)) ? 1 : 0;
    }
    if (count == 0) return make_float2(0.0f, 0.0f);
    auto at = [&](int r) {
        return __shfl(v, __ffsll(static_cast<long long>(__ballot(rank == r))) - 1);
    };
    float lo = at(count / 16), hi = at(count - 1 - count / 16);
    if (lo == hi) {
        lo = at(0);
        hi = at(count - 1);
    }
    const float wide = 0.25f * (hi - lo);
    return make_float2(lo - wide, (hi + wide) - (lo - wide));
}

// The ranges of samples 0 and 1 (even places in x, y), 2 and 3 (uneven ones), to
// the waves' slots.
__device__ __forceinline__ void sample_ranges(const PointIn& in, float2* range) {
    const int wid = threadIdx.x / WAVE;
    if (wid >= 4) return;
    const float2 r = sample_range(in, wid & 1 ? in.y : in.x, wid >= 2);
    if ((threadIdx.x & (WAVE - 1)) == 0) range[wid] = r;
}

// The grid of nx x ny cells over the sampled ranges: the even sample's, unless
// the uneven one shows more than twice as much.  (Sets that alternate between
// sources, the sensors of a vehicle or the rings of a sweep, at a period that
// divides n / 64 show one of them only at even places.)  Neither side of the range
// is taken as less than 1/16 of the other: along a wall the points of a leaf
// would otherwise be close across it and far apart along it (8192 points of a
// straight wall 20 m away, 2 cm thick: leaves 0.5 m long).
__device__ __forceinline__ Grid make_grid(const float2* range, int nx, int ny) {
    const float2 x = range[2].y > 2.0f * range[0].y ? range[2] : range[0];
    const float2 y = range[3].y > 2.0f * range[1].y ? range[3] : range[1];
    auto axis = [](float2 a, float least, int cells, float& lo, float& s) {
        const float span = fmaxf(a.y, least);
        lo = a.x - 0.5f * (span - a.y);
        s = span > 0.0f && span < 1e30f ? static_cast<float>(cells) / span : 0.0f;
    };
    Grid g;
    axis(x, y.y < 1e30f ? y.y * 0.0625f : 0.0f, nx, g.lox, g.sx);
    axis(y, x.y < 1e30f ? x.y * 0.0625f : 0.0f, ny, g.loy, g.sy);
    return g;
}

// Leaf over the points at(k) = (x, y, vx, vy), k < LEAF_POINTS (any repeated):
// the point nearest to the centre of their bounding box represents the leaf;
// radius = the largest distance to it.  Moving points: the box and the radius
// are those of time mid, in the nearest point's choice a velocity difference
// counts as the way it makes in mid; vel = the representative's velocity, rv =
// the largest velocity difference, mid, so that radius + rv |t - mid| bounds
// the distances at time t.
template <bool MOVING, typename At>
__device__ __forceinline__ void make_leaf(At&& at, float mid, float4& leaf, float4& vel) {
    float4 p[LEAF_POINTS];
    float x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
    float u0 = INFINITY, u1 = -INFINITY, w0 = INFINITY, w1 = -INFINITY;
#pragma unroll
    for (int k = 0; k < LEAF_POINTS; ++k) {
        p[k] = at(k);
        const float x = MOVING ? p[k].x + p[k].z * mid : p[k].x, y = MOVING ? p[k].y + p[k].w * mid : p[k].y;
        x0 = fminf(x0, x);
        x1 = fmaxf(x1, x);
        y0 = fminf(y0, y);
        y1 = fmaxf(y1, y);
        if (MOVING) {
            u0 = fminf(u0, p[k].z);
            u1 = fmaxf(u1, p[k].z);
            w0 = fminf(w0, p[k].w);
            w1 = fmaxf(w1, p[k].w);
        }
    }
    const float cx = 0.5f * x0 + 0.5f * x1, cy = 0.5f * y0 + 0.5f * y1;
    const float cu = 0.5f * u0 + 0.5f * u1, cw = 0.5f * w0 + 0.5f * w1;
    float best = INFINITY;
    float4 rep = p[0];
#pragma unroll
    for (int k = 0; k < LEAF_POINTS; ++k) {
        float dx = p[k].x - cx, dy = p[k].y - cy, d = dx * dx + dy * dy;
        if (MOVING) {
            dx = p[k].x + p[k].z * mid - cx;
            dy = p[k].y + p[k].w * mid - cy;
            const float du = (p[k].z - cu) * mid, dw = (p[k].w - cw) * mid;
            d = dx * dx + dy * dy + (du * du + dw * dw);
        }
        if (d < best) {
            best = d;
            rep = p[k];
        }
    }
    float r2 = 0.0f, v2 = 0.0f;
#pragma unroll
    for (int k = 0; k < LEAF_POINTS; ++k) {
        float dx = p[k].x - rep.x, dy = p[k].y - rep.y;
        if (MOVING) {
            // from the differences: points of equal velocity stay finite
            const float ux = p[k].z - rep.z, uy = p[k].w - rep.w;
            v2 = fmaxf(v2, ux * ux + uy * uy);
            dx += ux * mid;
            dy += uy * mid;
        }
        const float d = dx * dx + dy * dy;
        r2 = fmaxf(r2, MOVING && !(d == d) ? INFINITY : d);
    }
    // rounded up: the radius bounds the true distances (moving: the sum of a
    // difference and a way of opposite sign is exact to 2^-23 of the way)
    const float rv = __builtin_sqrtf(v2) * 1.00001f;
    leaf = make_float4(rep.x, rep.y, __builtin_sqrtf(r2) * 1.00001f, 0.0f);
    if (MOVING) {
        leaf.z += 2e-6f * rv * mid;
        vel = make_float4(rep.z, rep.w, rv, mid);
    }
}

// Super node over a wave's 64 leaves (lane = leaf, on: the leaf exists):
// centre and radius of a circle around them, and the largest speed.
template <bool MOVING>
__device__ __forceinline__ float4 make_super(bool on, float4 leaf, float4 vel) {
    const float x0 = wave_min(on ? leaf.x : INFINITY), x1 = -wave_min(on ? -leaf.x : INFINITY);
    const float y0 = wave_min(on ? leaf.y : INFINITY), y1 = -wave_min(on ? -leaf.y : INFINITY);
    const float cx = 0.5f * x0 + 0.5f * x1, cy = 0.5f * y0 + 0.5f * y1;
    const float dx = leaf.x - cx, dy = leaf.y - cy;
    // moving: at time 0
    float r = __builtin_sqrtf(dx * dx + dy * dy) * 1.00001f + (MOVING ? leaf.z + vel.z * vel.w * 1.00001f : leaf.z);
    if (MOVING) r = r == r ? r : INFINITY;  // velocities that overflow
    float v = 0.0f;
    if (MOVING) v = __builtin_sqrtf(vel.x * vel.x + vel.y * vel.y) * 1.00001f + vel.z;
    return make_float4(cx, cy, -wave_min(on ? -r : INFINITY), MOVING ? -wave_min(on ? -v : INFINITY) : 0.0f);
}

// ------------------------------------------------------------ few points
// Up to POINTS_DIRECT_MAX points keep the caller's order and get no
// hierarchy (the distance pass bounds every point of so small a set):
// order-preserving compaction, one point per thread.
__global__ __launch_bounds__(POINTS_DIRECT_MAX) void k_points_direct(PointIn in, PointSet out, bool moving) {
    __shared__ int wsum[POINTS_DIRECT_MAX / WAVE];
    const int t = threadIdx.x, lane = t & (WAVE - 1), wid = t / WAVE;
    const int i = min(t, max(in.n - 1, 0));
    float x = 0.f, y = 0.f, vx = 0.f, vy = 0.f;
    bool ok = t < in.n;
    if (in.n > 0) {
        x = in.x[i];
        y = in.y[i];
        vx = in.vx ? in.vx[i] : 0.0f;
        vy = in.vy ? in.vy[i] : 0.0f;
        const unsigned char va = in.valid ? in.valid[i] : 1;
        ok = ok && isfinite(x) && isfinite(y) && isfinite(vx) && isfinite(vy) && va != 0;
    }
    const unsigned long long m = __ballot(ok);
    if (lane == 0) wsum[wid] = __popcll(m);
    __syncthreads();
    int base = 0, total = 0;
    for (int w = 0; w < POINTS_DIRECT_MAX / WAVE; ++w) {
        base += w < wid ? wsum[w] : 0;
        total += wsum[w];
    }
    if (ok) {
        const int o = base + __popcll(m & ((1ull << lane) - 1ull));
        out.x[o] = x;
        out.y[o] = y;
        if (moving) {
            out.vx[o] = vx;
            out.vy[o] = vy;
            out.xyv[o] = make_float4(x, y, vx, vy);
        } else {
            out.xy[o] = make_float2(x, y);
        }
        out.idx[o] = i;
    }
    if (t == 0) *out.n_valid = total;
}

// ------------------------------------------------------------ one workgroup
// PT points per thread (n <= 1024 PT).  LDS: 16-bit cell counts (two per
// word) and the exclusive sums of their groups of 8; the counts' space is
// reused for the sorted points.  With PT <= 8 the points leave through LDS
// in sorted order, coalesced, and the leaves are formed there; above, the
// kernel stores every point's position (~0: masked) and k_points_place and
// k_points_nodes finish with many workgroups (one workgroup's scattered
// traffic would take longer than two more launches).
template <int PT, bool MOVING>
__global__ __launch_bounds__(SMALL_THREADS) void k_points_small(PointIn in, PointSet out, int cell_bits,
                                                                unsigned* __restrict__ positions) {
    constexpr bool PLACE = PT <= 8;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float2 range[4];
    __shared__ int wsum[SMALL_THREADS / WAVE];
    const int t = threadIdx.x, lane = t & (WAVE - 1), wid = t / WAVE;
    const int ncell = 1 << cell_bits;
    unsigned* hist = reinterpret_cast<unsigned*>(smem);
    uint4* h4 = reinterpret_cast<uint4*>(hist);
    unsigned short* group = reinterpret_cast<unsigned short*>(hist + ncell / 2);
    // the samples' ranges (waves 0 to 3) while the others clear the counts
    const int grid_bits = MOVING ? cell_bits - 1 : cell_bits;
    sample_ranges(in, range);
    for (int c = t; c < ncell / 8; c += SMALL_THREADS) h4[c] = make_uint4(0, 0, 0, 0);
    // every load of a batch is issued before the first result is used
    constexpr int HV = MOVING && PLACE ? PT : 1;  // velocities held
    constexpr int BATCH = PT < 8 ? PT : 8;
    float px[PT], py[PT], pvx[HV], pvy[HV];
    unsigned cr[PT];  // cell << 16 | rank within the cell; later the output position
    unsigned okm = 0, mvm = 0;
#pragma unroll
    for (int k0 = 0; k0 < PT; k0 += BATCH) {
        float vx[BATCH], vy[BATCH];
        unsigned char va[BATCH];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            const int i = min(t + (k0 + b) * SMALL_THREADS, max(in.n - 1, 0));
            if (in.n > 0) {
                px[k0 + b] = in.x[i];
                py[k0 + b] = in.y[i];
                vx[b] = MOVING && in.vx ? in.vx[i] : 0.0f;
                vy[b] = MOVING && in.vy ? in.vy[i] : 0.0f;
                va[b] = in.valid ? in.valid[i] : 1;
            }
        }
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            const int k = k0 + b;
            const bool ok = t + k * SMALL_THREADS < in.n && isfinite(px[k]) && isfinite(py[k]) && va[b] != 0 &&
                            (!MOVING || (isfinite(vx[b]) && isfinite(vy[b])));
            okm |= ok ? 1u << k : 0u;
            if (MOVING) mvm |= vx[b] != 0.0f || vy[b] != 0.0f ? 1u << k : 0u;
            if (HV == PT) {
                pvx[k % HV] = vx[b];
                pvy[k % HV] = vy[b];
            }
            if (MOVING && !PLACE) {  // the positions are only sorted by
                px[k] += vx[b] * in.mid;
                py[k] += vy[b] * in.mid;
            }
        }
    }
    __syncthreads();
    const Grid G = make_grid(range, 1 << ((grid_bits + 1) / 2), 1 << (grid_bits / 2));
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        cr[k] = 0;
        if (okm >> k & 1) {
            const unsigned c = cell_of(G, cell_bits, MOVING, mvm >> k & 1, HV == PT ? px[k] + pvx[k % HV] * in.mid : px[k],
                                       HV == PT ? py[k] + pvy[k % HV] * in.mid : py[k]);
            const unsigned sh = (c & 1) * 16;
            cr[k] = (c << 16) | ((atomicAdd(&hist[c >> 1], 1u << sh) >> sh) & 0xFFFFu);
        }
    }
    __syncthreads();
    // exclusive sums of the groups of 8 cells in cell order: wave w owns the
    // groups [w, w + 1) ncell / 128, one per lane and step (at most 8 steps)
    const int own = ncell / 8 / (SMALL_THREADS / WAVE);  // groups per wave
    const int per = min(own, WAVE);                      // groups per step
    int sum[8];
    int total = 0;
#pragma unroll
    for (int st = 0; st < 8; ++st) {
        sum[st] = 0;
        if (st * WAVE < own) {
            const uint4 v = lane < per ? h4[wid * own + st * WAVE + lane] : make_uint4(0, 0, 0, 0);
            // at most 2^15 points: the 16-bit halves cannot carry
            const unsigned p = v.x + v.y + v.z + v.w;
            sum[st] = static_cast<int>((p & 0xFFFFu) + (p >> 16));
            total += sum[st];
        }
    }
    total = wave_sum(total);
    if (lane == 0) wsum[wid] = total;
    __syncthreads();
    int base = 0, nv = 0;
    for (int w = 0; w < SMALL_THREADS / WAVE; ++w) {
        base += w < wid ? wsum[w] : 0;
        nv += wsum[w];
    }
#pragma unroll
    for (int st = 0; st < 8; ++st)
        if (st * WAVE < own) {
            const int incl = wave_scan(sum[st]);
            if (lane < per) group[wid * own + st * WAVE + lane] = static_cast<unsigned short>(base + incl - sum[st]);
            base += __builtin_amdgcn_readlane(incl, WAVE - 1);
        }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PT; ++k)
        if (okm >> k & 1) {
            // the group's sum, the counts of its cells before this one, the rank
            const unsigned c = cr[k] >> 16, in8 = c & 7;
            const uint4 v = h4[c >> 3];
            const unsigned odd = (in8 & 1) ? 0xFFFFu : 0u;  // the word of the cell: its lower half when odd
            const unsigned m0 = in8 >= 2 ? ~0u : odd, m1 = in8 >= 4 ? ~0u : in8 >= 2 ? odd : 0u;
            const unsigned m2 = in8 >= 6 ? ~0u : in8 >= 4 ? odd : 0u, m3 = in8 >= 6 ? odd : 0u;
            const unsigned p = (v.x & m0) + (v.y & m1) + (v.z & m2) + (v.w & m3);
            cr[k] = (cr[k] & 0xFFFFu) + group[c >> 3] + (p & 0xFFFFu) + (p >> 16);
        }
    if (t == 0) *out.n_valid = nv;
    if (!PLACE) {
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const int i = t + k * SMALL_THREADS;
            if (i < in.n) positions[i] = okm >> k & 1 ? cr[k] : ~0u;
        }
        return;
    }
    __syncthreads();  // the counts are no longer read
    // sorted points in LDS, WINDOW at a time, each array 16-byte aligned
    const int nleaf = (nv + LEAF_POINTS - 1) / LEAF_POINTS;
    constexpr int W = MOVING ? WINDOW / 2 : WINDOW;
    const int W8 = (min(W, in.n) + 7) & ~7;
    float* stx = reinterpret_cast<float*>(smem);
    float *sty = stx + W8, *stvx = stx + 2 * W8, *stvy = stx + 3 * W8;
    unsigned short* sti = reinterpret_cast<unsigned short*>(stx + (MOVING ? 4 : 2) * W8);
    for (int w0 = 0; w0 < nv; w0 += W) {
        const int wn = min(W, nv - w0);
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const int pos = static_cast<int>(cr[k]) - w0;
            if ((okm >> k & 1) && pos >= 0 && pos < wn) {
                stx[pos] = px[k];
                sty[pos] = py[k];
                if (MOVING) {
                    stvx[pos] = pvx[k % HV];
                    stvy[pos] = pvy[k % HV];
                }
                sti[pos] = static_cast<unsigned short>(t + k * SMALL_THREADS);
            }
        }
        __syncthreads();
        for (int j = t; j < wn; j += SMALL_THREADS) {
            out.x[w0 + j] = stx[j];
            out.y[w0 + j] = sty[j];
            if (MOVING) {
                out.vx[w0 + j] = stvx[j];
                out.vy[w0 + j] = stvy[j];
                out.xyv[w0 + j] = make_float4(stx[j], sty[j], stvx[j], stvy[j]);
            } else {
                out.xy[w0 + j] = make_float2(stx[j], sty[j]);
            }
            out.idx[w0 + j] = sti[j];
        }
        for (int l = t; l * LEAF_POINTS < wn; l += SMALL_THREADS) {
            // 8 points per leaf as two 16-byte reads per array
            float x[LEAF_POINTS], y[LEAF_POINTS], vx[LEAF_POINTS], vy[LEAF_POINTS];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                auto get = [&](const float* a, float* o) {
                    const float4 v = reinterpret_cast<const float4*>(a)[2 * l + h];
                    o[4 * h] = v.x;
                    o[4 * h + 1] = v.y;
                    o[4 * h + 2] = v.z;
                    o[4 * h + 3] = v.w;
                };
                get(stx, x);
                get(sty, y);
                if (MOVING) {
                    get(stvx, vx);
                    get(stvy, vy);
                }
            }
            const int m = min(LEAF_POINTS, wn - l * LEAF_POINTS);
            float4 leaf, vel = make_float4(0.f, 0.f, 0.f, 0.f);
            make_leaf<MOVING>([&](int k) {
                // past the end: the first point again
                const bool on = k < m;
                return make_float4(on ? x[k] : x[0], on ? y[k] : y[0], MOVING ? (on ? vx[k] : vx[0]) : 0.0f,
                                   MOVING ? (on ? vy[k] : vy[0]) : 0.0f);
            }, in.mid, leaf, vel);
            const int gl = w0 / LEAF_POINTS + l;
            out.leaf[gl] = leaf;
            if (MOVING) out.leaf_vel[gl] = vel;
        }
        __syncthreads();
    }
    for (int s = wid; s * SUPER_LEAVES < nleaf; s += SMALL_THREADS / WAVE) {
        const int l = s * SUPER_LEAVES + lane;
        const bool on = l < nleaf;
        const float4 leaf = on ? out.leaf[l] : make_float4(0.f, 0.f, 0.f, 0.f);
        const float4 vel = MOVING && on ? out.leaf_vel[l] : make_float4(0.f, 0.f, 0.f, 0.f);
        const float4 node = make_super<MOVING>(on, leaf, vel);
        if (lane == 0) out.super[s] = node;
    }
}

// ------------------------------------------------------------ many workgroups
// Cell counts cleared; the sample's range (workgroup 0).
__global__ __launch_bounds__(1024) void k_points_init(PointIn in, PointWork w) {
    for (int c = blockIdx.x * 1024 + threadIdx.x; c < (1 << LARGE_CELL_BITS); c += gridDim.x * 1024) w.cells[c] = 0;
    if (blockIdx.x == 0) sample_ranges(in, w.range);
}

// Cell and rank of every valid point ((~0, ~0) for the others).
__global__ __launch_bounds__(256) void k_points_count(PointIn in, PointWork w, bool moving) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= in.n) return;
    uint2 cr = make_uint2(~0u, ~0u);
    if (point_ok(in, i)) {
        const int bits = moving ? LARGE_CELL_BITS - 1 : LARGE_CELL_BITS;
        const Grid G = make_grid(w.range, 1 << ((bits + 1) / 2), 1 << (bits / 2));
        cr.x = cell_of(G, LARGE_CELL_BITS, moving, moving && point_moves(in, i),
                       in.x[i] + (in.vx ? in.vx[i] * in.mid : 0.0f), in.y[i] + (in.vy ? in.vy[i] * in.mid : 0.0f));
        cr.y = atomicAdd(&w.cells[cr.x], 1u);
    }
    w.cell_rank[i] = cr;
}

// Exclusive sums of 1024 cells per workgroup; totals to block_sums.
__global__ __launch_bounds__(1024) void k_points_scan(PointWork w) {
    __shared__ int sh[16];
    const int t = threadIdx.x, lane = t & (WAVE - 1), wid = t / WAVE;
    const int c = blockIdx.x * 1024 + t;
    const int v = static_cast<int>(w.cells[c]);
    const int incl = wave_scan(v);
    if (lane == WAVE - 1) sh[wid] = incl;
    __syncthreads();
    int base = 0, total = 0;
    for (int k = 0; k < 16; ++k) {
        base += k < wid ? sh[k] : 0;
        total += sh[k];
    }
    w.cells[c] = static_cast<unsigned>(base + incl - v);
    if (t == 0) w.block_sums[blockIdx.x] = total;
}

// Exclusive sums of the workgroup totals, and the valid count.
__global__ __launch_bounds__(256) void k_points_scan_top(PointWork w, int* n_valid) {
    __shared__ int sh[4];
    static_assert((1 << LARGE_CELL_BITS) / 1024 == 256, "one total per thread");
    const int t = threadIdx.x, lane = t & (WAVE - 1), wid = t / WAVE;
    const int v = w.block_sums[t];
    const int incl = wave_scan(v);
    if (lane == WAVE - 1) sh[wid] = incl;
    __syncthreads();
    int base = 0, total = 0;
    for (int k = 0; k < 4; ++k) {
        base += k < wid ? sh[k] : 0;
        total += sh[k];
    }
    w.block_sums[t] = base + incl - v;
    if (t == 0) *n_valid = total;
}

// Positions of the valid points from their cell's sum and rank.
__global__ __launch_bounds__(256) void k_points_positions(int n, PointWork w) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint2 cr = w.cell_rank[i];
    w.positions[i] = cr.x == ~0u ? ~0u : w.cells[cr.x] + cr.y + static_cast<unsigned>(w.block_sums[cr.x >> 10]);
}

// Every valid point to its position.
__global__ __launch_bounds__(256) void k_points_place(PointIn in, PointSet out,
                                                      const unsigned* __restrict__ positions, bool moving) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= in.n) return;
    const unsigned pos = positions[i];
    const float x = in.x[i], y = in.y[i];
    const float vx = in.vx ? in.vx[i] : 0.0f, vy = in.vy ? in.vy[i] : 0.0f;
    if (pos == ~0u) return;
    out.x[pos] = x;
    out.y[pos] = y;
    if (moving) {
        out.vx[pos] = vx;
        out.vy[pos] = vy;
        out.xyv[pos] = make_float4(x, y, vx, vy);
    } else {
        out.xy[pos] = make_float2(x, y);
    }
    out.idx[pos] = i;
}

// One wave per super node: lane = leaf.
template <bool MOVING>
__global__ __launch_bounds__(WAVE) void k_points_nodes(PointSet out, float mid) {
    const int nv = *out.n_valid;
    const int nleaf = (nv + LEAF_POINTS - 1) / LEAF_POINTS;
    if (static_cast<int>(blockIdx.x) * SUPER_LEAVES >= nleaf) return;
    const int l = blockIdx.x * SUPER_LEAVES + threadIdx.x;
    const bool on = l < nleaf;
    float4 leaf = make_float4(0.f, 0.f, 0.f, 0.f), vel = leaf;
    if (on) {
        const int j0 = l * LEAF_POINTS;
        make_leaf<MOVING>([&](int k) {
            const int j = min(j0 + k, nv - 1);
            if (MOVING) return out.xyv[j];
            const float2 o = out.xy[j];
            return make_float4(o.x, o.y, 0.0f, 0.0f);
        }, mid, leaf, vel);
        out.leaf[l] = leaf;
        if (MOVING) out.leaf_vel[l] = vel;
    }
    const float4 node = make_super<MOVING>(on, leaf, vel);
    if (threadIdx.x == 0) out.super[blockIdx.x] = node;
}

// Cells of the one-workgroup grid: about eight per point, since points
// crowd on walls (at least 256, the multiple of 16 cells per wave that the
// scan needs; at most 2^16, 128 KB).
int small_cell_bits(int n) {
    int b = 8;
    while (b < 16 && (1 << b) < 8 * n) ++b;
    return b;
}

size_t small_lds(int n, int cell_bits, bool moving) {
    const size_t hist = (sizeof(unsigned short) << cell_bits) + (sizeof(unsigned short) << cell_bits) / 8;
    if (n > 8 * SMALL_THREADS) return hist;
    const int W = moving ? WINDOW / 2 : WINDOW;
    const size_t W8 = static_cast<size_t>(((n < W ? n : W) + 7) & ~7);
    const size_t stage = W8 * ((moving ? 4 : 2) * sizeof(float) + sizeof(unsigned short));
    return ((hist > stage ? hist : stage) + 15) & ~static_cast<size_t>(15);
}

template <bool MOVING>
hipError_t launch_nodes(const PointSet& out, int n, float mid, hipStream_t s) {
    const int nsuper = (n + LEAF_POINTS * SUPER_LEAVES - 1) / (LEAF_POINTS * SUPER_LEAVES);
    hipLaunchKernelGGL((k_points_nodes<MOVING>), dim3(nsuper), dim3(WAVE), 0, s, out, mid);
    return hipGetLastError();
}

template <int PT, bool MOVING>
hipError_t launch_small(const PointIn& in, const PointSet& out, unsigned* positions, hipStream_t s) {
    const int bits = small_cell_bits(in.n);
    const size_t lds = small_lds(in.n, bits, MOVING);
    hipLaunchKernelGGL((k_points_small<PT, MOVING>), dim3(1), dim3(SMALL_THREADS), lds, s, in, out, bits,
                       positions);
    if (PT > 8) {
        hipLaunchKernelGGL(k_points_place, dim3((in.n + 255) / 256), dim3(256), 0, s, in, out, positions, MOVING);
        return launch_nodes<MOVING>(out, in.n, in.mid, s);
    }
    return hipGetLastError();
}

template <bool MOVING>
hipError_t launch_small_m(const PointIn& in, const PointSet& out, unsigned* positions, hipStream_t s) {
    const int pt = (in.n + SMALL_THREADS - 1) / SMALL_THREADS;
    if (pt <= 4) return launch_small<4, MOVING>(in, out, positions, s);
    if (pt <= 8) return launch_small<8, MOVING>(in, out, positions, s);
    return launch_small<32, MOVING>(in, out, positions, s);
}

}  // namespace

// Dynamic LDS beyond the default limit, on the current device (set_points
// would pay 14 us for it in each call).
hipError_t points_setup() {
    const void* k[] = {reinterpret_cast<const void*>(k_points_small<4, false>),
                       reinterpret_cast<const void*>(k_points_small<8, false>),
                       reinterpret_cast<const void*>(k_points_small<32, false>),
                       reinterpret_cast<const void*>(k_points_small<4, true>),
                       reinterpret_cast<const void*>(k_points_small<8, true>),
                       reinterpret_cast<const void*>(k_points_small<32, true>)};
    for (const void* f : k) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 152 * 1024);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

size_t points_work_bytes(int n) {
    if (n <= 8 * SMALL_THREADS) return 0;
    const size_t positions = sizeof(unsigned) * static_cast<size_t>(n);
    if (n <= POINTS_SMALL_MAX) return positions;
    return positions + sizeof(uint2) * static_cast<size_t>(n) + sizeof(unsigned) * (1 << LARGE_CELL_BITS) +
           sizeof(int) * 256 + sizeof(float) * 64;
}

hipError_t launch_points(const float* x, const float* y, const float* vx, const float* vy,
                         const unsigned char* valid, int n, float mid, const PointSet& out, void* work, hipStream_t s) {
    const PointIn in{x, y, vx, vy, valid, n, mid};
    const bool moving = vx || vy;
    if (n <= POINTS_DIRECT_MAX) {
        hipLaunchKernelGGL(k_points_direct, dim3(1), dim3(POINTS_DIRECT_MAX), 0, s, in, out, moving);
        return hipGetLastError();
    }
    PointWork w;
    char* p = static_cast<char*>(work);
    w.cell_rank = reinterpret_cast<uint2*>(p);  // first: 8-byte aligned
    if (n > POINTS_SMALL_MAX) p += sizeof(uint2) * static_cast<size_t>(n);
    w.positions = reinterpret_cast<unsigned*>(p);
    if (n <= POINTS_SMALL_MAX)
        return moving ? launch_small_m<true>(in, out, w.positions, s) : launch_small_m<false>(in, out, w.positions, s);
    p += sizeof(unsigned) * static_cast<size_t>(n);
    w.cells = reinterpret_cast<unsigned*>(p);
    p += sizeof(unsigned) * (1 << LARGE_CELL_BITS);
    w.block_sums = reinterpret_cast<int*>(p);
    p += sizeof(int) * 256;
    w.range = reinterpret_cast<float2*>((reinterpret_cast<uintptr_t>(p) + 7) & ~static_cast<uintptr_t>(7));
    const dim3 g((n + 255) / 256), b(256);
    hipLaunchKernelGGL(k_points_init, dim3(64), dim3(1024), 0, s, in, w);
    hipLaunchKernelGGL(k_points_count, g, b, 0, s, in, w, moving);
    hipLaunchKernelGGL(k_points_scan, dim3((1 << LARGE_CELL_BITS) / 1024), dim3(1024), 0, s, w);
    hipLaunchKernelGGL(k_points_scan_top, dim3(1), dim3(256), 0, s, w, out.n_valid);
    hipLaunchKernelGGL(k_points_positions, g, b, 0, s, n, w);
    hipLaunchKernelGGL(k_points_place, g, b, 0, s, in, out, w.positions, moving);
    return moving ? launch_nodes<true>(out, n, mid, s) : launch_nodes<false>(out, n, mid, s);
}

}  // namespace emppi
