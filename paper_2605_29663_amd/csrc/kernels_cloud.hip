// Point-cloud pre-processing (Section "Problem Statement": the obstacle set
// is the local point cloud restricted to a height band and downsampled to a
// fixed budget N).  One representative per occupied planar voxel (its
// lowest-index point), the N nearest representatives if there are more, in
// input order, padded with invalid slots.  Every decision is an exact
// integer or single-precision comparison, so the result does not depend on
// thread scheduling.
//
// The points are read once; after that the work is per voxel.  The range of
// the robot holds (2 r_max / voxel)^2 voxels, mostly far fewer than the
// points' hash table would have slots: then the voxels are a plain grid of
// lowest indices, in the L2, and a point costs one read and at times one
// atomic.  The budget's cut is found from one histogram of the
// representatives' ranges and an exact selection within one bin, and the kept
// points' bits, one per input point, give the input order by population
// counts.  What bounds it is the chain of six small launches.  2^20 points in
// 24 x 24 m, range 10 m, voxel 0.1 m, budget 8192: 116 -> 59 us with the call's overhead, 38 of them in
// the kernels (insertion 19), against nine launches with a hash insertion of
// 24 us and four histograms and a three-level scan over all the points.
#include <algorithm>
#include <climits>

#include "cloud.hpp"

namespace emppi {

namespace {

constexpr unsigned long long CELL_NONE = ~0ull;
// key of a cell without a point: above every squared range (the ranges are
// finite non-negative floats, whose bits stay below 0x7F800000)
constexpr uint32_t CLOUD_NONE = 0xFFFFFFFFu;
constexpr int CELL_BIAS = 1 << 30;  // voxel coordinates are stored biased, never all ones

// MurmurHash3's 64-bit finaliser (Appleby), used to spread voxel keys over
// the open-addressing table.
__device__ __forceinline__ uint32_t mix64(unsigned long long k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return static_cast<uint32_t>(k);
}

__device__ __forceinline__ float range2(const CloudArgs& a, float x, float y) {
    const float dx = x - a.cx, dy = y - a.cy;
    return dx * dx + dy * dy;
}

// Range bin of squared-range bits u <= umax (monotone): 128 bins an octave of
// the squared range for 8 octaves down from the largest, 32 for 24 more, then
// one.  With all of them in the first 16 octaves a range limit far above the
// points' ranges (1e4 m, points within 40 m) put most representatives into the
// last bin, which one workgroup then sorted out: 2^20 points 1180 us a call
// against 155.
__device__ __forceinline__ int range_bin(uint32_t u, uint32_t umax) {
    const int d = static_cast<int>((umax - u) >> 16);  // below 255 x 128
    return d < 1024 ? CLOUD_BINS - 1 - d : d < 4096 ? 1023 - ((d - 1024) >> 2) : 255 - ((d - 4096) >> 7);
}
static_assert(CLOUD_BINS == 2048, "1024 + 768 + at most 224 bins");

__global__ void k_cloud_init(CloudWork w, int words) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < w.cells) {
        if (w.nx == 0) w.keys[s] = CELL_NONE;
        w.first[s] = INT_MAX;
    }
    if (s < words) w.kept[s] = 0;
    if (s < CLOUD_BINS) w.hist[s] = 0;
    if (s < 8) w.state[s] = 0;
}

// Height band, range and finiteness test; the point's voxel keeps the minimum
// index of its points.  The grid is limited and its threads stride over the
// points, so that the indices rise with time: most points then find a lower
// index of their voxel and need no atomic (2^20 points in 31000 voxels: 22.6
// us with a thread per point, 19.2 so).  The reads before the atomics are plain
// cached ones: a slot's key is set once and its index only decreases, so a
// stale value costs an atomic and changes nothing.
constexpr int INSERT_BLOCKS = 1024;

__global__ __launch_bounds__(256) void k_cloud_insert(CloudArgs a, CloudWork w) {
    const int step = gridDim.x * 256;
    int i = blockIdx.x * 256 + threadIdx.x;
    float x = 0.f, y = 0.f, z = NAN;
    if (i < a.m) {
        x = a.xyz[3 * i];
        y = a.xyz[3 * i + 1];
        z = a.xyz[3 * i + 2];
    }
    for (; i < a.m; i += step) {
        float xn = 0.f, yn = 0.f, zn = NAN;
        const int in = i + step;
        if (in < a.m) {
            xn = a.xyz[3 * in];
            yn = a.xyz[3 * in + 1];
            zn = a.xyz[3 * in + 2];
        }
        const float r2 = range2(a, x, y);
        const bool ok = isfinite(x) && isfinite(y) && isfinite(z) && z >= a.z_min && z <= a.z_max &&
                        r2 <= a.rmax2;
        if (ok) {
            const int ix = static_cast<int>(floorf(x / a.voxel));
            const int iy = static_cast<int>(floorf(y / a.voxel));
            uint32_t slot;
            if (w.nx > 0) {
                // the grid's margins hold every point in range (the host's
                // rule); the limits only keep any other from leaving it
                slot = static_cast<uint32_t>(min(max(iy - w.y0, 0), w.ny - 1)) * static_cast<uint32_t>(w.nx) +
                       static_cast<uint32_t>(min(max(ix - w.x0, 0), w.nx - 1));
            } else {
                const unsigned long long key =
                    (static_cast<unsigned long long>(static_cast<uint32_t>(ix + CELL_BIAS)) << 32) |
                    static_cast<uint32_t>(iy + CELL_BIAS);
                const uint32_t mask = static_cast<uint32_t>(w.cells) - 1;
                slot = mix64(key) & mask;
                // the table holds at least twice as many slots as points: a
                // free slot is always reached
                for (;;) {
                    unsigned long long cur = w.keys[slot];
                    if (cur == CELL_NONE) cur = atomicCAS(&w.keys[slot], CELL_NONE, key);
                    if (cur == CELL_NONE || cur == key) break;
                    slot = (slot + 1) & mask;
                }
            }
            if (w.first[slot] > i) atomicMin(&w.first[slot], i);
        }
        x = xn;
        y = yn;
        z = zn;
    }
}

// Squared range of every voxel's representative, and their histogram.
__global__ __launch_bounds__(256) void k_cloud_ranges(CloudArgs a, CloudWork w) {
    __shared__ int h[CLOUD_BINS];
    for (int k = threadIdx.x; k < CLOUD_BINS; k += 256) h[k] = 0;
    __syncthreads();
    const uint32_t umax = __float_as_uint(a.rmax2);
    for (int c = blockIdx.x * 256 + threadIdx.x; c < w.cells; c += gridDim.x * 256) {
        const int i = w.first[c];
        uint32_t u = CLOUD_NONE;
        if (i != INT_MAX) {
            u = __float_as_uint(range2(a, a.xyz[3 * i], a.xyz[3 * i + 1]));
            atomicAdd(&h[range_bin(u, umax)], 1);
        }
        w.key[c] = u;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < CLOUD_BINS; k += 256)
        if (h[k]) atomicAdd(&w.hist[k], h[k]);
}

// The bin in which the cumulative count reaches need = min(representatives,
// n_out), by every workgroup for itself: representatives of the bins before
// it are kept, those of the bin are candidates.
__global__ __launch_bounds__(256) void k_cloud_mark(CloudArgs a, CloudWork w) {
    constexpr int PER = CLOUD_BINS / 256;
    __shared__ int wsum[4], s_bin, s_need;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    int c[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        c[k] = w.hist[PER * t + k];
        sum += c[k];
    }
    int incl = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wsum[wid] = incl;
    if (t == 0) s_bin = -1;
    __syncthreads();
    int before = incl - sum, total = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        before += k < wid ? wsum[k] : 0;
        total += wsum[k];
    }
    const int need = min(total, a.n_out);
    if (need > 0 && before < need && before + sum >= need) {
        int cum = before, b = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (cum < need && cum + c[k] >= need) {
                b = PER * t + k;
                s_need = need - cum;
            }
            cum += c[k];
        }
        s_bin = b;
    }
    __syncthreads();
    const int bin = s_bin;
    if (blockIdx.x == 0 && t == 0) {
        w.state[CLOUD_KEPT] = need;
        w.state[CLOUD_BIN] = bin;
        w.state[CLOUD_NEED] = bin >= 0 ? s_need : 0;
    }
    if (bin < 0) return;
    const uint32_t umax = __float_as_uint(a.rmax2);
    for (int k = blockIdx.x * 256 + t; k < w.cells; k += gridDim.x * 256) {
        const uint32_t u = w.key[k];
        if (u == CLOUD_NONE) continue;
        const int b = range_bin(u, umax);
        if (b > bin) continue;
        const int i = w.first[k];
        if (b < bin)
            atomicOr(&w.kept[i >> 5], 1u << (i & 31));
        else
            w.cand[atomicAdd(&w.state[CLOUD_CAND], 1)] = make_uint2(u, static_cast<uint32_t>(i));
    }
}

// The `need` candidates of lowest (range, index), one workgroup: up to 1024
// candidates by counting each one's predecessors, more by a radix selection
// of 12 bits a pass from the highest bit in which they differ (one bin's
// candidates share most of their 64 bits) until a bucket is taken whole.
constexpr int PICK_THREADS = 1024;
constexpr int PICK_BITS = 12;

__global__ __launch_bounds__(PICK_THREADS) void k_cloud_pick(CloudWork w) {
    __shared__ unsigned long long v[PICK_THREADS];
    __shared__ int h[1 << PICK_BITS];
    __shared__ int wsum[PICK_THREADS / 64];
    __shared__ unsigned long long s_prefix;
    __shared__ int s_need;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int n = w.state[CLOUD_CAND], need = w.state[CLOUD_NEED];
    auto value = [&](int k) {
        const uint2 q = w.cand[k];
        return (static_cast<unsigned long long>(q.x) << 32) | q.y;
    };
    auto keep = [&](unsigned long long x) {
        const uint32_t i = static_cast<uint32_t>(x);
        atomicOr(&w.kept[i >> 5], 1u << (i & 31));
    };
    if (n <= need) {
        for (int k = t; k < n; k += PICK_THREADS) keep(value(k));
        return;
    }
    if (n <= PICK_THREADS) {
        const unsigned long long x = t < n ? value(t) : 0;
        v[t] = x;
        __syncthreads();
        int rank = 0;
        for (int k = 0; k < n; ++k) rank += v[k] < x ? 1 : 0;
        if (t < n && rank < need) keep(x);
        return;
    }
    // bits that are not the same in all of them
    unsigned long long all = ~0ull, any = 0;
#pragma unroll 4
    for (int k = t; k < n; k += PICK_THREADS) {
        const unsigned long long x = value(k);
        all &= x;
        any |= x;
    }
    for (int o = 32; o > 0; o >>= 1) {
        all &= __shfl_xor(all, o);
        any |= __shfl_xor(any, o);
    }
    if (lane == 0) {
        v[wid] = all;
        v[PICK_THREADS / 64 + wid] = any;
    }
    __syncthreads();
    for (int k = 0; k < PICK_THREADS / 64; ++k) {
        all &= v[k];
        any |= v[PICK_THREADS / 64 + k];
    }
    int shift = max(64 - __clzll(all ^ any) - PICK_BITS, 0);  // (they differ: the indices do)
    unsigned long long mask = shift + PICK_BITS < 64 ? ~0ull << (shift + PICK_BITS) : 0;
    unsigned long long prefix = all & mask;
    int left = need;
    for (;;) {
        for (int k = t; k < (1 << PICK_BITS); k += PICK_THREADS) h[k] = 0;
        __syncthreads();
#pragma unroll 4
        for (int k = t; k < n; k += PICK_THREADS) {
            const unsigned long long x = value(k);
            if ((x & mask) == prefix) atomicAdd(&h[static_cast<int>(x >> shift) & ((1 << PICK_BITS) - 1)], 1);
        }
        __syncthreads();
        constexpr int PER = (1 << PICK_BITS) / PICK_THREADS;
        int c[PER], sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            c[k] = h[PER * t + k];
            sum += c[k];
        }
        int incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(incl, o);
            if (lane >= o) incl += u;
        }
        if (lane == 63) wsum[wid] = incl;
        __syncthreads();
        int before = incl - sum;
        for (int k = 0; k < wid; ++k) before += wsum[k];
        if (before < left && before + sum >= left) {
            int cum = before;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                if (cum < left && cum + c[k] >= left) {
                    s_prefix = prefix | (static_cast<unsigned long long>(PER * t + k) << shift);
                    s_need = cum + c[k] == left ? 0 : left - cum;  // 0: the bucket whole
                }
                cum += c[k];
            }
        }
        __syncthreads();
        prefix = s_prefix;
        left = s_need;
        __syncthreads();
        if (left == 0 || shift == 0) break;
        // the next bits (those of the last pass may overlap ones already fixed)
        mask = ~0ull << shift;
        shift = max(shift - PICK_BITS, 0);
    }
    const unsigned long long limit = prefix | ((1ull << shift) - 1);  // the need-th smallest value, or above it
#pragma unroll 4
    for (int k = t; k < n; k += PICK_THREADS) {
        const unsigned long long x = value(k);
        if (x <= limit) keep(x);
    }
}

// Kept points in input order: a workgroup takes 256 words of bits, counts
// those before it, and each thread writes the points of a byte.  Slots [kept,
// n_out) are cleared.
constexpr int OUT_THREADS = 1024, OUT_WORDS = OUT_THREADS / 4;

__global__ __launch_bounds__(OUT_THREADS) void k_cloud_out(CloudArgs a, CloudWork w, int words, float* ox,
                                                           float* oy, unsigned char* valid, int* n_kept) {
    __shared__ int wsum[2][OUT_THREADS / 64];
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int kept = w.state[CLOUD_KEPT];
    if (blockIdx.x == 0 && t == 0 && n_kept) *n_kept = kept;
    for (int g = kept + static_cast<int>(blockIdx.x) * OUT_THREADS + t; g < a.n_out; g += gridDim.x * OUT_THREADS) {
        ox[g] = 0.0f;
        oy[g] = 0.0f;
        valid[g] = 0;
    }
    const int w0 = blockIdx.x * OUT_WORDS;
    if (w0 >= words) return;
    int prev = 0;
    const uint4* q = reinterpret_cast<const uint4*>(w.kept);
#pragma unroll 8
    for (int k = t; k < w0 / 4; k += OUT_THREADS) {
        const uint4 b = q[k];
        prev += __popc(b.x) + __popc(b.y) + __popc(b.z) + __popc(b.w);
    }
    uint32_t bits = w0 + t / 4 < words ? (w.kept[w0 + t / 4] >> (8 * (t & 3))) & 255u : 0;
    const int own = __popc(bits);
    for (int o = 32; o > 0; o >>= 1) prev += __shfl_xor(prev, o);
    int incl = own;
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    if (lane == 63) {
        wsum[0][wid] = prev;
        wsum[1][wid] = incl;
    }
    __syncthreads();
    int pos = incl - own;
    for (int k = 0; k < OUT_THREADS / 64; ++k) pos += wsum[0][k] + (k < wid ? wsum[1][k] : 0);
    while (bits) {
        const int i = 32 * w0 + 8 * t + __ffs(bits) - 1;
        bits &= bits - 1;
        ox[pos] = a.xyz[3 * i];
        oy[pos] = a.xyz[3 * i + 1];
        valid[pos] = 1;
        ++pos;
    }
}

}  // namespace

// The whole pre-processing pass on stream s (6 launches; 2 when m = 0).
hipError_t launch_cloud(const CloudArgs& a, const CloudWork& w, float* ox, float* oy,
                        unsigned char* valid, int* n_kept, hipStream_t s) {
    const int m = a.m, words = (m + 127) / 128 * 4;
    const int n_init = std::max({m > 0 ? w.cells : 0, words, CLOUD_BINS});
    hipLaunchKernelGGL(k_cloud_init, dim3((n_init + 255) / 256), dim3(256), 0, s, w, words);
    if (m > 0) {
        hipLaunchKernelGGL(k_cloud_insert, dim3(std::min((m + 255) / 256, INSERT_BLOCKS)), dim3(256), 0, s, a, w);
        const dim3 g(std::min((w.cells + 255) / 256, 1024));
        hipLaunchKernelGGL(k_cloud_ranges, g, dim3(256), 0, s, a, w);
        hipLaunchKernelGGL(k_cloud_mark, g, dim3(256), 0, s, a, w);
        hipLaunchKernelGGL(k_cloud_pick, dim3(1), dim3(PICK_THREADS), 0, s, w);
    }
    const int blocks = std::max({(words + OUT_WORDS - 1) / OUT_WORDS, std::min((a.n_out + OUT_THREADS - 1) / OUT_THREADS, 256), 1});
    hipLaunchKernelGGL(k_cloud_out, dim3(blocks), dim3(OUT_THREADS), 0, s, a, w, words, ox, oy, valid, n_kept);
    return hipGetLastError();
}

}  // namespace emppi
