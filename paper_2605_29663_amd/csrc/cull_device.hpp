// Minimum signed distance over the points by bounded search, shared by the
// single-scene kernels and the batched one.
//
// Paper: Section "Batched Rollout and Distance Computation" (K x T x N
// queries, masked min).  The minimum is exact and the same bits as over all
// N points: a point is passed over only when a lower bound of its distance
// exceeds an upper bound of the pose's minimum.
//
// Evaluating every point costs about 11 instructions per (pose, point,
// edge); but only the few points next to the footprint can be nearest.  One
// workgroup takes NW x P poses (P per wave):
//   1. the workgroup drops the super nodes and then the leaves of the point
//      hierarchy that no pose of it can need, by bounding circles (rotation
//      invariant, so the poses' headings do not matter);
//   2. each wave, pose by pose, bounds the remaining leaves (one per lane)
//      and then the points of the leaves that are left (one per lane) by a
//      table of the footprint's signed distance in the body frame, about 25
//      instructions per 64 of them whatever the number of edges; the points
//      whose lower bound does not exceed the pose's upper bound (a handful)
//      are queued.  The table's bounds are loose far from the footprint; a pose
//      that keeps many leaves or points goes through them once more with the
//      corner that reaches furthest in the point's direction (FootTable::far);
//   3. when the queue fills, and at the end, the wave evaluates the queued
//      points exactly, 16 lanes per pose with the edges split among them
//      (the same operations on the same operands, hence the same bits, as an
//      evaluation of every point by one lane); many points of one pose go one
//      per lane where the footprint is boxes.
// It is bound by issue, about 800 vector instructions a pose at 39 to 54 % of the
// peak rate, and by the latency of the short dependent phases of step 2, hence
// many waves with few poses each, LDS for everything that is read at random
// and one pass over memory for the points.  Measured against evaluating every
// point (which ran at 86 - 92 % of the VALU issue rate): 81920 poses, 8192
// corridor points, 16 vertices 1800 -> 135 us; 204800 poses, 20000 points of
// which 30 % move, 4 boxes 2700 -> 500 us.  Sets that the bounds cannot thin out
// cost more than every point would: 20480 poses against 8192 points, with 16
// edges / 4 boxes, a field 60 / 57 us, a wall 20 m away 370 / 325, a ring of 5 m
// 640 / 365, all in one place 2740 / 815, every point evaluated 510 - 620 / 122
// (before FootTable::far: wall 2300 / 1760, ring 2430 / 2010).
#pragma once
#include "sdf_device.hpp"
#include "wave_ops.hpp"

namespace emppi {

constexpr int CULL_WAVES = 8;          // most waves per workgroup
constexpr int CULL_POSES = 16;         // most poses per wave and tile
constexpr int CULL_LEAVES = 320;       // leaves listed at a time (LDS)
constexpr int CULL_QUEUE = 256;        // queued points per wave (LDS)
constexpr int CULL_CHUNK = 2;          // 64-point batches bounded before they are filtered
constexpr int CULL_REFILTER = 8;       // a pose's queued points worth a second filter
// Queued points and kept leaves of a pose that call for the closer bounds: a
// field's or corridor's poses keep about 3 and 30 and pay only the comparison;
// 48 leaves instead of 128 took the corridor from 230 to 276 us a step.
constexpr int CULL_FAR = 48;
constexpr int CULL_FAR_LEAVES = 128;
constexpr int CULL_EACH = 24;          // a pose's queued points that are evaluated one per lane (boxes)
constexpr int CULL_SUPERS = 512;       // super nodes examined at a time

// LDS of a workgroup.
struct CullShared {
    float4 leaf[CULL_LEAVES];                 // x, y, radius, leaf index (no hierarchy: the static points)
    float4 far[FAR_BINS];                     // FootTable::far
    unsigned short supers[CULL_SUPERS];
    float group[8];                           // centre x, y, spread, tau centre, spread, max |tau|, table's centre x, y
    unsigned ub_super, ub_leaf;               // ordered keys of the workgroup's upper bounds
    int n_super, n_leaf, flags;
};
struct CullWave {
    float4 pose[CULL_POSES];
    float tau[CULL_POSES];
    float best[CULL_POSES];                   // signed squared distance so far
    float2 queue[CULL_QUEUE];                 // points (at the pose's time), pose after pose
    unsigned short leaf[CULL_LEAVES];         // list positions of the leaves a pose keeps
    unsigned short begin[CULL_POSES], end[CULL_POSES];  // each pose's part of the queue
};

// Order of the dynamic LDS: footprint table, CullShared, one CullWave per
// wave, then (moving points) the listed leaves' velocities, then (argmin) the
// queued points' caller's indices and those attaining the poses' minima.
__host__ __device__ inline size_t cull_lds_bytes(int nw, bool moving, bool argmin) {
    return sizeof(uint32_t) * FOOT_CELLS + sizeof(CullShared) + sizeof(CullWave) * nw +
           (moving ? sizeof(float4) * CULL_LEAVES : 0) + (argmin ? sizeof(int) * (CULL_QUEUE + CULL_POSES) * nw : 0);
}

// One launch's view of a pass: poses, points, footprint.
struct CullArgs {
    const float4* poses;
    int npose;
    PoseTime pt;
    PointArgs pts;
    const FootTable* foot;
    unsigned int* key;
    unsigned long long* key64;
};

// LDS writes of this wave are visible to its later reads (one wave's LDS
// operations complete in order; this keeps the compiler from reordering).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same value, opaque to the compiler: what is computed from it is not
// hoisted out of the loops around it (held across the whole search, the
// phases' invariant addresses cost more registers than they save
// instructions).
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ unsigned lanes_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(mask), 0));
}

// Signed distance of a signed square, to 1 ulp (for bounds).
__device__ __forceinline__ float signed_sqrt_fast(float s) {
    return copysignf(__builtin_amdgcn_sqrtf(fabsf(s)), s);
}

// Upper bounds are kept as unsigned keys in the order of the floats (dkey).
__device__ __forceinline__ float threshold(float ub, float slack) {
    // every bound and distance is computed with relative errors of a few
    // 2^-24 of the distance or of the footprint's size; 1e-4 covers them
    // with a wide margin (and rotations up to 1e-5 off unit length).  Errors of
    // the coordinates' size (a group's centre, a moving point's position) are in
    // the group's spread and in the caller's slack.
    return ub + 1e-4f * fabsf(ub) + slack;
}

// c^2 + s^2 of a rotation, up to this
constexpr float ROTATION_TOL = 1e-5f;

// Bounds of the signed distance from the footprint table for points given
// relative to the pose position.
struct PoseBounds {
    float ax, bx, ay, by, ox, oy;  // cell coordinates: fma(dx, ax, fma(dy, bx, ox)), ...
    float dx, dy, gdx, gdy, base, quantum, err_step, err_linear, mx, my;
    unsigned nx;

    __device__ __forceinline__ void init(const FootTable& F, float c, float s) {
        ax = c * F.sx;
        bx = s * F.sx;
        ay = -s * F.sy;
        by = c * F.sy;
        ox = F.ox;
        oy = F.oy;
        dx = F.dx;
        dy = F.dy;
        gdx = F.dx * (1.0f / 127.0f);
        gdy = F.dy * (1.0f / 127.0f);
        base = F.base;
        quantum = F.quantum;
        err_step = (F.err_cell - F.err_linear) * (1.0f / 7.0f);
        err_linear = F.err_linear;
        nx = F.nx;
        mx = static_cast<float>(F.nx) - 0.01f;
        my = static_cast<float>(F.ny) - 0.01f;
    }

    // For (c, s) of length k that is no rotation (the caller's poses may be
    // anything, a rotation rounded to 16 bits for one).  The evaluators then see
    // the footprint scaled by k (SCALED: a polygon, whose vertices are turned by
    // (c, s)) or the points scaled by k (a cover): the table at (c, s) / k^2,
    // its distances times k, or the table at (c, s), points k times as far apart.
    // Without bounds (NaN) where k is no size to calculate with.
    template <bool SCALED>
    __device__ __forceinline__ void rescale(float c, float s, float& pslack, float& apart) {
        const float k2 = __builtin_fmaf(c, c, s * s);
        const bool usable = k2 > 1e-6f && k2 < 1e6f;
        const float k = fabsf(k2 - 1.0f) <= ROTATION_TOL ? 1.0f : usable ? __builtin_amdgcn_sqrtf(k2) : NAN;
        if (SCALED) {
            const float inv = k == 1.0f ? 1.0f : 1.0f / k2;
            ax *= inv;
            bx *= inv;
            ay *= inv;
            by *= inv;
            dx *= k;
            dy *= k;
            gdx *= k;
            gdy *= k;
            base *= k;
            quantum *= k;
            err_step *= k;
            err_linear *= k;
        } else {
            base = k == k ? base : k;
            apart = wave_uniform(k);
        }
        pslack *= wave_uniform(fmaxf(k, 1.0f));
    }

    __device__ __forceinline__ void operator()(const uint32_t* cells, float px, float py, float& lb,
                                               float& ub) const {
        const float fx = __builtin_fmaf(px, ax, __builtin_fmaf(py, bx, ox));
        const float fy = __builtin_fmaf(px, ay, __builtin_fmaf(py, by, oy));
        const float qx = __builtin_amdgcn_fmed3f(fx, 0.0f, mx), qy = __builtin_amdgcn_fmed3f(fy, 0.0f, my);
        // within the grid for every input (of NaN, v_med3 returns the lower
        // limit), and the bounds of a NaN coordinate are NaN
        const uint32_t w = cells[__umul24(static_cast<unsigned>(qy), nx) + static_cast<unsigned>(qx)];
        const float tx = (__builtin_amdgcn_fractf(qx) - 0.5f) * gdx, ty = (__builtin_amdgcn_fractf(qy) - 0.5f) * gdy;
        float est = __builtin_fmaf(static_cast<float>(w & 0xFFFFu), quantum, base);
        est = __builtin_fmaf(static_cast<float>(static_cast<int>(w << 8) >> 24), tx, est);
        est = __builtin_fmaf(static_cast<float>(static_cast<int>(w) >> 24), ty, est);
        const float err = __builtin_fmaf(static_cast<float>(w & 7u), err_step, err_linear);
        const float l = est - err;
        lb = l;
        ub = est + err;
        if (__ballot(fx != qx || fy != qy)) {  // some point is off the grid
            const float gx = (fx - qx) * dx, gy = (fy - qy) * dy;
            const float a2 = __builtin_fmaf(gx, gx, gy * gy);
            lb = l > 0.0f ? __builtin_amdgcn_sqrtf(__builtin_fmaf(l, l, a2)) : l;
            ub += __builtin_amdgcn_sqrtf(a2);
        }
    }
};

// Interval of FootTable::far that holds the direction of (x, y): the
// pseudo-angle y / (|x| + |y|), continued over the left half plane, from -1 to 3.
__device__ __forceinline__ int far_bin(float x, float y) {
    const float t = y * __builtin_amdgcn_rcpf(fabsf(x) + fabsf(y));
    const float a = x >= 0.0f ? t : 2.0f - t;
    return static_cast<int>(__builtin_fmaf(a, FAR_BINS / 4.0f, FAR_BINS / 4.0f)) & (FAR_BINS - 1);  // (NaN: 0)
}

// Bounds of the signed distance from FootTable::far for a point relative to
// the pose q (a rotation).
__device__ __forceinline__ void far_bounds(const CullShared& S, float4 q, float px, float py, float& lb, float& ub) {
    const float x = __builtin_fmaf(q.z, px, __builtin_fmaf(q.w, py, -S.group[6]));
    const float y = __builtin_fmaf(q.z, py, __builtin_fmaf(-q.w, px, -S.group[7]));
    const float4 v = S.far[far_bin(x, y)];
    const float b2 = __builtin_fmaf(x, x, y * y);
    // (NaN where the square overflows: neither drops a point nor bounds)
    lb = (b2 - __builtin_fmaf(v.x, x, v.y * y)) * __builtin_amdgcn_rsqf(b2) - v.z;
    const float ex = x - v.x, ey = y - v.y;
    ub = __builtin_amdgcn_sqrtf(__builtin_fmaf(ex, ex, ey * ey));
}

// Exact evaluation of one point by a row of 16 lanes, each with 1 / 16 of
// the footprint in the pose's frame (the row's first lane returns the
// distance).  The search queues a handful of points per pose, so what counts
// is the set-up per pose and the registers it takes from the search's waves
// (6 per edge and lane), not the combine's dozen instructions per point.
constexpr int EVAL_LANES = 16;
constexpr int DPP_ROR1 = 0x121, DPP_ROR2 = 0x122, DPP_ROR4 = 0x124, DPP_ROR8 = 0x128;  // within a row

// Polygon of n <= 16 HB edges.  The edges above n (repeats of vertex 0) never
// cross the ray; their distance is made infinite, so that they are no minimum
// at any distance.
template <int HB>
struct EvalPoly {
    static constexpr int WAVES = HB <= 2 ? 6 : 4;  // per SIMD, without scratch in the loops
    static constexpr bool SCALED = true;           // PoseBounds::rescale
    static constexpr bool EACH = false;            // has each()
    PolyPart<HB, EVAL_LANES> F;
    __device__ __forceinline__ void init(const float2* verts, const float4*, int n, int part, float4 q) {
        F.init(verts, part * HB, q.z, q.w);
#pragma unroll
        for (int b = 0; b < HB; ++b)
            if (part * HB + b >= n) F.CV[b] = INFINITY;
    }
    __device__ __forceinline__ float operator()(float dx, float dy) const {
        float m;
        unsigned long long odd;
        F.eval(dx, dy, m, odd);
        // parity of the row's 16 lanes in the bit of its first lane
        odd ^= odd >> 8;
        odd ^= odd >> 4;
        odd ^= odd >> 2;
        odd ^= odd >> 1;
        const bool neg = __builtin_amdgcn_inverse_ballot_w64(odd);
        // the minima are non-negative: their integer order is their order
        int mi = __float_as_int(m);
        mi = min(mi, dpp_or<DPP_ROR8>(0x7FFFFFFF, mi));
        mi = min(mi, dpp_or<DPP_ROR4>(0x7FFFFFFF, mi));
        mi = min(mi, dpp_or<DPP_ROR2>(0x7FFFFFFF, mi));
        mi = min(mi, dpp_or<DPP_ROR1>(0x7FFFFFFF, mi));
        const float mm = __int_as_float(mi);
        return neg ? -mm : mm;
    }
};
// Cover of n <= 16 NB boxes (missing ones repeat box 0).
template <int NB>
struct EvalRect {
    static constexpr int WAVES = 6;
    static constexpr bool SCALED = false;
    static constexpr bool EACH = true;
    float4 bx[NB];
    float c, s;
    __device__ __forceinline__ void init(const float2*, const float4* rects, int n, int part, float4 q) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int k = part + j * EVAL_LANES;
            bx[j] = rects[k < n ? k : 0];
        }
        c = q.z;
        s = q.w;
    }
    __device__ __forceinline__ float operator()(float dx, float dy) const {
        const float px = __builtin_fmaf(c, dx, s * dy);
        const float py = __builtin_fmaf(c, dy, -(s * dx));
        float v = box_s(px, py, bx[0]);
#pragma unroll
        for (int j = 1; j < NB; ++j) v = fminf(v, box_s(px, py, bx[j]));
        v = fminf(v, dpp_or<DPP_ROR8>(v, v));
        v = fminf(v, dpp_or<DPP_ROR4>(v, v));
        v = fminf(v, dpp_or<DPP_ROR2>(v, v));
        v = fminf(v, dpp_or<DPP_ROR1>(v, v));
        return v;
    }
    // One point per lane, every box in turn.
    static __device__ __forceinline__ float each(const float4* __restrict__ rects, int n, float4 q, float dx, float dy) {
        const float px = __builtin_fmaf(q.z, dx, q.w * dy);
        const float py = __builtin_fmaf(q.z, dy, -(q.w * dx));
        float v = box_s(px, py, rects[0]);
        for (int j = 1; j < n; ++j) v = fminf(v, box_s(px, py, rects[j]));
        return v;
    }
};

enum { CULL_ANY = 1, CULL_SCALED = 2 };  // a finite pose exists; one whose (cos, sin) is no rotation

// `tiles` tiles of nw P poses of A from g0, gstep apart (P per wave, wave w the
// w-th P of a tile), against the leaves of the super nodes [s0, s1): each pose's minimum
// is merged into its key.  Every thread of the workgroup calls it.
template <typename Eval, bool MOVING, bool ARGMIN>
__device__ __forceinline__ void cull_block(const CullArgs& A, const float2* __restrict__ verts,
                                           const float4* __restrict__ rects, int nprim, int g0, int gstep, int P, int tiles,
                                           int s0, int s1, unsigned char* lds) {
    uint32_t* cells = reinterpret_cast<uint32_t*>(lds);
    CullShared& S = *reinterpret_cast<CullShared*>(lds + sizeof(uint32_t) * FOOT_CELLS);
    CullWave* waves = reinterpret_cast<CullWave*>(reinterpret_cast<unsigned char*>(&S) + sizeof(CullShared));
    const int nthreads = static_cast<int>(blockDim.x), nw = nthreads / WAVE;
    const int t = static_cast<int>(threadIdx.x), lane = t & (WAVE - 1);
    const int wid = __builtin_amdgcn_readfirstlane(t / WAVE);
    CullWave& Wv = waves[wid];
    float4* leaf_vel = reinterpret_cast<float4*>(waves + nw);
    int* ids = reinterpret_cast<int*>(leaf_vel + (MOVING ? CULL_LEAVES : 0));
    int* queue_id = ids + wid * CULL_QUEUE;
    int* besti_of = ids + nw * CULL_QUEUE;  // CULL_POSES a wave
    int* wave_besti = besti_of + wid * CULL_POSES;
    const FootTable& F = *A.foot;
    const int nv = *A.pts.n_valid;
    const int nleaf = (nv + LEAF_POINTS - 1) / LEAF_POINTS;
    s1 = min(s1, (nleaf + SUPER_LEAVES - 1) / SUPER_LEAVES);
    // without a hierarchy every point is a candidate of every pose; static
    // points are read from LDS
    const bool direct = A.pts.leaf == nullptr;
    float2* lds_xy = reinterpret_cast<float2*>(S.leaf);
    static_assert(sizeof(float2) * POINTS_DIRECT_MAX <= sizeof(float4) * CULL_LEAVES, "the points fit the list");

    // one lane: into the minimum of one of the wave's poses
    auto merge = [&](int o, float d, int id) {
        const float old = Wv.best[o];
        if (ARGMIN) {
            if (d < old || (d == old && d < INFINITY && id < wave_besti[o])) {
                Wv.best[o] = d;
                wave_besti[o] = id;
            }
        } else {
            Wv.best[o] = fminf(old, d);
        }
    };

    // ---- poses, footprint table, the group's bounding circle
    {
        const uint4* src = reinterpret_cast<const uint4*>(&F + 1);
        const int n16 = (F.nx * F.ny + 3) / 4;
        for (int i = t; i < n16; i += nthreads) reinterpret_cast<uint4*>(cells)[i] = src[i];
        if (t < FAR_BINS) S.far[t] = F.far[t];
        if (direct && !MOVING)
            for (int i = t; i < nv; i += nthreads) lds_xy[i] = A.pts.xy[i];
    }
    for (int tile = 0; tile < tiles; ++tile, g0 += gstep) {
    if (g0 >= A.npose) break;
    if (wid == 0) {
        const int ln = opaque(lane);
        float xmin = INFINITY, xmax = INFINITY, ymin = INFINITY, ymax = INFINITY;  // maxima negated
        float tmin = INFINITY, tmax = INFINITY;
        bool any = false, scaled = false;
        float ccx[CULL_WAVES * CULL_POSES / WAVE], ccy[CULL_WAVES * CULL_POSES / WAVE];
        bool ok[CULL_WAVES * CULL_POSES / WAVE];
#pragma unroll
        for (int k = 0; k < CULL_WAVES * CULL_POSES / WAVE; ++k) {
            const int p = ln + k * WAVE, g = g0 + p;
            ok[k] = false;
            if (p < nw * P) {
                const bool live = g < A.npose;
                const float4 q = live ? A.poses[g] : make_float4(NAN, 0.f, 1.f, 0.f);
                // a pose with a non-finite entry has no finite distance
                ok[k] = isfinite(q.x) && isfinite(q.y) && isfinite(q.z) && isfinite(q.w);
                const float tau = MOVING ? pose_tau(A.pt, live ? g : 0) : 0.0f;
                CullWave& O = waves[p / P];
                const int o = p % P;
                O.pose[o] = ok[k] ? q : make_float4(NAN, NAN, NAN, NAN);
                O.tau[o] = tau;
                O.best[o] = INFINITY;
                if (ARGMIN) besti_of[p / P * CULL_POSES + o] = -1;
                if (ok[k]) {
                    any = true;
                    // no rotation: the group's circles do not hold
                    if (!(fabsf(__builtin_fmaf(q.z, q.z, q.w * q.w) - 1.0f) <= ROTATION_TOL)) scaled = true;
                    ccx[k] = q.x + (q.z * F.cx - q.w * F.cy);
                    ccy[k] = q.y + (q.w * F.cx + q.z * F.cy);
                    xmin = fminf(xmin, ccx[k]);
                    xmax = fminf(xmax, -ccx[k]);
                    ymin = fminf(ymin, ccy[k]);
                    ymax = fminf(ymax, -ccy[k]);
                    tmin = fminf(tmin, tau);
                    tmax = fminf(tmax, -tau);
                }
            }
        }
        xmin = wave_min(xmin);
        xmax = -wave_min(xmax);
        ymin = wave_min(ymin);
        ymax = -wave_min(ymax);
        const float gx = 0.5f * xmin + 0.5f * xmax, gy = 0.5f * ymin + 0.5f * ymax;
        float spread = 0.0f;  // negated maximum of the squared distances
#pragma unroll
        for (int k = 0; k < CULL_WAVES * CULL_POSES / WAVE; ++k)
            if (ok[k]) spread = fminf(spread, -((ccx[k] - gx) * (ccx[k] - gx) + (ccy[k] - gy) * (ccy[k] - gy)));
        spread = __builtin_sqrtf(-wave_min(spread));
        float tc = 0.0f, ts = 0.0f, ta = 0.0f;
        if (MOVING) {
            tmin = wave_min(tmin);
            tmax = -wave_min(tmax);
            tc = 0.5f * tmin + 0.5f * tmax;
            ts = 0.5f * (tmax - tmin);
            ta = fmaxf(fabsf(tmin), fabsf(tmax));
        }
        const int fl = (__ballot(any) ? CULL_ANY : 0) | (__ballot(scaled) ? CULL_SCALED : 0);
        if (lane == 0) {
            S.group[0] = gx;
            S.group[1] = gy;
            // rounding of the centres (2^-24 of each coordinate) and of the moving
            // points' positions grows with the coordinates
            S.group[2] = spread * 1.0001f + (MOVING ? 2e-6f : 5e-7f) * (fabsf(gx) + fabsf(gy) + spread);
            S.group[3] = tc;
            S.group[4] = ts * 1.0001f;
            S.group[5] = ta * 1.0001f;
            S.group[6] = F.cx;
            S.group[7] = F.cy;
            S.flags = fl;
            S.ub_super = S.ub_leaf = DKEY_INIT;
            S.n_super = S.n_leaf = 0;
        }
    }
    __syncthreads();
    const int flags = __builtin_amdgcn_readfirstlane(S.flags);
    const float slack = 1e-4f * F.reach;
    if (flags & CULL_ANY) {
        const float gx = S.group[0], gy = S.group[1], spread = S.group[2];
        const float tc = S.group[3], ts = S.group[4], ta = S.group[5];
        const bool scaled = flags & CULL_SCALED;
        // distance bounds of a circle (x, y, r) to any pose of the group:
        // >= D - r - spread - radius and <= D + r + spread + centre_d
        const float lo_off = spread + F.radius, hi_off = spread + F.centre_d;
        // up to 64 leaves: list them as they are
        const bool few = s1 - s0 <= 1 || direct;
        if (!few && !scaled) {
            float m = INFINITY;
            for (int s = s0 + opaque(t); s < s1; s += nthreads) {
                const float4 c = A.pts.super[s];
                const float dx = c.x - gx, dy = c.y - gy;
                m = fminf(m, __builtin_sqrtf(dx * dx + dy * dy) + (c.z + c.w * ta) + hi_off);
            }
            m = wave_min(m);
            if (lane == 0) atomicMin(&S.ub_super, dkey(m));
        }
        // super nodes CULL_SUPERS at a time; their leaves listed at most
        // CULL_LEAVES at a time
        for (int sb = s0; sb < s1; sb += CULL_SUPERS) {
            if (!direct) __syncthreads();
            const float thr_s = scaled ? INFINITY : threshold(dkey_value(S.ub_super), slack);
            const int se = min(sb + CULL_SUPERS, s1);
            for (int s = sb + opaque(t); s < se && !direct; s += nthreads) {
                bool keep = true;
                if (!few && !scaled) {
                    const float4 c = A.pts.super[s];
                    const float dx = c.x - gx, dy = c.y - gy;
                    keep = !(__builtin_sqrtf(dx * dx + dy * dy) - (c.z + c.w * ta) - lo_off > thr_s);
                }
                if (keep) S.supers[atomicAdd(&S.n_super, 1)] = static_cast<unsigned short>(s - sb);
            }
            if (!direct) __syncthreads();
            const int ns = direct ? 1 : __builtin_amdgcn_readfirstlane(S.n_super);
            // the leaf nearest to the group bounds every pose's minimum
            if (!few && !scaled) {
                float m = INFINITY;
                for (int k = wid; k < ns; k += nw) {
                    const int l = (sb + S.supers[k]) * SUPER_LEAVES + opaque(lane);
                    if (l < nleaf) {
                        const float4 c = A.pts.leaf[l];
                        float x = c.x, y = c.y, r = 0.0f;
                        if (MOVING) {
                            const float4 v = A.pts.leaf_vel[l];
                            x = __builtin_fmaf(v.x, tc, x);
                            y = __builtin_fmaf(v.y, tc, y);
                            r = ts * (fabsf(v.x) + fabsf(v.y));
                        }
                        const float dx = x - gx, dy = y - gy;
                        m = fminf(m, __builtin_sqrtf(dx * dx + dy * dy) + r + hi_off);
                    }
                }
                m = wave_min(m);
                if (lane == 0) atomicMin(&S.ub_leaf, dkey(m));
                __syncthreads();
            }
            const float thr_l = scaled ? INFINITY : threshold(dkey_value(S.ub_leaf), slack);
            for (int k0 = 0; k0 < ns;) {
                // list leaves while the next super node's certainly fit
                int k1 = k0, nlist = 0;
                if (direct) {
                    k1 = 1;
                } else for (;;) {
                    nlist = __builtin_amdgcn_readfirstlane(S.n_leaf);
                    __syncthreads();
                    const int kn = min(ns, k1 + (CULL_LEAVES - nlist) / SUPER_LEAVES);
                    if (kn == k1) break;
                    for (int k = k1 + wid; k < kn; k += nw) {
                        const int l = (sb + S.supers[k]) * SUPER_LEAVES + opaque(lane);
                        bool keep = l < nleaf;
                        float4 c = make_float4(0.f, 0.f, 0.f, 0.f), v = c;
                        if (keep) {
                            c = A.pts.leaf[l];
                            if (MOVING) v = A.pts.leaf_vel[l];
                            if (!few && !scaled) {
                                float x = c.x, y = c.y, r = c.z;
                                if (MOVING) {
                                    x = __builtin_fmaf(v.x, tc, x);
                                    y = __builtin_fmaf(v.y, tc, y);
                                    r += v.z * (fabsf(tc - v.w) + ts) + ts * (fabsf(v.x) + fabsf(v.y));
                                }
                                const float dx = x - gx, dy = y - gy;
                                keep = !(__builtin_sqrtf(dx * dx + dy * dy) - r - lo_off > thr_l);
                            }
                        }
                        const unsigned long long mask = __ballot(keep);
                        int at = 0;
                        if (lane == 0) at = atomicAdd(&S.n_leaf, __popcll(mask));
                        at = __builtin_amdgcn_readfirstlane(at);
                        if (keep) {
                            const int o = at + static_cast<int>(lanes_below(mask));
                            S.leaf[o] = make_float4(c.x, c.y, c.z, __int_as_float(l));
                            if (MOVING) leaf_vel[o] = v;
                        }
                    }
                    k1 = kn;
                    __syncthreads();
                }
                k0 = k1;

                // ---- each wave: its poses against the listed leaves
                int p = 0, pf = 0;         // pose in progress, first pose with queued points
                int nq = 0, nq0 = 0, nkeep = 0, c0 = 0;  // queued in all, before this pose
                float ub = INFINITY, pslack = slack, tau = 0.0f, apart = 1.0f;
                float4 q = make_float4(0.f, 0.f, 1.f, 0.f);
                PoseBounds B;
                int far_min = 0;  // queued points of the pose that call for closer bounds
                bool fresh = true;
                while (pf < P) {
                    while (p < P) {
                        if (fresh) {
                            q = wave_uniform(Wv.pose[p]);
                            tau = MOVING ? wave_uniform(Wv.tau[p]) : 0.0f;
                            pslack = slack + (MOVING ? 2e-6f * (fabsf(q.x) + fabsf(q.y)) : 0.0f);
                            B.init(F, q.z, q.w);
                            if (__builtin_expect(scaled, 0)) B.template rescale<Eval::SCALED>(q.z, q.w, pslack, apart);
                            nkeep = 0;
                            c0 = 0;
                            nq0 = nq;
                            far_min = scaled ? CULL_QUEUE : CULL_FAR;
                            if (lane == 0) Wv.begin[p] = static_cast<unsigned short>(nq);
                            if (direct) {
                                fresh = false;
                                ub = signed_sqrt_fast(Wv.best[p]);
                                nkeep = (nv + LEAF_POINTS - 1) / LEAF_POINTS;
                            }
                            if (!(q.x == q.x)) {
                                // no finite distance
                                if (lane == 0) Wv.end[p] = static_cast<unsigned short>(nq);
                                ++p;
                                fresh = true;
                                continue;
                            }
                        }
                        if (fresh) {
                            // bounds of the listed leaves, one per lane
                            const int ln = opaque(lane);
                            float lbs[CULL_LEAVES / WAVE];
                            float m = INFINITY;
#pragma unroll
                            for (int b = 0; b < CULL_LEAVES / WAVE; ++b) {
                                lbs[b] = 0.0f;
                                if (b * WAVE < nlist) {
                                    const int i = min(b * WAVE + ln, nlist - 1);
                                    const float4 c = S.leaf[i];
                                    float x = c.x, y = c.y, r = c.z;
                                    if (MOVING) {
                                        const float4 v = leaf_vel[i];
                                        x = __builtin_fmaf(v.x, tau, x);
                                        y = __builtin_fmaf(v.y, tau, y);
                                        r = __builtin_fmaf(v.z, fabsf(tau - v.w), r);
                                    }
                                    float lb, u;
                                    B(cells, x - q.x, y - q.y, lb, u);
                                    lbs[b] = __builtin_fmaf(-r, apart, lb);
                                    m = fminf(m, u);
                                    // one batch at a time: interleaved, the
                                    // batches' registers would spill
                                    __builtin_amdgcn_sched_barrier(0);
                                }
                            }
                            ub = fminf(wave_min(m), signed_sqrt_fast(Wv.best[p]));
                            const float thr = threshold(ub, pslack);
#pragma unroll
                            for (int b = 0; b < CULL_LEAVES / WAVE; ++b)
                                if (b * WAVE < nlist) {
                                    const bool keep = b * WAVE + ln < nlist && !(lbs[b] > thr);
                                    const unsigned long long mask = __ballot(keep);
                                    if (keep)
                                        Wv.leaf[nkeep + lanes_below(mask)] = static_cast<unsigned short>(b * WAVE + ln);
                                    nkeep += __popcll(mask);
                                }
                            wave_lds_fence();
                            fresh = false;
                            if (__builtin_expect(nkeep > CULL_FAR_LEAVES && far_min < CULL_QUEUE, 0)) {
                                // most are far away, where the table's bounds
                                // say little: the closer ones
                                // (the pose again: it need not stay in registers)
                                const float4 qc = Wv.pose[p];
                                auto bounds = [&](int i, float& lb, float& u) {
                                    const float4 c = S.leaf[Wv.leaf[i]];
                                    float x = c.x, y = c.y, r = c.z;
                                    if (MOVING) {
                                        const float4 v = leaf_vel[Wv.leaf[i]];
                                        x = __builtin_fmaf(v.x, tau, x);
                                        y = __builtin_fmaf(v.y, tau, y);
                                        r = __builtin_fmaf(v.z, fabsf(tau - v.w), r);
                                    }
                                    far_bounds(S, qc, x - qc.x, y - qc.y, lb, u);
                                    lb -= r;
                                };
                                const int n = nkeep;
                                nkeep = 0;
                                for (int b = 0; b < n; b += WAVE) {
                                    const int i = b + opaque(lane);
                                    float lb, u;
                                    bounds(min(i, n - 1), lb, u);
                                    const unsigned short l = Wv.leaf[min(i, n - 1)];
                                    ub = fminf(ub, wave_min(u));
                                    const bool keep = i < n && !(lb > threshold(ub, pslack));
                                    const unsigned long long mask = __ballot(keep);
                                    if (keep) Wv.leaf[nkeep + lanes_below(mask)] = l;
                                    nkeep += __popcll(mask);
                                    wave_lds_fence();
                                }
                            }
                        }
                        // the points of the kept leaves, CULL_CHUNK batches of 64
                        // bounded before they are filtered
                        bool full = false;
                        while (c0 < nkeep * LEAF_POINTS) {
                            if (nq + CULL_CHUNK * WAVE > CULL_QUEUE) {
                                full = true;
                                break;
                            }
                            const int ln = opaque(lane);
                            float lbs[CULL_CHUNK];
                            float2 xy[CULL_CHUNK];
                            int idx[CULL_CHUNK];  // -1: no point
                            float m = INFINITY;
#pragma unroll
                            for (int k = 0; k < CULL_CHUNK; ++k) {
                                idx[k] = -1;
                                lbs[k] = 0.0f;
                                if (c0 + k * WAVE < nkeep * LEAF_POINTS) {
                                    const unsigned j = static_cast<unsigned>(c0 + k * WAVE + ln);
                                    if (j < static_cast<unsigned>(nkeep * LEAF_POINTS)) {
                                        unsigned i = j;
                                        if (!direct) {
                                            const unsigned l = __float_as_uint(S.leaf[Wv.leaf[j / LEAF_POINTS]].w);
                                            i = l * LEAF_POINTS + (j & (LEAF_POINTS - 1));
                                        }
                                        if (i < static_cast<unsigned>(nv)) {
                                            idx[k] = static_cast<int>(i);
                                            float x, y;
                                            if (MOVING) {
                                                const float4 o = A.pts.xyv[i];
                                                x = __builtin_fmaf(o.z, tau, o.x);
                                                y = __builtin_fmaf(o.w, tau, o.y);
                                            } else {
                                                const float2 o = direct ? lds_xy[i] : A.pts.xy[i];
                                                x = o.x;
                                                y = o.y;
                                            }
                                            xy[k] = make_float2(x, y);
                                            float u;
                                            B(cells, x - q.x, y - q.y, lbs[k], u);
                                            m = fminf(m, u);
                                        }
                                    }
                                }
                            }
                            ub = fminf(ub, wave_min(m));
                            const float thr = threshold(ub, pslack);
#pragma unroll
                            for (int k = 0; k < CULL_CHUNK; ++k)
                                if (c0 + k * WAVE < nkeep * LEAF_POINTS) {
                                    const bool keep = idx[k] >= 0 && !(lbs[k] > thr);
                                    const unsigned long long mask = __ballot(keep);
                                    if (keep) {
                                        const int o = nq + static_cast<int>(lanes_below(mask));
                                        Wv.queue[o] = xy[k];
                                        if (ARGMIN) queue_id[o] = A.pts.idx[idx[k]];
                                    }
                                    nq += __popcll(mask);
                                }
                            c0 += CULL_CHUNK * WAVE;
                        }
                        if (!full && nq - nq0 > CULL_REFILTER) {
                            // most were queued before the pose's bound was
                            // final: filter them once more
                            wave_lds_fence();
                            const float thr = threshold(ub, pslack);
                            const int n = nq;
                            nq = nq0;
                            for (int b = nq0; b < n; b += WAVE) {
                                const int ln = opaque(lane);
                                const int i = min(b + ln, n - 1);
                                const float2 o = Wv.queue[i];
                                const int id = ARGMIN ? queue_id[i] : 0;
                                float lb, u;
                                B(cells, o.x - q.x, o.y - q.y, lb, u);
                                const bool keep = b + ln < n && !(lb > thr);
                                const unsigned long long mask = __ballot(keep);
                                if (keep) {
                                    const int to = nq + static_cast<int>(lanes_below(mask));
                                    Wv.queue[to] = o;
                                    if (ARGMIN) queue_id[to] = id;
                                }
                                nq += __popcll(mask);
                            }
                        }
                        if (__builtin_expect(nq - nq0 > far_min, 0)) {
                            // still many: the closer bounds of far points
                            wave_lds_fence();
                            const float4 qc = Wv.pose[p];
                            const int n = nq;
                            nq = nq0;
                            for (int b = nq0; b < n; b += WAVE) {
                                const int i = b + opaque(lane);
                                const float2 o = Wv.queue[min(i, n - 1)];
                                const int id = ARGMIN ? queue_id[min(i, n - 1)] : 0;
                                float lb, u;
                                far_bounds(S, qc, o.x - qc.x, o.y - qc.y, lb, u);
                                ub = fminf(ub, wave_min(u));
                                const bool keep = i < n && !(lb > threshold(ub, pslack));
                                const unsigned long long mask = __ballot(keep);
                                if (keep) {
                                    const int to = nq + static_cast<int>(lanes_below(mask));
                                    Wv.queue[to] = o;
                                    if (ARGMIN) queue_id[to] = id;
                                }
                                nq += __popcll(mask);
                                wave_lds_fence();
                            }
                            if (4 * (nq - nq0) > 3 * (n - nq0)) far_min = CULL_QUEUE;  // of no use here
                            if (full && nq + CULL_CHUNK * WAVE <= CULL_QUEUE) continue;  // with the pose's other points
                        }
                        if constexpr (Eval::EACH)
                            if (__builtin_expect(nq - nq0 >= CULL_EACH, 0)) {
                                // many: one per lane costs 10 instructions a box
                                // for 64 of them (the row's 80 for 4)
                                wave_lds_fence();
                                const float4 qc = Wv.pose[p];
                                float best = INFINITY;
                                int besti = 0x7FFFFFFF;
                                const int ln = opaque(lane);
                                for (int b = nq0; b < nq; b += WAVE) {
                                    // (lanes past the end take the last point again)
                                    const int i = min(b + ln, nq - 1);
                                    const float2 o = Wv.queue[i];
                                    const float sd = Eval::each(rects, nprim, qc, o.x - qc.x, o.y - qc.y);
                                    if (ARGMIN) {
                                        const int id = queue_id[i];
                                        if (sd < best || (sd == best && id < besti)) {
                                            best = sd;
                                            besti = id;
                                        }
                                    } else {
                                        best = fminf(best, sd);
                                    }
                                }
                                const float d = wave_min(best);
                                if (ARGMIN) besti = static_cast<int>(wave_umin(best == d ? static_cast<unsigned>(besti) : ~0u));
                                if (ln == 0) merge(p, d, besti);
                                wave_lds_fence();
                                nq = nq0;
                                if (full && nq + CULL_CHUNK * WAVE <= CULL_QUEUE) {
                                    ub = fminf(ub, signed_sqrt_fast(Wv.best[p]));
                                    continue;  // with the pose's other points
                                }
                            }
                        if (lane == 0) Wv.end[p] = static_cast<unsigned short>(nq);
                        if (full) break;
                        ++p;
                        fresh = true;
                    }
                    wave_lds_fence();
                    // ---- exact distances of the queued points of poses [pf, pe),
                    // a row of lanes per pose (several for one or two poses)
                    const int pe = p < P ? p + 1 : P;
                    if (nq > 0)
                        for (int p0 = pf; p0 < pe; p0 += WAVE / EVAL_LANES) {
                            const int ln = opaque(lane);
                            const int np = pe - p0;
                            const int lsh = np <= 1 ? 6 : np <= 2 ? 5 : 4;
                            const int per = 1 << lsh;
                            const int slot = ln >> lsh;
                            const int pp = p0 + min(slot, np - 1);
                            const float4 qe = Wv.pose[pp];
                            int i = Wv.begin[pp] + (ln & (per - 1)) / EVAL_LANES;
                            const int e = slot < np ? Wv.end[pp] : 0;
                            Eval E;
                            E.init(verts, rects, nprim, ln & (EVAL_LANES - 1), qe);
                            float best = INFINITY;
                            int besti = 0x7FFFFFFF;
                            while (__ballot(i < e)) {
                                const bool on = i < e;
                                const int j = on ? i : 0;
                                const float2 o = Wv.queue[j];
                                const float sd = E(o.x - qe.x, o.y - qe.y);
                                if (ARGMIN) {
                                    // the lowest caller's index among equal distances
                                    const int id = queue_id[j];
                                    if (on && (sd < best || (sd == best && id < besti))) {
                                        best = sd;
                                        besti = id;
                                    }
                                } else {
                                    best = on ? fminf(best, sd) : best;
                                }
                                i += per / EVAL_LANES;
                            }
                            for (int o = EVAL_LANES; o < per; o <<= 1) {
                                const float ob = __shfl_xor(best, o);
                                if (ARGMIN) {
                                    const int oi = __shfl_xor(besti, o);
                                    if (ob < best || (ob == best && oi < besti)) {
                                        best = ob;
                                        besti = oi;
                                    }
                                } else {
                                    best = fminf(best, ob);
                                }
                            }
                            if (slot < np && (ln & (per - 1)) == 0) merge(pp, best, besti);
                        }
                    wave_lds_fence();
                    // a pose cut by the full queue goes on with its exact
                    // distance so far
                    pf = p;
                    nq = nq0 = 0;
                    if (p < P) {
                        if (lane == 0) Wv.begin[p] = 0;
                        ub = fminf(ub, signed_sqrt_fast(Wv.best[p]));
                    }
                }
                __syncthreads();
                if (t == 0) S.n_leaf = 0;
                __syncthreads();
            }
            __syncthreads();
            if (t == 0) S.n_super = 0;
        }
    }
    wave_lds_fence();
    const int ln = opaque(lane), g = g0 + wid * P + ln;
    if (ln < P && g < A.npose) {
        const float b = Wv.best[ln];
        if (ARGMIN) {
            const int i = wave_besti[ln];
            const unsigned idx = i < 0 ? 0xFFFFFFFFu : static_cast<unsigned>(i);
            atomicMin(&A.key64[g], (static_cast<unsigned long long>(dkey(b)) << 32) | idx);
        } else {
            atomicMin(&A.key[g], dkey(b));
        }
    }
    __syncthreads();  // the next tile's poses replace these
    }
}

}  // namespace emppi
