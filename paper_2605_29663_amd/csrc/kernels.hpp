// Internal interface between the C ABI layer and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace emppi {

constexpr int WAVE = 64;
constexpr int DMIN_TILE = 1024;      // points staged in LDS per tile
// Bounding hierarchy over the spatially ordered points (kernels_points.hip).
// 8 points per leaf: with 16, the leaves that survive a pose's test hold
// about twice as many points, with 4 the leaf tests cost as much as the
// point tests they save.  64 leaves per super node: one per lane.
constexpr int LEAF_POINTS = 8;
constexpr int SUPER_LEAVES = 64;
// Sets without a hierarchy: bounding all of 512 points takes a pose 8 lane
// batches, about as many as the hierarchy's tests and the points they leave,
// and the order costs set_points 4 us.
constexpr int POINTS_DIRECT_MAX = 512;
constexpr int POINTS_SMALL_MAX = 1 << 15;  // sets prepared by one workgroup
constexpr int MPPI_MAX_T_DEV = 128;  // horizon capacity (MPPI_MAX_T of the C ABI)
// Per-step result record: u*_0, u*_1, u*_2, valid, J_nom (noise-free cost of
// the validated nominal), then padding.
constexpr int OUT_FLOATS = 8;

// Step parameters as the kernels see them (POD, passed by value).
struct StepArgs {
    int K, Kpad, T, nu, model, state_offset;
    float dt, lambda, wheelbase;
    float sigma[3], umin[3], umax[3];
    float d_safe, w_coll, w_rep, w_inf, w_goal, w_ctrl[3], goal[2];
    float q0[3];
    uint64_t seed, step, stream;
    const float2* path;  // guidance waypoints (planning frame)
    int n_path;
    float w_path;
};

// Valid obstacle points, compacted in spatial order (the count lives on the
// device so that a mask change needs no host round trip), with their
// bounding hierarchy: leaf l covers points [8 l, 8 l + 8): (x, y) of one of
// them, the largest distance from it to the others, unused; leaf_vel: that
// point's velocity, the largest velocity difference to it, and the time at
// which the points were sorted and the leaf's distance holds; super node s
// covers leaves [64 s, 64 s + 64): centre and radius of a circle around
// them at time 0, and their largest speed.
struct PointArgs {
    const float* x;
    const float* y;
    const float* vx;  // nullptr for static point sets
    const float* vy;
    const int* idx;   // caller's index of each compacted point
    const int* n_valid;
    const float2* xy;        // static sets: (x, y) of each point
    const float4* xyv;       // moving sets: (x, y, vx, vy)
    const float4* leaf;      // nullptr: no hierarchy (at most POINTS_DIRECT_MAX points)
    const float4* leaf_vel;  // moving sets only
    const float4* super;
};

// The same buffers as set_points fills them.
struct PointSet {
    float *x, *y, *vx, *vy;
    int *idx, *n_valid;
    float2* xy;   // one of xy and xyv
    float4 *xyv, *leaf, *leaf_vel, *super;
};

// Workspace of the many-workgroup preparation.
struct PointWork {
    unsigned* positions;  // output position per point, ~0 if masked (above 8192 points)
    uint2* cell_rank;     // this and the rest above POINTS_SMALL_MAX
    unsigned* cells;
    int* block_sums;
    float2* range;  // sampled ranges (lo, length)
};
size_t points_work_bytes(int n);
hipError_t points_setup();  // once per device, before the first launch_points
hipError_t launch_points(const float* x, const float* y, const float* vx, const float* vy,
                         const unsigned char* valid, int n, float mid, const PointSet& out, void* work, hipStream_t s);

// Bounds of a footprint's signed distance on a grid of cells in the body
// frame, at the head of a device buffer that the cells follow.  A cell is one
// word, (v, gx, gy) in bits 0-15, 16-23 and 24-31 (gx, gy signed): est = base
// + quantum v + (gx, gy) / 127 . offset from the centre is the distance up to
// err_linear + c (err_cell - err_linear) / 7, where c is v's lowest 3 bits (the
// others are the distance at the centre, 8 quantum the step).  c = 0 where the
// distance is linear in the cell; 1 .. 6 where it bends slowly (beside a
// corner, the more the nearer); 7 with no gradient elsewhere: err_cell is half
// the cell's diagonal, and the distance changes by at most the way travelled.
// The grid covers the footprint's
// bounding box and a margin around it, in which every border cell's lower
// bound is positive; a point outside projects onto the grid's rectangle,
// which is convex, so with the distance a to the projection and the
// projection's bounds [lb, ub] its distance lies in
// [sqrt(lb^2 + a^2), ub + a].  That interval is as wide as the margin; far[k]
// bounds points outside closely: in directions u (from the box's centre) of
// the k-th of FAR_BINS intervals of the pseudo-angle (far_bin), the footprint
// reaches at most v . u + eps, where v is one of its corners, so the distance
// of a point b at |b| u lies in [|b| - v . u - eps, |b - v|].
constexpr int FAR_BINS = 64;
struct FootHead {
    float cx, cy;      // centre of the bounding box
    float radius;      // of a circle around (cx, cy) that holds the footprint
    float centre_d;    // signed distance at (cx, cy), rounded up
    float reach;       // largest distance of the footprint from the body origin
    float sx, sy;      // cells per metre
    float ox, oy;      // cell coordinate of the body origin
    float dx, dy;      // metres per cell
    float base, quantum, err_cell, err_linear;
    int nx, ny;
    int pad_[15];
};
struct FootTable : FootHead {
    float4 far[FAR_BINS];  // v (from the centre), eps, unused
};
static_assert(sizeof(FootTable) == 128 + 16 * FAR_BINS, "the cells start on 128 bytes of the buffer");
constexpr int FOOT_CELLS = 4096;  // most cells of a table (16 KB of LDS)
inline size_t foot_table_bytes() { return sizeof(FootTable) + sizeof(uint32_t) * FOOT_CELLS; }
constexpr int FOOT_EDGES = 64, FOOT_BOXES = 32;  // most edges of a polygon, boxes of a cover
// Fill the table at `table`, from its head, the point-wise tables of the
// footprint (launch_sdf_points) and a polygon's vertices.
hipError_t launch_foot_table(int kind, const FootHead& head, FootTable* table, const float4* tab_a,
                             const float4* tab_b, const float2* verts, int count, hipStream_t s);

// Time of pose g for moving points: h = (g / div) % mod, t = (h + off) dt.
struct PoseTime {
    int div, mod, off;
    float dt;
};

// Order-preserving keys of the signed squared distance s: the unsigned order
// of key(s) is the order of s (sign bit flipped for s >= 0, all bits for
// s < 0).  Chunks of points merge their minima with atomicMin on these keys
// (exact and order-independent, hence deterministic); with the argmin, the
// 64-bit key is key(s) << 32 | point index, so ties go to the lowest index.
constexpr unsigned int DKEY_INIT = 0xFF800000u;                 // key(+inf)
constexpr unsigned long long DKEY64_INIT = 0xFF800000FFFFFFFFull;  // (+inf, index -1)

__device__ __forceinline__ unsigned int dkey(float s) {
    const unsigned int u = __float_as_uint(s);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float dkey_value(unsigned int k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
// Signed distance sign(s) sqrt|s| of a merged key (one square root per pose).
__device__ __forceinline__ float dkey_distance(unsigned int k) {
    const float sq = dkey_value(k);
    return sq < 0.0f ? -__builtin_sqrtf(-sq) : __builtin_sqrtf(sq);
}

// The distance pass evaluates every point (kernels_sdf_every.hip) where that is
// faster than the bounded search (cull_device.hpp): (10.75 padded + 6) / 64
// instructions per pose and point, against about 1000 per pose (static sets; up
// to 4000 moving ones) and some 6 us more for the search's chain of phases, which
// weigh the more the fewer poses there are.  Microseconds, every point / search,
// of 1280, 5120 and 81920 poses: 4 edges, 1000 points 8 / 12, 11 / 16, 69 / 82,
// 2000 points 12 / 12, 17 / 15, 129 / 73; 16 edges, 300 points 10 / 10, 14 / 14,
// 85 / 72, 600 points 11 / 12, 20 / 16, 152 / 77; moving, 8 edges, 1000 points
// 12 / 16, 18 / 27, 132 / 210, 16 edges, 600 points 11 / 15, 21 / 25, 158 / 157.
// Above 16 primitives a lane's share of the work is too long a chain for few
// poses (32 edges, 300 points: 12 / 10, 22 / 14).
constexpr int EVERY_MAX_POINTS = 2048;
inline bool dmin_every(int padded, int n_points, long long npose, bool moving) {
    double limit = 50000.0;
    if (padded <= 16) limit = npose <= 2048 ? 100000.0 : moving ? 80000.0 : npose <= 8192 ? 60000.0 : limit;
    return n_points <= EVERY_MAX_POINTS && n_points * (10.75 * padded + 6.0) <= limit;
}

// One launch of the fused transform + signed distance + min-over-points
// stage over npose poses.  Search: a workgroup of `waves` waves takes `tiles`
// tiles of poses_per_wave poses per wave; the point hierarchy is split into
// nchunk ranges of `supers` super nodes.  Every point: one lane (group) per
// pose, `block` threads, nchunk chunks of `chunk` points.  Each (pose, chunk
// or range) minimum is merged into key[g] (or key64[g]).
struct DminLaunch {
    const float4* poses;
    int npose;
    PoseTime pt;
    PointArgs pts;
    bool every;
    int waves, poses_per_wave, tiles, supers;
    int block, chunk;
    int nchunk;
    int kind;          // 0 polygon, 1 rectangle cover
    const float2* verts;  // polygon, padded to `padded` vertices and to 16, 32 or 64 (repeats of v0)
    const float4* rects;  // rectangle cover, padded to `padded` boxes (repeats of box 0)
    const FootTable* foot;  // bound table of that footprint
    int padded;
    bool argmin;
    unsigned int* key;         // [npose], initialised to DKEY_INIT
    unsigned long long* key64; // [npose], initialised to DKEY64_INIT (argmin)
};

hipError_t launch_dmin(const DminLaunch& L, hipStream_t s);
hipError_t launch_dmin_every(const DminLaunch& L, hipStream_t s);
int dmin_padded_count(int kind, int count);  // bucket a footprint size is padded to

hipError_t launch_key_init(unsigned int* key, unsigned long long* key64, int n, hipStream_t s);
hipError_t launch_dmin_finalize(const unsigned int* key, const unsigned long long* key64, int npose,
                                float* d_out, int* idx_out, hipStream_t s);

hipError_t launch_sdf_points(int kind, const float* px, const float* py, int n,
                             const float4* tab_a, const float4* tab_b, int count, float* out,
                             hipStream_t s);

struct RolloutOut {
    const float* useq = nullptr;  // [K][T][nu] given control sequences (no noise), or nullptr
    float* eps_ws;   // [T][nu][Kpad] (may be nullptr with useq)
    float4* poses;   // [T][Kpad]
    float* jbase;    // [Kpad]
    unsigned int* key;          // [T][Kpad] distance keys to initialise (or nullptr)
    unsigned long long* key64;  // [T][Kpad] (argmin variant, or nullptr)
    float* diag_poses;  // [K][T][4] or nullptr
    float* diag_eps;    // [K][T][nu]
    float* diag_u;      // [K][T][nu]
};

hipError_t launch_rollout(const StepArgs& P, const float* U, const RolloutOut& o, hipStream_t s);

hipError_t launch_cost(const StepArgs& P, const unsigned int* key, const unsigned long long* key64,
                       const float* jbase, float* jt, float* diag_dmin, int* diag_argmin,
                       hipStream_t s);

hipError_t launch_update(const StepArgs& P, const float* jt, const float* eps_ws, const float* U,
                         float* Unew, float* diag_w, hipStream_t s);

hipError_t launch_nominal(const StepArgs& P, const float* Unew, float4* nom_poses,
                          unsigned int* key_nom, hipStream_t s);

hipError_t launch_finalize(const StepArgs& P, int validate, const unsigned int* key_nom,
                           const float4* nom, const float* Unew, float* U, float* out,
                           float* diag_unew, float* diag_dnom, float* diag_jnom, hipStream_t s);

// Small steps (the single-scene path): cost + update in one launch when
// cost_update_fused(Kpad, T), and nominal + validation distances +
// validation in one single-workgroup launch when the footprint needs one lane
// per pose (polygons of up to 16 vertices, rectangle covers) and T N
// (padded primitives) <= VAL_SMALL_MAX_PAIRS.  Bit-identical to the separate
// launches.
constexpr int COST_UPDATE_MAX_KPAD = 512;               // LDS: 21 Kpad floats' worth
constexpr long long COST_UPDATE_MAX_POSES = 1ll << 15;  // Kpad T: every workgroup decodes them all
inline bool cost_update_fused(int Kpad, int T) {
    return Kpad <= COST_UPDATE_MAX_KPAD && static_cast<long long>(Kpad) * T <= COST_UPDATE_MAX_POSES;
}
constexpr int VAL_SMALL_THREADS = 1024;
constexpr long long VAL_SMALL_MAX_PAIRS = 1ll << 18;
hipError_t launch_cost_update(const StepArgs& P, const unsigned int* key,
                              const unsigned long long* key64, const float* jbase,
                              const float* eps_ws, const float* U, float* Unew, float* jt,
                              float* diag_w, float* diag_dmin, int* diag_argmin, hipStream_t s);
bool validate_small_supported(int kind, int padded);
hipError_t launch_validate_small(const StepArgs& P, int kind, int padded, const PointArgs& pts,
                                 const float2* verts, const float4* rects, const float* Unew,
                                 float* U, float* out, float* diag_unew, float* diag_dnom,
                                 float* diag_jnom, hipStream_t s);

// ---------------------------------------------------------------- batched path
// Per-step arguments of one scene (refreshed by one host-to-device copy per
// step, so a captured graph replays with new poses, seeds and nominals).
struct SceneStep {
    StepArgs P;
    float* U;  // the scene's T x nu nominal (device), updated in place
};

// Static per-scene workspaces.
struct SceneBufs {
    float* eps_ws;   // [T][nu][Kpad]
    float4* poses;   // [T][Kpad]
    float* jbase;    // [Kpad]
    float* jt;       // [Kpad]
    unsigned int* key;      // [T*Kpad] distance keys
    float* unew;     // [T][nu]
    float4* nom;     // [T]
    unsigned int* key_nom;  // [T]
    float* out;      // OUT_FLOATS floats
    int validate;    // run Algorithm 1 step 4 for this scene
};

// One (scene, pass) for the persistent signed-distance kernel.
struct SceneDmin {
    const float4* poses;
    int npose;
    PoseTime pt;
    PointArgs pts;
    int chunk;
    int kind, padded;
    const float2* verts;
    const float4* rects;
    const FootTable* foot;
    unsigned int* key;
};

// One workgroup's share of the batched bounded search: `tiles` tiles of
// SEARCH_WAVES P consecutive poses of SceneDmin sd from g0.
struct SearchItem {
    int sd, g0, P, tiles;
};
constexpr int SEARCH_WAVES = 8;  // waves per workgroup
// Kernel variant of the search: evaluator (edges or boxes per lane) and
// static or moving points.
constexpr int SEARCH_CLASSES = 10;
inline int search_class(int kind, int padded, bool moving) {
    const int e = kind == 1 ? (padded <= 16 ? 3 : 4) : padded <= 16 ? 0 : padded <= 32 ? 1 : 2;
    return 2 * e + (moving ? 1 : 0);
}

// One work item: pose tile [g0, g0 + blockDim) of SceneDmin sd against the
// compacted points [c0, c1) (clipped to the valid count on the device).
struct DminItem {
    int sd, g0, c0, c1;
};

// Register class of a footprint bucket (padded primitive count) in the
// persistent kernel, each compiled for the occupancy its largest bucket
// allows without spilling in the point loop: 0 polygons of 3..8 vertices
// (6 waves per SIMD), 1 polygons of 9..16 (4 waves), 2 polygons padded to
// 18..30 with a lane pair per pose (4 waves), 3 polygons padded to 32 with a
// lane pair per pose (3 waves), 4 rectangle covers up to 12 boxes (8
// waves), 5 larger covers (2 waves), 6 polygons padded to 36..64 with a lane
// quad per pose (3 waves).
constexpr int DMIN_CLASSES = 7;
inline int dmin_class(int kind, int padded) {
    if (kind == 1) return padded <= 12 ? 4 : 5;
    return padded <= 8 ? 0 : padded <= 16 ? 1 : padded <= 30 ? 2 : padded <= 32 ? 3 : 6;
}
// Lanes that share one pose in a register class.
constexpr int dmin_class_lanes(int cls) { return cls == 2 || cls == 3 ? 2 : cls == 6 ? 4 : 1; }

hipError_t launch_batch_reset(int* counters, int n, hipStream_t s);
hipError_t launch_rollout_batched(const SceneStep* steps, const SceneBufs* bufs, const int2* blk,
                                  int nblk, hipStream_t s);
hipError_t launch_dmin_persistent(int cls, int block, int grid, const SceneDmin* sds,
                                  const DminItem* items, int n_items, int* counter, hipStream_t s);
hipError_t launch_search_batched(int cls, const SceneDmin* sds, const SearchItem* items, int n_items,
                                 hipStream_t s);
hipError_t launch_cost_batched(const SceneStep* steps, const SceneBufs* bufs, const int2* blk,
                               int nblk, hipStream_t s);
hipError_t launch_update_batched(const SceneStep* steps, const SceneBufs* bufs, const int2* blk,
                                 int nblk, hipStream_t s);
hipError_t launch_nominal_batched(const SceneStep* steps, const SceneBufs* bufs, int n,
                                  hipStream_t s);
hipError_t launch_finalize_batched(const SceneStep* steps, const SceneBufs* bufs, int n,
                                   hipStream_t s);
// Diagnostics of one scene of the last batched step in the caller's [r][h]
// layouts (any output may be nullptr): d_min decoded from the merged keys,
// scored poses, clipped perturbations, J~, the updated nominal, d_nom
// (validation pass) and J_nom.
struct SceneDiag {
    float *d_min, *poses, *eps, *J, *U_upd, *d_nom, *J_nom;
};
hipError_t launch_scene_diag(const SceneBufs& B, int K, int Kpad, int T, int nu,
                             const SceneDiag& d, hipStream_t s);
// Workgroups of k_dmin_persistent<cls> (block threads) resident per compute
// unit on the current device, from the occupancy calculator (registers and
// the LDS tile); 0 on error.
int dmin_persistent_blocks_per_cu(int cls, int block);
int dmin_persistent_lanes_per_pose(int cls);

// ---------------------------------------------------------------- hybrid modes
constexpr int HYB_MAX_MODES = 8;

// Mode selection and actuator post-processing of one hybrid-mode cycle
// (Algorithm 2, steps 2 and 3), from the per-mode result records.
struct HybridArgs {
    int n_modes, m_prev, tau_cool, cool_max;
    float lambda_switch, v_min, w_min, noise_v, noise_w;
    int model[HYB_MAX_MODES];
    int nu[HYB_MAX_MODES];
};

// res = (u*_0, u*_1, u*_2, m*, tau_cool', safe_stop, Jbar(m*), 0).
hipError_t launch_hybrid_select(const float* out, const HybridArgs& a, float* res, hipStream_t s);

}  // namespace emppi
