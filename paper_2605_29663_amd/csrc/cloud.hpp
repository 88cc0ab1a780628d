// Internal interface of the point-cloud pre-processing kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace emppi {

constexpr int CLOUD_MAX_POINTS = 1 << 20;
constexpr int CLOUD_BINS = 2048;         // of the squared range (range_bin)
constexpr int CLOUD_DENSE_MIN = 1 << 18;  // cells always held as a plain grid

struct CloudArgs {
    const float* xyz;  // m x 3, row-major
    int m;
    float cx, cy;      // robot position (planning frame)
    float z_min, z_max, rmax2, voxel;
    int n_out;
};

// Device workspace of one pre-processing call (sizes in elements).
struct CloudWork {
    int nx, ny, x0, y0;        // nx > 0: the cells are the voxels [x0, x0 + nx) x [y0, y0 + ny)
    unsigned long long* keys;  // nx == 0: the cells are a hash table's slots, these its keys (a power of two >= 2 m)
    int cells;
    int* first;                // cells: lowest point index of the voxel
    uint32_t* key;             // cells: squared range bits of that point, or CLOUD_NONE (in the keys' place)
    uint32_t* kept;            // one bit per point, a multiple of 4 words
    int* hist;                 // CLOUD_BINS: representatives per range bin
    int* state;                // 8 (CLOUD_*)
    uint2* cand;               // m at most: (range bits, point) of the bin that the budget cuts
};
enum { CLOUD_KEPT = 0, CLOUD_BIN = 1, CLOUD_NEED = 2, CLOUD_CAND = 3 };

hipError_t launch_cloud(const CloudArgs& a, const CloudWork& w, float* ox, float* oy,
                        unsigned char* valid, int* n_kept, hipStream_t s);

}  // namespace emppi
