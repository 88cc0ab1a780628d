// Batched bounded search of the distance pass: one workgroup per item, the
// search of cull_device.hpp on the item's scene.
#include "cull_device.hpp"

namespace emppi {

namespace {

// The items are queued longest first and are many times the resident
// workgroups, so the dispatcher balances scenes of uneven cost.
template <typename Eval, bool MOVING>
__global__ __launch_bounds__(SEARCH_WAVES * WAVE) __attribute__((amdgpu_waves_per_eu(Eval::WAVES)))
void k_search_b(const SceneDmin* __restrict__ sds, const SearchItem* __restrict__ items) {
    extern __shared__ __align__(16) unsigned char lds[];
    const SearchItem it = items[blockIdx.x];
    const SceneDmin& S = sds[it.sd];
    const CullArgs A{S.poses, S.npose, S.pt, S.pts, S.foot, S.key, nullptr};
    cull_block<Eval, MOVING, false>(A, S.verts, S.rects, S.padded, it.g0, SEARCH_WAVES * it.P, it.P, it.tiles,
                                    0, 0x7FFFFFFF, lds);
}

using SearchKernel = void (*)(const SceneDmin*, const SearchItem*);
constexpr SearchKernel SEARCH[SEARCH_CLASSES] = {
    k_search_b<EvalPoly<1>, false>, k_search_b<EvalPoly<1>, true>, k_search_b<EvalPoly<2>, false>,
    k_search_b<EvalPoly<2>, true>,  k_search_b<EvalPoly<4>, false>, k_search_b<EvalPoly<4>, true>,
    k_search_b<EvalRect<1>, false>, k_search_b<EvalRect<1>, true>, k_search_b<EvalRect<2>, false>,
    k_search_b<EvalRect<2>, true>};

}  // namespace

hipError_t launch_search_batched(int cls, const SceneDmin* sds, const SearchItem* items, int n_items,
                                 hipStream_t s) {
    if (n_items <= 0) return hipSuccess;
    if (cls < 0 || cls >= SEARCH_CLASSES) return hipErrorInvalidValue;
    hipLaunchKernelGGL(SEARCH[cls], dim3(n_items), dim3(SEARCH_WAVES * WAVE),
                       cull_lds_bytes(SEARCH_WAVES, cls & 1, false), s, sds, items);
    return hipGetLastError();
}

}  // namespace emppi
