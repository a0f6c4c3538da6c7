// Device code of a batch's groups (one orbital count and one kind each), shared
// by the kernel that runs one group and the one that runs several.
#pragma once

#include "mc_apply.h"
#include "mc_direct.h"
#include "mc_split.h"
#include "mc_tiles.h"

namespace mc {

constexpr int kBatchMaxN = 255;

// Work item i of a group: a tile of its instance.  j: position in the group,
// which only rises (prefix is non-decreasing and a worker visits items in
// increasing order, so the search resumes where it stopped).
template <int MT, int KIND, class PT>
__device__ __forceinline__ void batch_item(const PT &part, int64_t i, int &j,
                                           const BatchInst *__restrict__ inst,
                                           const int64_t *__restrict__ prefix, int first, int count,
                                           const double *sq, double2 *red,
                                           const double2 *__restrict__ coef,
                                           const double2 *__restrict__ Cb,
                                           double2 *__restrict__ HCb)
{
    while (j + 1 < count && prefix[first + j + 1] <= i) ++j;
    const BatchInst I = inst[first + j];
    const int64_t tile = i - prefix[first + j];
    const double2 *C = Cb + I.vec_off, *gp = coef + I.gp_off, *hp = coef + I.hp_off;
    double2 v;
    if constexpr (KIND == kDirect || KIND == kDirectLarge)
        v = apply_tile_direct<MT, false>(part, tile, I.N, I.dim, sq, gp, C);
    else
        v = apply_tile_tables<MT, uint8_t, KIND>(part, tile, I.dim, I.cap, sq, I.occ, I.t1, I.pmask,
                                                 I.t2_off, I.t2,
                                                 KIND == kPaperMap || KIND == kPaperChain ? hp : gp,
                                                 gp, C);
    store_tile<PT::kWaves>(v, part.part, tile, I.dim, red, HCb + I.vec_off);
}

// Calls item(i, j) for `grab` items at a time from the group's counter (a vector
// atomic of one lane; the count is zeroed before each apply).  A worker is a
// wavefront, with NP > 1 a block.
template <int NP, class Item>
__device__ __forceinline__ void batch_take(uint32_t *__restrict__ counter, int64_t items, int grab,
                                           uint32_t *taken, const Item &item)
{
    int j = 0;
    for (;;) {
        uint32_t base = 0;
        if constexpr (NP == 1) {
            if ((threadIdx.x & 63) == 0) base = atomicAdd(counter, (uint32_t)grab);
            base = __builtin_amdgcn_readfirstlane(base);
        } else {
            __syncthreads();   // the last value is read
            if (threadIdx.x == 0) *taken = atomicAdd(counter, (uint32_t)grab);
            __syncthreads();
            base = __builtin_amdgcn_readfirstlane(*taken);
        }
        if ((int64_t)base >= items) break;
        const int64_t end = (int64_t)base + grab < items ? (int64_t)base + grab : items;
        for (int64_t i = base; i < end; ++i) item(i, j);
    }
}

}  // namespace mc
