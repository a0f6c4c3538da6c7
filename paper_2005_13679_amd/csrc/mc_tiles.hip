// Kernels with one row per lane for MC_TILES_M orbitals.  Compiled once per
// orbital count, and in parts (MC_TILES_PART: 0 table-driven, 1 table-free, 2
// groups of a batch, 3 its groups of many small instances), so that the long
// compilations run side by side.
#include "mc_tiles.h"

#include "mc_apply.h"
#include "mc_direct.h"
#include "mc_group.h"
#include "mc_split.h"

#define MC_TILES_NAME2(what, M) tiles_##what##_##M
#define MC_TILES_NAME1(what, M) MC_TILES_NAME2(what, M)
#define MC_TILES_NAME0(what, M) MC_TILES_NAME1(what, M)
#define MC_TILES_NAME(what) MC_TILES_NAME0(what, MC_TILES_M)

namespace mc {

#if MC_TILES_PART == 0

// H.C through the tables in small spaces (at most kSmallTiles tiles): from
// M = 5 on the kTileParts wavefronts of a block share a tile, below one
// wavefront does it and a block has four.
template <int MT, typename OccT, int KIND>
__global__ __launch_bounds__(kSmallParts<MT> == 1 ? 256 : kSmallParts<MT> * 64)
__attribute__((amdgpu_waves_per_eu(MC_APPLY_WAVES)))
void k_apply_tables(int N, int64_t D, int64_t tiles, int64_t cap, const OccT *__restrict__ occ,
                    const int32_t *__restrict__ t1, const uint64_t *__restrict__ pmask,
                    const int64_t *__restrict__ t2_off, const int32_t *__restrict__ t2,
                    const double2 *__restrict__ ca, const double2 *__restrict__ cb,
                    const double2 *__restrict__ C, double2 *__restrict__ HC)
{
    constexpr int NP = kSmallParts<MT>;
    extern __shared__ double sq[];
    __shared__ double2 red[NP > 1 ? NP * kTile : 1];
    if constexpr (kLdsRoots<MT>) fill_sqrt_table(sq, N + 3);
    const int64_t tile = NP == 1 ? (int64_t)blockIdx.x * 4 + wave_in_block() : blockIdx.x;
    if (tile >= tiles) return;
    const Part<NP> part{NP == 1 ? 0 : wave_in_block(), nullptr};
    store_tile<NP>(apply_tile_tables<MT, OccT, KIND>(part, tile, D, cap, sq, occ, t1, pmask, t2_off,
                                                     t2, ca, cb, C),
                   part.part, tile, D, red, HC);
}

template <typename OccT, int KIND>
static int tables_launch(const TablesCall &c)
{
    constexpr int MT = MC_TILES_M, NP = kSmallParts<MT>;
    const mc_tables *t = c.t;
    hipLaunchKernelGGL((k_apply_tables<MT, OccT, KIND>),
                       dim3(NP == 1 ? (t->tiles + 3) / 4 : t->tiles), dim3(NP == 1 ? 256 : NP * 64),
                       kLdsRoots<MT> ? (size_t)(c.N + 3) * 8 : 0, c.s, c.N, t->dim, t->tiles,
                       t->t2_entries, (const OccT *)t->occ_d, t->t1_d, t->pmask_d, t->t2_off_d,
                       t->t2_d, c.ca, c.cb, c.C, c.HC);
    return launch_status();
}

template <typename OccT>
static int tables_kind(const TablesCall &c)
{
    switch (c.kind) {
    case kPaperMap: return tables_launch<OccT, kPaperMap>(c);
    case kPaperChain: return tables_launch<OccT, kPaperChain>(c);
    case kSplitMap: return tables_launch<OccT, kSplitMap>(c);
    case kSplitChain: return tables_launch<OccT, kSplitChain>(c);
    default: return MC_EINVAL;
    }
}

int MC_TILES_NAME(tables)(const TablesCall &c)
{
    if (occ_width(c.N) == 1) return tables_kind<uint8_t>(c);
    // more than 255 particles are no small space from M = 4 on
#if MC_TILES_M <= 3
    return tables_kind<uint16_t>(c);
#else
    return MC_EINVAL;
#endif
}

#elif MC_TILES_PART == 1

// H.C with no table, one row per lane (mc_direct.h): one wavefront per 64-row
// tile and four tiles per block, or the NP wavefronts of a block on one tile.
template <int MT, bool BIGC, int NP>
__global__ __launch_bounds__(NP == 1 ? 256 : NP * 64) __attribute__((amdgpu_waves_per_eu(MC_APPLY_WAVES)))
void k_apply_direct(int N, int64_t D, int64_t tiles, int64_t nblocks,
                    const double2 *__restrict__ cf, const double2 *__restrict__ C,
                    double2 *__restrict__ HC)
{
    extern __shared__ double sq[];
    __shared__ double2 red[NP > 1 ? NP * kTile : 1];
    if constexpr (kLdsRoots<MT>) fill_sqrt_table(sq, N + 3);
    const int64_t block = xcd_block_as<kDirectRemap<MT>>(blockIdx.x, nblocks);
    const int64_t tile = NP == 1 ? block * 4 + wave_in_block() : block;
    if (tile >= tiles) return;
    const Part<NP> part{NP == 1 ? 0 : wave_in_block(), nullptr};
    store_tile<NP>(apply_tile_direct<MT, BIGC>(part, tile, N, D, sq, cf, C), part.part, tile, D, red,
                   HC);
}

template <bool BIGC, int NP>
static int direct_launch(const DirectCall &c)
{
    constexpr int MT = MC_TILES_M;
    const int64_t tiles = (c.D + kTile - 1) / kTile, nblocks = NP == 1 ? (tiles + 3) / 4 : tiles;
    hipLaunchKernelGGL((k_apply_direct<MT, BIGC, NP>), dim3(nblocks), dim3(NP == 1 ? 256 : NP * 64),
                       kLdsRoots<MT> ? (size_t)(c.N + 3) * 8 : 0, c.s, c.N, c.D, tiles, nblocks,
                       c.cf, c.C, c.HC);
    return launch_status();
}

int MC_TILES_NAME(direct)(const DirectCall &c)
{
    if (c.D * 16 > (int64_t)0xFFFFFFFFu) return direct_launch<true, 1>(c);
    if (c.small) return direct_launch<false, kSmallParts<MC_TILES_M>>(c);
    return direct_launch<false, 1>(c);
}

#else

// Persistent H.C over one group (one orbital count and one kind).
// Work item i of the group is tile (i - prefix[j]) of the group's j-th
// instance; with order 0 wavefront w takes items w, w + W, w + 2W, ...
// (neighbouring tiles on neighbouring wavefronts), with order 1 a contiguous
// range of items, with order 2 each XCD a contiguous share of the items,
// interleaved over its wavefronts; with order 3 wavefronts take a few items
// at a time from a per-group counter (dynamic balance, like a plain launch).
// With NP > 1 a worker is a block, whose wavefronts share each tile, instead of
// a wavefront, which keeps NC sums of a row.
template <int MT, int KIND, int NP, int NC>
__global__ __launch_bounds__(NP == 1 ? 256 : NP * 64) __attribute__((amdgpu_waves_per_eu(MC_APPLY_WAVES)))
void k_batch_apply(const BatchInst *__restrict__ inst, const int64_t *__restrict__ prefix,
                   int first, int count, int64_t items, int64_t nblocks, int order, int grab,
                   uint32_t *__restrict__ counter, const double2 *__restrict__ coef,
                   const double2 *__restrict__ Cb, double2 *__restrict__ HCb)
{
    __shared__ double sq[kLdsRoots<MT> ? kBatchMaxN + 3 : 1];
    if constexpr (kLdsRoots<MT>) fill_sqrt_table(sq, kBatchMaxN + 3);
    // the paper's map at M = 5 has the registers for the sums
    using PT = Part<NP, NC, !(MT == 5 && KIND == kPaperMap)>;
    __shared__ double2 red[NP > 1 ? NP * kTile : (PT::kLds ? 4 * NC * kTile : 1)];
    __shared__ uint32_t taken;
    const PT part{NP == 1 ? 0 : wave_in_block(),
                  PT::kLds ? red + wave_in_block() * NC * kTile + (threadIdx.x & 63) : nullptr};
    auto tile_body = [&](int64_t i, int &j) __attribute__((always_inline)) {
        batch_item<MT, KIND>(part, i, j, inst, prefix, first, count, sq, red, coef, Cb, HCb);
    };
    int j = 0;
    constexpr int WB = NP == 1 ? 4 : 1;   // workers per block
    if (order == 3) {
        batch_take<NP>(counter, items, grab, &taken, tile_body);
        return;
    }
    const int64_t W = nblocks * WB;
    const int wb = NP == 1 ? wave_in_block() : 0;
    const int64_t w = xcd_block(blockIdx.x, nblocks) * WB + wb;
    int64_t i0, step, iend;
    if (order == 2) {
        // blocks go to XCD b % 8; this XCD's blocks own items [ib, ie)
        const int64_t xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
        const int64_t bper = nblocks >> 3, brem = nblocks & 7;
        const int64_t nbx = bper + (xcd < brem ? 1 : 0);
        const int64_t fb = xcd * bper + (xcd < brem ? xcd : brem);
        const int64_t ib = items * fb / nblocks, ie = items * (fb + nbx) / nblocks;
        i0 = ib + local * WB + wb;
        step = nbx * WB;
        iend = ie;
    } else if (order == 1) {
        const int64_t per = (items + W - 1) / W;
        i0 = w * per;
        step = 1;
        iend = i0 + per < items ? i0 + per : items;
    } else {
        i0 = w;
        step = W;
        iend = items;
    }
    for (int64_t i = i0; i < iend; i += step) tile_body(i, j);
}

template <int KIND, int NP, int NC>
static int group_launch(const GroupCall &c)
{
    hipLaunchKernelGGL((k_batch_apply<MC_TILES_M, KIND, NP, NC>), dim3(c.blocks),
                       dim3(NP == 1 ? 256 : NP * 64), 0, c.s, c.inst, c.prefix, c.first, c.count,
                       c.items, c.blocks, c.order, c.grab, c.counter, c.coef, c.C, c.HC);
    return launch_status();
}

#if MC_TILES_PART == 2
#define MC_GROUP_NAME group
constexpr int kGroupWaves = kSmallParts<MC_TILES_M>, kGroupSums = 1;
#else
#define MC_GROUP_NAME many
constexpr int kGroupWaves = 1, kGroupSums = kTileParts;
#endif

int MC_TILES_NAME(MC_GROUP_NAME)(const GroupCall &c)
{
    constexpr int NP = kGroupWaves, NC = kGroupSums;
    switch (c.kind) {
    case kPaperMap: return group_launch<kPaperMap, NP, NC>(c);
    case kPaperChain: return group_launch<kPaperChain, NP, NC>(c);
    case kSplitMap: return group_launch<kSplitMap, NP, NC>(c);
    case kSplitChain: return group_launch<kSplitChain, NP, NC>(c);
    case kDirect: return group_launch<kDirect, NP, NC>(c);
#if MC_TILES_PART == 2 && MC_TILES_M >= 5
    case kDirectLarge: return group_launch<kDirectLarge, 1, 1>(c);
#endif
    default: return MC_EINVAL;
    }
}

#endif

}  // namespace mc
