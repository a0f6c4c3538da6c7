// Several small groups of a batch, of one kind (MC_JOINT_KIND) and 3 to 6
// orbitals, in one launch.  Compiled once per kind.
#include "mc_group.h"

#define MC_JOINT_NAME2(K) tiles_joint_##K
#define MC_JOINT_NAME1(K) MC_JOINT_NAME2(K)
#define MC_JOINT_NAME MC_JOINT_NAME1(MC_JOINT_KIND)

namespace mc {

// Bound: the chain of one tile's loads, once per tile a worker takes: a small
// group takes that long however few its tiles are (three groups of 24 instances,
// N 8..20, M 3..5, through the map: 24.5, 17.2 and 8.0 us one after another), and
// the groups overlap here.  Ten Lanczos steps of that batch: 820 -> 707 us.
template <int KIND>
__global__ __launch_bounds__(kTileParts * 64) __attribute__((amdgpu_waves_per_eu(MC_APPLY_WAVES)))
void k_batch_joint(const BatchInst *__restrict__ inst, const int64_t *__restrict__ prefix,
                   JointGroups groups, uint32_t *__restrict__ counters,
                   const double2 *__restrict__ coef, const double2 *__restrict__ Cb,
                   double2 *__restrict__ HCb)
{
    __shared__ double sq[kBatchMaxN + 3];
    __shared__ double2 red[kTileParts * kTile];
    __shared__ uint32_t taken;
    int gi = 0;
    while (gi + 1 < groups.n && (int)blockIdx.x >= groups.g[gi + 1].block0) ++gi;
    const JointGroup G = groups.g[gi];
    auto run = [&](auto m) __attribute__((always_inline)) {
        constexpr int MT = decltype(m)::value, NP = kSmallParts<MT>;
        if constexpr (kLdsRoots<MT>) fill_sqrt_table(sq, kBatchMaxN + 3);
        const Part<NP> part{NP == 1 ? 0 : wave_in_block(), nullptr};
        batch_take<NP>(counters + G.counter, G.items, G.grab, &taken, [&](int64_t i, int &j)
                       __attribute__((always_inline)) {
            batch_item<MT, KIND>(part, i, j, inst, prefix, G.first, G.count, sq, red, coef, Cb,
                                     HCb);
        });
    };
    switch (G.M) {
    case 3: run(std::integral_constant<int, 3>{}); break;
    case 4: run(std::integral_constant<int, 4>{}); break;
    case 5: run(std::integral_constant<int, 5>{}); break;
    default: run(std::integral_constant<int, 6>{}); break;
    }
}

int MC_JOINT_NAME(const JointCall &c)
{
    hipLaunchKernelGGL((k_batch_joint<MC_JOINT_KIND>), dim3(c.blocks), dim3(kTileParts * 64), 0,
                       c.s, c.inst, c.prefix, *c.groups, c.counters, c.coef, c.C, c.HC);
    return launch_status();
}

}  // namespace mc
