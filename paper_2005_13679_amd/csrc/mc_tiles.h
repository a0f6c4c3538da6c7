// Kernels with one row per lane: their launches, one function per orbital count
// (mc_tiles.hip, compiled once per count and part), and what they share with
// the batched plan.
#pragma once

#include "mc_internal.h"

namespace mc {

// How a row is summed: the paper's sum through its map or chained, the
// case-split sum through the reduced map, chained, or with no table (kDirect
// in small spaces, kDirectLarge above kSmallTiles).
enum ApplyKind : int32_t {
    kPaperMap = 0,
    kPaperChain = 1,
    kSplitMap = 2,
    kSplitChain = 3,
    kDirect = 4,
    kDirectLarge = 5,
};

// Spaces of at most this many tiles (65,536 rows) are small: there are fewer
// tiles than the GPU has room for wavefronts.  Without tables, one wavefront
// per tile against eight (us): M = 5, N = 30 (725 tiles) 21 / 18, N = 38 (1,749)
// 22 / 30; M = 6, N = 20 (831) 37 / 32, N = 24 (1,856) 38 / 54; M = 7, N = 16
// (1,166) 55 / 50; M = 8, N = 10 (304) 85 / 36, N = 14 (1,817) 85 / 114.
constexpr int64_t kSmallTiles = 1024;

struct BatchInst {
    int32_t N, M;
    int32_t kind, chunk0;  // chunk0: first chunk of the instance
    int64_t dim, tiles, cap, vec_off;
    const uint8_t *occ;
    const int32_t *t1;
    const uint64_t *pmask;
    const int64_t *t2_off;
    const int32_t *t2;   // null: chain single jumps
    const double2 *h, *g;
    double2 *hp, *gp;    // staged h' and G' (paper form) / gp: case-split constants
    int64_t hp_off, gp_off;  // the same, as offsets into the plan's coefficient region
    int32_t *btab;           // tables of the four-row kernel (instances that take it)
};

// Pointers read from a descriptor are generic (flat loads); the staged
// constants are therefore reached through the __restrict__ coefficient-region
// kernel argument, which keeps their loads scalar.

// One table-driven apply of a small space.
struct TablesCall {
    int32_t N, kind;
    const mc_tables *t;
    const double2 *ca, *cb;   // staged: case-split constants, or h and G'
    const double2 *C;
    double2 *HC;
    hipStream_t s;
};
// One table-free apply, one row per lane.
struct DirectCall {
    int32_t N;
    bool small;   // at most kSmallTiles
    int64_t D;
    const double2 *cf, *C;
    double2 *HC;
    hipStream_t s;
};
// One group of a batch.
struct GroupCall {
    int32_t kind, first, count, order, grab;
    int64_t items, blocks;
    const BatchInst *inst;
    const int64_t *prefix;
    uint32_t *counter;
    const double2 *coef, *C;
    double2 *HC;
    hipStream_t s;
};

#define MC_TILES_DECLARE(M)                \
    int tiles_tables_##M(const TablesCall &); \
    int tiles_direct_##M(const DirectCall &); \
    int tiles_group_##M(const GroupCall &);
MC_TILES_DECLARE(1)
MC_TILES_DECLARE(2)
MC_TILES_DECLARE(3)
MC_TILES_DECLARE(4)
MC_TILES_DECLARE(5)
MC_TILES_DECLARE(6)
MC_TILES_DECLARE(7)
MC_TILES_DECLARE(8)
#undef MC_TILES_DECLARE
int tiles_many_5(const GroupCall &);
int tiles_many_6(const GroupCall &);
int tiles_many_7(const GroupCall &);
int tiles_many_8(const GroupCall &);

// Calls tiles_<what>_<M> (1 <= M <= 8).
#define MC_TILES_CALL(what, M, call)                                                     \
    ((M) == 1 ? tiles_##what##_1(call) : (M) == 2 ? tiles_##what##_2(call)                \
     : (M) == 3 ? tiles_##what##_3(call) : (M) == 4 ? tiles_##what##_4(call)              \
     : (M) == 5 ? tiles_##what##_5(call) : (M) == 6 ? tiles_##what##_6(call)              \
     : (M) == 7 ? tiles_##what##_7(call) : tiles_##what##_8(call))

// Groups of one kind in one launch (mc_joint.hip): group i has the blocks from
// block0 on, up to the next group's.
struct JointGroup {
    int32_t M, first, count, grab, counter, block0;
    int64_t items;
};
constexpr int kJointMinM = 3, kJointMaxM = 6, kJointKinds = 5;
struct JointGroups {
    int32_t n;
    JointGroup g[kJointMaxM - kJointMinM + 1];
};
struct JointCall {
    const JointGroups *groups;
    int64_t blocks;
    const BatchInst *inst;
    const int64_t *prefix;
    uint32_t *counters;
    const double2 *coef, *C;
    double2 *HC;
    hipStream_t s;
};
int tiles_joint_0(const JointCall &);
int tiles_joint_1(const JointCall &);
int tiles_joint_2(const JointCall &);
int tiles_joint_3(const JointCall &);
int tiles_joint_4(const JointCall &);
inline int tiles_joint(int kind, const JointCall &c)
{
    switch (kind) {
    case kPaperMap: return tiles_joint_0(c);
    case kPaperChain: return tiles_joint_1(c);
    case kSplitMap: return tiles_joint_2(c);
    case kSplitChain: return tiles_joint_3(c);
    case kDirect: return tiles_joint_4(c);
    default: return MC_EINVAL;
    }
}

// Whether instances of this kind are summed in kTileParts parts (from M = 5 on, in
// small spaces; mc_apply.h has the reason).
inline bool small_parts(int M, int kind) { return M >= 5 && kind != kDirectLarge; }

// Groups of such instances with at most this many tiles have a block per tile,
// whose wavefronts share it, larger ones a wavefront per tile, which keeps the
// sums.  One apply in the better of orders 0 and 2, us, shared / kept, at the tiles
// given: M = 5, N = 20, without tables 498 17 / 22, 996 25 / 21, 1,992 40 / 23, 8,134
// 130 / 66; reduced map 19 / 28, 31 / 31, 51 / 34, 178 / 101; chained 13 / 27, 19 / 27,
// 29 / 30, 88 / 83.  M = 6, N = 14, 910 35 / 35, 2,002 62 / 40, 8,190 216 / 121.  M = 8,
// N = 8, 505 40 / 75, 1,010 68 / 75, 2,020 126 / 88, 8,181 456 / 308.  With order 3 the
// counter costs more the more workers take from it, and sharing is level up to
// 4,000 tiles and within 1.3 above.
inline int64_t shared_tiles(int M, int kind, int order)
{
    if (order == 3) return INT64_MAX;
    if (M == 5) return kind == kSplitChain ? 1600 : 768;
    return M == 6 && kind == kDirect ? 768 : 1300;
}

}  // namespace mc
