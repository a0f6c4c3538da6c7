// Batched H.C over many (N, M, h, g) instances of uneven size, and the
// segmented vector operations a batched Lanczos recurrence needs.
//
// A batch vector is the concatenation of the instances' coefficient vectors
// (instance i at offset vec_off[i]).  The plan, built once into a caller
// buffer, holds per-instance descriptors and staged coefficients, the
// instances grouped by orbital count and kind, and a chunk table for segmented
// reductions.  Each group runs as one persistent kernel whose wavefronts walk
// the group's (instance, tile) work list; an instance that fills the GPU with
// four rows per lane has a launch of its own (mc_plan.h).  Every call only enqueues kernels (no
// host synchronisation, no memset), so a sequence of calls can be captured
// into a HIP graph and replayed.
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "mc_block.h"
#include "mc_plan.h"
#include "mc_tiles.h"

namespace mc {

// An item whose descriptor holds sizes but no buffers runs table-free.
static bool table_free(const mc_tables *t)
{
    return !t->binom_d && !t->occ_d && !t->t1_d && !t->pmask_d && !t->t2_off_d && !t->t2_d;
}

// Staged complex constants of an instance of M orbitals, enough for either
// form, and with the tables of the four-row kernel behind them where the
// instance takes it (as mc_apply_H and mc_apply_H_direct would).
inline int64_t batch_const_elems(int M)
{
    const int64_t paper = (int64_t)npairs(M) * M * M + (int64_t)M * M;
    const int64_t split = split_total(M);
    return paper > split ? paper : split;
}
inline bool batch_block(const mc_tables *t)
{
    return block_serves(t->N, t->M, t->dim);
}
inline int64_t batch_coef_elems(const mc_tables *t)
{
    return batch_const_elems(t->M) + (batch_block(t) ? (block_table_ints(t->N, t->M) + 3) / 4 : 0);
}

struct BatchChunk {
    int32_t inst;
    int32_t first, count;   // the instance's chunks
    int32_t pad;
    int64_t start, len;     // in batch-vector elements
};

// Elements per chunk of the segmented vector operations: a chunk is one
// block's work, so enough of them to fill the GPU, between 2,048 and 65,536
// (24 instances of together 8e4 elements ran one block each, 11 us per
// reduction where 4 us do).
inline int64_t batch_chunk(int64_t total)
{
    int64_t c = 2048;
    while (c < (1 << 16) && total / c > 2048) c <<= 1;
    return c;
}
constexpr int kMaxGroups = 48;   // 8 orbital counts x 6 kinds
// Tiles a wavefront takes per counter increment (order 3): 8, fewer where the
// group has no 8 per wavefront (8 small instances at M = 5: 165 us with 8 tiles
// in a row on an eighth of the wavefronts, 25 us with one each).
inline int batch_grab(int64_t items, int64_t workers)
{
    const int64_t per = items / workers;
    return per >= 8 ? 8 : (per > 1 ? (int)per : 1);
}

// An instance that the four-row kernel serves: a launch of its own.
struct OwnLaunch {
    int32_t j;      // sorted position (index into the plan's descriptors)
    int32_t M, N;
    int64_t dim, vec_off, gp_off;
    const int32_t *btab;
};

}  // namespace mc

struct mc_batch {
    int32_t count;
    int32_t ngroups;
    int32_t group_M[48];
    int32_t group_kind[48];   // ApplyKind of the group's instances
    int32_t group_first[48];  // first entry in the sorted instance order
    int32_t group_count[48];
    int64_t group_tiles[48];
    int64_t group_blocks[48];
    bool group_shared[48];    // its tiles are shared by blocks (shared_tiles)
    bool group_joined[48];    // runs with others of its kind in one launch
    mc::JointGroups joint[mc::kJointKinds];   // those groups, by kind
    int64_t joint_blocks[mc::kJointKinds];
    int64_t nchunks;
    int64_t total_len;        // batch-vector length
    int32_t order;
    mc::BatchInst *inst_d;    // [count], in sorted order
    int64_t *tile_prefix_d;   // [count + 1] per sorted instance, restarting per group
    mc::BatchChunk *chunks_d; // [nchunks]
    double2 *partials_d;      // [2][nchunks]
    int32_t *sorted_d;        // [count] sorted position -> caller index
    int32_t *pos_d;           // [count] caller index -> sorted position
    uint32_t *counters_d;     // [kMaxGroups] work counters of order 3, zeroed per apply
    double2 *coef_d;          // staged coefficients of all instances
    int32_t nown;             // instances with launches of their own
    mc::OwnLaunch *own;       // [nown] (host)
};

namespace mc {

// Puts small groups of one kind, the one with the most orbitals first, into one
// launch, two at least.  Small: at most 64 tiles per CU and eight wavefronts, 16
// for the chained case-split sum.  One apply of a batch, us, each group a launch
// / up to 16 / up to 64, without tables, through the map, chained: 24 instances
// (N 8..20, M 3..5) 45 / 36 / 36, 55 / 45 / 45, 50 / 37 / 37; 30 (8..20, 3..6)
// 127 / 106 / 106, 180 / 139 / 139, 139 / 114 / 114; 100 (8..28, 3..5) 170 / 165
// / 135, 232 / 224 / 191, 166 / 155 / 163; 80 (20..40, 4..5) 454 / 448 / 433, 561
// / 561 / 532, 447 / 448 / 486; 300 (40..120, 3..4) 1,095 / 1,096 / 1,093, 1,252 /
// 1,206 / 1,206, 1,278 / 1,239 / 1,236.
static void batch_join(mc_batch *b, int cus)
{
    memset(b->group_joined, 0, sizeof b->group_joined);
    memset(b->joint, 0, sizeof b->joint);
    for (int kind = 0; kind < kJointKinds; ++kind) {
        JointGroups &J = b->joint[kind];
        int64_t blocks = 0;
        int member[48], n = 0;
        for (int gi = b->ngroups - 1; gi >= 0; --gi) {
            const int M = b->group_M[gi];
            if (b->group_kind[gi] != kind || M < kJointMinM || M > kJointMaxM || b->order != 3)
                continue;
            const bool parts = b->group_shared[gi];
            const int64_t tiles = b->group_tiles[gi];
            const int64_t need = parts ? tiles : (tiles + kTileParts - 1) / kTileParts;
            if (need > (int64_t)(kind == kSplitChain ? 16 : 64) * cus) continue;
            const int64_t own = parts ? b->group_blocks[gi]
                                      : (b->group_blocks[gi] * 4 + kTileParts - 1) / kTileParts;
            J.g[n] = JointGroup{M, b->group_first[gi], b->group_count[gi],
                                batch_grab(tiles, parts ? own : own * kTileParts), gi,
                                (int32_t)blocks, tiles};
            member[n++] = gi;
            blocks += own;
        }
        if (n < 2) continue;
        J.n = n;
        b->joint_blocks[kind] = blocks;
        for (int i = 0; i < n; ++i) b->group_joined[member[i]] = true;
    }
}

__global__ void k_batch_prep(const BatchInst *__restrict__ inst, uint32_t *__restrict__ counters)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kMaxGroups) counters[threadIdx.x] = 0;
    const BatchInst I = inst[blockIdx.y];
    const int M = I.M;
    // the last block of an instance makes its tables, the others its constants
    if (blockIdx.x + 1 == gridDim.x) {
        __shared__ int sum[256];
        if (I.btab) stage_block_tables(I.N, M, I.btab, sum);
        return;
    }
    const int first = blockIdx.x * blockDim.x + threadIdx.x;
    const int stride = (gridDim.x - 1) * blockDim.x;
    if (I.kind >= kSplitMap || I.btab) {   // every kind but the paper's sum
        stage_split_constants(M, 0, I.g, I.h, I.gp, first, stride);
        return;
    }
    const int P = M * (M + 1) / 2;
    const int total = P * M * M;
    for (int idx = first; idx < total + M * M; idx += stride) {
        if (idx >= total) {
            const int e = idx - total;
            I.hp[e] = I.h[e];
            continue;
        }
        const int p = idx / (M * M), ql = idx % (M * M);
        int k = 0, rem = p;
        while (rem >= M - k) {
            rem -= M - k;
            ++k;
        }
        const int s = k + rem;
        const int q = ql / M, l = ql % M;
        double2 a = I.g[((k * M + s) * M + q) * M + l];
        if (k != s) {
            const double2 b = I.g[((s * M + k) * M + q) * M + l];
            a.x += b.x;
            a.y += b.y;
        }
        I.gp[idx] = make_double2(0.5 * a.x, 0.5 * a.y);
    }
}

// conj(a) b added to (r, i); every reduction below adds its terms this way.
__device__ __forceinline__ void dot_add(const double2 &a, const double2 &b, double &r, double &i)
{
    r = fma(a.x, b.x, fma(a.y, b.y, r));
    i = fma(a.x, b.y, fma(-a.y, b.x, i));
}

// The block's sum of (ar, ai) over 256 threads, on every thread.
__device__ __forceinline__ double2 block_sum2(double ar, double ai, double *s)
{
    ar = wave_sum(ar);
    ai = wave_sum(ai);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        s[wave_in_block()] = ar;
        s[4 + wave_in_block()] = ai;
    }
    __syncthreads();
    return make_double2((s[0] + s[1]) + (s[2] + s[3]), (s[4] + s[5]) + (s[6] + s[7]));
}

// The sum of an instance's chunk partials, on every thread of a block of 256:
// a fixed strided split over the threads and a fixed tree.
__device__ __forceinline__ double2 seg_total(const double2 *__restrict__ part, int first,
                                             int count, double *s)
{
    double ar = 0.0, ai = 0.0;
    for (int c = threadIdx.x; c < count; c += 256) {
        const double2 v = part[first + c];
        ar += v.x;
        ai += v.y;
    }
    return block_sum2(ar, ai, s);
}

// Segmented conj(x).y: partials per chunk.
__global__ __launch_bounds__(256) void k_seg_dot_partial(const BatchChunk *__restrict__ ch,
                                                          int64_t nchunks,
                                                          const double2 *__restrict__ x,
                                                          const double2 *__restrict__ y,
                                                          double2 *__restrict__ part)
{
    __shared__ double s[8];
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const BatchChunk C = ch[c];
        double ar = 0.0, ai = 0.0;
        for (int64_t i = C.start + threadIdx.x; i < C.start + C.len; i += 256)
            dot_add(x[i], y[i], ar, ai);
        const double2 v = block_sum2(ar, ai, s);
        if (threadIdx.x == 0) part[c] = v;
    }
}

// out[caller index] = sum of the instance's chunk partials (one block per
// instance); out_norm: sqrt(Re) as double.
__global__ __launch_bounds__(256) void k_seg_final(const BatchInst *__restrict__ inst,
                                                    const BatchChunk *__restrict__ ch,
                                                    const int32_t *__restrict__ sorted,
                                                    const double2 *__restrict__ part,
                                                    double2 *__restrict__ out_c,
                                                    double *__restrict__ out_norm)
{
    __shared__ double s[8];
    const BatchChunk C = ch[inst[blockIdx.x].chunk0];
    const double2 v = seg_total(part, C.first, C.count, s);
    if (threadIdx.x) return;
    const int dst = sorted[blockIdx.x];
    if (out_c) out_c[dst] = v;
    if (out_norm) out_norm[dst] = sqrt(v.x);
}

// w - a v - b v_prev at element i
__device__ __forceinline__ double2 seg_orth_at(double2 x, const double2 &y,
                                               const double2 *__restrict__ vp, int64_t i, double a,
                                               double b)
{
    x.x = fma(-a, y.x, x.x);
    x.y = fma(-a, y.y, x.y);
    if (b != 0.0) {
        const double2 z = vp[i];
        x.x = fma(-b, z.x, x.x);
        x.y = fma(-b, z.y, x.y);
    }
    return x;
}

// One three-term step on a chunk's instance, as k_seg_final(alpha), k_seg_orth
// and k_seg_dot_partial(w, w) leave it, in one pass: alpha from the partials of
// <v|w>, w -= Re(alpha) v + beta v_prev, and the partials of the norm.
__global__ __launch_bounds__(256) void k_seg_step(const BatchChunk *__restrict__ ch,
                                                   int64_t nchunks,
                                                   const int32_t *__restrict__ sorted,
                                                   double2 *__restrict__ w,
                                                   const double2 *__restrict__ v,
                                                   const double2 *__restrict__ vp,
                                                   const double2 *__restrict__ part,
                                                   double2 *__restrict__ alpha,
                                                   const double *__restrict__ beta,
                                                   double2 *__restrict__ norm)
{
    __shared__ double s[8];
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const BatchChunk C = ch[c];
        const int dst = sorted[C.inst];
        const double2 al = seg_total(part, C.first, C.count, s);
        if (c == C.first && threadIdx.x == 0) alpha[dst] = al;
        const double a = al.x, b = vp ? beta[dst] : 0.0;
        double ar = 0.0, ai = 0.0;
        for (int64_t i = C.start + threadIdx.x; i < C.start + C.len; i += 256) {
            const double2 x = seg_orth_at(w[i], v[i], vp, i, a, b);
            w[i] = x;
            dot_add(x, x, ar, ai);
        }
        const double2 n = block_sum2(ar, ai, s);
        if (threadIdx.x == 0) norm[c] = n;
    }
}

// out = w / beta per instance, beta from the partials of the norm (as
// k_seg_final and k_seg_scale leave it).  `counters`, if any, are zeroed for
// the apply that follows.
__global__ __launch_bounds__(256) void k_seg_norm_scale(const BatchChunk *__restrict__ ch,
                                                         int64_t nchunks,
                                                         const int32_t *__restrict__ sorted,
                                                         const double2 *__restrict__ w,
                                                         const double2 *__restrict__ norm,
                                                         double *__restrict__ beta,
                                                         double2 *__restrict__ out,
                                                         uint32_t *__restrict__ counters)
{
    __shared__ double s[8];
    if (blockIdx.x == 0 && threadIdx.x < kMaxGroups) counters[threadIdx.x] = 0;
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const BatchChunk C = ch[c];
        const double b = sqrt(seg_total(norm, C.first, C.count, s).x);
        if (c == C.first && threadIdx.x == 0) beta[sorted[C.inst]] = b;
        const double inv = b > 0.0 ? 1.0 / b : 0.0;
        for (int64_t i = C.start + threadIdx.x; i < C.start + C.len; i += 256) {
            const double2 x = w[i];
            out[i] = make_double2(x.x * inv, x.y * inv);
        }
    }
}

// w -= Re(alpha_i) v + beta_i v_prev per instance segment (three-term step)
__global__ __launch_bounds__(256) void k_seg_orth(const BatchChunk *__restrict__ ch,
                                                   int64_t nchunks,
                                                   const int32_t *__restrict__ sorted,
                                                   double2 *__restrict__ w,
                                                   const double2 *__restrict__ v,
                                                   const double2 *__restrict__ vp,
                                                   const double2 *__restrict__ alpha,
                                                   const double *__restrict__ beta)
{
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const BatchChunk C = ch[c];
        const int dst = sorted[C.inst];
        const double a = alpha[dst].x;
        const double b = (vp && beta) ? beta[dst] : 0.0;
        for (int64_t i = C.start + threadIdx.x; i < C.start + C.len; i += blockDim.x)
            w[i] = seg_orth_at(w[i], v[i], vp, i, a, b);
    }
}

// out = w / beta_i per instance segment (0 where beta_i = 0)
__global__ __launch_bounds__(256) void k_seg_scale(const BatchChunk *__restrict__ ch,
                                                    int64_t nchunks,
                                                    const int32_t *__restrict__ sorted,
                                                    const double2 *__restrict__ w,
                                                    const double *__restrict__ beta,
                                                    double2 *__restrict__ out)
{
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const BatchChunk C = ch[c];
        const double b = beta[sorted[C.inst]];
        const double inv = b > 0.0 ? 1.0 / b : 0.0;
        for (int64_t i = C.start + threadIdx.x; i < C.start + C.len; i += blockDim.x) {
            const double2 x = w[i];
            out[i] = make_double2(x.x * inv, x.y * inv);
        }
    }
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct PlanLayout {
    size_t inst, prefix, chunks, partials, sorted, pos, counters, coef, total;
};

static int plan_layout(int32_t count, const mc_batch_item *items, int64_t *nchunks_out,
                       int64_t *chunk_out, int64_t *coef_elems_out, PlanLayout *L)
{
    int64_t nchunks = 0, coef = 0, total = 0;
    for (int i = 0; i < count; ++i) {
        if (!items[i].tables) return MC_EINVAL;
        total += items[i].tables->dim;
    }
    const int64_t chunk = batch_chunk(total);
    *chunk_out = chunk;
    for (int i = 0; i < count; ++i) {
        const mc_tables *t = items[i].tables;
        nchunks += (t->dim + chunk - 1) / chunk;
        coef += batch_coef_elems(t);
    }
    L->inst = 0;
    L->prefix = align256(L->inst + sizeof(BatchInst) * count);
    L->chunks = align256(L->prefix + sizeof(int64_t) * (count + 1));
    L->partials = align256(L->chunks + sizeof(BatchChunk) * nchunks);
    L->sorted = align256(L->partials + sizeof(double2) * 2 * nchunks);
    L->pos = align256(L->sorted + sizeof(int32_t) * count);
    L->counters = align256(L->pos + sizeof(int32_t) * count);
    L->coef = align256(L->counters + sizeof(uint32_t) * kMaxGroups);
    L->total = align256(L->coef + sizeof(double2) * coef);
    *nchunks_out = nchunks;
    *coef_elems_out = coef;
    return MC_OK;
}

}  // namespace mc

using namespace mc;

extern "C" {

int mc_batch_plan_size(int32_t count, const mc_batch_item *items, size_t *bytes)
{
    if (count < 1 || !items || !bytes) return MC_EINVAL;
    PlanLayout L;
    int64_t nch, chunk, coef;
    const int st = plan_layout(count, items, &nch, &chunk, &coef, &L);
    if (st) return st;
    *bytes = L.total;
    return MC_OK;
}

int mc_batch_create(int32_t count, const mc_batch_item *items, const mc_batch_schedule *sched,
                    void *plan_d, size_t plan_bytes, mc_stream stream, mc_batch **out)
{
    if (count < 1 || !items || !out || !plan_d) return MC_EINVAL;
    *out = nullptr;
    for (int i = 0; i < count; ++i) {
        const mc_tables *t = items[i].tables;
        if (!t || !items[i].h_d || !items[i].g_d) return MC_EINVAL;
        int st = check_nm(t->N, t->M);
        if (st) return st;
        if (table_free(t)) {
            // sizes only: they must be those of (N, M)
            const int64_t D = dim_checked(t->N, t->M);
            if (D < 0 || t->dim != D || t->tiles != (D + kTile - 1) / kTile) return MC_EINVAL;
        } else {
            st = check_tables(t->N, t->M, t, t->t2_d != nullptr);
            if (st) return st;
        }
        // batched instances: M <= 8, N <= 255, D < 2^28 (range-checked gathers)
        if (t->M > 8 || occ_width(t->N) != 1 || t->dim * 16 > (int64_t)0xFFFFFFFFu) return MC_EINVAL;
    }
    PlanLayout L;
    int64_t nchunks, chunk, coef_elems;
    int st = plan_layout(count, items, &nchunks, &chunk, &coef_elems, &L);
    if (st) return st;
    if (plan_bytes < L.total) return MC_ENOMEM;
    const int bpc = sched && sched->blocks_per_cu > 0 ? sched->blocks_per_cu : 2;
    const int order = sched ? sched->order : 0;
    if (order < 0 || order > 3) return MC_EINVAL;

    auto kind_of = [](const mc_tables *t) -> int32_t {
        // above kSmallTiles, what the four-row kernel does not serve runs
        // table-free as in mc_apply_H
        if (table_free(t) || t->tiles > kSmallTiles)
            return t->tiles > kSmallTiles && t->M >= 5 ? kDirectLarge : kDirect;
        const bool split = t->form == MC_FORM_REDUCED, map = t->t2_d != nullptr;
        return split ? (map ? kSplitMap : kSplitChain) : (map ? kPaperMap : kPaperChain);
    };
    std::vector<PlanItem> plan(count);
    for (int i = 0; i < count; ++i) {
        const mc_tables *t = items[i].tables;
        plan[i] = PlanItem{t->M, kind_of(t), t->dim, t->tiles, batch_block(t)};
    }
    std::vector<int32_t> sorted;
    std::vector<int64_t> prefix;
    const std::vector<PlanGroup> groups = plan_groups(plan, sorted, prefix);
    mc_batch *b = (mc_batch *)calloc(1, sizeof(mc_batch));
    if (!b) return MC_ENOMEM;
    b->own = (OwnLaunch *)calloc((size_t)count, sizeof(OwnLaunch));
    if (!b->own) {
        free(b);
        return MC_ENOMEM;
    }
    b->count = count;
    b->order = order;
    std::vector<int32_t> pos(count);
    std::vector<BatchInst> inst(count);
    std::vector<BatchChunk> chunks;
    chunks.reserve(nchunks);
    char *base = (char *)plan_d;
    double2 *coef = (double2 *)(base + L.coef);
    int64_t voff = 0, cpos = 0;
    for (int j = 0; j < count; ++j) {
        const int i = sorted[j];
        pos[i] = j;
        const mc_tables *t = items[i].tables;
        BatchInst &I = inst[j];
        I.N = t->N;
        I.M = t->M;
        I.kind = plan[i].kind;
        I.dim = t->dim;
        I.tiles = t->tiles;
        I.cap = t->t2_d ? t->t2_entries : 0;
        I.vec_off = 0;
        I.occ = (const uint8_t *)t->occ_d;
        I.t1 = t->t1_d;
        I.pmask = t->pmask_d;
        I.t2_off = t->t2_off_d;
        I.t2 = t->t2_d;
        I.h = (const double2 *)items[i].h_d;
        I.g = (const double2 *)items[i].g_d;
        I.gp = coef + cpos;
        I.hp = coef + cpos + (int64_t)npairs(t->M) * t->M * t->M;
        I.gp_off = cpos;
        I.hp_off = cpos + (int64_t)npairs(t->M) * t->M * t->M;
        const bool block = plan[i].own;
        I.btab = block ? (int32_t *)(coef + cpos + batch_const_elems(t->M)) : nullptr;
        cpos += batch_coef_elems(t);
        // an instance of the four-row kernel gets a launch of its own; the
        // rest join groups
        if (block) {
            OwnLaunch &o = b->own[b->nown++];
            o.j = j;
            o.M = t->M;
            o.N = t->N;
            o.dim = t->dim;
            o.gp_off = I.gp_off;
            o.btab = I.btab;
        }
    }
    for (const PlanGroup &g : groups) {
        const int gi = b->ngroups++;
        b->group_M[gi] = g.M;
        b->group_kind[gi] = g.kind;
        b->group_first[gi] = g.first;
        b->group_count[gi] = g.count;
        b->group_tiles[gi] = g.tiles;
    }
    // vector offsets follow the caller's order so that batch vectors are laid
    // out instance by instance as the caller listed them
    {
        std::vector<int64_t> off(count);
        for (int i = 0; i < count; ++i) {
            off[i] = voff;
            voff += items[i].tables->dim;
        }
        for (int j = 0; j < count; ++j) inst[j].vec_off = off[sorted[j]];
        for (int k = 0; k < b->nown; ++k) b->own[k].vec_off = inst[b->own[k].j].vec_off;
        for (int j = 0; j < count; ++j) {
            const int64_t D = inst[j].dim;
            const int32_t first = (int32_t)chunks.size();
            inst[j].chunk0 = first;
            for (int64_t s = 0; s < D; s += chunk) {
                BatchChunk c;
                c.inst = j;
                c.first = first;
                c.count = (int32_t)((D + chunk - 1) / chunk);
                c.pad = 0;
                c.start = inst[j].vec_off + s;
                c.len = D - s < chunk ? D - s : chunk;
                chunks.push_back(c);
            }
        }
    }
    b->total_len = voff;
    b->nchunks = (int64_t)chunks.size();
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) == hipSuccess) cus = prop.multiProcessorCount;
    }
    for (int gi = 0; gi < b->ngroups; ++gi) {
        const bool parts = small_parts(b->group_M[gi], b->group_kind[gi]) &&
                           b->group_tiles[gi] <= shared_tiles(b->group_M[gi], b->group_kind[gi], order);
        b->group_shared[gi] = parts;
        const int64_t need = parts ? b->group_tiles[gi] : (b->group_tiles[gi] + 3) / 4;
        const int64_t cap_blocks = (int64_t)bpc * cus;
        b->group_blocks[gi] = need < cap_blocks ? need : cap_blocks;
        if (b->group_blocks[gi] < 1) b->group_blocks[gi] = 1;
    }
    batch_join(b, cus);
    b->inst_d = (BatchInst *)(base + L.inst);
    b->tile_prefix_d = (int64_t *)(base + L.prefix);
    b->chunks_d = (BatchChunk *)(base + L.chunks);
    b->partials_d = (double2 *)(base + L.partials);
    b->sorted_d = (int32_t *)(base + L.sorted);
    b->pos_d = (int32_t *)(base + L.pos);
    b->counters_d = (uint32_t *)(base + L.counters);
    b->coef_d = (double2 *)(base + L.coef);
    hipStream_t s = (hipStream_t)stream;
    st = set_hip_error(hipMemcpyAsync(b->inst_d, inst.data(), sizeof(BatchInst) * count,
                                      hipMemcpyHostToDevice, s));
    if (!st) st = set_hip_error(hipMemcpyAsync(b->tile_prefix_d, prefix.data(),
                                                sizeof(int64_t) * (count + 1),
                                                hipMemcpyHostToDevice, s));
    if (!st) st = set_hip_error(hipMemcpyAsync(b->chunks_d, chunks.data(),
                                                sizeof(BatchChunk) * chunks.size(),
                                                hipMemcpyHostToDevice, s));
    if (!st) st = set_hip_error(hipMemcpyAsync(b->sorted_d, sorted.data(), sizeof(int32_t) * count,
                                                hipMemcpyHostToDevice, s));
    if (!st) st = set_hip_error(hipMemcpyAsync(b->pos_d, pos.data(), sizeof(int32_t) * count,
                                                hipMemcpyHostToDevice, s));
    // host staging vectors go out of scope: wait for the copies
    if (!st) st = set_hip_error(hipStreamSynchronize(s));
    if (st) {
        free(b->own);
        free(b);
        return st;
    }
    *out = b;
    return MC_OK;
}

int mc_batch_destroy(mc_batch *b)
{
    if (b) free(b->own);
    free(b);
    return MC_OK;
}

int64_t mc_batch_vector_length(const mc_batch *b) { return b ? b->total_len : (int64_t)MC_EINVAL; }

static void batch_stage(const mc_batch *b, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_prep, dim3(5, b->count), dim3(256), 0, s, b->inst_d, b->counters_d);
}

// The apply on staged constants and zeroed counters.
static int batch_apply_staged(const mc_batch *b, const double *C_d, double *HC_d, hipStream_t s)
{
    for (int k = 0; k < b->nown; ++k) {
        const OwnLaunch &o = b->own[k];
        const int st = apply_block_run(o.N, o.M, o.dim, b->coef_d + o.gp_off, o.btab,
                                       C_d + 2 * o.vec_off, HC_d + 2 * o.vec_off, s);
        if (st) return st;
    }
    for (int kind = 0; kind < kJointKinds; ++kind) {
        if (!b->joint[kind].n) continue;
        const JointCall c{&b->joint[kind], b->joint_blocks[kind], b->inst_d, b->tile_prefix_d,
                          b->counters_d, b->coef_d, (const double2 *)C_d, (double2 *)HC_d, s};
        const int st = tiles_joint(kind, c);
        if (st) return st;
    }
    for (int gi = 0; gi < b->ngroups; ++gi) {
        if (b->group_joined[gi]) continue;
        const int M = b->group_M[gi];
        const int64_t blocks = b->group_blocks[gi];
        const int64_t workers = b->group_shared[gi] ? blocks : blocks * 4;
        const GroupCall c{b->group_kind[gi], b->group_first[gi], b->group_count[gi], b->order,
                          batch_grab(b->group_tiles[gi], workers), b->group_tiles[gi], blocks,
                          b->inst_d, b->tile_prefix_d, b->counters_d + gi, b->coef_d,
                          (const double2 *)C_d, (double2 *)HC_d, s};
        int st;
        if (b->group_shared[gi] || !small_parts(M, c.kind))
            st = MC_TILES_CALL(group, M, c);
        else
            st = M == 5 ? tiles_many_5(c) : M == 6 ? tiles_many_6(c) : M == 7 ? tiles_many_7(c)
                                                                        : tiles_many_8(c);
        if (st) return st;
    }
    return launch_status();
}

int mc_batch_apply_H(const mc_batch *b, const double *C_d, double *HC_d, mc_stream stream)
{
    if (!b || !C_d || !HC_d) return MC_EINVAL;
    if (overlaps(C_d, (size_t)b->total_len * 16, HC_d, (size_t)b->total_len * 16)) return MC_EINVAL;
    batch_stage(b, (hipStream_t)stream);
    return batch_apply_staged(b, C_d, HC_d, (hipStream_t)stream);
}

int mc_batch_dot(const mc_batch *b, const double *x_d, const double *y_d, double *out_d,
                 mc_stream stream)
{
    if (!b || !x_d || !y_d || !out_d) return MC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const int64_t grid = b->nchunks < 4096 ? b->nchunks : 4096;
    hipLaunchKernelGGL(k_seg_dot_partial, dim3(grid), dim3(256), 0, s, b->chunks_d, b->nchunks,
                       (const double2 *)x_d, (const double2 *)y_d, b->partials_d);
    hipLaunchKernelGGL(k_seg_final, dim3(b->count), dim3(256), 0, s, b->inst_d, b->chunks_d,
                       b->sorted_d, b->partials_d, (double2 *)out_d, (double *)nullptr);
    return launch_status();
}

int mc_batch_lanczos_orth(const mc_batch *b, double *w_d, const double *v_d,
                          const double *vprev_d, const double *alpha_d, const double *beta_d,
                          mc_stream stream)
{
    if (!b || !w_d || !v_d || !alpha_d) return MC_EINVAL;
    const int64_t grid = b->nchunks < 8192 ? b->nchunks : 8192;
    hipLaunchKernelGGL(k_seg_orth, dim3(grid), dim3(256), 0, (hipStream_t)stream, b->chunks_d,
                       b->nchunks, b->sorted_d, (double2 *)w_d, (const double2 *)v_d,
                       (const double2 *)vprev_d, (const double2 *)alpha_d, beta_d);
    return launch_status();
}

int mc_batch_normalize(const mc_batch *b, const double *w_d, double *out_d, double *beta_d,
                       mc_stream stream)
{
    if (!b || !w_d || !out_d || !beta_d) return MC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const int64_t grid = b->nchunks < 4096 ? b->nchunks : 4096;
    hipLaunchKernelGGL(k_seg_dot_partial, dim3(grid), dim3(256), 0, s, b->chunks_d, b->nchunks,
                       (const double2 *)w_d, (const double2 *)w_d, b->partials_d);
    hipLaunchKernelGGL(k_seg_final, dim3(b->count), dim3(256), 0, s, b->inst_d, b->chunks_d,
                       b->sorted_d, b->partials_d, (double2 *)nullptr, beta_d);
    const int64_t grid2 = b->nchunks < 8192 ? b->nchunks : 8192;
    hipLaunchKernelGGL(k_seg_scale, dim3(grid2), dim3(256), 0, s, b->chunks_d, b->nchunks,
                       b->sorted_d, (const double2 *)w_d, beta_d, (double2 *)out_d);
    return launch_status();
}

struct mc_graph {
    hipGraph_t graph;
    hipGraphExec_t exec;
};

int mc_batch_lanczos_graph(const mc_batch *b, int32_t steps, const double *v0_d, double *V_d,
                           double *w_d, double *alpha_d, double *beta_d, mc_stream stream,
                           mc_graph **out)
{
    if (!b || steps < 1 || !v0_d || !V_d || !w_d || !alpha_d || !beta_d || !out || !stream)
        return MC_EINVAL;
    *out = nullptr;
    const int64_t n = b->total_len;
    double *V[3] = {V_d, V_d + 2 * n, V_d + 4 * n};
    for (int i = 0; i < 3; ++i)
        if (overlaps(V[i], (size_t)n * 16, w_d, (size_t)n * 16)) return MC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    int st = set_hip_error(hipStreamIsCapturing(s, &cs));
    if (st) return st;
    if (cs != hipStreamCaptureStatusNone) return MC_EINVAL;
    st = set_hip_error(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    if (st) return st;
    // the recurrence; every call below only enqueues kernels.  The constants
    // are staged once per replay, and a step after its product takes three
    // passes with the sums of the calls it stands for (mc_batch_dot,
    // mc_batch_lanczos_orth, mc_batch_normalize: seven launches).
    const int64_t nch = b->nchunks, grid = nch < 8192 ? nch : 8192;
    double2 *dots = b->partials_d, *norms = dots + nch;
    batch_stage(b, s);
    int rec = mc_batch_normalize(b, v0_d, V[0], beta_d + (int64_t)steps * b->count, stream);
    for (int32_t j = 0; j < steps && rec == MC_OK; ++j) {
        double *cur = V[j % 3], *prev = V[(j + 2) % 3], *nxt = V[(j + 1) % 3];
        double *alpha_j = alpha_d + (int64_t)2 * j * b->count;
        rec = batch_apply_staged(b, cur, w_d, s);
        if (rec != MC_OK) break;
        hipLaunchKernelGGL(k_seg_dot_partial, dim3(grid), dim3(256), 0, s, b->chunks_d, nch,
                           (const double2 *)cur, (const double2 *)w_d, dots);
        hipLaunchKernelGGL(k_seg_step, dim3(grid), dim3(256), 0, s, b->chunks_d, nch, b->sorted_d,
                           (double2 *)w_d, (const double2 *)cur,
                           j > 0 ? (const double2 *)prev : (const double2 *)nullptr,
                           (const double2 *)dots, (double2 *)alpha_j,
                           j > 0 ? (const double *)beta_d + (int64_t)(j - 1) * b->count
                                 : (const double *)nullptr,
                           norms);
        hipLaunchKernelGGL(k_seg_norm_scale, dim3(grid), dim3(256), 0, s, b->chunks_d, nch,
                           b->sorted_d, (const double2 *)w_d, (const double2 *)norms,
                           beta_d + (int64_t)j * b->count, (double2 *)nxt, b->counters_d);
        rec = launch_status();
    }
    hipGraph_t graph = nullptr;
    st = set_hip_error(hipStreamEndCapture(s, &graph));
    if (rec != MC_OK || st != MC_OK) {
        if (graph) hipGraphDestroy(graph);
        return rec != MC_OK ? rec : st;
    }
    hipGraphExec_t exec = nullptr;
    st = set_hip_error(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
    if (st) {
        hipGraphDestroy(graph);
        return st;
    }
    mc_graph *gr = (mc_graph *)malloc(sizeof(mc_graph));
    if (!gr) {
        hipGraphExecDestroy(exec);
        hipGraphDestroy(graph);
        return MC_ENOMEM;
    }
    gr->graph = graph;
    gr->exec = exec;
    *out = gr;
    return MC_OK;
}

int mc_graph_launch(const mc_graph *g, mc_stream stream)
{
    if (!g) return MC_EINVAL;
    return set_hip_error(hipGraphLaunch(g->exec, (hipStream_t)stream));
}

int mc_graph_destroy(mc_graph *g)
{
    if (!g) return MC_OK;
    int st = set_hip_error(hipGraphExecDestroy(g->exec));
    const int st2 = set_hip_error(hipGraphDestroy(g->graph));
    free(g);
    return st ? st : st2;
}

}  // extern "C"
