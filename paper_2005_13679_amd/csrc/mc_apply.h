// Device-side building blocks of H.C (Eq. Haction) shared by the plain and
// batched kernels: one 64-row tile per wavefront, lane = row, through either
// the double-jump map or two chained single jumps.
#pragma once

#include <utility>

#include "mc_internal.h"

#ifndef MC_SLOT_BATCH
#define MC_SLOT_BATCH 13
#endif
// Occupancy the apply kernels are compiled for (wavefronts per SIMD); the
// register allocator caps VGPRs accordingly (512 / waves).
#ifndef MC_APPLY_WAVES
#define MC_APPLY_WAVES 2
#endif

namespace mc {

// Vectors of up to 2^28 entries go through a range-checked buffer resource
// (any t outside [0, D) reads zero); larger ones (BIGC) use 64-bit addresses
// with an explicit range test.
template <bool BIGC>
struct Gather {
    __amdgpu_buffer_rsrc_t r;
    const double2 *__restrict__ p;
    int64_t n;
    __device__ __forceinline__ Gather(const double2 *C, int64_t D)
    {
        p = C;
        n = D;
        if (!BIGC) r = make_rsrc(C, (uint32_t)(D * 16));
    }
    __device__ __forceinline__ double2 operator()(int32_t t) const
    {
        if (!BIGC) return buf_ld_c128(r, (uint32_t)t << 4);
        const bool ok = t >= 0 && t < n;
        const double2 v = p[ok ? t : 0];
        return ok ? v : make_double2(0.0, 0.0);
    }
};

// Per-row square roots of small integers used by the jump amplitudes:
// root<d>(m) = sqrt(n_m + d) for d in {-1, 0, 1, 2} (0 where n_m + d < 0).
// Either the four tables live in registers (8M VGPRs), or only the
// occupations do and the roots come from an LDS table of sqrt(i),
// i = 0 .. N+2, filled once per block: from M = 5 on, where the registers
// are worth more as waves in flight.
#ifndef MC_LDS_ROOTS_FROM
#define MC_LDS_ROOTS_FROM 5
#endif
template <int MT>
constexpr bool kLdsRoots = MT >= MC_LDS_ROOTS_FROM;
// The chained paper-form body keeps its roots in registers up to M = 5
// (measured: the LDS table slowed it by a fifth at M = 5, while it sped the
// map and case-split bodies up by 2-6 %, their registers going to waves).
template <int MT>
constexpr bool kLdsRootsChained = MT >= 6;

template <int MT, bool LDS = kLdsRoots<MT>>
struct RowSq;

template <int MT>
struct RowSq<MT, false> {
    double sm1[MT], s0[MT], sp1[MT], sp2[MT];
    __device__ __forceinline__ void init(const int (&n)[MT], const double *)
    {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const double x = (double)n[m];
            s0[m] = sqrt(x);
            sm1[m] = sqrt(x > 1.0 ? x - 1.0 : 0.0);
            sp1[m] = sqrt(x + 1.0);
            sp2[m] = sqrt(x + 2.0);
        }
    }
    template <int d>
    __device__ __forceinline__ double root(int m) const
    {
        static_assert(d >= -1 && d <= 2, "root offset");
        return d == -1 ? sm1[m] : (d == 0 ? s0[m] : (d == 1 ? sp1[m] : sp2[m]));
    }
};

template <int MT>
struct RowSq<MT, true> {
    int nn[MT];
    const double *sq;
    __device__ __forceinline__ void init(const int (&n)[MT], const double *tab)
    {
#pragma unroll
        for (int m = 0; m < MT; ++m) nn[m] = n[m];
        sq = tab;
    }
    template <int d>
    __device__ __forceinline__ double root(int m) const
    {
        const int i = nn[m] + d;
        return sq[i > 0 ? i : 0];
    }
};

// sqrt(i) for i = 0 .. n-1 into LDS (block-wide; every thread must call it)
__device__ __forceinline__ void fill_sqrt_table(double *tab, int n)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) tab[i] = sqrt((double)i);
    __syncthreads();
}

template <int MT, typename OccT, bool LDS>
__device__ __forceinline__ void load_row(const OccT *__restrict__ occ, int64_t tile, int lane,
                                         int (&n)[MT], RowSq<MT, LDS> &R, const double *sq)
{
#pragma unroll
    for (int m = 0; m < MT; ++m) n[m] = (int)occ[(tile * MT + m) * kTile + lane];
    R.init(n, sq);
}

// A wave-uniform true that the compiler cannot see through.  Branching on
// it puts each batch of a long straight-line stream into a basic block of its
// own; within one huge block the instruction scheduler issues every load of
// the stream first and keeps all gathered values live (hundreds of spilled
// registers), across blocks it cannot move them.
__device__ __forceinline__ bool opaque_true()
{
    int v;
    asm volatile("s_mov_b32 %0, 1" : "=s"(v));
    return v != 0;
}

// A tile's terms come in units that are basic blocks of their own (a batch of
// slots, a removal pair).  In a large space one wavefront does them all; in a
// small one, where there are fewer tiles than the GPU has room for wavefronts
// and a tile's chain of loads is all the time there is, kTileParts wavefronts
// of one block share the tile, unit I going to wavefront I mod kTileParts, and
// their sums are added in order.  Whole calls without tables: N=6, M=8 94 us with
// one wavefront per tile, 21 with eight; N=8, M=7 59 and 15; N=10, M=5 18.6 and
// 14.7 (15 us is the caller's own time); through the paper's map 161 and 25, 97
// and 20, 28 and 15.
// A group of a batch with many tiles has the wavefronts without that, and a tile
// would be decoded eight times; but its sums have to have the same bits, so one
// wavefront keeps the kTileParts sums itself.
constexpr int kTileParts = 8;
template <int MT>
constexpr int kSmallParts = MT >= 5 ? kTileParts : 1;   // M <= 4: at most 55 slots

// A wavefront's part of a tile: one of NP, or all with NC sums kept apart, in LDS
// (in registers they spilled through the maps from M = 6 on) or in registers.
template <int NP, int NC = 1, bool LDS = true>
struct Part {
    static constexpr int kWaves = NP, kSums = NC;
    static constexpr bool kSplit = NP * NC > 1;   // units are summed apart
    static constexpr bool kLds = NC > 1 && LDS;
    int part;        // wave-uniform, 0 .. NP-1
    double2 *sums;   // kLds: the lane's first sum, the others every kTile
    template <int I>
    __device__ __forceinline__ bool has() const
    {
        if constexpr (NP == 1) return opaque_true();
        else return part == I % NP;
    }
    // the row's own term
    __device__ __forceinline__ bool own() const { return NP == 1 || part == NP - 1; }
};

// The sums that a wavefront keeps of a row; unit I goes into number I mod NC, the
// row's own term into the last.
template <class PT>
struct RowSum {
    static constexpr int NC = PT::kSums;
    double2 v[PT::kLds ? 1 : NC];
    double2 *s;
    // own: the row's own term (zero where another wavefront has it)
    __device__ __forceinline__ RowSum(const PT &part, double2 own)
    {
        s = part.sums;
#pragma unroll
        for (int c = 0; c < NC; ++c) put(c, c + 1 < NC ? make_double2(0.0, 0.0) : own);
    }
    __device__ __forceinline__ double2 get(int unit) const
    {
        if constexpr (PT::kLds) return s[unit % NC * kTile];
        else return v[unit % NC];
    }
    __device__ __forceinline__ void put(int unit, double2 u)
    {
        if constexpr (PT::kLds) s[unit % NC * kTile] = u;
        else v[unit % NC] = u;
    }
    __device__ __forceinline__ double2 total() const
    {
        double2 t = get(0);
#pragma unroll
        for (int c = 1; c < NC; ++c) {
            const double2 u = get(c);
            t.x += u.x;
            t.y += u.y;
        }
        return t;
    }
};

// Adds the parts of a tile (`red` holds NP * 64 double2) and stores its rows.
// Block-uniform; with NP > 1 the block is one tile's wavefronts.
template <int NP>
__device__ __forceinline__ void store_tile(double2 v, int part, int64_t tile, int64_t D,
                                           double2 *red, double2 *__restrict__ HC)
{
    const int lane = threadIdx.x & 63;
    const int64_t g = tile * kTile + lane;
    if constexpr (NP > 1) {
        __syncthreads();   // the last tile's sums are read
        red[part * kTile + lane] = v;
        __syncthreads();
        if (part != 0) return;
#pragma unroll
        for (int p = 1; p < NP; ++p) {
            v.x += red[p * kTile + lane].x;
            v.y += red[p * kTile + lane].y;
        }
    }
    if (g < D) HC[g] = v;
}

// Removal pair p (lexicographic k <= s) -> (k, s), for compile-time use.
__host__ __device__ constexpr int pair_k(int M, int p)
{
    for (int k = 0; k < M; ++k) {
        if (p < M - k) return k;
        p -= M - k;
    }
    return -1;
}
__host__ __device__ constexpr int pair_s(int M, int p)
{
    for (int k = 0; k < M; ++k) {
        if (p < M - k) return k + p;
        p -= M - k;
    }
    return -1;
}

// Slots of one removal pair handled per batch: a batch issues all its table
// loads, then all its gathers, then the arithmetic.
template <int MT>
constexpr int kSlotBatch = MT * MT < MC_SLOT_BATCH ? MT * MT : MC_SLOT_BATCH;
// Double-jump blocks of the paper form: a whole M*M block per batch up to
// M * M = MC_T2_WHOLE_BLOCK (larger M would spill).
#ifndef MC_T2_WHOLE_BLOCK
#define MC_T2_WHOLE_BLOCK 25
#endif
template <int MT>
constexpr int kT2Batch = MT * MT <= MC_T2_WHOLE_BLOCK ? MT * MT : kSlotBatch<MT>;

// The paper's double-jump block holds one column per ordered creation pair
// (q, l); (q, l) and (l, q) reach one configuration, so the per-pair walk
// reads the columns with q <= l only and weights them by G'_{P,ql} +
// G'_{P,lq}.  Slot j of the walk is column t2_col(j) of the block.
#ifndef MC_PAPER_TRIANGLE
#define MC_PAPER_TRIANGLE 1
#endif
template <int MT>
constexpr int kT2Slots = MC_PAPER_TRIANGLE ? MT * (MT + 1) / 2 : MT * MT;

template <int MT>
__host__ __device__ constexpr int t2_col(int j)
{
    if (!MC_PAPER_TRIANGLE) return j;
    for (int q = 0; q < MT; ++q) {
        if (j < MT - q) return q * MT + q + j;
        j -= MT - q;
    }
    return 0;
}

// Indices of walk slots [J0, J0 + SB) of a double-jump block (one per lane).
template <int MT, int SB, int J0>
__device__ __forceinline__ void load_t2_batch(int32_t (&t)[SB], __amdgpu_buffer_rsrc_t r, int lane)
{
#pragma unroll
    for (int i = 0; i < SB; ++i)
        if (J0 + i < kT2Slots<MT>)
            t[i] = buf_ld_i32(r, (uint32_t)((t2_col<MT>(J0 + i) * kTile + lane) * 4), 0);
}

// Contribution of removal pair P = (K, S), K <= S, to one row:
//   A_KS * sum_{q,l} G'_{P,ql} B_ql(m) C[T2 slot],   m = n - e_K - e_S,
// for the pair's block at `pos` (M*M*64 entries).  Lanes whose row cannot
// lose (K, S) hold -1 entries (gathers read 0) and get A = 0.
template <int MT, int B, int NB>
__device__ __forceinline__ void pair_batches(int lane, __amdgpu_buffer_rsrc_t r2,
                                             const double (&rq)[MT], const double (&dq)[MT],
                                             const double2 *__restrict__ G,
                                             const Gather<false> &ldc, double &br, double &bi)
{
    if constexpr (B < NB) {
        constexpr int NS = kT2Slots<MT>, SB = kT2Batch<MT>, J0 = B * SB;
        int32_t t[SB];
        double2 c[SB];
        load_t2_batch<MT, SB, J0>(t, r2, lane);
#pragma unroll
        for (int i = 0; i < SB; ++i)
            if (J0 + i < NS) c[i] = ldc(t[i]);
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int j = J0 + i;
            if (j >= NS) break;
            const int col = t2_col<MT>(j), q = col / MT, l = col % MT;
            const double Bf = q == l ? rq[q] * dq[q] : rq[q] * rq[l];
            const double cr = c[i].x * Bf, ci = c[i].y * Bf;
            double2 Gv = G[col];
            if (MC_PAPER_TRIANGLE && q != l) {
                Gv.x += G[l * MT + q].x;
                Gv.y += G[l * MT + q].y;
            }
            br = fma(Gv.x, cr, br);
            br = fma(-Gv.y, ci, br);
            bi = fma(Gv.x, ci, bi);
            bi = fma(Gv.y, cr, bi);
        }
        pair_batches<MT, B + 1, NB>(lane, r2, rq, dq, G, ldc, br, bi);
    }
}

template <int MT, int P>
__device__ __forceinline__ void pair_term(const int32_t *t2, int64_t pos, int lane,
                                          const int (&n)[MT], const RowSq<MT> &R,
                                          const double2 *__restrict__ gp, const Gather<false> &ldc,
                                          double &ar, double &ai)
{
    constexpr int K = pair_k(MT, P), S = pair_s(MT, P);
    constexpr int NS = MT * MT, SB = kT2Batch<MT>;
    constexpr int NB = (kT2Slots<MT> + SB - 1) / SB;
    const __amdgpu_buffer_rsrc_t r2 = make_rsrc(t2 + pos, (uint32_t)(NS * kTile * 4));
    const bool valid = K == S ? n[K] >= 2 : (n[K] >= 1 && n[S] >= 1);
    const double A =
        valid ? R.template root<0>(K) * (K == S ? R.template root<-1>(K) : R.template root<0>(S))
              : 0.0;
    // creation amplitudes on m: rq = sqrt(m_q + 1), dq = sqrt(m_q + 2)
    double rq[MT], dq[MT];
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        const int d = (q == K) + (q == S);
        rq[q] = d == 0 ? R.template root<1>(q) : (d == 1 ? R.template root<0>(q) : R.template root<-1>(q));
        dq[q] = d == 0 ? R.template root<2>(q) : (d == 1 ? R.template root<1>(q) : R.template root<0>(q));
    }
    double br = 0.0, bi = 0.0;
    pair_batches<MT, 0, NB>(lane, r2, rq, dq, gp + P * NS, ldc, br, bi);
    ar = fma(A, br, ar);
    ai = fma(A, bi, ai);
}

// All removal pairs in order; each present pair is its own basic block
// (uniform branch on the tile's pair mask), which keeps the scheduler from
// hoisting later pairs' loads.
template <int MT, class PT, int... Ps>
__device__ __forceinline__ void all_pairs(std::integer_sequence<int, Ps...>, PT part,
                                          const uint64_t *pm, const int32_t *t2, int64_t off0,
                                          int64_t off1, int lane, const int (&n)[MT],
                                          const RowSq<MT> &R, const double2 *__restrict__ gp,
                                          const Gather<false> &ldc, RowSum<PT> &A)
{
    int64_t pos = off0;
    (
        [&] {
            constexpr int NSB = MT * MT * kTile;
            if (((pm[Ps >> 6] >> (Ps & 63)) & 1) && pos + NSB <= off1) {
                if (PT::kWaves == 1 || part.template has<Ps>()) {
                    double2 u = A.get(Ps);
                    pair_term<MT, Ps>(t2, pos, lane, n, R, gp, ldc, u.x, u.y);
                    A.put(Ps, u);
                }
                pos += NSB;
            }
        }(),
        ...);
}

// One 64-row tile of H.C for a compile-time orbital count MT (1..8) through
// the single- and double-jump maps; every orbital, pair and slot index is a
// compile-time constant.  Called by one whole wavefront.
template <int MT, typename OccT, class PT>
__device__ __forceinline__ double2 apply_tile_t2(PT part, int64_t tile, int64_t D, int64_t cap, const double *sq,
                                              const OccT *__restrict__ occ,
                                              const int32_t *__restrict__ t1,
                                              const uint64_t *__restrict__ pmask,
                                              const int64_t *__restrict__ t2_off,
                                              const int32_t *__restrict__ t2,
                                              const double2 *__restrict__ h,
                                              const double2 *__restrict__ gp,
                                              const double2 *__restrict__ C)
{
    constexpr int M = MT;
    constexpr int P = M * (M + 1) / 2;
    constexpr int W = (P + 63) / 64;
    const int lane = threadIdx.x & 63;
    const int64_t g = tile * kTile + lane;
    const bool live = g < D;

    int64_t off0, off1;
    t2_block(t2_off, tile, cap, off0, off1);
    int n[M];
    RowSq<M> R;
    load_row<MT, OccT>(occ, tile, lane, n, R, sq);
    const Gather<false> ldc(C, D);

    // diagonal one-body part: sum_k h_kk n_k C_g
    const double2 cg = ldc(live ? (int32_t)g : -1);
    double2 own = make_double2(0.0, 0.0);
    if (part.own()) {
        double dr = 0.0, di = 0.0;
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const double2 hk = h[k * M + k];
            dr = fma(hk.x, (double)n[k], dr);
            di = fma(hk.y, (double)n[k], di);
        }
        own.x = dr * cg.x - di * cg.y;
        own.y = dr * cg.y + di * cg.x;
    }
    RowSum<PT> A(part, own);

    // single jumps k -> l (k != l): h_kl sqrt(n_k (n_l + 1)) C[T1], in
    // batches of kSlotBatch slots (table loads, then gathers, then FMAs)
    {
        constexpr int NS = M * M, SB = kSlotBatch<MT>;
        const __amdgpu_buffer_rsrc_t r1 =
            make_rsrc(t1 + tile * NS * kTile, (uint32_t)(NS * kTile * 4));
#pragma unroll
        for (int j0 = 0; j0 < NS; j0 += SB) {
            if (PT::kWaves > 1 && part.part != j0 / SB % PT::kWaves) continue;
            double2 u = A.get(j0 / SB);
            double &ar = u.x, &ai = u.y;
            int32_t t[SB];
            double2 c[SB];
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                const int j = j0 + i;
                if (j < NS && j / M != j % M)
                    t[i] = buf_ld_i32(r1, (uint32_t)((j * kTile + lane) * 4), 0);
            }
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                const int j = j0 + i;
                if (j < NS && j / M != j % M) c[i] = ldc(t[i]);
            }
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                const int j = j0 + i;
                if (j >= NS) break;
                const int k = j / M, l = j % M;
                if (k == l) continue;
                const double f = R.template root<0>(k) * R.template root<1>(l);
                const double2 hv = h[j];
                const double cr = c[i].x * f, ci = c[i].y * f;
                ar = fma(hv.x, cr, ar);
                ar = fma(-hv.y, ci, ar);
                ai = fma(hv.x, ci, ai);
                ai = fma(hv.y, cr, ai);
            }
            A.put(j0 / SB, u);
        }
    }

    // double jumps: one block of M*M*64 entries per pair present in the tile
    all_pairs<MT>(std::make_integer_sequence<int, P>{}, part, pmask + tile * W, t2, off0, off1,
                        lane, n, R, gp, ldc, A);
    return A.total();
}


// ---------------------------------------------------------------------------
// H.C without the double-jump map: a double jump (k, s) -> (q, l) is two
// single jumps, first k -> q from the row, then s -> l from that
// intermediate configuration,
//     T2[g][(k,s)][q*M + l] = T1[T1[g][k][q]][s][l],
// which holds for every valid removal pair (the intermediate still has a
// particle in s).  For q = k the first hop leaves the row unchanged and the
// target is the single jump T1[g][s][l].  First hops and q = k targets come
// from the tile's own single-jump block (coalesced, cache-resident); the
// second hop is a gather from rows near g.
// ---------------------------------------------------------------------------
template <int MT, int P>
__device__ __forceinline__ void pair_term_chained(int64_t D, const int32_t *__restrict__ t1,
                                                  __amdgpu_buffer_rsrc_t r1, int lane,
                                                  const int (&n)[MT], const RowSq<MT, kLdsRootsChained<MT>> &R,
                                                  const double2 *__restrict__ gp,
                                                  const Gather<false> &ldc, double &ar, double &ai)
{
    constexpr int K = pair_k(MT, P), S = pair_s(MT, P);
    constexpr int NS = MT * MT, SB = kSlotBatch<MT>;
    const bool valid = K == S ? n[K] >= 2 : (n[K] >= 1 && n[S] >= 1);
    if (!__ballot(valid)) return;   // no row of the tile can lose (K, S)
    const double A =
        valid ? R.template root<0>(K) * (K == S ? R.template root<-1>(K) : R.template root<0>(S))
              : 0.0;
    double rq[MT], dq[MT];
#pragma unroll
    for (int q = 0; q < MT; ++q) {
        const int d = (q == K) + (q == S);
        rq[q] = d == 0 ? R.template root<1>(q) : (d == 1 ? R.template root<0>(q) : R.template root<-1>(q));
        dq[q] = d == 0 ? R.template root<2>(q) : (d == 1 ? R.template root<1>(q) : R.template root<0>(q));
    }
    // first hops K -> q of this row
    int32_t fh[MT];
#pragma unroll
    for (int q = 0; q < MT; ++q)
        fh[q] = q == K ? 0 : buf_ld_i32(r1, (uint32_t)(((K * MT + q) * kTile + lane) * 4), 0);
    const double2 *G = gp + P * NS;
    double br = 0.0, bi = 0.0;
#pragma unroll
    for (int j0 = 0; j0 < NS; j0 += SB) {
        int32_t t[SB];
        double2 c[SB];
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int j = j0 + i;
            if (j >= NS) break;
            const int q = j / MT, l = j % MT;
            if (q == K) {
                const int32_t v = buf_ld_i32(r1, (uint32_t)(((S * MT + l) * kTile + lane) * 4), 0);
                t[i] = valid ? v : -1;
            } else {
                const int32_t b = fh[q];
                const bool ok = valid && b >= 0 && b < D;
                const int64_t bb = ok ? b : 0;
                const int32_t v = t1[((bb >> 6) * NS + S * MT + l) * kTile + (bb & 63)];
                t[i] = ok ? v : -1;
            }
        }
#pragma unroll
        for (int i = 0; i < SB; ++i)
            if (j0 + i < NS) c[i] = ldc(t[i]);
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int j = j0 + i;
            if (j >= NS) break;
            const int q = j / MT, l = j % MT;
            const double B = q == l ? rq[q] * dq[q] : rq[q] * rq[l];
            const double cr = c[i].x * B, ci = c[i].y * B;
            const double2 Gv = G[j];
            br = fma(Gv.x, cr, br);
            br = fma(-Gv.y, ci, br);
            bi = fma(Gv.x, ci, bi);
            bi = fma(Gv.y, cr, bi);
        }
    }
    ar = fma(A, br, ar);
    ai = fma(A, bi, ai);
}

// The same double jumps for M >= 6 with the removal pairs as a loop: the
// compile-time fold over M(M+1)/2 pairs of M^2 slots each keeps too many
// values live at once there.  K and S are wave-uniform loop counters; q and
// l stay compile-time, so the per-row occupations are picked with selects and
// the roots come from the block's sqrt table.
template <int MT, class PT>
__device__ __forceinline__ void pairs_chained_loop(PT part, int64_t D, int64_t g,
                                                   const int32_t *__restrict__ t1,
                                                   __amdgpu_buffer_rsrc_t r1, int lane,
                                                   const int (&n)[MT], const double *sq,
                                                   const double2 *__restrict__ gp,
                                                   const Gather<false> &ldc, RowSum<PT> &sum)
{
    constexpr int NS = MT * MT, SB = kSlotBatch<MT>;
    int P = 0;
#pragma unroll 1
    for (int K = 0; K < MT; ++K) {
#pragma unroll 1
        for (int S = K; S < MT; ++S, ++P) {
            if (PT::kWaves > 1 && part.part != P % PT::kWaves) continue;
            int nK = 0, nS = 0;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                nK = m == K ? n[m] : nK;
                nS = m == S ? n[m] : nS;
            }
            const bool valid = K == S ? nK >= 2 : (nK >= 1 && nS >= 1);
            if (!__ballot(valid)) continue;
            const double A = valid ? sq[nK] * (K == S ? sq[nK > 0 ? nK - 1 : 0] : sq[nS]) : 0.0;
            // first hops K -> q (q = K: the row itself)
            int32_t b[MT];
#pragma unroll
            for (int q = 0; q < MT; ++q) {
                const int32_t f = buf_ld_i32(r1, (uint32_t)(((K * MT + q) * kTile + lane) * 4), 0);
                b[q] = q == K ? (int32_t)g : f;
            }
            double rq[MT];
#pragma unroll
            for (int q = 0; q < MT; ++q) {
                const int i = n[q] + 1 - (q == K) - (q == S);
                rq[q] = sq[i > 0 ? i : 0];
            }
            const double2 *G = gp + (int64_t)P * NS;
            double br = 0.0, bi = 0.0;
#pragma unroll
            for (int j0 = 0; j0 < NS; j0 += SB) {
                int32_t t[SB];
                double2 c[SB];
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    const int j = j0 + i;
                    if (j >= NS) break;
                    const int q = j / MT, l = j % MT;
                    const int32_t bq = b[q];
                    const bool ok = valid && bq >= 0 && bq < D;
                    const int64_t bb = ok ? bq : 0;
                    const int32_t v = t1[((bb >> 6) * NS + S * MT + l) * kTile + (bb & 63)];
                    t[i] = ok ? v : -1;
                }
#pragma unroll
                for (int i = 0; i < SB; ++i)
                    if (j0 + i < NS) c[i] = ldc(t[i]);
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    const int j = j0 + i;
                    if (j >= NS) break;
                    const int q = j / MT, l = j % MT;
                    double Bv;
                    if (q == l) {
                        const int i2 = n[q] + 2 - (q == K) - (q == S);
                        Bv = rq[q] * sq[i2 > 0 ? i2 : 0];
                    } else {
                        Bv = rq[q] * rq[l];
                    }
                    const double cr = c[i].x * Bv, ci = c[i].y * Bv;
                    const double2 Gv = G[j];
                    br = fma(Gv.x, cr, br);
                    br = fma(-Gv.y, ci, br);
                    bi = fma(Gv.x, ci, bi);
                    bi = fma(Gv.y, cr, bi);
                }
            }
            double2 u = sum.get(P);
            u.x = fma(A, br, u.x);
            u.y = fma(A, bi, u.y);
            sum.put(P, u);
        }
    }
}

template <int MT, class PT, int... Ps>
__device__ __forceinline__ void all_pairs_chained(std::integer_sequence<int, Ps...>, PT part, int64_t D,
                                                  const int32_t *__restrict__ t1,
                                                  __amdgpu_buffer_rsrc_t r1, int lane,
                                                  const int (&n)[MT], const RowSq<MT, kLdsRootsChained<MT>> &R,
                                                  const double2 *__restrict__ gp,
                                                  const Gather<false> &ldc, RowSum<PT> &A)
{
    (
        [&] {
            if (PT::kWaves == 1 || part.template has<Ps>()) {
                double2 u = A.get(Ps);
                pair_term_chained<MT, Ps>(D, t1, r1, lane, n, R, gp, ldc, u.x, u.y);
                A.put(Ps, u);
            }
        }(),
        ...);
}

// One 64-row tile of H.C through single jumps only (see above).
template <int MT, typename OccT, class PT>
__device__ __forceinline__ double2 apply_tile_chained(PT part, int64_t tile, int64_t D, const double *sq,
                                                   const OccT *__restrict__ occ,
                                                   const int32_t *__restrict__ t1,
                                                   const double2 *__restrict__ h,
                                                   const double2 *__restrict__ gp,
                                                   const double2 *__restrict__ C)
{
    constexpr int M = MT;
    constexpr int P = M * (M + 1) / 2;
    constexpr int NS = M * M, SB = kSlotBatch<MT>;
    const int lane = threadIdx.x & 63;
    const int64_t g = tile * kTile + lane;
    const bool live = g < D;
    int n[M];
    RowSq<M, kLdsRootsChained<MT>> R;
    load_row<MT, OccT>(occ, tile, lane, n, R, sq);
    const Gather<false> ldc(C, D);
    const __amdgpu_buffer_rsrc_t r1 =
        make_rsrc(t1 + tile * NS * kTile, (uint32_t)(NS * kTile * 4));
    const double2 cg = ldc(live ? (int32_t)g : -1);
    double2 own = make_double2(0.0, 0.0);
    if (part.own()) {
        double dr = 0.0, di = 0.0;
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const double2 hk = h[k * M + k];
            dr = fma(hk.x, (double)n[k], dr);
            di = fma(hk.y, (double)n[k], di);
        }
        own.x = dr * cg.x - di * cg.y;
        own.y = dr * cg.y + di * cg.x;
    }
    RowSum<PT> A(part, own);
    // single jumps k -> l (k != l), in batches
#pragma unroll
    for (int j0 = 0; j0 < NS; j0 += SB) {
        if (PT::kWaves > 1 && part.part != j0 / SB % PT::kWaves) continue;
        double2 u = A.get(j0 / SB);
        double &ar = u.x, &ai = u.y;
        int32_t t[SB];
        double2 c[SB];
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int j = j0 + i;
            if (j < NS && j / M != j % M) t[i] = buf_ld_i32(r1, (uint32_t)((j * kTile + lane) * 4), 0);
        }
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int j = j0 + i;
            if (j < NS && j / M != j % M) c[i] = ldc(t[i]);
        }
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int j = j0 + i;
            if (j >= NS) break;
            const int k = j / M, l = j % M;
            if (k == l) continue;
            const double f = R.template root<0>(k) * R.template root<1>(l);
            const double2 hv = h[j];
            const double cr = c[i].x * f, ci = c[i].y * f;
            ar = fma(hv.x, cr, ar);
            ar = fma(-hv.y, ci, ar);
            ai = fma(hv.x, ci, ai);
            ai = fma(hv.y, cr, ai);
        }
        A.put(j0 / SB, u);
    }
    if constexpr (kLdsRootsChained<MT>)
        pairs_chained_loop<MT>(part, D, g, t1, r1, lane, n, sq, gp, ldc, A);
    else
        all_pairs_chained<MT>(std::make_integer_sequence<int, P>{}, part, D, t1, r1, lane, n, R,
                                    gp, ldc, A);
    return A.total();
}

}  // namespace mc
