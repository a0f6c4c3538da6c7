// H.C with no table, four rows per lane (large spaces; 4 <= M <= 8, and M = 3 in
// the apply over non-zero constants only).
//
// One row per lane (mc_direct.h) gathers every configuration that H reaches
// from that row: 131 at M = 5.  Rows that differ by particles moved between
// two orbitals reach mostly the same configurations, so here a lane holds
// R = 4 rows of a chain between the two highest orbitals a = M-2, b = M-1,
//
//   row j = (n_0, ..., n_a - j, n_b + j),   j = 0 .. R-1,
//
// and gathers each configuration that any of them reaches once: 296 for four
// rows at M = 5 (74 per row), 664 at M = 6 (166 instead of 271).
//
// Classes.  Two jumps from the rows of a lane belong to one class when they
// change the outer orbitals 0 .. M-3 alike (particles leave c1, c2 and enter
// d1, d2); a class then differs only in how the inner orbitals a, b take
// part.  With delta = #removed - #created outer particles, member Delta_a of
// a class changes n_a by Delta_a and n_b by delta - Delta_a, so from row j it
// reaches the configuration u = Delta_a - j of the class
// (n_a + u, n_b + delta - u).  Each class loads u = lo - (R-1) .. hi once and
// uses each value for every row and member that meets it.
//
// Amplitudes.  The amplitude of a jump is a product of an outer factor (the
// same for the rows of a lane, taken into the coefficient once) and an inner
// factor f(n_a, n_b) that depends on the row and on the member's kind only.
// So values are summed per inner factor with four multiply-adds each and the
// factor multiplies the sum: about 1,100 vector instructions per row instead
// of 2,300 at M = 5.
//
// Rows.  A lane's item is a row with n_b divisible by R (its row 0).  The
// index rises with n_b first, so the items of one n_b are consecutive rows:
// lanes of a wavefront gather consecutive elements of C for nearly every
// jump.  Row j exists where n_a >= j.  With the prefix sums S_m of mc_direct.h
// row j's index is D - 1 - sum_{m < a} G_m(S_m) - G_a(S_a - j).
//
// Impossible jumps.  A configuration with a negative occupation is gathered
// out of range (zero), so a value that is not finite reaches only the rows
// that H couples to it.  A jump is possible exactly when its configuration
// has no negative occupation (removed and created orbitals are disjoint).
#pragma once

#include "mc_direct.h"

namespace mc {

constexpr int kBlockRows = 4;
// Values loaded per basic block: as many as the registers hold beside the
// accumulators without spilling (measured: 20 against 12 at M = 5 0.97x the
// time, 16 against 12 at M = 6 1.09x, within 1 % at M = 7, 0.90x at M = 8).
__host__ __device__ constexpr int block_loads(int M) { return M <= 5 ? 20 : (M == 6 ? 12 : 16); }

// Kinds of classes, in the order of the walk.
enum BlockKind {
    kBkMove = 0,    // c -> d                 Delta_a in {-1, 0, 1}
    kBkTwo,         // c c' -> d d'           {0}
    kBkIn,          // c -> inner             {-1, 0, 1, 2}
    kBkInMove,      // c c' -> d inner        {0, 1}
    kBkOut,         // inner -> d             {-2, -1, 0, 1}
    kBkOutMove,     // c inner -> d d'        {-1, 0}
    kBkIn2,         // c c' -> inner inner    {0, 1, 2}
    kBkOut2,        // inner inner -> d d'    {-2, -1, 0}
    kBkKinds
};

struct BlockClass {
    int kind, c1, c2, d1, d2, lo, hi;
};

template <int MT>
struct BlockPlan {
    static constexpr int R = kBlockRows;
    static constexpr int MAXC = 520;
    BlockClass cls[MAXC] = {};
    int n = 0;
    int seg[kBkKinds + 1] = {};    // first class of each kind
    int bstart[MAXC + 1] = {};     // batches of classes of one kind
    int bseg[kBkKinds + 1] = {};   // first batch of each kind
    int nb = 0;

    static constexpr bool outer(int o) { return o < MT - 2; }
    constexpr void add(int kind, int c1, int c2, int d1, int d2, int lo, int hi)
    {
        cls[n] = BlockClass{kind, c1, c2, d1, d2, lo, hi};
        ++n;
    }
    constexpr int loads(int i) const { return cls[i].hi - cls[i].lo + R; }

    constexpr BlockPlan()
    {
        for (int kind = 0; kind < kBkKinds; ++kind) {
            seg[kind] = n;
            const int nc = kind == kBkMove || kind == kBkIn || kind == kBkOutMove  ? 1
                           : kind == kBkTwo || kind == kBkInMove || kind == kBkIn2 ? 2
                                                                                   : 0;
            const int nd = kind == kBkMove || kind == kBkOut || kind == kBkInMove   ? 1
                           : kind == kBkTwo || kind == kBkOutMove || kind == kBkOut2 ? 2
                                                                                     : 0;
            const int lo = kind == kBkMove || kind == kBkIn || kind == kBkOutMove ? -1
                           : kind == kBkOut || kind == kBkOut2                     ? -2
                                                                                   : 0;
            const int hi = kind == kBkMove || kind == kBkInMove || kind == kBkOut ? 1
                           : kind == kBkIn || kind == kBkIn2                      ? 2
                                                                                  : 0;
            for (int c1 = nc > 0 ? 0 : -1; c1 < (nc > 0 ? MT : 0); ++c1) {
                if (nc > 0 && !outer(c1)) continue;
                for (int c2 = nc > 1 ? c1 : -1; c2 < (nc > 1 ? MT : 0); ++c2) {
                    if (nc > 1 && !outer(c2)) continue;
                    for (int d1 = nd > 0 ? 0 : -1; d1 < (nd > 0 ? MT : 0); ++d1) {
                        if (nd > 0 && (!outer(d1) || d1 == c1 || d1 == c2)) continue;
                        for (int d2 = nd > 1 ? d1 : -1; d2 < (nd > 1 ? MT : 0); ++d2) {
                            if (nd > 1 && (!outer(d2) || d2 == c1 || d2 == c2)) continue;
                            add(kind, c1, c2, d1, d2, lo, hi);
                        }
                    }
                }
            }
        }
        seg[kBkKinds] = n;
        for (int kind = 0; kind < kBkKinds; ++kind) {
            bseg[kind] = nb;
            int i = seg[kind];
            while (i < seg[kind + 1]) {
                bstart[nb++] = i;
                int sum = loads(i++);
                while (i < seg[kind + 1] && sum + loads(i) <= block_loads(MT)) sum += loads(i++);
            }
        }
        bstart[nb] = n;
        bseg[kBkKinds] = nb;
    }
};

template <int MT>
constexpr BlockPlan<MT> kBlockPlan{};

// Accumulator of member Delta_a of a class: slot 0 is the row's sum itself
// (inner factor 1), the others are multiplied by block_factor.
__host__ __device__ constexpr int block_slot(int kind, int d1)
{
    switch (kind) {
    case kBkMove: return d1 == 0 ? 0 : (d1 < 0 ? 1 : 2);
    case kBkTwo: return 0;
    case kBkIn: return d1 == 1 ? 1 : (d1 == 0 ? 2 : (d1 == -1 ? 3 : 4));
    case kBkInMove: return d1 == 1 ? 1 : 2;
    case kBkOut: return d1 == -1 ? 1 : (d1 == 0 ? 2 : (d1 == -2 ? 3 : 4));
    case kBkOutMove: return d1 == -1 ? 1 : 2;
    case kBkIn2: return d1 == 2 ? 1 : (d1 == 1 ? 2 : 3);
    default: return d1 == -2 ? 1 : (d1 == -1 ? 2 : 3);
    }
}

// The kinds with many classes (240, 90 and 90 at M = 8) sum into a second
// level, slot 3 for slot 0 and 3, 4 for 1, 2 (free at that time), which is
// added to the first every kBlockFlush batches: short chains of additions
// round less (relative error against 64 bits, one row per lane / one chain /
// so: N=200, M=5 3.8e-16 / 3.9e-16 / 3.4e-16; N=24, M=8 4.8e-16 / 7.1e-16 /
// 4.7e-16, at the same time).
constexpr int kBlockFlush = 6;
__host__ __device__ constexpr bool block_two_level(int M, int kind)
{
    return M >= 5 && (kind == kBkTwo || kind == kBkInMove || kind == kBkOutMove);
}
__host__ __device__ constexpr int block_level_slot(int M, int kind, int d1)
{
    const int s = block_slot(kind, d1);
    return block_two_level(M, kind) ? (s == 0 ? 3 : s + 2) : s;
}

// Index of the true double jump {r1, r2} -> {a1, a2} among the staged GD.
__host__ __device__ constexpr int block_gd(int M, int r1, int r2, int a1, int a2)
{
    const int K = r1 < r2 ? r1 : r2, S = r1 < r2 ? r2 : r1;
    const int q = a1 < a2 ? a1 : a2, l = a1 < a2 ? a2 : a1;
    const int p = K * M - K * (K - 1) / 2 + (S - K);
    return reduced_pair_offset(M, p) + reduced_rank(M, K, S, q, l);
}

// Tables of one (N, M) space behind the staged constants, int32 each:
// G_m(s) = C(s + m, m + 1), s = 0 .. N, for m = 1 .. M-2, then the number of
// items with n_b < R q, q = 0 .. floor(N / R) + 1.
__host__ __device__ constexpr int block_table_ints(int N, int M)
{
    return (M - 2) * (N + 1) + N / kBlockRows + 2;
}

// The tables of (N, M), by one block of 256 threads; `sum` holds 256 int.
__device__ inline void stage_block_tables(int N, int M, int *__restrict__ tab, int *sum)
{
    const int t = threadIdx.x;
    for (int i = t; i < (M - 2) * (N + 1); i += 256) {
        const int m = 1 + i / (N + 1), s = i % (N + 1);
        double f = 1.0;
        for (int k = 2; k <= m + 1; ++k) f *= (double)k;
        tab[i] = (int)rint(direct_prod(m, (double)s) / f);
    }
    // rows with n_b = R i number C(S + M - 2, M - 2) = G_{M-3}(S + 1), S = N - R i;
    // their exclusive prefix sums
    double f = 1.0;
    for (int k = 2; k <= M - 2; ++k) f *= (double)k;
    int *first = tab + (M - 2) * (N + 1);
    const int nq = N / kBlockRows + 1;
    int carry = 0;
    for (int q0 = 0; q0 <= nq; q0 += 256) {
        const int q = q0 + t, S = N - kBlockRows * q;
        const int v = S >= 0 ? (int)rint(direct_prod(M - 3, (double)(S + 1)) / f) : 0;
        sum[t] = v;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {
            const int u = t >= o ? sum[t - o] : 0;
            __syncthreads();
            sum[t] += u;
            __syncthreads();
        }
        if (q <= nq) first[q] = carry + sum[t] - v;
        carry += sum[255];
        __syncthreads();
    }
}

// One lane: its rows, and what their targets and amplitudes come from.
template <int MT>
struct BlockLane {
    static constexpr int R = kBlockRows;
    static constexpr int IA = MT - 2, IB = MT - 1;
    static constexpr int NX = R + 4;                    // S_a + x, x = -(R+1) .. 2
    static constexpr int NG = MT > 3 ? MT - 3 : 1;      // m = 1 .. M-3
    int n[MT];            // occupations of row 0
    uint32_t base;        // 16 (D - 1 - n_0)
    uint32_t ga[NX];      // 16 G_a(S_a + x) (S_a + x clamped to [0, N])
    uint32_t gm[NG][5];   // 16 G_m(S_m + d), d = -2 .. 2 (clamped likewise)
    const double *sq;

    __device__ __forceinline__ void init(int item, int64_t D, int N, const int *__restrict__ tab,
                                         const double *sqrt_tab)
    {
        sq = sqrt_tab;
        int S[MT];
        S[IB] = N;
        const int nbits = 32 - __builtin_clz(N);
        // largest q with first[q] <= item
        const int *first = tab + (MT - 2) * (N + 1);
        int q = 0;
        for (int b = nbits - 1; b >= 0; --b) {
            const int c = q | (1 << b);
            if (c <= N / R && first[c] <= item) q = c;
        }
        S[IA] = N - R * q;
        // what is left of the index below: items rise with the index
        int J = first[q + 1] - 1 - item;
#pragma unroll
        for (int m = IA - 1; m >= 1; --m) {
            // largest s <= S_{m+1} with G_m(s) <= J
            const int *G = tab + (m - 1) * (N + 1);
            int s = 0;
            for (int b = nbits - 1; b >= 0; --b) {
                const int c = s | (1 << b);
                if (c <= S[m + 1] && G[c] <= J) s = c;
            }
            J -= G[s];
            S[m] = s;
        }
        S[0] = J;
        n[0] = J;
#pragma unroll
        for (int m = 1; m < MT; ++m) n[m] = S[m] - S[m - 1];
        base = (uint32_t)(D - 1 - n[0]) << 4;
        auto at = [&](int m, int s) {
            s = s < 0 ? 0 : (s > N ? N : s);
            return (uint32_t)tab[(m - 1) * (N + 1) + s] << 4;
        };
#pragma unroll
        for (int k = 0; k < NX; ++k) ga[k] = at(IA, S[IA] + k - (R + 1));
#pragma unroll
        for (int m = 1; m < IA; ++m)
#pragma unroll
            for (int d = -2; d <= 2; ++d) gm[m - 1][d + 2] = at(m, S[m] + d);
    }

    __device__ __forceinline__ double root(int m, int d) const
    {
        const int i = n[m] + d;
        return sq[i > 0 ? i : 0];
    }

    // change of S_m, m < a, when particles leave C1, C2 and enter D1, D2
    template <int m, int C1, int C2, int D1, int D2>
    static constexpr int shift()
    {
        return prefix_delta(m, C1, C2, D1, D2);
    }

    template <int C1, int C2, int D1, int D2, int... Ks>
    __device__ __forceinline__ uint32_t class_base_fold(std::integer_sequence<int, Ks...>) const
    {
        constexpr int d0 = shift<0, C1, C2, D1, D2>();
        const uint32_t b0 = base - (uint32_t)(16 * d0);
        return (b0 - ... - gm[Ks][shift<Ks + 1, C1, C2, D1, D2>() + 2]);
    }

    // 16 x (index + G_a term) of a class; out of range where an outer
    // orbital cannot lose its particles
    template <int C1, int C2, int D1, int D2>
    __device__ __forceinline__ uint32_t class_base() const
    {
        const uint32_t b =
            class_base_fold<C1, C2, D1, D2>(std::make_integer_sequence<int, (MT > 3 ? MT - 3 : 0)>{});
        if constexpr (C1 < 0) return b;
        else if constexpr (C2 < 0) return n[C1] >= 1 ? b : 0xFFFFFFF0u;
        else if constexpr (C1 == C2) return n[C1] >= 2 ? b : 0xFFFFFFF0u;
        else return n[C1] >= 1 && n[C2] >= 1 ? b : 0xFFFFFFF0u;
    }

    // byte offset of configuration u of a class
    template <int DELTA, int U>
    __device__ __forceinline__ uint32_t address(uint32_t cb) const
    {
        constexpr int x = U - DELTA;   // change of S_a
        static_assert(x >= -(R + 1) && x <= 2, "chain offset out of range");
        const uint32_t v = cb - ga[x + R + 1];
        constexpr int w = DELTA - U;
        if constexpr (U < 0 && w < 0) return n[IA] >= -U && n[IB] >= -w ? v : 0xFFFFFFF0u;
        else if constexpr (U < 0) return n[IA] >= -U ? v : 0xFFFFFFF0u;
        else if constexpr (w < 0) return n[IB] >= -w ? v : 0xFFFFFFF0u;
        else return v;
    }

    // amplitude of the outer orbitals
    template <int C1, int C2, int D1, int D2>
    __device__ __forceinline__ double outer_amp() const
    {
        double a = 1.0;
        if constexpr (C1 >= 0) a = root(C1, 0);
        if constexpr (C2 >= 0) a *= root(C2, C1 == C2 ? -1 : 0);
        if constexpr (D1 >= 0) a = C1 >= 0 ? a * root(D1, 1) : root(D1, 1);
        if constexpr (D2 >= 0) a *= root(D2, D1 == D2 ? 2 : 1);
        return a;
    }
};

template <int MT>
struct BlockAcc {
    double x[5][kBlockRows], y[5][kBlockRows];
};

// Loads of class I: v[OFF + k] = configuration u = lo - (R-1) + k.
template <int MT, int I, int OFF, int... Ks>
__device__ __forceinline__ void block_class_loads(std::integer_sequence<int, Ks...>,
                                                  const BlockLane<MT> &L,
                                                  const Gather<false> &ldc, double2 *v)
{
    constexpr BlockClass c = kBlockPlan<MT>.cls[I];
    constexpr int delta = (c.c1 >= 0) + (c.c2 >= 0) - (c.d1 >= 0) - (c.d2 >= 0);
    const uint32_t cb = L.template class_base<c.c1, c.c2, c.d1, c.d2>();
    ((v[OFF + Ks] = buf_ld_c128(
          ldc.r, L.template address<delta, c.lo - (kBlockRows - 1) + Ks>(cb))),
     ...);
}

// Configurations u = -(R+1) .. 2 of the class of the rows themselves.
template <int MT, int... Ks>
__device__ __forceinline__ void block_own_loads(std::integer_sequence<int, Ks...>,
                                                const BlockLane<MT> &L, uint32_t cb,
                                                const Gather<false> &ldc, double2 *v)
{
    ((v[Ks] = buf_ld_c128(ldc.r, L.template address<0, Ks - (kBlockRows + 1)>(cb))), ...);
}

// Member Delta_a = D1 of class I: its terms on every row of the lane.
template <int MT, int I, int OFF, int D1>
__device__ __forceinline__ void block_member(const BlockLane<MT> &L, double amp,
                                             const double2 *__restrict__ HS,
                                             const double2 *__restrict__ GS,
                                             const double2 *__restrict__ GD, const double2 *v,
                                             BlockAcc<MT> &A)
{
    constexpr int R = kBlockRows, IA = MT - 2, IB = MT - 1;
    constexpr BlockClass c = kBlockPlan<MT>.cls[I];
    constexpr int slot = block_level_slot(MT, c.kind, D1);
    constexpr int at = OFF + D1 - (c.lo - (R - 1));   // value of row j: v[at - j]
    // a single jump a -> b: spectators add to its coefficient
    constexpr int sa = c.kind == kBkMove && D1 == 0  ? c.c1
                       : c.kind == kBkIn && (D1 == 0 || D1 == 1) ? c.c1
                       : c.kind == kBkOut && D1 == -1            ? IA
                       : c.kind == kBkOut && D1 == 0             ? IB
                                                                 : -1;
    if constexpr (sa >= 0) {
        constexpr int sb = c.kind == kBkIn ? (D1 == 1 ? IA : IB) : c.d1;
        constexpr int j0 = sa * MT + sb;
        double er = HS[j0].x, ei = HS[j0].y;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const double x = (double)L.n[m];
            er = fma(GS[j0 * MT + m].x, x, er);
            ei = fma(GS[j0 * MT + m].y, x, ei);
        }
        const double dr = (GS[j0 * MT + IB].x - GS[j0 * MT + IA].x) * amp;
        const double di = (GS[j0 * MT + IB].y - GS[j0 * MT + IA].y) * amp;
        er *= amp;
        ei *= amp;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            cmac(er, ei, v[at - j], A.x[slot][j], A.y[slot][j]);
            er += dr;
            ei += di;
        }
    } else {
        // inner orbitals removed and created by the member
        constexpr int k = c.kind;
        constexpr int r1 = k == kBkMove ? (D1 < 0 ? IA : IB)
                           : k == kBkIn ? (D1 == -1 ? IA : IB)
                           : k == kBkOut ? (D1 == -2 ? IA : IB)
                           : k == kBkOutMove ? (D1 == -1 ? IA : IB)
                           : k == kBkOut2 ? (D1 == 0 ? IB : IA)
                                          : -1;
        constexpr int r2 = k == kBkOut ? r1 : (k == kBkOut2 ? (D1 == -2 ? IA : IB) : -1);
        constexpr int a1 = k == kBkMove ? (D1 < 0 ? IB : IA)
                           : k == kBkIn ? (D1 == -1 ? IB : IA)
                           : k == kBkOut ? (D1 == -2 ? IB : IA)
                           : k == kBkInMove ? (D1 == 1 ? IA : IB)
                           : k == kBkIn2 ? (D1 == 0 ? IB : IA)
                                         : -1;
        constexpr int a2 = k == kBkIn ? a1 : (k == kBkIn2 ? (D1 == 2 ? IA : IB) : -1);
        constexpr int R1 = c.c1 >= 0 ? c.c1 : r1, R2 = c.c1 >= 0 ? (c.c2 >= 0 ? c.c2 : r1) : r2;
        constexpr int A1 = c.d1 >= 0 ? c.d1 : a1, A2 = c.d1 >= 0 ? (c.d2 >= 0 ? c.d2 : a1) : a2;
        static_assert(R1 >= 0 && R2 >= 0 && A1 >= 0 && A2 >= 0, "two particles leave and enter");
        constexpr int gd = block_gd(MT, R1, R2, A1, A2);
        const double2 G = GD[gd];
        const double er = G.x * amp, ei = G.y * amp;
#pragma unroll
        for (int j = 0; j < R; ++j) cmac(er, ei, v[at - j], A.x[slot][j], A.y[slot][j]);
    }
}

template <int MT, int I, int OFF, int... Ms>
__device__ __forceinline__ void block_class_terms(std::integer_sequence<int, Ms...>,
                                                  const BlockLane<MT> &L,
                                                  const double2 *__restrict__ HS,
                                                  const double2 *__restrict__ GS,
                                                  const double2 *__restrict__ GD,
                                                  const double2 *v, BlockAcc<MT> &A)
{
    constexpr BlockClass c = kBlockPlan<MT>.cls[I];
    const double amp = L.template outer_amp<c.c1, c.c2, c.d1, c.d2>();
    (block_member<MT, I, OFF, c.lo + Ms>(L, amp, HS, GS, GD, v, A), ...);
}

// First value of class I within its batch that starts at class I0.
template <int MT>
__host__ __device__ constexpr int block_off(int I0, int I)
{
    int o = 0;
    for (int i = I0; i < I; ++i) o += kBlockPlan<MT>.loads(i);
    return o;
}

template <int MT, int I0, int... Is>
__device__ __forceinline__ void block_batch(std::integer_sequence<int, Is...>,
                                            const BlockLane<MT> &L, const Gather<false> &ldc,
                                            const double2 *__restrict__ HS,
                                            const double2 *__restrict__ GS,
                                            const double2 *__restrict__ GD, BlockAcc<MT> &A)
{
    constexpr int NV = block_off<MT>(I0, I0 + (int)sizeof...(Is));
    double2 v[NV];
    (block_class_loads<MT, I0 + Is, block_off<MT>(I0, I0 + Is)>(
         std::make_integer_sequence<int, kBlockPlan<MT>.loads(I0 + Is)>{}, L, ldc, v),
     ...);
    (block_class_terms<MT, I0 + Is, block_off<MT>(I0, I0 + Is)>(
         std::make_integer_sequence<int, kBlockPlan<MT>.cls[I0 + Is].hi -
                                             kBlockPlan<MT>.cls[I0 + Is].lo + 1>{},
         L, HS, GS, GD, v, A),
     ...);
}

// sum of slot s into the row's sum with its inner factor f
template <int MT>
__device__ __forceinline__ void block_fold(BlockAcc<MT> &A, int s, int j, double f)
{
    A.x[0][j] = fma(f, A.x[s][j], A.x[0][j]);
    A.y[0][j] = fma(f, A.y[s][j], A.y[0][j]);
    A.x[s][j] = 0.0;
    A.y[s][j] = 0.0;
}

// slot s of the second level into slot t
template <int MT>
__device__ __forceinline__ void block_flush(BlockAcc<MT> &A, int s, int t)
{
#pragma unroll
    for (int j = 0; j < kBlockRows; ++j) {
        A.x[t][j] += A.x[s][j];
        A.y[t][j] += A.y[s][j];
        A.x[s][j] = 0.0;
        A.y[s][j] = 0.0;
    }
}

template <int MT, int KIND, int... Bs>
__device__ __forceinline__ void block_batches(std::integer_sequence<int, Bs...>,
                                              const BlockLane<MT> &L, const Gather<false> &ldc,
                                              const double2 *__restrict__ HS,
                                              const double2 *__restrict__ GS,
                                              const double2 *__restrict__ GD, BlockAcc<MT> &A)
{
    constexpr int B0 = kBlockPlan<MT>.bseg[KIND];
    (
        [&] {
            constexpr int b = B0 + Bs;
            // each batch in a basic block of its own (see opaque_true)
            if (opaque_true()) {
                block_batch<MT, kBlockPlan<MT>.bstart[b]>(
                    std::make_integer_sequence<int, kBlockPlan<MT>.bstart[b + 1] -
                                                        kBlockPlan<MT>.bstart[b]>{},
                    L, ldc, HS, GS, GD, A);
                if constexpr (block_two_level(MT, KIND) &&
                              (Bs % kBlockFlush == kBlockFlush - 1 || Bs + 1 == sizeof...(Bs))) {
                    block_flush(A, 3, KIND == kBkTwo ? 0 : 1);
                    if constexpr (KIND != kBkTwo) block_flush(A, 4, 2);
                }
            }
        }(),
        ...);
}

template <int MT, int KIND>
__device__ __forceinline__ void block_kind(const BlockLane<MT> &L, const Gather<false> &ldc,
                                           const double2 *__restrict__ HS,
                                           const double2 *__restrict__ GS,
                                           const double2 *__restrict__ GD, BlockAcc<MT> &A)
{
    block_batches<MT, KIND>(
        std::make_integer_sequence<int, kBlockPlan<MT>.bseg[KIND + 1] -
                                            kBlockPlan<MT>.bseg[KIND]>{},
        L, ldc, HS, GS, GD, A);
}

// The rows of item `item` (0 <= item < items, clamped by the caller).
template <int MT>
__device__ __forceinline__ void apply_block(int item, bool live, int64_t D, int N,
                                            const int *__restrict__ tab, const double *sq,
                                            const double2 *__restrict__ cf,
                                            const double2 *__restrict__ C,
                                            double2 *__restrict__ HC)
{
    constexpr int M = MT, R = kBlockRows, IA = M - 2, IB = M - 1;
    const double2 *DL = cf + split_dl_offset(M);
    const double2 *GI = cf + split_gi_offset(M);
    const double2 *HS = cf + split_hs_offset(M);
    const double2 *GS = cf + split_gs_offset(M);
    const double2 *GD = cf + split_gd_offset(M);
    BlockLane<MT> L;
    L.init(item, D, N, tab, sq);
    const Gather<false> ldc(C, D);
    BlockAcc<MT> A;
#pragma unroll
    for (int s = 0; s < 5; ++s)
#pragma unroll
        for (int j = 0; j < R; ++j) A.x[s][j] = A.y[s][j] = 0.0;

    auto r1 = [&](int d) { return L.root(IA, d); };
    auto r2 = [&](int d) { return L.root(IB, d); };

    // the rows themselves and the jumps within orbitals a, b
    if (opaque_true()) {
        const uint32_t cb = L.template class_base<-1, -1, -1, -1>();
        double2 v[R + 4];   // u = -(R+1) .. 2
        block_own_loads<MT>(std::make_integer_sequence<int, R + 4>{}, L, cb, ldc, v);
        // row coefficient: alpha + n_a beta_a + n_b beta_b + quadratic part
        double cr = 0.0, ci = 0.0, b1r = DL[IA].x, b1i = DL[IA].y, b2r = DL[IB].x, b2i = DL[IB].y;
        auto gi = [&](int a, int b) { return GI[a * M - a * (a - 1) / 2 + (b - a)]; };
#pragma unroll
        for (int o = 0; o < IA; ++o) {
            const double x = (double)L.n[o];
            double tr = DL[o].x, ti = DL[o].y;
#pragma unroll
            for (int p = o; p < IA; ++p) {
                tr = fma(gi(o, p).x, (double)L.n[p], tr);
                ti = fma(gi(o, p).y, (double)L.n[p], ti);
            }
            cr = fma(tr, x, cr);
            ci = fma(ti, x, ci);
            const double2 g1 = gi(o, IA), g2 = gi(o, IB);
            b1r = fma(g1.x, x, b1r);
            b1i = fma(g1.y, x, b1i);
            b2r = fma(g2.x, x, b2r);
            b2i = fma(g2.y, x, b2i);
        }
        double e12r = HS[IA * M + IB].x, e12i = HS[IA * M + IB].y;
        double e21r = HS[IB * M + IA].x, e21i = HS[IB * M + IA].y;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const double x = (double)L.n[m];
            e12r = fma(GS[(IA * M + IB) * M + m].x, x, e12r);
            e12i = fma(GS[(IA * M + IB) * M + m].y, x, e12i);
            e21r = fma(GS[(IB * M + IA) * M + m].x, x, e21r);
            e21i = fma(GS[(IB * M + IA) * M + m].y, x, e21i);
        }
        constexpr int gab = block_gd(M, IA, IA, IB, IB), gba = block_gd(M, IB, IB, IA, IA);
        const double2 Gaabb = GD[gab], Gbbaa = GD[gba];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const double x1 = (double)(L.n[IA] - j), x2 = (double)(L.n[IB] + j);
            double dr = fma(b1r, x1, cr), di = fma(b1i, x1, ci);
            dr = fma(b2r, x2, dr);
            di = fma(b2i, x2, di);
            const double x11 = x1 * x1, x12 = x1 * x2, x22 = x2 * x2;
            dr = fma(gi(IA, IA).x, x11, dr);
            di = fma(gi(IA, IA).y, x11, di);
            dr = fma(gi(IA, IB).x, x12, dr);
            di = fma(gi(IA, IB).y, x12, di);
            dr = fma(gi(IB, IB).x, x22, dr);
            di = fma(gi(IB, IB).y, x22, di);
            const int own = R + 1 - j;   // u = -j
            cmac(dr, di, v[own], A.x[0][j], A.y[0][j]);
            cmac(e12r, e12i, v[own - 1], A.x[1][j], A.y[1][j]);
            cmac(e21r, e21i, v[own + 1], A.x[2][j], A.y[2][j]);
            e12r += GS[(IA * M + IB) * M + IB].x - GS[(IA * M + IB) * M + IA].x;
            e12i += GS[(IA * M + IB) * M + IB].y - GS[(IA * M + IB) * M + IA].y;
            e21r += GS[(IB * M + IA) * M + IB].x - GS[(IB * M + IA) * M + IA].x;
            e21i += GS[(IB * M + IA) * M + IB].y - GS[(IB * M + IA) * M + IA].y;
            const double f1 = r1(-j) * r1(-j - 1) * r2(j + 1) * r2(j + 2);
            const double f2 = r2(j) * r2(j - 1) * r1(-j + 1) * r1(-j + 2);
            cmac(Gaabb.x * f1, Gaabb.y * f1, v[own - 2], A.x[0][j], A.y[0][j]);
            cmac(Gbbaa.x * f2, Gbbaa.y * f2, v[own + 2], A.x[0][j], A.y[0][j]);
        }
    }
    block_kind<MT, kBkMove>(L, ldc, HS, GS, GD, A);
    block_kind<MT, kBkTwo>(L, ldc, HS, GS, GD, A);
    if (opaque_true())
#pragma unroll
        for (int j = 0; j < R; ++j) {
            block_fold(A, 1, j, r1(-j) * r2(j + 1));
            block_fold(A, 2, j, r2(j) * r1(-j + 1));
        }
    block_kind<MT, kBkIn>(L, ldc, HS, GS, GD, A);
    if (opaque_true())
#pragma unroll
        for (int j = 0; j < R; ++j) {
            block_fold(A, 3, j, r1(-j) * r2(j + 1) * r2(j + 2));
            block_fold(A, 4, j, r2(j) * r1(-j + 1) * r1(-j + 2));
        }
    block_kind<MT, kBkInMove>(L, ldc, HS, GS, GD, A);
    if (opaque_true())
#pragma unroll
        for (int j = 0; j < R; ++j) {
            block_fold(A, 1, j, r1(-j + 1));
            block_fold(A, 2, j, r2(j + 1));
        }
    block_kind<MT, kBkOut>(L, ldc, HS, GS, GD, A);
    if (opaque_true())
#pragma unroll
        for (int j = 0; j < R; ++j) {
            block_fold(A, 3, j, r1(-j) * r1(-j - 1) * r2(j + 1));
            block_fold(A, 4, j, r2(j) * r2(j - 1) * r1(-j + 1));
        }
    block_kind<MT, kBkOutMove>(L, ldc, HS, GS, GD, A);
    if (opaque_true())
#pragma unroll
        for (int j = 0; j < R; ++j) {
            block_fold(A, 1, j, r1(-j));
            block_fold(A, 2, j, r2(j));
        }
    block_kind<MT, kBkIn2>(L, ldc, HS, GS, GD, A);
    if (opaque_true())
#pragma unroll
        for (int j = 0; j < R; ++j) {
            block_fold(A, 1, j, r1(-j + 1) * r1(-j + 2));
            block_fold(A, 2, j, r1(-j + 1) * r2(j + 1));
            block_fold(A, 3, j, r2(j + 1) * r2(j + 2));
        }
    block_kind<MT, kBkOut2>(L, ldc, HS, GS, GD, A);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        block_fold(A, 1, j, r1(-j) * r1(-j - 1));
        block_fold(A, 2, j, r1(-j) * r2(j));
        block_fold(A, 3, j, r2(j) * r2(j - 1));
    }
    const uint32_t own = L.template class_base<-1, -1, -1, -1>();
#pragma unroll
    for (int j = 0; j < R; ++j)
        if (live && L.n[IA] >= j)
            HC[(own - L.ga[R + 1 - j]) >> 4] = make_double2(A.x[0][j], A.y[0][j]);
}

}  // namespace mc
