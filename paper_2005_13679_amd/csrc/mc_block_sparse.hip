// H.C over non-zero constants only, four rows per lane (the rows and tables of
// mc_block.h), and the lists of those constants.
#include "mc_block.h"
#include "mc_sparse.h"

namespace mc {
namespace {

// The lists of the staged constants cf (layout in mc_sparse.h), by one block of
// 1,024 threads: a wavefront per removal pair, its slots found with one ballot.
__global__ __launch_bounds__(1024) void k_sparse_lists(int M, const double2 *__restrict__ cf,
                                                      int32_t *__restrict__ sl)
{
    __shared__ uint64_t mask[36];
    const double2 *HS = cf + split_hs_offset(M), *GS = cf + split_gs_offset(M);
    const double2 *GD = cf + split_gd_offset(M);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t below = (1ull << lane) - 1;
    if (wave == 0) {
        bool any = false;
        if (lane < M * M && lane / M != lane % M) {
            any = nonzero(HS[lane]);
            for (int c = 0; c < M; ++c) any = nonzero(GS[lane * M + c]) || any;
        }
        const uint64_t w = __ballot(any);
        if (any) sl[kSlSingles + __popcll(w & below)] = lane;
        if (lane == 0) sl[0] = __popcll(w);
    }
    int p = 0, co = 0;
    for (int k = 0; k < M; ++k)
        for (int s = k; s < M; ++s, ++p) {
            const int nd = reduced_slots(M, k, s);
            if ((p & 15) == wave) {
                const uint64_t w = __ballot(lane < nd && nonzero(GD[co + (lane < nd ? lane : 0)]));
                if (lane == 0) mask[p] = w;
            }
            co += nd;
        }
    __syncthreads();
    int e = 0;
    p = co = 0;
    for (int k = 0; k < M; ++k)
        for (int s = k; s < M; ++s, ++p) {
            const int nd = reduced_slots(M, k, s);
            const uint64_t w = mask[p];
            if ((p & 15) == wave) {
                if (lane == 0) {
                    sl[kSlPairs + 2 * p] = e;
                    sl[kSlPairs + 2 * p + 1] = __popcll(w);
                }
                if (w >> lane & 1) {
                    // creation pair number `lane` outside {k, s}
                    int r = 0;
                    for (int q = 0; q < M; ++q)
                        for (int l = q; l < M; ++l) {
                            if (q == k || q == s || l == k || l == s) continue;
                            if (r++ == lane)
                                sl[kSlEntries + e + __popcll(w & below)] =
                                    (co + lane) | q << 10 | l << 13 | k << 16 | s << 19;
                        }
                }
            }
            e += __popcll(w);
            co += nd;
        }
}

// Additions of one chain before it is added to the row's sum (short chains of
// additions round less).
constexpr int kSparseFlush = 8;

// Roots below the square root table of a block: read at the rows of a lane that
// do not exist, or that have no such jump (smallest index -4).
constexpr int kRootPad = 8;

// Zeros below the space's tables: what load() reads at prefix sums below 0, on
// rows without such a jump (smallest -5).  With three orbitals these words are
// subtracted from the index that stands for "past the vector".
constexpr int kTablePad = 8;

// Three bits of every orbital from o on: a particle entering o adds one to
// each S_m, m >= o.
__device__ __forceinline__ uint32_t from_orbital(int o) { return 0x249249u << 3 * o; }
constexpr uint32_t kNothingMoved = 2u * 0x249249u;

// A lane's rows and where their targets lie, for jumps known at run time only.
// Row j has n_a - j and n_b + j; a row that does not exist (j > n_a) is summed
// like the others and not stored.
template <int MT>
struct SparseLane {
    static constexpr int R = kBlockRows, IA = MT - 2, IB = MT - 1;
    const int *G[MT];   // where G_m(S_m) of row 0 lies, m = 1 .. a
    int top;            // D - 1 - S_0
    const int *occ;     // occupations of row 0, one orbital every 256
    const double *sq;

    // change of an orbital's occupation from row to row, two bits each plus 1
    static constexpr uint32_t kStep = (0x5555u & ~(3u << 2 * IA) & ~(3u << 2 * IB)) | 2u << 2 * IB;
    static __device__ __forceinline__ int step(int o) { return (int)(kStep >> 2 * o & 3) - 1; }

    // Values of the targets of a jump; `sh`: the change of each S_m plus 2,
    // three bits each; zero where n1 + j c1 or n2 + j c2 is below 1.  Offsets
    // below 16 (2^28 - 1) - 16 G_a lie past the vector.
    __device__ __forceinline__ void load(uint32_t sh, int n1, int c1, int n2, int c2,
                                         const Gather<false> &ldc, double2 (&v)[R]) const
    {
        int i = top + 2 - (int)(sh & 7);
#pragma unroll
        for (int m = 1; m < IA; ++m) i -= G[m][(int)(sh >> 3 * m & 7) - 2];
        const int *ga = G[IA] + (int)(sh >> 3 * IA & 7) - 2;
        if ((c1 | c2) == 0) {
            i = (n1 < n2 ? n1 : n2) >= 1 ? i : 0x0FFFFFFF;
#pragma unroll
            for (int j = 0; j < R; ++j) v[j] = buf_ld_c128(ldc.r, (uint32_t)(i - ga[-j]) << 4);
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int m1 = n1 + j * c1, m2 = n2 + j * c2;
                const uint32_t at = (uint32_t)(i - ga[-j]) << 4;
                v[j] = buf_ld_c128(ldc.r, (m1 < m2 ? m1 : m2) >= 1 ? at : 0xFFFFFFF0u);
            }
        }
    }
    // f[j] *= the root of n + j c, c = 1 or -1
    __device__ __forceinline__ void times_roots(int n, int c, double (&f)[R]) const
    {
        const double *r = sq + n;
        if (c > 0)
#pragma unroll
            for (int j = 0; j < R; ++j) f[j] *= r[j];
        else
#pragma unroll
            for (int j = 0; j < R; ++j) f[j] *= r[-j];
    }
};

// Bound: the vector ALU is busy for 75 % of the cycles (201 M instructions at
// N=40, M=7 on a ring), the L1's look-ups for 52 %; what is left is the latency
// of a jump's chain (list entry, occupations, index, gather) at six wavefronts
// per SIMD.  The walk is a loop over the list: the compile-time walk of
// mc_block.h with a flag per jump gathers whole classes for one member and
// took 1,053 us where this takes 533; one row per lane through the map, 1,558.
// N=100, M=5 347 -> 100 us; N=20, M=7 202 -> 57; with no zero constants
// N=30, M=7 2.25 -> 1.24 ms.
template <int MT>
__global__ __launch_bounds__(256) void k_sparse_block(
    int N, int64_t D, int items, int64_t nblocks, const int32_t *__restrict__ sl,
    const int *__restrict__ tab, const double2 *__restrict__ cf, const double2 *__restrict__ C,
    double2 *__restrict__ HC)
{
    constexpr int M = MT, R = kBlockRows, IA = M - 2, IB = M - 1, NP = M * (M + 1) / 2;
    extern __shared__ double lds[];   // roots, the space's tables, the occupations
    double *sq = lds + kRootPad;
    int *lt = (int *)(sq + N + 3 + kBlockRows) + kTablePad;
    const int nt = block_table_ints(N, M);
    int *occ = lt + nt + threadIdx.x;
    if (threadIdx.x < kRootPad) lds[threadIdx.x] = 0.0;
    if (threadIdx.x < kTablePad) lt[(int)threadIdx.x - kTablePad] = 0;
    for (int i = threadIdx.x; i < nt; i += 256) lt[i] = tab[i];
    fill_sqrt_table(sq, N + 3 + kBlockRows);
    const int64_t it = xcd_block(blockIdx.x, nblocks) * 256 + threadIdx.x;
    const bool live = it < items;
    BlockLane<MT> B;
    B.init(live ? (int)it : items - 1, D, N, lt, sq);
    SparseLane<MT> L;
    L.top = (int)(D - 1) - B.n[0];
    L.sq = sq;
    L.occ = occ;
    double x[M];
    int S = 0;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        occ[m * 256] = B.n[m];
        x[m] = (double)B.n[m];
        S += B.n[m];
        if (m >= 1 && m <= IA) L.G[m] = lt + (m - 1) * (N + 1) + S;
    }
    const int na = B.n[IA];
    const Gather<false> ldc(C, D);
    const double2 *DL = cf + split_dl_offset(M), *GI = cf + split_gi_offset(M);
    const double2 *HS = cf + split_hs_offset(M), *GS = cf + split_gs_offset(M);
    const double2 *GD = cf + split_gd_offset(M);
    double ar[R], ai[R];

    // the rows themselves: alpha + n_a beta_a + n_b beta_b + quadratic part
    {
        double2 v[R];
        L.load(kNothingMoved, 1, 0, 1, 0, ldc, v);
        double cr = 0.0, ci = 0.0, b1r = DL[IA].x, b1i = DL[IA].y, b2r = DL[IB].x, b2i = DL[IB].y;
        auto gi = [&](int a, int b) { return GI[a * M - a * (a - 1) / 2 + (b - a)]; };
#pragma unroll
        for (int o = 0; o < IA; ++o) {
            double tr = DL[o].x, ti = DL[o].y;
#pragma unroll
            for (int p = o; p < IA; ++p) {
                tr = fma(gi(o, p).x, x[p], tr);
                ti = fma(gi(o, p).y, x[p], ti);
            }
            cr = fma(tr, x[o], cr);
            ci = fma(ti, x[o], ci);
            b1r = fma(gi(o, IA).x, x[o], b1r);
            b1i = fma(gi(o, IA).y, x[o], b1i);
            b2r = fma(gi(o, IB).x, x[o], b2r);
            b2i = fma(gi(o, IB).y, x[o], b2i);
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const double x1 = x[IA] - j, x2 = x[IB] + j;
            double dr = fma(b1r, x1, cr), di = fma(b1i, x1, ci);
            dr = fma(b2r, x2, dr);
            di = fma(b2i, x2, di);
            dr = fma(gi(IA, IA).x, x1 * x1, dr);
            di = fma(gi(IA, IA).y, x1 * x1, di);
            dr = fma(gi(IA, IB).x, x1 * x2, dr);
            di = fma(gi(IA, IB).y, x1 * x2, di);
            dr = fma(gi(IB, IB).x, x2 * x2, dr);
            di = fma(gi(IB, IB).y, x2 * x2, di);
            ar[j] = dr * v[j].x - di * v[j].y;
            ai[j] = dr * v[j].y + di * v[j].x;
        }
    }

    const int ns = sl[0];
    const int nd = sl[kSlPairs + 2 * (NP - 1)] + sl[kSlPairs + 2 * (NP - 1) + 1];
    double br[R], bi[R];
    auto clear = [&] {
#pragma unroll
        for (int j = 0; j < R; ++j) br[j] = bi[j] = 0.0;
    };
    auto flush = [&] {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            ar[j] += br[j];
            ai[j] += bi[j];
        }
    };
    // the root of an orbital's occupation that is the same on every row
    auto outer = [&](int n, int c) { return c == 0 ? sq[n] : 1.0; };
#pragma unroll 1
    for (int e0 = 0; e0 < ns; e0 += kSparseFlush) {
        clear();
#pragma unroll 1
        for (int e = e0; e < ns && e < e0 + kSparseFlush; ++e) {
            const int s = sl[kSlSingles + e], a = s / M, b = s % M;
            const int nA = occ[a * 256], nB = occ[b * 256] + 1;
            const int ca = L.step(a), cb = L.step(b);
            double2 v[R];
            L.load(kNothingMoved - from_orbital(a) + from_orbital(b), nA, ca, 1, 0, ldc, v);
            const double fo = outer(nA, ca) * outer(nB, cb);
            double f[R];
#pragma unroll
            for (int j = 0; j < R; ++j) f[j] = fo;
            if (ca) L.times_roots(nA, ca, f);
            if (cb) L.times_roots(nB, cb, f);
            double er = HS[s].x, ei = HS[s].y;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                er = fma(GS[s * M + m].x, x[m], er);
                ei = fma(GS[s * M + m].y, x[m], ei);
            }
            const double gr = GS[s * M + IB].x - GS[s * M + IA].x;
            const double gi = GS[s * M + IB].y - GS[s * M + IA].y;
#pragma unroll
            for (int j = 0; j < R; ++j)
                cmac(fma(gr, (double)j, er) * f[j], fma(gi, (double)j, ei) * f[j], v[j], br[j],
                     bi[j]);
        }
        flush();
    }
    int next = sl[kSlEntries];
#pragma unroll 1
    for (int e0 = 0; e0 < nd; e0 += kSparseFlush) {
        clear();
#pragma unroll 1
        for (int e = e0; e < nd && e < e0 + kSparseFlush; ++e) {
            const int w = next;
            next = sl[kSlEntries + e + 1];   // one past the last may be read
            const int q = w >> 10 & 7, l = w >> 13 & 7, k = w >> 16 & 7, s = w >> 19 & 7;
            const int nk = occ[k * 256], ns2 = occ[s * 256] - (k == s);
            const int nq = occ[q * 256] + 1, nl = occ[l * 256] + 1 + (q == l);
            const int ck = L.step(k), cs = L.step(s), cq = L.step(q), cl = L.step(l);
            double2 v[R];
            L.load(kNothingMoved - from_orbital(k) - from_orbital(s) + from_orbital(q) +
                       from_orbital(l),
                   nk, ck, ns2, cs, ldc, v);
            const double2 G = GD[w & 1023];
            const double fo = (outer(nk, ck) * outer(ns2, cs)) * (outer(nq, cq) * outer(nl, cl));
            if (ck | cs | cq | cl) {
                double f[R];
#pragma unroll
                for (int j = 0; j < R; ++j) f[j] = fo;
                if (ck) L.times_roots(nk, ck, f);
                if (cs) L.times_roots(ns2, cs, f);
                if (cq) L.times_roots(nq, cq, f);
                if (cl) L.times_roots(nl, cl, f);
#pragma unroll
                for (int j = 0; j < R; ++j) cmac(G.x * f[j], G.y * f[j], v[j], br[j], bi[j]);
            } else {
                const double er = G.x * fo, ei = G.y * fo;
#pragma unroll
                for (int j = 0; j < R; ++j) cmac(er, ei, v[j], br[j], bi[j]);
            }
        }
        flush();
    }

    if (live) {
        int i = L.top;
#pragma unroll
        for (int m = 1; m < IA; ++m) i -= L.G[m][0];
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (na >= j) HC[i - L.G[IA][-j]] = make_double2(ar[j], ai[j]);
    }
}

}  // namespace

void launch_sparse_lists(int32_t M, const double2 *cf, int32_t *sl, hipStream_t s)
{
    hipLaunchKernelGGL(k_sparse_lists, dim3(1), dim3(1024), 0, s, M, cf, sl);
}

static size_t lists_offset(int32_t N, int32_t M)
{
    return (size_t)split_total(M) * 16 + (size_t)block_table_ints(N, M) * 4;
}

// the lists and one entry past them
size_t block_sparse_workspace(int32_t N, int32_t M)
{
    return lists_offset(N, M) + (kSlInts + 1) * 4;
}

static size_t sparse_lds(int32_t N, int32_t M)
{
    return (size_t)(kRootPad + N + 3 + kBlockRows) * 8 +
           (size_t)(kTablePad + block_table_ints(N, M) + 256 * M) * 4;
}

// Spaces served: from above those of the four-row kernel; from below 131,072
// rows, where the four rows of a lane stop costing more in wavefronts than they
// save.  One row through the map, one row chained, four rows (us; on a ring, and
// without zero constants): M = 5, N = 33 (66 k rows) 26, 27, 27 and 89, 80, 99;
// M = 7, N = 16 (75 k) 51, 56, 55 and 347, 316, 347; M = 8, N = 14 (116 k) 88,
// 91, 79 and 617, 658, 578; M = 8, N = 17 (346 k) 121, 135, 88 and 787, 1,013,
// 732; M = 8, N = 19 (658 k) 188, 215, 99 and 1,348, 1,750, 870.
bool block_sparse_serves(int32_t N, int32_t M, int64_t D)
{
    return block_fits(N, M, D) && D >= 131072 && sparse_lds(N, M) <= 65536;
}

int apply_block_sparse_launch(int32_t N, int32_t M, int64_t D, const double *h_d,
                              const double *g_d, const double *C_d, double *HC_d, void *ws_d,
                              hipStream_t s)
{
    double2 *cf = (double2 *)ws_d;
    int32_t *tab = (int32_t *)(cf + split_total(M));
    int32_t *sl = (int32_t *)((char *)ws_d + lists_offset(N, M));
    launch_prep_block(N, M, 0, g_d, h_d, cf, tab, s);
    launch_sparse_lists(M, cf, sl, s);
    const int64_t items = block_items(N, M), nblocks = (items + 255) / 256;
    MC_DISPATCH_M(M, if constexpr (MT >= 3 && MT <= 8) {
        hipLaunchKernelGGL((k_sparse_block<MT>), dim3(nblocks), dim3(256), sparse_lds(N, M), s, N,
                           D, (int)items, nblocks, (const int32_t *)sl, (const int *)tab,
                           (const double2 *)cf, (const double2 *)C_d, (double2 *)HC_d);
    });
    return launch_status();
}

}  // namespace mc
