// Table-free H.C with four rows per lane: staging and launch (mc_block.h).
#include "mc_block.h"

namespace mc {
namespace {

// The constants of the case-split sum (blocks 0 .. gridDim - 2) and the
// tables of the space (the last block).
__global__ __launch_bounds__(256) void k_prep_block(int N, int M, int adjoint,
                                                    const double2 *__restrict__ g,
                                                    const double2 *__restrict__ h,
                                                    double2 *__restrict__ cf,
                                                    int *__restrict__ tab)
{
    __shared__ int sum[256];
    if (blockIdx.x + 1 < gridDim.x)
        stage_split_constants(M, adjoint, g, h, cf, blockIdx.x * 256 + threadIdx.x,
                              (gridDim.x - 1) * 256);
    else
        stage_block_tables(N, M, tab, sum);
}

// Bound: the L1's look-ups.  At M = 5 a wavefront's 296 gathers make 21
// look-ups each (16 when they start on 64 bytes), 95 % of the kernel's cycles;
// the vector ALU is at 73 % and HBM reads are 5.4 GB (C is 1.1).  One item per lane, 256
// consecutive items per block, blocks in XCD chunks as in the one-row kernel.
// N=200, M=5 (70,058,751 rows): 5.50 ms with one row per lane, 3.44 so;
// N=50, M=6: 0.56 -> 0.40; N=29, M=7: 0.46 -> 0.37; N=24, M=8: 1.60 -> 1.24;
// N=40, M=8 (62,891,499 rows): 39.9 -> 26.9 ms.
template <int MT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MC_APPLY_WAVES)))
void k_apply_block(int N, int64_t D, int items, int64_t nblocks, const int *__restrict__ tab,
                   const double2 *__restrict__ cf, const double2 *__restrict__ C,
                   double2 *__restrict__ HC)
{
    extern __shared__ double sq[];   // roots, then the space's tables
    int *lt = (int *)(sq + N + 3 + kBlockRows);
    const int nt = block_table_ints(N, MT);
    for (int i = threadIdx.x; i < nt; i += 256) lt[i] = tab[i];
    fill_sqrt_table(sq, N + 3 + kBlockRows);
    const int64_t i = xcd_block(blockIdx.x, nblocks) * 256 + threadIdx.x;
    const bool live = i < items;
    apply_block<MT>(live ? (int)i : items - 1, live, D, N, lt, sq, cf, C, HC);
}

}  // namespace

// Rows whose n_b is divisible by R.
int64_t block_items(int32_t N, int32_t M)
{
    int64_t items = 0;
    for (int S = N; S >= 0; S -= kBlockRows) items += dim_checked(S, M - 1);
    return items;
}

size_t block_workspace(int32_t N, int32_t M)
{
    return (size_t)split_total(M) * 16 + (size_t)block_table_ints(N, M) * 4;
}

// What the kernel's addresses allow: every offset of a gather, the out-of-range
// ones included, has to fit 32 bits (16 D plus 16 G_a, G_a < D), and the root
// table 64 KB of LDS.
bool block_fits(int32_t N, int32_t M, int64_t D)
{
    return M >= 3 && M <= 8 && N < 4096 && D * 32 <= (int64_t)0xFFFFFFF0u;
}

// Which spaces the four-row kernel serves.  Its lanes hold four rows, so it fills
// the GPU at four times the rows of the one-row kernel, and its wavefronts take
// longer.  Measured against that kernel (us, one row / four rows): M = 4, N = 110
// (234 k rows) 15 / 18, N = 130 (383 k) 21 / 19; M = 5, N = 42 (163 k) 24 / 31,
// N = 48 (271 k) 35 / 35, N = 52 (367 k) 39 / 35; M = 6, N = 28 (237 k) 53 / 56,
// N = 30 (325 k) 58 / 56; M = 7, N = 18 (135 k) 81 / 80, N = 22 (377 k) 126 / 102;
// M = 8, N = 19 (658 k) 415 / 414, N = 21 (1,184 k) 720 / 621.  Just past a whole
// number of wavefronts per SIMD it can lose a few per cent above the line (M = 6,
// N = 32, 436 k rows, 77 / 82; M = 5, N = 56, 48 / 49).
// Three orbitals stay with the one-row kernel, whose error is the smaller there:
// against 64 bits, N = 900, mean of eight states, 2.77e-16 and 2.94e-16 (in each of
// the eight), for 18 and 15 us at N = 1,000.
bool block_serves(int32_t N, int32_t M, int64_t D)
{
    return M >= 4 && block_fits(N, M, D) && D >= (M <= 6 ? 262144 : M == 7 ? 131072 : 786432);
}

void launch_prep_block(int32_t N, int32_t M, int adjoint, const double *g_d, const double *h_d,
                       double2 *cf, int32_t *tab, hipStream_t s)
{
    hipLaunchKernelGGL(k_prep_block, dim3(5), dim3(256), 0, s, N, M, adjoint,
                       (const double2 *)g_d, (const double2 *)h_d, cf, tab);
}

int apply_block_run(int32_t N, int32_t M, int64_t D, const double2 *cf, const int32_t *tab,
                    const double *C_d, double *HC_d, hipStream_t s)
{
    const int64_t items = block_items(N, M);
    const int64_t nblocks = (items + 255) / 256;
    const size_t lds = (size_t)(N + 3 + kBlockRows) * 8 + (size_t)block_table_ints(N, M) * 4;
    MC_DISPATCH_M(M, if constexpr (MT >= 4 && MT <= 8) {
        hipLaunchKernelGGL((k_apply_block<MT>), dim3(nblocks), dim3(256), lds, s, N, D, (int)items,
                           nblocks, tab, cf, (const double2 *)C_d, (double2 *)HC_d);
    });
    return launch_status();
}

int apply_block_launch(int32_t N, int32_t M, int64_t D, const double *h_d, const double *g_d,
                       int adjoint, const double *C_d, double *HC_d, void *ws_d, hipStream_t s)
{
    double2 *cf = (double2 *)ws_d;
    int *tab = (int *)(cf + split_total(M));
    launch_prep_block(N, M, adjoint, g_d, h_d, cf, tab, s);
    return apply_block_run(N, M, D, cf, tab, C_d, HC_d, s);
}

}  // namespace mc
