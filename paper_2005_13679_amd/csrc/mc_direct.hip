// Table-free H.C: its entry points, and the staging of the case-split
// constants.
#include <mutex>

#include "mc_split.h"
#include "mc_tiles.h"

namespace mc {

// Staged constants of the case-split apply (layout in mc_split.h).
__global__ void k_prep_split(int M, int adjoint, const double2 *__restrict__ g,
                             const double2 *__restrict__ h, double2 *__restrict__ cf)
{
    stage_split_constants(M, adjoint, g, h, cf, blockIdx.x * blockDim.x + threadIdx.x,
                          gridDim.x * blockDim.x);
}

void launch_prep_split(int32_t M, int adjoint, const double *g_d, const double *h_d, double2 *cf,
                       hipStream_t s)
{
    hipLaunchKernelGGL(k_prep_split, dim3(4), dim3(256), 0, s, M, adjoint, (const double2 *)g_d,
                       (const double2 *)h_d, cf);
}

int apply_direct_launch(int32_t N, int32_t M, int64_t D, const double *h_d, const double *g_d,
                        int adjoint, const double *C_d, double *HC_d, void *ws_d, hipStream_t s)
{
    double2 *cf = (double2 *)ws_d;
    launch_prep_split(M, adjoint, g_d, h_d, cf, s);
    const DirectCall c{N, D <= kSmallTiles * kTile, D, cf, (const double2 *)C_d, (double2 *)HC_d, s};
    return MC_TILES_CALL(direct, M, c);
}

}  // namespace mc

using namespace mc;

extern "C" {

// Scratch of mc_apply_H_direct_noalloc: the staged constants of the apply
// live in this file-scope device array (one copy per GPU, held until the
// process ends) instead of a caller workspace.  Host code never passes the
// array's name to a kernel: its device address is looked up once per device
// (with that device current) and kept per device.
static __device__ __align__(256) unsigned char scratch[MC_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

static int noalloc_scratch(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return set_hip_error(e);
    if (dev < 0 || dev >= kMaxDevices) return MC_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return set_hip_error(e != hipSuccess ? e : hipErrorUnknown);
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return MC_OK;
}

static int apply_direct_common(int32_t N, int32_t M, const double *h_d, const double *g_d,
                               const double *C_d, double *HC_d, void *ws_d, size_t ws_bytes,
                               int adjoint, mc_stream stream)
{
    int st = check_nm(N, M);
    if (st) return st;
    if (M > 8) return MC_EINVAL;
    const int64_t D = dim_checked(N, M);
    if (D < 0 || D >= ((int64_t)1 << 31)) return MC_ERANGE;
    if (!h_d || !g_d || !C_d || !HC_d || !ws_d) return MC_EINVAL;
    if (overlaps(C_d, (size_t)D * 16, HC_d, (size_t)D * 16)) return MC_EINVAL;
    if (ws_bytes < apply_workspace_least(M)) return MC_ENOMEM;
    const size_t sqb = (size_t)(N + 3) * 8;
    if (M >= MC_LDS_ROOTS_FROM && sqb > 65536) return MC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    if (block_serves(N, M, D) && ws_bytes >= block_workspace(N, M))
        return apply_block_launch(N, M, D, h_d, g_d, adjoint, C_d, HC_d, ws_d, s);
    return apply_direct_launch(N, M, D, h_d, g_d, adjoint, C_d, HC_d, ws_d, s);
}

int mc_apply_H_direct(int32_t N, int32_t M, const double *h_d, const double *g_d,
                      const double *C_d, double *HC_d, void *ws_d, size_t ws_bytes,
                      mc_stream stream)
{
    return apply_direct_common(N, M, h_d, g_d, C_d, HC_d, ws_d, ws_bytes, 0, stream);
}

int mc_apply_H_direct_noalloc(int32_t N, int32_t M, const double *h_d, const double *g_d,
                              const double *C_d, double *HC_d, mc_stream stream)
{
    size_t need = 0;
    int st = mc_workspace_size(N, M, MC_OP_APPLY, &need);
    if (st) return st;
    if (need > (size_t)MC_NOALLOC_SCRATCH_BYTES) return MC_ENOMEM;
    void *ws = nullptr;
    st = noalloc_scratch(&ws);
    if (st) return st;
    return apply_direct_common(N, M, h_d, g_d, C_d, HC_d, ws, MC_NOALLOC_SCRATCH_BYTES, 0,
                               stream);
}

int mc_apply_H_direct_adjoint(int32_t N, int32_t M, const double *h_d, const double *g_d,
                              const double *C_d, double *HC_d, void *ws_d, size_t ws_bytes,
                              mc_stream stream)
{
    return apply_direct_common(N, M, h_d, g_d, C_d, HC_d, ws_d, ws_bytes, 1, stream);
}

}  // extern "C"
