// One Lanczos vector with full reorthogonalisation (Sec. VI): classical
// Gram-Schmidt twice against the basis V_0 .. V_{K-1}, then normalisation.
//
// Bound: memory.  Composed of one call per operation this read V four times
// and w once per basis vector and pass; here V is read three times and w four
// times in all:
//   1. c1 = V^H w                       (k_proj)
//   2. w -= V c1, and c2 = V^H w of the updated w while the elements of V are
//      still in registers               (k_sub_proj, K <= 12; two passes above)
//   3. out = w - V c2, and its norm     (k_sub_norm)
//   4. out /= norm                      (k_scale)
// Each block keeps one contiguous part of the vectors in every pass, and the
// passes sweep it in alternating directions, so a pass starts on what the
// last one left in the 256 MB memory-side cache.  Sums are taken in a fixed
// order.  Eight vectors at N=100, M=5 (4,598,126 rows), without the products
// H.V: 4.3 -> 2.1 ms.
#include "mc_internal.h"

namespace mc {
namespace {

constexpr int kKryTile = 8;     // basis vectors per pass over w in k_proj
constexpr int kKryFused = 12;   // most basis vectors k_sub_proj holds

// Sums v over the block's 256 threads into s[0] (fixed order).
__device__ __forceinline__ double block_sum(double v, double *s)
{
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    return (s[0] + s[1]) + (s[2] + s[3]);
}

// part[k G + b] = sum over part b of conj(V_k) w, for the KT vectors k from
// first + KT blockIdx.y on.
template <int KT>
__global__ __launch_bounds__(256) void k_proj(int64_t n, int64_t len, int first,
                                              const double2 *__restrict__ V, int64_t ldv,
                                              const double2 *__restrict__ w,
                                              double2 *__restrict__ part)
{
    __shared__ double s[4];
    const int64_t lo = blockIdx.x * len, hi = lo + len < n ? lo + len : n;
    const int K0 = first + KT * (int)blockIdx.y;
    const double2 *v = V + K0 * ldv;
    double ar[KT], ai[KT];
#pragma unroll
    for (int k = 0; k < KT; ++k) ar[k] = ai[k] = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
        const double2 x = w[i];
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            const double2 a = v[k * ldv + i];
            ar[k] = fma(a.x, x.x, fma(a.y, x.y, ar[k]));
            ai[k] = fma(a.x, x.y, fma(-a.y, x.x, ai[k]));
        }
    }
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const double r = block_sum(ar[k], s), c = block_sum(ai[k], s);
        if (threadIdx.x == 0)
            part[(int64_t)(K0 + k) * gridDim.x + blockIdx.x] = make_double2(r, c);
    }
}

// c[k] = sum of part k over the blocks; alpha (if any) = c[K-1].
__global__ __launch_bounds__(256) void k_proj_sum(int G, const double2 *__restrict__ part,
                                                  double2 *__restrict__ c,
                                                  double2 *__restrict__ alpha)
{
    __shared__ double s[4];
    double ar = 0.0, ai = 0.0;
    for (int b = threadIdx.x; b < G; b += 256) {
        const double2 v = part[(int64_t)blockIdx.x * G + b];
        ar += v.x;
        ai += v.y;
    }
    const double r = block_sum(ar, s), i = block_sum(ai, s);
    if (threadIdx.x == 0) {
        c[blockIdx.x] = make_double2(r, i);
        if (alpha && blockIdx.x + 1 == gridDim.x) alpha[0] = make_double2(r, i);
    }
}

// w -= V c, then part = V^H w as in k_proj, for all K basis vectors.
template <int K>
__global__ __launch_bounds__(256) void k_sub_proj(int64_t n, int64_t len,
                                                  const double2 *__restrict__ V, int64_t ldv,
                                                  const double2 *__restrict__ c,
                                                  double2 *__restrict__ w,
                                                  double2 *__restrict__ part)
{
    __shared__ double s[4];
    const int64_t lo = blockIdx.x * len, hi = lo + len < n ? lo + len : n;
    double ar[K], ai[K];
#pragma unroll
    for (int k = 0; k < K; ++k) ar[k] = ai[k] = 0.0;
    for (int64_t i = hi - 1 - threadIdx.x; i >= lo; i -= 256) {
        double2 a[K];
#pragma unroll
        for (int k = 0; k < K; ++k) a[k] = V[k * ldv + i];
        double2 x = w[i];
        double sr = 0.0, si = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double2 b = c[k];
            sr = fma(a[k].x, b.x, fma(-a[k].y, b.y, sr));
            si = fma(a[k].x, b.y, fma(a[k].y, b.x, si));
        }
        x.x -= sr;
        x.y -= si;
        w[i] = x;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            ar[k] = fma(a[k].x, x.x, fma(a[k].y, x.y, ar[k]));
            ai[k] = fma(a[k].x, x.y, fma(-a[k].y, x.x, ai[k]));
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const double r = block_sum(ar[k], s), i = block_sum(ai[k], s);
        if (threadIdx.x == 0) part[(int64_t)k * gridDim.x + blockIdx.x] = make_double2(r, i);
    }
}

// out = w - V c (out may be w), norm[b] = sum over part b of |out|^2 (if any).
template <bool FORWARD>
__global__ __launch_bounds__(256) void k_sub_norm(int K, int64_t n, int64_t len,
                                                  const double2 *__restrict__ V, int64_t ldv,
                                                  const double2 *__restrict__ c,
                                                  const double2 *w, double2 *out,
                                                  double *__restrict__ norm)
{
    __shared__ double s[4];
    const int64_t lo = blockIdx.x * len, hi = lo + len < n ? lo + len : n;
    double q = 0.0;
    for (int64_t j = lo + threadIdx.x; j < hi; j += 256) {
        const int64_t i = FORWARD ? j : hi - 1 - (j - lo);
        const double2 x0 = w[i];
        double sr = 0.0, si = 0.0;
#pragma unroll 8
        for (int k = 0; k < K; ++k) {
            const double2 a = V[k * ldv + i], b = c[k];
            sr = fma(a.x, b.x, fma(-a.y, b.y, sr));
            si = fma(a.x, b.y, fma(a.y, b.x, si));
        }
        const double2 x = make_double2(x0.x - sr, x0.y - si);
        out[i] = x;
        q = fma(x.x, x.x, fma(x.y, x.y, q));
    }
    if (!norm) return;
    q = block_sum(q, s);
    if (threadIdx.x == 0) norm[blockIdx.x] = q;
}

// beta = sqrt(sum of norm), out /= beta (0 if beta = 0).
__global__ __launch_bounds__(256) void k_scale(int G, int64_t n, int64_t len,
                                               const double *__restrict__ norm,
                                               double2 *__restrict__ out,
                                               double *__restrict__ beta)
{
    __shared__ double s[4];
    double q = 0.0;
    for (int b = threadIdx.x; b < G; b += 256) q += norm[b];
    const double b = sqrt(block_sum(q, s));
    if (blockIdx.x == 0 && threadIdx.x == 0) beta[0] = b;
    const double inv = b > 0.0 ? 1.0 / b : 0.0;
    const int64_t lo = blockIdx.x * len, hi = lo + len < n ? lo + len : n;
    for (int64_t i = hi - 1 - threadIdx.x; i >= lo; i -= 256) {
        const double2 x = out[i];
        out[i] = make_double2(x.x * inv, x.y * inv);
    }
}

// `sets` sets of kt vectors each from vector `first` on
template <int KT>
void proj_launch(int kt, int sets, int G, int64_t n, int64_t len, int first, const double2 *V,
                 int64_t ldv, const double2 *w, double2 *part, hipStream_t s)
{
    if (kt == KT)
        hipLaunchKernelGGL((k_proj<KT>), dim3(G, sets), dim3(256), 0, s, n, len, first, V, ldv, w,
                           part);
    else if constexpr (KT > 1)
        proj_launch<KT - 1>(kt, sets, G, n, len, first, V, ldv, w, part, s);
}

template <int K>
void sub_proj_launch(int k, int G, int64_t n, int64_t len, const double2 *V, int64_t ldv,
                     const double2 *c, double2 *w, double2 *part, hipStream_t s)
{
    if (k == K)
        hipLaunchKernelGGL((k_sub_proj<K>), dim3(G), dim3(256), 0, s, n, len, V, ldv, c, w, part);
    else if constexpr (K > 1) sub_proj_launch<K - 1>(k, G, n, len, V, ldv, c, w, part, s);
}

}  // namespace
}  // namespace mc

using namespace mc;

extern "C" {

int mc_lanczos_reorth(int32_t K, int64_t n, const double *V_d, int64_t ldv, double *w_d,
                      double *out_d, double *alpha_d, double *beta_d, void *ws_d,
                      size_t ws_bytes, mc_stream stream)
{
    if (K < 1 || n < 1 || ldv < n || !V_d || !w_d || !out_d || !beta_d || !ws_d) return MC_EINVAL;
    if (ws_bytes < (size_t)(K + 1) * (MC_REORTH_BLOCKS + 2) * 16) return MC_ENOMEM;
    const size_t vb = (size_t)((K - 1) * ldv + n) * 16, nb = (size_t)n * 16;
    if (overlaps(V_d, vb, w_d, nb) || overlaps(V_d, vb, out_d, nb) ||
        (out_d != w_d && overlaps(w_d, nb, out_d, nb)))
        return MC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    // parts of whole kilobytes, none smaller than a block's width
    int64_t len = ((n + MC_REORTH_BLOCKS - 1) / MC_REORTH_BLOCKS + 255) / 256 * 256;
    const int G = (int)((n + len - 1) / len);
    const double2 *V = (const double2 *)V_d;
    double2 *w = (double2 *)w_d, *out = (double2 *)out_d;
    double2 *part = (double2 *)ws_d, *c = part + (size_t)K * MC_REORTH_BLOCKS;
    double *norm = (double *)(c + K);
    // Projections of many vectors: one launch for every whole set of kKryTile
    // and one for the rest (with a launch per set a step waited for the host),
    // on longer parts, since a block sums 16 numbers over its threads at the
    // end: up to 2,048 elements while there are 1,024 blocks.  100 vectors made
    // one after another, ms, as four calls per vector / a launch per set / so:
    // N=20, M=7 24.3 / 31.3 / 24.0; N=30, M=5 10.8 / 12.1 / 8.5; N=60, M=5 47.5 / 54.4
    // / 44.3.
    const int sets = K / kKryTile, rest = K % kKryTile;
    int64_t plen = len;
    if (K > kKryFused)
        while (plen < 2048 && (n + 2 * plen - 1) / (2 * plen) * sets >= 1024) plen *= 2;
    const int PG = (int)((n + plen - 1) / plen);
    auto project = [&](double2 *alpha) {
        if (sets) proj_launch<kKryTile>(kKryTile, sets, PG, n, plen, 0, V, ldv, w, part, s);
        if (rest) proj_launch<kKryTile>(rest, 1, PG, n, plen, K - rest, V, ldv, w, part, s);
        hipLaunchKernelGGL(k_proj_sum, dim3(K), dim3(256), 0, s, PG, (const double2 *)part, c, alpha);
    };
    project((double2 *)alpha_d);
    if (K <= kKryFused) {
        sub_proj_launch<kKryFused>(K, G, n, len, V, ldv, c, w, part, s);
        hipLaunchKernelGGL(k_proj_sum, dim3(K), dim3(256), 0, s, G, (const double2 *)part, c,
                           (double2 *)nullptr);
    } else {
        hipLaunchKernelGGL(k_sub_norm<false>, dim3(G), dim3(256), 0, s, K, n, len, V, ldv,
                           (const double2 *)c, (const double2 *)w, w, (double *)nullptr);
        project(nullptr);
    }
    hipLaunchKernelGGL(k_sub_norm<true>, dim3(G), dim3(256), 0, s, K, n, len, V, ldv,
                       (const double2 *)c, (const double2 *)w, out, norm);
    hipLaunchKernelGGL(k_scale, dim3(G), dim3(256), 0, s, G, n, len, (const double *)norm, out,
                       beta_d);
    return launch_status();
}

}  // extern "C"
