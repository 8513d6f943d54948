// Kernels around the scalar arithmetic of attn_simple.hpp, on bf16 storage: the second implementation of
// the bf16 path (L2A_FLAG_SCALAR) and its only one for head size 64, which the bf16 matrix-core kernels
// are not built for.
#include "attn_simple.hpp"

namespace l2a {
namespace {

constexpr int kThreads = 256;
constexpr int kRowsPerBlock = kThreads / 4;

__device__ __forceinline__ int block_row() { return blockIdx.x * kRowsPerBlock + (threadIdx.x >> 2); }

template <typename E, int DL>
__global__ __launch_bounds__(kThreads) void simple_fwd_kernel(Geom gm, RowSet rs, const E* __restrict__ q,
                                                              const E* __restrict__ k, const E* __restrict__ v,
                                                              FwdOut out) {
    simple_fwd_row<E, DL>(gm, rs, q, k, v, out, blockIdx.y, block_row(), threadIdx.x & 3);
}

template <typename E, int DL>
__global__ __launch_bounds__(kThreads) void simple_bwd_dq_kernel(Geom gm, RowSet rs, const E* __restrict__ q,
                                                                 const E* __restrict__ k, const E* __restrict__ v,
                                                                 const E* __restrict__ dO,
                                                                 const float* __restrict__ lse, float* delta,
                                                                 E* dq, int accumulate) {
    simple_dq_row<E, DL>(gm, rs, q, k, v, dO, lse, delta, dq, accumulate, blockIdx.y, block_row(), threadIdx.x & 3);
}

template <typename E, int DL>
__global__ __launch_bounds__(kThreads) void simple_bwd_dkdv_kernel(Geom gm, DkdvSets sets, const E* __restrict__ q,
                                                                   const E* __restrict__ k, const E* __restrict__ v,
                                                                   const E* __restrict__ dO, E* dk, E* dv) {
    simple_dkdv_key<E, DL>(gm, sets, q, k, v, dO, dk, dv, blockIdx.y, block_row(), threadIdx.x & 3);
}

inline dim3 row_grid(const Geom& g) {
    const long long rows = (long long)g.T * g.G;
    return dim3((unsigned)((rows + kRowsPerBlock - 1) / kRowsPerBlock), g.B * g.Hkv);
}

}  // namespace

template <typename T>
static const T* cp(const void* p) { return (const T*)p; }

int simple_fwd(const Geom& g, const RowSet& rs, const void* q, const void* k, const void* v,
               const FwdOut& out, hipStream_t st) {
    const dim3 grid = row_grid(g);
    KernelTimer kt(rs.local ? "scalar_fwd_local" : "scalar_fwd_global", st);
    if (g.D == 64)
        hipLaunchKernelGGL((simple_fwd_kernel<__bf16, 16>), grid, dim3(kThreads), 0, st, g, rs, cp<__bf16>(q), cp<__bf16>(k), cp<__bf16>(v), out);
    else if (g.D == 128)
        hipLaunchKernelGGL((simple_fwd_kernel<__bf16, 32>), grid, dim3(kThreads), 0, st, g, rs, cp<__bf16>(q), cp<__bf16>(k), cp<__bf16>(v), out);
    else
        return L2A_ERR_UNSUPPORTED;
    return launch_status();
}

int simple_bwd_dq(const Geom& g, const RowSet& rs, const void* q, const void* k, const void* v,
                  const void* dO, const float* lse, float* delta, void* dq, int accumulate, hipStream_t st) {
    const dim3 grid = row_grid(g);
    KernelTimer kt(rs.local ? "scalar_bwd_dq_local" : "scalar_bwd_dq_global", st);
    if (g.D == 64)
        hipLaunchKernelGGL((simple_bwd_dq_kernel<__bf16, 16>), grid, dim3(kThreads), 0, st, g, rs, cp<__bf16>(q), cp<__bf16>(k), cp<__bf16>(v), cp<__bf16>(dO), lse, delta, (__bf16*)dq, accumulate);
    else if (g.D == 128)
        hipLaunchKernelGGL((simple_bwd_dq_kernel<__bf16, 32>), grid, dim3(kThreads), 0, st, g, rs, cp<__bf16>(q), cp<__bf16>(k), cp<__bf16>(v), cp<__bf16>(dO), lse, delta, (__bf16*)dq, accumulate);
    else
        return L2A_ERR_UNSUPPORTED;
    return launch_status();
}

int simple_bwd_dkdv(const Geom& g, const RowSet* sets, int nsets, const void* q, const void* k,
                    const void* v, const void* dO, const float* const* lse, const float* const* delta, void* dk,
                    void* dv, hipStream_t st) {
    DkdvSets s;
    s.n = nsets;
    for (int i = 0; i < nsets; ++i) {
        s.rs[i] = sets[i];
        s.lse[i] = lse[i];
        s.delta[i] = delta[i];
    }
    const dim3 grid((g.T + kRowsPerBlock - 1) / kRowsPerBlock, g.B * g.Hkv);
    KernelTimer kt("scalar_bwd_dkdv", st);
    if (g.D == 64)
        hipLaunchKernelGGL((simple_bwd_dkdv_kernel<__bf16, 16>), grid, dim3(kThreads), 0, st, g, s, cp<__bf16>(q), cp<__bf16>(k), cp<__bf16>(v), cp<__bf16>(dO), (__bf16*)dk, (__bf16*)dv);
    else if (g.D == 128)
        hipLaunchKernelGGL((simple_bwd_dkdv_kernel<__bf16, 32>), grid, dim3(kThreads), 0, st, g, s, cp<__bf16>(q), cp<__bf16>(k), cp<__bf16>(v), cp<__bf16>(dO), (__bf16*)dk, (__bf16*)dv);
    else
        return L2A_ERR_UNSUPPORTED;
    return launch_status();
}

}  // namespace l2a
