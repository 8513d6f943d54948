// Small memory-bound helpers: the backward pass's per-row dot products and fills.
#include "mfma.hpp"

#include <algorithm>

namespace l2a {
namespace {

// delta_l[b,h,t] = <dO, S>, delta_g[b,h,t] = <dO, A>  (the "D" vector of the FlashAttention
// backward, one per branch; delta_g is also the task-loss part of the router-score gradient,
// Sec. 3.3 Eq. 7).  A workgroup takes `tok` consecutive tokens of one sequence -- a contiguous
// stretch of [t, h, D] rows, sixteen lanes per row -- and transposes its results through LDS, so
// that the [b, h, t] outputs are written in runs of consecutive t instead of one scattered float
// per row.
template <typename E, int DL>
__global__ __launch_bounds__(kThreads) void row_deltas_kernel(Geom gm, const E* __restrict__ dO,
                                                              const E* __restrict__ S, const E* __restrict__ A,
                                                              float* __restrict__ delta_l,
                                                              float* __restrict__ delta_g,
                                                              float* __restrict__ share_zero, int tok) {
    extern __shared__ float stage[];  // [2][Hq][tok]
    const int b = blockIdx.y, t0 = blockIdx.x * tok;
    const int ntok = min(tok, gm.T - t0);
    const int part = threadIdx.x & 15;
    float* sa = stage;
    float* sc = stage + gm.Hq * tok;
    const size_t row0 = ((size_t)b * gm.T + t0) * gm.Hq;
    for (int r = threadIdx.x >> 4; r < ntok * gm.Hq; r += kThreads / 16) {
        const size_t off = (row0 + r) * gm.D + part * DL;
        float a = 0.f, c = 0.f;
        // one 16- or 32-byte load per array and lane
        typedef E Vec __attribute__((ext_vector_type(DL)));
        const Vec gv = *reinterpret_cast<const Vec*>(dO + off);
        if (S) {
            const Vec sv = *reinterpret_cast<const Vec*>(S + off);
#pragma unroll
            for (int i = 0; i < DL; ++i) a += (float)gv[i] * (float)sv[i];
        }
        if (A) {
            const Vec av = *reinterpret_cast<const Vec*>(A + off);
#pragma unroll
            for (int i = 0; i < DL; ++i) c += (float)gv[i] * (float)av[i];
        }
        for (int o = 8; o > 0; o >>= 1) {
            a += __shfl_xor(a, o);
            c += __shfl_xor(c, o);
        }
        if (part == 0) {
            const int tt = r / gm.Hq, h = r - tt * gm.Hq;
            sa[h * tok + tt] = a;
            sc[h * tok + tt] = c;
        }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < gm.Hq * tok; idx += kThreads) {
        const int h = idx / tok, tt = idx - h * tok;
        if (tt >= ntok) continue;
        const size_t so = ((size_t)b * gm.Hq + h) * gm.T + t0 + tt;
        if (delta_l) delta_l[so] = sa[idx];
        if (delta_g) delta_g[so] = sc[idx];
        if (share_zero) share_zero[so] = 0.f;
    }
}

// Shared inputs: in its window a routed row's two branches have the same scores, so that their weights differ by a
// constant, p_g = a p_l with a = exp(lse_l - lse_g) <= 1, and what they add up to there is one row's gradient:
//     p_l + p_g = p',   p_l (dP - delta_l) + p_g (dP - delta_g) = p' (dP - delta'),
//     p' = exp(s - lse_l + log(1 + a)),   delta' = (delta_l + a delta_g) / (1 + a).
// The Local pass runs over these rows, and the Global pass only over the keys before the window: the window's
// (row, key) pairs are computed once instead of twice.  Training step, W = 4096, 20 % routed, before / after: T = 16379
// (32 / 8 heads) 6389 / 5740 us, T = 131072 (28 / 4 heads) 125.9 / 121.2 ms.  dK and dV take one rounding of the sum of
// two weights where they took two independent ones: their error against 64 bits at T = 16379 is 1.4 % and 0.9 % larger
// (2.83e-3 -> 2.87e-3, 2.31e-3 -> 2.33e-3 of the norm); dQ, whose two parts are now added in fp32, 2.381e-3 -> 2.380e-3.
// One thread per routed row.
__global__ __launch_bounds__(kThreads) void fold_rows_kernel(Geom gm, RowSet rs, const float* __restrict__ lse_l,
                                                             const float* __restrict__ lse_g, float* __restrict__ delta_l,
                                                             const float* __restrict__ delta_g, float* __restrict__ share) {
    const int bh = blockIdx.y, b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    const int r = blockIdx.x * kThreads + threadIdx.x;
    if (r >= rows_total(rs, gm, bh)) return;
    const int code = row_code(rs, gm, bh, r), p = code / gm.G;
    const size_t so = ((size_t)b * gm.Hq + hk * gm.G + (code - p * gm.G)) * gm.T + p;
    float a = expf(lse_l[so] - lse_g[so]);
    a = a < 1e-30f ? 1e-30f : a;  // not zero: that marks the rows that are not folded (a NaN stays one)
    share[so] = a;
    delta_l[so] = (delta_l[so] + a * delta_g[so]) / (1.f + a);
}

// delta of the first tokens of a sequence, from its definition instead of from the saved outputs:
//     delta_t = sum_j p_tj <dO_t, v_j>,   p_tj = exp(scale <q_t, k_j> - lse_t)     (= <dO_t, out_t>).
// The saved outputs are bf16: <dO_t, out_t> then carries an error of about 2^-9 sqrt(D) |dO_t| |out_t|,
// which enters dq_t as  scale * error * sum_j p_tj k_j.  Both factors shrink like 1 / sqrt(keys) for
// rows that average many keys, but for the first few tokens they do not (token 2 with N(0,1) inputs:
// up to 1.2e-2 per branch, twice that when both branches read the same tensors, since s_t = a_t
// there), so the first kHeadTokens deltas are recomputed exactly.  A row whose log-sum-exp is -inf (not routed: a_t = 0)
// gets delta = 0.  Workgroup = (branch, head, sequence), wavefront = 32 tokens, on the matrix cores: S^T = K Q^T and dP^T
// = V dO^T of 32 keys at a time, a lane owns a token.  With a wavefront per token and a lane per key the 64 separate cache
// lines of every load set the time: 30 us for two sequences of 28 heads, both branches, now 12.
constexpr int kHeadTokens = 64;

struct HeadBranch {
    const __bf16 *q, *k, *v;
    const float* lse;
    float* delta;
    int local;
};

__global__ __launch_bounds__(128) void head_deltas_kernel(Geom gm, HeadBranch br0, HeadBranch br1,
                                                          const __bf16* __restrict__ dO) {
    const HeadBranch br = blockIdx.x ? br1 : br0;
    const int h = blockIdx.y, b = blockIdx.z, hk = h / gm.G;
    const int lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
    const int t0 = (int)(threadIdx.x >> 6) * 32, nt = min(gm.T, kHeadTokens);
    if (t0 >= nt) return;
    const int t = min(t0 + n, nt - 1);  // lanes past the end repeat the last token and write nothing
    const size_t row = (((size_t)b * gm.T + t) * gm.Hq + h) * gm.D + 8 * half;
    const size_t so = ((size_t)b * gm.Hq + h) * gm.T + t;
    const float l = br.lse[so];
    float sum = 0.f;
    for (int k0 = 0; k0 <= min(t0 + 31, nt - 1); k0 += 32) {
        const int j = min(k0 + n, gm.T - 1);  // keys past the end: out of every token's reach
        const size_t key = (((size_t)b * gm.T + j) * gm.Hkv + hk) * gm.D + 8 * half;
        f32x16 s, dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
        for (int c0 = 0; c0 < gm.D; c0 += 64) {  // D = 64 or 128
            bf16x8 q8[4], g8[4], k8[4], v8[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = c0 + 16 * i;
                q8[i] = *reinterpret_cast<const bf16x8*>(br.q + row + c), k8[i] = *reinterpret_cast<const bf16x8*>(br.k + key + c);
                g8[i] = *reinterpret_cast<const bf16x8*>(dO + row + c), v8[i] = *reinterpret_cast<const bf16x8*>(br.v + key + c);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) s = mfma32(k8[i], q8[i], s), dp = mfma32(v8[i], g8[i], dp);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int kr = k0 + c_row(r, half);
            const bool in_reach = kr <= t && (!br.local || t - kr <= gm.W);
            sum += in_reach && l != -INFINITY ? expf(s[r] * gm.scale - l) * dp[r] : 0.f;
        }
    }
    sum += __shfl_xor(sum, 32);
    if (half == 0 && t0 + n < nt) br.delta[so] = sum;
}

// 16-byte stores from an aligned address, a few per thread (57 MB with a 4-byte store per thread 18 us, now 11)
__global__ __launch_bounds__(kThreads) void fill_u32_kernel(uint32_t* p, size_t n, uint32_t value) {
    size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * kThreads;
    if (((uintptr_t)p & 15) == 0) {
        const u32x4 v = {value, value, value, value};
        for (size_t q = i; q < n / 4; q += stride) reinterpret_cast<u32x4*>(p)[q] = v;
        i += n / 4 * 4;
    }
    for (; i < n; i += stride) p[i] = value;
}

}  // namespace

int row_deltas(const Geom& g, int dtype, const void* dO, const void* S, const void* A, float* delta_l,
               float* delta_g, float* share_zero, hipStream_t st) {
    int tok = 64;  // tokens per workgroup: as many as fit 64 KB of LDS with Hq heads
    while (tok > 1 && sizeof(float) * 2 * g.Hq * tok > 64 * 1024) tok /= 2;
    // short sequences: fewer tokens per workgroup rather than a grid that leaves most of the chip idle
    while (tok > 8 && (long long)((g.T + tok - 1) / tok) * g.B < 2048) tok /= 2;
    const size_t lds = sizeof(float) * 2 * g.Hq * tok;
    if (lds > 64 * 1024) return L2A_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)((g.T + tok - 1) / tok), (unsigned)g.B);
    KernelTimer kt("row_deltas", st);
    if (dtype == L2A_FP32 && g.D == 64)
        hipLaunchKernelGGL((row_deltas_kernel<float, 4>), grid, dim3(kThreads), lds, st, g, (const float*)dO, (const float*)S, (const float*)A, delta_l, delta_g, share_zero, tok);
    else if (dtype == L2A_FP32 && g.D == 128)
        hipLaunchKernelGGL((row_deltas_kernel<float, 8>), grid, dim3(kThreads), lds, st, g, (const float*)dO, (const float*)S, (const float*)A, delta_l, delta_g, share_zero, tok);
    else if (dtype == L2A_BF16 && g.D == 64)
        hipLaunchKernelGGL((row_deltas_kernel<__bf16, 4>), grid, dim3(kThreads), lds, st, g, (const __bf16*)dO, (const __bf16*)S, (const __bf16*)A, delta_l, delta_g, share_zero, tok);
    else if (dtype == L2A_BF16 && g.D == 128)
        hipLaunchKernelGGL((row_deltas_kernel<__bf16, 8>), grid, dim3(kThreads), lds, st, g, (const __bf16*)dO, (const __bf16*)S, (const __bf16*)A, delta_l, delta_g, share_zero, tok);
    else
        return L2A_ERR_UNSUPPORTED;
    return launch_status();
}

int fold_rows(const Geom& g, const RowSet& rs, const float* lse_l, const float* lse_g, float* delta_l, const float* delta_g,
              float* share, hipStream_t st) {
    const long long rows = (long long)g.T * g.G;
    KernelTimer kt("fold_rows", st);
    hipLaunchKernelGGL(fold_rows_kernel, dim3((unsigned)((rows + kThreads - 1) / kThreads), g.B * g.Hkv), dim3(kThreads), 0, st, g,
                       rs, lse_l, lse_g, delta_l, delta_g, share);
    return launch_status();
}

int head_deltas(const Geom& g, const HeadDeltas* branches, int n, const void* dO, hipStream_t st) {
    static_assert(kHeadTokens <= 64, "two wavefronts of 32 tokens");
    HeadBranch br[2] = {};
    for (int i = 0; i < n; ++i)
        br[i] = HeadBranch{(const __bf16*)branches[i].q, (const __bf16*)branches[i].k, (const __bf16*)branches[i].v,
                           branches[i].lse, branches[i].delta, branches[i].local};
    KernelTimer kt("head_deltas", st);
    hipLaunchKernelGGL(head_deltas_kernel, dim3((unsigned)n, (unsigned)g.Hq, (unsigned)g.B), dim3(128), 0, st, g, br[0], br[1],
                       (const __bf16*)dO);
    return launch_status();
}

static size_t fill_blocks(size_t n) { return std::min<size_t>((n / 4 + kThreads - 1) / kThreads + 1, 4096); }

// bytes must be a multiple of 4 (every tensor here is)
int fill_zero(void* ptr, size_t bytes, hipStream_t st) {
    const size_t n = bytes / 4;
    if (n == 0) return L2A_OK;
    const size_t blocks = fill_blocks(n);
    KernelTimer kt("fill", st);
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, st, (uint32_t*)ptr, n, 0u);
    return launch_status();
}

int fill_f32(float* ptr, size_t n, float value, hipStream_t st) {
    if (n == 0) return L2A_OK;
    const size_t blocks = fill_blocks(n);
    uint32_t bits;
    __builtin_memcpy(&bits, &value, 4);
    KernelTimer kt("fill", st);
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, st, (uint32_t*)ptr, n, bits);
    return launch_status();
}

}  // namespace l2a
