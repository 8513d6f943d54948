// Small memory-bound helpers: the backward pass's per-row dot products and fills.
#include "mfma.hpp"

#include <algorithm>

namespace l2a {
namespace {

// The per-row statistics of the backward, one launch:
//     delta_l[b,h,t] = <dO, S>, delta_g[b,h,t] = <dO, A>  (the "D" vector of the FlashAttention backward, one per branch;
//     delta_g is also the task-loss part of the router-score gradient, Sec. 3.3 Eq. 7),
// for bf16 those of the first tokens from their definition, and for fp32 with shared inputs the fold of the routed rows.
//
// Fold.  In its window a routed row's two branches have the same scores, so that their weights differ by a
// constant, p_g = a p_l with a = exp(lse_l - lse_g) <= 1, and what they add up to there is one row's gradient:
//     p_l + p_g = p',   p_l (dP - delta_l) + p_g (dP - delta_g) = p' (dP - delta'),
//     p' = exp(s - lse_l + log(1 + a)),   delta' = (delta_l + a delta_g) / (1 + a).
// dK and dV take these rows for the Local ones, and of the Global rows only the keys before the window: the window's
// (row, key) pairs are computed once instead of twice.  fp32 only: in bf16 dK and dV would take one rounding of the sum of two
// weights where they take two independent ones, and their error against 64 bits at 16379 tokens would be 1.4 % and 0.9 % larger
// (2.83e-3 -> 2.87e-3, 2.31e-3 -> 2.33e-3 of the norm).  Not dQ (but where s = a to the bit): the two branches' sums over the window
// would share their roundings, which their sum does not average out (up to 2.6 % more error at 4096 tokens).
//
// Memory-bound: a workgroup takes `tok` consecutive tokens of one sequence -- a contiguous
// stretch of [t, h, D] rows, sixteen lanes per row, four rows of each in flight -- and transposes its results through
// LDS, so that the [b, h, t] outputs are written in runs of consecutive t instead of one scattered float
// per row.  Which rows are routed comes from the lists: the entries of the 64 positions around.  As three launches
// (products, first tokens, fold) with one row in flight this took 36 us at 1000 tokens of 28 heads, now 15; 2 x 4000 tokens
// of separate modules (two launches) 51, now 43 (172 MB).
struct StatsBranch {
    const void *q, *k, *v, *out;  // out: the saved s or a (null: the branch is not run)
    const float* lse;
    float* delta;
    int local;
};
struct StatsArgs {
    Geom gm;
    StatsBranch br[2];
    const void* dO;
    int tok;         // tokens per workgroup, a power of two up to 64
    int row_blocks;  // workgroups per sequence that take rows; the ones behind them the first tokens, one head each
    RowSet routed;   // share: the routed rows and kblk_first_row
    float* share;    // fold: a, 0 on rows that are not routed (null: no fold)
    bool fold_delta;
};

// Marks the routed rows of positions t0 .. t0 + n - 1 (inside one block of 64): flags[head * n + t - t0].  The KV heads side
// by side, 64 or 16 lanes each: one after the other their three dependent loads were the workgroup's time where there are many.
__device__ __forceinline__ void mark_routed(const Geom& gm, const RowSet& rs, int b, int t0, int n, unsigned char* flags) {
    const int lanes = gm.Hkv >= kThreads / 16 ? 16 : 64;
    for (int hk = (int)threadIdx.x / lanes; hk < gm.Hkv; hk += kThreads / lanes) {
        const int bh = b * gm.Hkv + hk, total = rows_total(rs, gm, bh);
        const int32_t* first = rs.kblk_first_row + (size_t)bh * ((gm.T + 63) / 64 + 1) + (t0 >> 6);
        const int f0 = min(max(first[0], 0), total), f1 = min(max(first[1], f0), total);
        for (int i = f0 + (int)threadIdx.x % lanes; i < f1; i += lanes) {
            const int code = row_code(rs, gm, bh, i), p = code / gm.G, t = p - t0;
            if (t >= 0 && t < n) flags[(hk * gm.G + code - p * gm.G) * n + t] = 1;
        }
    }
}

__device__ __forceinline__ void store_stats(const StatsArgs& a, size_t so, float dl, float dg, bool routed) {
    if (a.share) {
        float f = 0.f;
        if (routed) {
            f = expf(a.br[0].lse[so] - a.br[1].lse[so]);
            if (a.fold_delta) dl = (dl + f * dg) / (1.f + f);
        }
        a.share[so] = f;
    }
    if (a.br[0].out) a.br[0].delta[so] = dl;
    if (a.br[1].out) a.br[1].delta[so] = dg;
}

// delta of the first tokens of a sequence, from its definition instead of from the saved outputs:
//     delta_t = sum_j p_tj <dO_t, v_j>,   p_tj = exp(scale <q_t, k_j> - lse_t)     (= <dO_t, out_t>).
// The saved outputs are bf16: <dO_t, out_t> then carries an error of about 2^-9 sqrt(D) |dO_t| |out_t|,
// which enters dq_t as  scale * error * sum_j p_tj k_j.  Both factors shrink like 1 / sqrt(keys) for
// rows that average many keys, but for the first few tokens they do not (token 2 with N(0,1) inputs:
// up to 1.2e-2 per branch, twice that when both branches read the same tensors, since s_t = a_t
// there), so the first kHeadTokens deltas are recomputed exactly.  A row whose log-sum-exp is -inf (not routed: a_t = 0)
// gets delta = 0.  Workgroup = (head, sequence), wavefront = 32 tokens of a branch, on the matrix cores: S^T = K Q^T and
// dP^T = V dO^T of 32 keys at a time, a lane owns a token.  With a wavefront per token and a lane per key the 64 separate
// cache lines of every load set the time: 30 us for two sequences of 28 heads, both branches, now 12.
constexpr int kHeadTokens = 64;

__device__ __forceinline__ void head_deltas(const StatsArgs& a, const StatsBranch& br, int b, int h, int t0, float* out) {
    const Geom& gm = a.gm;
    const int hk = h / gm.G, lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
    const int nt = min(gm.T, kHeadTokens);
    const int t = min(t0 + n, nt - 1);  // lanes past the end repeat the last token and write nothing
    const size_t row = (((size_t)b * gm.T + t) * gm.Hq + h) * gm.D + 8 * half;
    const float l = br.lse[((size_t)b * gm.Hq + h) * gm.T + t];
    const __bf16 *q = (const __bf16*)br.q, *k = (const __bf16*)br.k, *v = (const __bf16*)br.v, *dO = (const __bf16*)a.dO;
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
                q8[i] = *reinterpret_cast<const bf16x8*>(q + row + c), k8[i] = *reinterpret_cast<const bf16x8*>(k + key + c);
                g8[i] = *reinterpret_cast<const bf16x8*>(dO + row + c), v8[i] = *reinterpret_cast<const bf16x8*>(v + key + c);
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
    if (half == 0) out[t0 + n] = sum;
}

constexpr int kFlight = 4;  // rows of sixteen lanes whose loads are in flight together
template <typename E, int DL>
__global__ __launch_bounds__(kThreads) void row_stats_kernel(StatsArgs a) {
    extern __shared__ float stage[];  // [2][Hq][tok] products; fold: then one byte per row, routed
    const Geom& gm = a.gm;
    const int b = blockIdx.y;
    if constexpr (sizeof(E) == 2) {
        if ((int)blockIdx.x >= a.row_blocks) {  // the first tokens of one head
            const int h = (int)blockIdx.x - a.row_blocks, nt = min(gm.T, kHeadTokens);
            const int which = (int)threadIdx.x >> 7, t0 = (int)(threadIdx.x >> 6 & 1) * 32;
            if (a.br[which].out && t0 < nt) head_deltas(a, a.br[which], b, h, t0, stage + which * kHeadTokens);
            __syncthreads();
            const int t = threadIdx.x;
            if (t < nt) store_stats(a, ((size_t)b * gm.Hq + h) * gm.T + t, stage[t], stage[kHeadTokens + t], false);
            return;
        }
    }
    const int tok = a.tok, t0 = blockIdx.x * tok;
    const int ntok = min(tok, gm.T - t0), rows = ntok * gm.Hq;
    const int part = threadIdx.x & 15;
    float* sa = stage;
    float* sc = stage + gm.Hq * tok;
    unsigned char* flags = reinterpret_cast<unsigned char*>(stage + 2 * gm.Hq * tok);  // [Hq][ntok]
    if (a.share) {
        for (int i = threadIdx.x; i < rows; i += kThreads) flags[i] = 0;
        __syncthreads();
        mark_routed(gm, a.routed, b, t0, ntok, flags);
    }
    const size_t row0 = ((size_t)b * gm.T + t0) * gm.Hq;
    typedef E Vec __attribute__((ext_vector_type(DL)));  // one 16- or 32-byte load per array and lane
    const E* dO = (const E*)a.dO;
    const E *S = (const E*)a.br[0].out, *A = (const E*)a.br[1].out;
    for (int rr = threadIdx.x >> 4; rr < rows; rr += kFlight * (kThreads / 16)) {
        Vec gv[kFlight], sv[kFlight], av[kFlight];
#pragma unroll
        for (int j = 0; j < kFlight; ++j) {
            const size_t off = (row0 + min(rr + j * (kThreads / 16), rows - 1)) * gm.D + part * DL;
            gv[j] = *reinterpret_cast<const Vec*>(dO + off);
            if (S) sv[j] = *reinterpret_cast<const Vec*>(S + off);
            if (A) av[j] = *reinterpret_cast<const Vec*>(A + off);
        }
#pragma unroll
        for (int j = 0; j < kFlight; ++j) {
            float x = 0.f, y = 0.f;
            if (S)
#pragma unroll
                for (int i = 0; i < DL; ++i) x += (float)gv[j][i] * (float)sv[j][i];
            if (A)
#pragma unroll
                for (int i = 0; i < DL; ++i) y += (float)gv[j][i] * (float)av[j][i];
            for (int o = 8; o > 0; o >>= 1) {
                x += __shfl_xor(x, o);
                y += __shfl_xor(y, o);
            }
            const int r = rr + j * (kThreads / 16);
            if (part == 0 && r < rows) {
                const int tt = r / gm.Hq, h = r - tt * gm.Hq;
                sa[h * tok + tt] = x;
                sc[h * tok + tt] = y;
            }
        }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < gm.Hq * tok; idx += kThreads) {
        const int h = idx / tok, tt = idx - h * tok;
        if (tt >= ntok || (sizeof(E) == 2 && t0 + tt < kHeadTokens)) continue;
        store_stats(a, ((size_t)b * gm.Hq + h) * gm.T + t0 + tt, sa[idx], sc[idx], a.share && flags[h * ntok + tt]);
    }
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

namespace {
constexpr size_t kStatsLds = 64 * 1024;
size_t stats_lds(const Geom& g, int tok, bool fold) { return (size_t)g.Hq * tok * (2 * sizeof(float) + (fold ? 1 : 0)); }
}  // namespace

bool row_stats_can_fold(const Geom& g) { return stats_lds(g, 1, true) <= kStatsLds; }

int row_stats(const Geom& g, int dtype, const void* dO, const RowStats* local, const RowStats* global, const RowSet& routed,
              float* share, bool fold_delta, hipStream_t st) {
    auto lds_bytes = [&](int tok) { return stats_lds(g, tok, share != nullptr); };
    int tok = 64;  // tokens per workgroup: as many as fit 64 KB of LDS with Hq heads
    while (tok > 1 && lds_bytes(tok) > kStatsLds) tok /= 2;
    // short sequences: fewer tokens per workgroup rather than a grid that leaves most of the chip idle
    while (tok > 2 && tok * g.Hq > kFlight * (kThreads / 16) && (long long)((g.T + tok - 1) / tok) * g.B < 1024) tok /= 2;
    if (lds_bytes(tok) > kStatsLds) return L2A_ERR_UNSUPPORTED;
    StatsArgs a{};
    a.gm = g;
    a.dO = dO;
    a.tok = tok;
    a.row_blocks = (g.T + tok - 1) / tok;
    a.routed = routed;
    a.share = share;
    a.fold_delta = fold_delta;
    if (local) a.br[0] = StatsBranch{local->q, local->k, local->v, local->out, local->lse, local->delta, 1};
    if (global) a.br[1] = StatsBranch{global->q, global->k, global->v, global->out, global->lse, global->delta, 0};
    // bf16: the first tokens of a head need 2 x 64 floats
    const size_t head_lds = 2 * sizeof(float) * kHeadTokens, row_lds = lds_bytes(tok);
    const size_t lds = dtype == L2A_BF16 && head_lds > row_lds ? head_lds : row_lds;
    const dim3 grid((unsigned)(a.row_blocks + (dtype == L2A_BF16 ? g.Hq : 0)), (unsigned)g.B);
    KernelTimer kt("row_stats", st);
    if (dtype == L2A_FP32 && g.D == 64) hipLaunchKernelGGL((row_stats_kernel<float, 4>), grid, dim3(kThreads), lds, st, a);
    else if (dtype == L2A_FP32 && g.D == 128) hipLaunchKernelGGL((row_stats_kernel<float, 8>), grid, dim3(kThreads), lds, st, a);
    else if (dtype == L2A_BF16 && g.D == 64) hipLaunchKernelGGL((row_stats_kernel<__bf16, 4>), grid, dim3(kThreads), lds, st, a);
    else if (dtype == L2A_BF16 && g.D == 128) hipLaunchKernelGGL((row_stats_kernel<__bf16, 8>), grid, dim3(kThreads), lds, st, a);
    else return L2A_ERR_UNSUPPORTED;
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
