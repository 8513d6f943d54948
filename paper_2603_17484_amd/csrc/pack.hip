// Layout pre-passes of the matrix-core kernels (memory-bound, one pass over the tensor).
//
//   pack_token_minor : copies of a tensor whose rows are either the tokens of a KV head (V, for
//                      the forward kernel: the token-minor copy XT[b, kv head, channel, row], rows
//                      inside each group of 16 in the order the matrix-core operands want, see
//                      tiles.hpp) or the rows of a branch's row set (Q and dO, for the dK/dV
//                      kernel: compact row-major copies together with the rows' saved statistics
//                      -- for the Global branch this is the consolidation of the active queries
//                      into a contiguous buffer Q_c, App. C Alg. 1 step 1).
// The transpose itself is done by ds_read_b64_tr_b16: sixteen lanes hand in four rows of sixteen
// channels and each lane gets back four rows of one channel.
#include "tiles.hpp"

namespace l2a {
namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

struct PackArgs {
    Geom gm;
    RowSet rs;
    int kv_rows;  // 1: rows are the tokens of a KV head, tensors are [B,T,Hkv,D]; 0: rows of rs, tensors [B,T,Hq,D]
    const __bf16* x[2];   // up to two tensors share the row list (Q and dO); x[1] may be null
    __bf16* xt[2];        // optional token-minor copies [B*Hkv][128][cap]
    __bf16* xc[2];        // optional compact row-major copies [B*Hkv][cap][128]
    const float* lse;     // optional per-row statistics of the row set, [B,Hq,T]
    const float* delta;
    float* lse2_c;        // [B*Hkv][cap]: lse * log2(e)
    float* delta_c;
    int32_t* pos_c;       // position, -1 for padding
    int cap;              // rows per (b, kv head) in the outputs; multiple of 64
    Fill fill[3];         // buffers to be filled on the way
    RoutedFlags routed;   // kv_rows: which rows are routed, marked on the way (routed.flags may be null)
};

// A launch costs a short forward as much as the kernel it carries (about 3 us each), so the constants that its
// kernels expect are written by the workgroups of the one that runs first.  16-byte stores where the buffer allows.
__device__ __forceinline__ void run_fill(const Fill& f) {
    const size_t step = (size_t)gridDim.x * gridDim.y * kThreads;
    size_t i = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kThreads + threadIdx.x;
    size_t done = 0;
    if (((uintptr_t)f.p & 15) == 0) {
        const u32x4 v = {f.value, f.value, f.value, f.value};
        for (size_t j = i; j < f.n / 4; j += step) reinterpret_cast<u32x4*>(f.p)[j] = v;
        done = f.n / 4 * 4;
    }
    for (i += done; i < f.n; i += step) f.p[i] = f.value;
}

// Which rows of positions 64 kb .. 64 kb + 63 are routed: gathered as bits from the list's entries first[kb] .. first[kb+1]
constexpr int kMaxG = 16;  // Hq / Hkv at most
__device__ __forceinline__ void mark_routed(const Geom& gm, const RoutedFlags& rf, int bh, int kb, unsigned long long (&bits)[kMaxG]) {
    const int nkb = (gm.T + 63) / 64, n = rows_total(rf.routed, gm, bh);
    if (kb >= nkb) return;
    const int32_t* first = rf.routed.kblk_first_row + (size_t)bh * (nkb + 1) + kb;
    const int f0 = min(max(first[0], 0), n), f1 = min(max(first[1], f0), n);
    const int c0 = kb * 64 * gm.G, codes = min(64, gm.T - kb * 64) * gm.G;
    if (threadIdx.x < kMaxG) bits[threadIdx.x] = 0;
    __syncthreads();
    for (int i = f0 + (int)threadIdx.x; i < f1; i += kThreads) {
        const int c = row_code(rf.routed, gm, bh, i) - c0;
        if (c >= 0 && c < codes) atomicOr(&bits[c >> 6], 1ull << (c & 63));
    }
    __syncthreads();
    for (int c = threadIdx.x; c < codes; c += kThreads) rf.flags[(size_t)bh * gm.T * gm.G + c0 + c] = bits[c >> 6] >> (c & 63) & 1;
}

__global__ __launch_bounds__(kThreads) void pack_token_minor_kernel(PackArgs a) {
    __shared__ __attribute__((aligned(16))) __bf16 lds[2][kTileRows * kRowPad];
    __shared__ unsigned long long routed_bits[kMaxG];
    const Geom& gm = a.gm;
    const int bh = blockIdx.y, b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    const int r0 = blockIdx.x * 64;
    const int n_rows = a.kv_rows ? gm.T : rows_total(a.rs, gm, bh);

    // global element offset of row r's channel 0, or -1 for padding
    auto row_offset = [&](int r, int* pos_out, size_t* stat_out) -> long long {
        if (r >= n_rows) return -1;
        if (a.kv_rows) return (((long long)b * gm.T + r) * gm.Hkv + hk) * kD;
        const int code = row_code(a.rs, gm, bh, r);
        const int p = code / gm.G;
        const int head = hk * gm.G + (code - p * gm.G);
        if (pos_out) *pos_out = p;
        if (stat_out) *stat_out = ((size_t)b * gm.Hq + head) * gm.T + p;
        return (((long long)b * gm.T + p) * gm.Hq + head) * kD;
    };

    // ---- 64 rows, on their way while the constants and the flags are written: a workgroup's time is the chain of its dependent
    // loads (list bounds, list, then the rows), T = 1001 with 4 KV heads 6.9 -> 5.7 us; the rows of two tensors in flight
    // together, 2 x 4000 tokens with 4 KV heads 47.2 + 19.3 -> 42.0 + 17.1 us (5.4 TB/s).
    const int r4 = (threadIdx.x >> 4) * 4, c8 = (threadIdx.x & 15) * 8;
    long long offs[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) offs[i] = row_offset(r0 + r4 + i, nullptr, nullptr);
    u32x4 v[2][4] = {};
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (a.x[t] && offs[i] >= 0) v[t][i] = *reinterpret_cast<const u32x4*>(a.x[t] + offs[i] + c8);

#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (a.fill[i].n) run_fill(a.fill[i]);
    if (a.routed.flags) mark_routed(gm, a.routed, bh, (int)blockIdx.x, routed_bits);
    if (r0 >= n_rows) return;  // the readers stop at the last row's tile

    // ---- -> LDS (row-major, padded), and the compact row-major copy
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        if (!a.x[t]) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (a.xt[t]) *reinterpret_cast<u32x4*>(&lds[t][(r4 + i) * kRowPad + c8]) = v[t][i];
            if (a.xc[t])
                *reinterpret_cast<u32x4*>(a.xc[t] + ((size_t)bh * a.cap + r0 + r4 + i) * kD + c8) = v[t][i];
        }
    }
    if (a.lse2_c && threadIdx.x < 64) {
        int p = -1;
        size_t so = 0;
        const long long off = row_offset(r0 + (int)threadIdx.x, &p, &so);
        const size_t o = (size_t)bh * a.cap + r0 + threadIdx.x;
        a.lse2_c[o] = off >= 0 ? a.lse[so] * kLog2e : 0.f;
        a.delta_c[o] = off >= 0 ? -a.delta[so] : 0.f;  // stored negated: dP accumulators start from it
        a.pos_c[o] = off >= 0 ? p : -1;
    }
    __syncthreads();

    // ---- token-minor copy.  A group of 16 lanes transposes 4 rows x 16 channels at a time; two
    // such reads (rows R..R+3 and R+8..R+11) are one 16-byte chunk of a channel's row.
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, gi = lane >> 4;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        if (!a.x[t] || !a.xt[t]) continue;
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const int combo = (wave * 4 + tt) * 4 + gi;
            const int cb = combo >> 3, lc = combo & 7;   // 16-channel block, chunk of the 64-token row
            const int grp = lc >> 1, hh = lc & 1;
            const int R = 16 * grp + 4 * hh;
            const __bf16* p1 = &lds[t][(R + (j >> 2)) * kRowPad + cb * 16 + 4 * (j & 3)];
            const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (s16x4 __attribute__((address_space(3)))*)(__attribute__((address_space(3))) const void*)p1);
            const s16x4 v2 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (s16x4 __attribute__((address_space(3)))*)(__attribute__((address_space(3))) const void*)(p1 + 8 * kRowPad));
            const s16x8 v = __builtin_shufflevector(v1, v2, 0, 1, 2, 3, 4, 5, 6, 7);
            __bf16* dst = a.xt[t] + ((size_t)bh * kD + cb * 16 + j) * a.cap + r0 + 16 * grp + 8 * hh;
            *reinterpret_cast<s16x8*>(dst) = v;
        }
    }
}

// O = S + A on the rows of a set (Sec. 3.2 Eq. 5), for the forward that runs both branches in one
// launch: O holds S, A the Global branch's rows in fp32, so that the sum is rounded once.  Sixteen
// lanes per row, sixteen rows per workgroup.
__global__ __launch_bounds__(kThreads) void merge_rows_kernel(Geom gm, RowSet rs, const float* __restrict__ A,
                                                              __bf16* __restrict__ O) {
    const int bh = blockIdx.y, b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    const int r = blockIdx.x * (kThreads / 16) + (threadIdx.x >> 4);
    if (r >= rows_total(rs, gm, bh)) return;
    const int code = row_code(rs, gm, bh, r);
    const int p = code / gm.G;
    const int head = hk * gm.G + (code - p * gm.G);
    const size_t off = (((size_t)b * gm.T + p) * gm.Hq + head) * kD + (threadIdx.x & 15) * 8;
    const f32x8 x = *reinterpret_cast<const f32x8*>(A + off);
    const bf16x8 y = *reinterpret_cast<const bf16x8*>(O + off);
    *reinterpret_cast<bf16x8*>(O + off) = __builtin_convertvector(x + __builtin_convertvector(y, f32x8), bf16x8);
}

}  // namespace

// rows = tokens of each KV head: x[i] [B,T,Hkv,128] -> xt[i] [B*Hkv][128][cap], cap = round_up(T, 64)
int pack_kv(const Geom& g, int n, const void* const* x, void* const* xt, int cap, const Fill* fills, int nfills,
            const RoutedFlags* flags, hipStream_t st) {
    if (n < 1 || n > 2 || nfills < 0 || nfills > 3) return L2A_ERR_UNSUPPORTED;
    PackArgs a{};
    a.gm = g;
    a.rs = RowSet{nullptr, nullptr, nullptr, 0};
    a.kv_rows = 1;
    for (int i = 0; i < n; ++i) {
        a.x[i] = (const __bf16*)x[i];
        a.xt[i] = (__bf16*)xt[i];
    }
    for (int i = 0; i < nfills; ++i) a.fill[i] = fills[i];
    a.cap = cap;
    if (flags) a.routed = *flags;
    KernelTimer kt("pack_kv", st);
    hipLaunchKernelGGL(pack_token_minor_kernel, dim3(cap / 64, g.B * g.Hkv), dim3(kThreads), 0, st, a);
    return launch_status();
}

// rows of a branch: Q and dO -> compact row-major copies + per-row statistics
int pack_rows(const Geom& g, const RowSet& rs, const void* q, const void* dO, const float* lse, const float* delta,
              void* qc, void* gc, float* lse2_c, float* delta_c, int32_t* pos_c, int cap, hipStream_t st) {
    PackArgs a{};
    a.gm = g;
    a.rs = rs;
    a.kv_rows = 0;
    a.x[0] = (const __bf16*)q;
    a.x[1] = (const __bf16*)dO;
    a.xc[0] = (__bf16*)qc;
    a.xc[1] = (__bf16*)gc;
    a.lse = lse;
    a.delta = delta;
    a.lse2_c = lse2_c;
    a.delta_c = delta_c;
    a.pos_c = pos_c;
    a.cap = cap;
    KernelTimer kt(rs.local ? "pack_rows_local" : "pack_rows_global", st);
    hipLaunchKernelGGL(pack_token_minor_kernel, dim3(cap / 64, g.B * g.Hkv), dim3(kThreads), 0, st, a);
    return launch_status();
}

int merge_rows(const Geom& g, const RowSet& rs, const float* A, void* O, hipStream_t st) {
    if (g.D != kD) return L2A_ERR_UNSUPPORTED;
    const long long rows = (long long)g.T * g.G;
    KernelTimer kt("merge_rows", st);
    hipLaunchKernelGGL(merge_rows_kernel, dim3((unsigned)((rows + kThreads / 16 - 1) / (kThreads / 16)), g.B * g.Hkv),
                       dim3(kThreads), 0, st, g, rs, A, (__bf16*)O);
    return launch_status();
}

}  // namespace l2a
