// Forward attention kernel, bf16 on the matrix cores (gfx950), for both branches of the layer:
//   GLOBAL rows = compacted routed (position, head-in-group) pairs, keys 0..pos
//          (App. C Alg. 1: tiles of Q_c, causal mask with the original positions Q_idx, K/V tiles
//          beyond the tile's largest position skipped), or all rows in the dense mode;
//   LOCAL  rows = all (position, head) pairs, keys pos-W..pos (Sec. 2 sliding-window mask).
// The epilogue writes the log-sum-exp and merges into O (Sec. 3.1 Eq. 5), so the scatter of
// Alg. 1's last step costs no extra pass.
//
// Layers whose branches share q, k, v take every row once while the window spans the sequence (kWhole, fwd_whole_kernel).
//
// Work decomposition.  One workgroup = 8 wavefronts of 32 rows = a tile of 256 consecutive rows of
// one (batch, KV head); the rows of the G query heads of the group are interleaved, so every row of
// a tile reads the same K/V.  K and the token-minor copy of V are streamed through LDS in blocks
// of 64 keys by direct global->LDS loads (three and two buffers, one barrier per block).  With 32 rows
// a wavefront needs 256 registers, so two share a SIMD (measured 2-5 % faster than 4 wavefronts of 64
// rows at 500 registers).  Short sequences (half_tiles) have workgroups of 4
// wavefronts and 128 rows, half a tile each, and both branches in one launch.
//
// Everything is computed transposed so that a lane owns a query row:
//   S^T[key, row]  = K Q^T     A = K block (LDS), B = Q (registers, loaded once)
//   O^T[ch,  row] += V^T P^T   A = V block (LDS, token-minor), B = P^T = the S^T accumulators
// A lane holds 32 scores of one row per block (the lane 32 apart holds the other 32): row max
// and row sum are in-register reductions plus one cross-lane exchange, and rescaling O is a
// per-lane scalar.
//
// Software pipeline (per wavefront and half-block of 32 keys: 16 matrix-core instructions per 32 rows,
// issued as numbered slots): while half-block j's scores go through the softmax on the VALU, the
// matrix cores first compute half-block j+1's scores and then accumulate P_j V_j (in the order the
// softmax finishes the 16-key groups).  LDS operand reads run a few slots ahead.
#include "tiles.hpp"

namespace l2a {
namespace {

constexpr int kBK = 64;  // keys per block
constexpr int kFwdNW = 8;  // wavefronts of 32 rows: two per SIMD, so that one's softmax can overlap the other's matrix instructions
constexpr int kBQ = 256;                // rows of a tile
constexpr int kAhead = 2;  // operand look-ahead, in operands (each feeds two instructions)

#define L2A_FENCE() __builtin_amdgcn_sched_barrier(0)

struct FwdArgs {
    Geom gm;
    RowSet rs;
    const __bf16* q;
    const __bf16* k;
    const __bf16* v;   // V as given (running_max_body only)
    const __bf16* vt;  // token-minor copy of V: [B*Hkv][128][vt_cap]
    int vt_cap;
    int32_t* redo;  // [B*Hkv][redo_stride]: set to 1 for a tile of 256 rows that was left to running_max_body (for diagnosis only)
    int redo_stride;
    FwdOut out;
    // kWhole: `out` is where a goes (main_out: o); s and its log-sum-exp
    __bf16* s_out = nullptr;
    float* s_lse = nullptr;
    const unsigned char* routed = nullptr;  // kWhole: [B*Hkv][T*G], by row code
};

template <int V>
using Int = std::integral_constant<int, V>;

// What a workgroup computes for its rows.  kWhole: all rows of a layer whose branches share their inputs while the window
// spans the sequence: s = a, and which rows are routed only matters to what is written.  (A shorter window is computed for each
// branch: in one walk over the window and then the keys before it s and a share the roundings of the window's weights,
// which their sum does not average out -- error of O against 64 bits at 32768 tokens 1.2 % larger -- and s of a token would
// depend, in its last bits, on which other tokens are routed.)
enum Kind { kGlobal, kLocal, kWhole };

// Which tile of which (b, KV head) a workgroup takes; (bx, by) of (gx, nbh): its index in its branch's part of the grid (a
// launch may carry both branches).
//
// Workgroups are dispatched in the order of their linear index and dealt round-robin to the 8 XCDs
// (the grid's width is a multiple of 8).  Global rows: longest prefixes first; every tile starts
// at key block 0, so the tiles resident on an XCD read the same K/V blocks at about the same time
// whatever their order.  While the K and V of all heads together about fit the last-level cache, the
// order runs over all (b, KV head) together (rotated, so that no XCD is tied to one head) -- with
// a few hundred tiles in all, a head whose long tiles started last would set the kernel's time;
// beyond that the heads go one after the other, so that the chip streams one head's K and V at a time.
// Local rows: each XCD takes a contiguous range of a head's tiles, so that the tiles resident on it
// have overlapping windows and share their K/V blocks through its L2 -- when the sequence is
// several windows long, so that the ranges cost the same; otherwise the tiles' costs grow with
// their position like the Global ones' and they are ordered the same way.
struct Tile {
    int bh, tile, n_rows;
};
__device__ __forceinline__ bool windows_by_range(const Geom& gm) { return gm.T / 4 > gm.W; }
__device__ __forceinline__ void head_and_rank(const Geom& gm, int bx, int by, int gx, int nbh, int& bh, int& rank) {
    if ((long long)nbh * gm.T <= kAllHeadsMaxTokens) {
        const int lin = by * gx + bx;
        rank = lin / nbh;
        bh = (lin - rank * nbh + rank) % nbh;
    } else {
        bh = by;
        rank = bx;
    }
}
template <int BQ>
__device__ __forceinline__ Tile tile_of(const Geom& gm, const RowSet& rs, bool windows, int bx, int by, int gx, int nbh) {
    Tile t;
    int rank;
    if (windows && windows_by_range(gm)) {
        t.bh = by;
        t.n_rows = rows_total(rs, gm, t.bh);
        const int n = (t.n_rows + BQ - 1) / BQ, x = bx & 7, j = bx >> 3;
        t.tile = j < n / 8 + (x < (n & 7) ? 1 : 0) ? x * (n / 8) + min(x, n & 7) + j : -1;
        return t;
    }
    head_and_rank(gm, bx, by, gx, nbh, t.bh, rank);
    t.n_rows = rows_total(rs, gm, t.bh);
    t.tile = (t.n_rows + BQ - 1) / BQ - 1 - rank;
    return t;
}

// The same tile by the classical streaming softmax with a running maximum and rescaling (App. C Alg. 1 as printed, with the
// rescaling factor read as exp(m_old - m_new)): for tiles the pipeline below gives up on, because a score exceeded
// a row's fixed reference by so much that a sum left the safe range.  V is transposed on its way into LDS.  A launch of its own
// for such tiles cost 3 to 5 us per branch where there were none.  Inside the pipeline's kernels it takes the registers that they
// have, and 14 to 36 of a kernel's are spilled (3 to 5 without it): in the prologue and in this walk, none in the pipeline's loops.
// Whole forward, us, launch of its own / inside: dense 1001 tokens 82.1 / 72.4, 32768 tokens 8298 / 8263, routed rows alone 32768
// tokens 1447 / 1441, windows alone 32768 tokens 1805 / 1781, 60000 tokens with W = 1024 1140 / 1113, separate modules 32768 tokens
// 3233 / 3202.
struct FwdLds {
    __bf16 k[3][kBK * 128];
    __bf16 v[2][kD * kBK];
};
// kWhole: four channels x of s, which is a where the row is routed; the row's log-sum-exp
__device__ __forceinline__ void store_whole(const FwdArgs& a, size_t off, const f32x4& x, bool routed) {
    const bf16x4 y = __builtin_convertvector(x, bf16x4), z = {(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
    if (a.s_out) *reinterpret_cast<bf16x4*>(a.s_out + off) = y;
    if (a.out.copy_out) *reinterpret_cast<bf16x4*>((__bf16*)a.out.copy_out + off) = routed ? y : z;
    const f32x4 both = __builtin_convertvector(y, f32x4) + x;
    *reinterpret_cast<bf16x4*>((__bf16*)a.out.main_out + off) = routed ? __builtin_convertvector(both, bf16x4) : y;
}
__device__ __forceinline__ void store_whole_lse(const FwdArgs& a, size_t so, float lse, bool routed) {
    a.s_lse[so] = lse;
    a.out.lse_out[so] = routed ? lse : -INFINITY;
}

template <bool LOCAL, int NW>
__device__ __forceinline__ void running_max_body(const FwdArgs& a, const Tile t, FwdLds& lds, bool whole) {
    const FwdOut& out = a.out;
    constexpr int RW = 32, BQ = NW * RW;
    typedef __bf16 K2[2][kTileRows * kRowPad];
    typedef __bf16 V2[2][kD * kColPad];
    static_assert(sizeof(K2) + sizeof(V2) <= sizeof(FwdLds), "both fit the pipeline's buffers");
    K2& lds_k = *reinterpret_cast<K2*>(&lds);
    V2& lds_v = *reinterpret_cast<V2*>(reinterpret_cast<char*>(&lds) + sizeof(K2));
    const Geom& gm = a.gm;
    const int bh = t.bh, tile = t.tile, n_rows = t.n_rows;
    const int b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    __syncthreads();  // the buffers are free

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 31, h = lane >> 5;

    // ---- rows of this workgroup / wavefront / lane
    const int wg_r0 = tile * BQ;
    const int wg_r1 = min(wg_r0 + BQ, n_rows);  // exclusive
    const int wg_pmin = row_code(a.rs, gm, bh, wg_r0) / gm.G;
    const int wg_pmax = row_code(a.rs, gm, bh, wg_r1 - 1) / gm.G;
    const int wv_r0 = wg_r0 + wave * RW;
    const bool wave_active = wv_r0 < n_rows;
    const int wv_r1 = min(wv_r0 + RW, n_rows);
    int wv_pmin = 0, wv_pmax = 0;
    if (wave_active) {
        wv_pmin = row_code(a.rs, gm, bh, wv_r0) / gm.G;
        wv_pmax = row_code(a.rs, gm, bh, wv_r1 - 1) / gm.G;
    }

    const bool valid = wv_r0 + n < n_rows;
    // rows past the end repeat the last row: computed, never written
    const int code = row_code(a.rs, gm, bh, min(wv_r0 + n, n_rows - 1));
    const int pos = code / gm.G, head = hk * gm.G + (code - pos * gm.G);
    bf16x8 qreg[8];
    const __bf16* qp = a.q + (((size_t)b * gm.T + pos) * gm.Hq + head) * kD + 8 * h;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);

    // ---- K/V block range of the workgroup
    const int jb0 = LOCAL ? max(wg_pmin - gm.W, 0) / kBK : 0;
    const int jb1 = wg_pmax / kBK;  // inclusive

    const size_t kv_row = (size_t)gm.Hkv * kD;
    const __bf16* kbase = a.k + ((size_t)b * gm.T * gm.Hkv + hk) * kD;
    const __bf16* vbase = a.v + ((size_t)b * gm.T * gm.Hkv + hk) * kD;
    const int r4 = (threadIdx.x >> 4) * 4;
    TileRegs kr, vr;
    const bool loads = threadIdx.x < kThreads;  // 256 threads stage a tile
    auto load_block = [&](int jb) {
        if (!loads) return;
        const int k0 = jb * kBK + r4;
        // keys past the end of the sequence are clamped: always masked, never out of bounds
        tile_load(kr, [&](int i) { return kbase + (size_t)min(k0 + i, gm.T - 1) * kv_row; });
        tile_load(vr, [&](int i) { return vbase + (size_t)min(k0 + i, gm.T - 1) * kv_row; });
    };
    auto store_block = [&](int buf) {
        if (!loads) return;
        tile_store_rowmajor(kr, lds_k[buf]);
        tile_store_transposed(vr, lds_v[buf]);
    };

    f32x16 oacc[4];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] = 0.f;

    load_block(jb0);
    store_block(0);
    __syncthreads();

    for (int jb = jb0; jb <= jb1; ++jb) {
        const int cur = (jb - jb0) & 1;
        if (jb < jb1) load_block(jb + 1);

        const int k0 = jb * kBK;
        bool skip = !wave_active || k0 > wv_pmax;
        if (LOCAL) skip = skip || (k0 + kBK - 1 < wv_pmin - gm.W);
        if (!skip) {
            bool need_mask = k0 + kBK - 1 > wv_pmin;
            if (LOCAL) need_mask = need_mask || (k0 < wv_pmax - gm.W);
            const __bf16* ks_ = lds_k[cur];
            const __bf16* vs_ = lds_v[cur];

            // S^T = K Q^T
            f32x16 s[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                const bf16x8 a0 = lds_rowmajor(ks_, n, ks, h);
                const bf16x8 a1 = lds_rowmajor(ks_, 32 + n, ks, h);
                s[0] = mfma32(a0, qreg[ks], s[0]);
                s[1] = mfma32(a1, qreg[ks], s[1]);
            }

            // streaming softmax, one row per lane
            bf16x8 pb[4];
            if (need_mask) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int key = k0 + kb * 32 + c_row(r, h);
                        bool ok = key <= pos;
                        if (LOCAL) ok = ok && (key >= pos - gm.W);
                        s[kb][r] = ok ? s[kb][r] : -INFINITY;
                    }
            }
            float mx = s[0][0];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            // A row may have seen only masked keys so far (sliding window): its running max is
            // then -inf and must not enter a subtraction.
            const float mnew = fmaxf(m, mx * gm.scale_log2);
            const bool grow = mnew > m;
            if (__any(grow)) {
                const float alpha = grow ? fast_exp2(m - mnew) : 1.f;
                l *= alpha;
#pragma unroll
                for (int d = 0; d < 4; ++d)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[d][r] *= alpha;
                m = mnew;
            }
            const float negm = (m == -INFINITY) ? 0.f : -m;
            float rsum = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float p = fast_exp2(fmaf(s[kb][r], gm.scale_log2, negm));
                    s[kb][r] = p;
                    rsum += p;
                }
            l += rsum;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                pb[kb * 2 + 0] = pack8(s[kb], 0);
                pb[kb * 2 + 1] = pack8(s[kb], 1);
            }

            // O^T += V^T P^T
#pragma unroll
            for (int step = 0; step < 4; ++step)
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const bf16x8 av = lds_transposed(vs_, d * 32 + n, step, h);
                    oacc[d] = mfma32(av, pb[step], oacc[d]);
                }
        }

        if (jb < jb1) store_block(cur ^ 1);
        __syncthreads();
    }

    // ---- epilogue: normalise, log-sum-exp, merge / scatter
    if (!wave_active) return;
    __bf16* mo = (__bf16*)out.main_out;
    __bf16* co = (__bf16*)out.copy_out;
    __bf16* zf = (__bf16*)out.zero_fill;
    const float lt = l + __shfl_xor(l, 32);
    if (!valid) return;
    const float inv = 1.f / lt;
    const size_t base = (((size_t)b * gm.T + pos) * gm.Hq + head) * kD + 4 * h;
    const bool routed = whole && a.routed[(size_t)bh * gm.T * gm.G + wv_r0 + n];
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            const size_t off = base + d * 32 + 8 * rg;
            f32x4 x = {oacc[d][4 * rg + 0] * inv, oacc[d][4 * rg + 1] * inv,
                       oacc[d][4 * rg + 2] * inv, oacc[d][4 * rg + 3] * inv};
            if (whole) {
                store_whole(a, off, x, routed);
                continue;
            }
            if (co) *reinterpret_cast<bf16x4*>(co + off) = __builtin_convertvector(x, bf16x4);
            if (out.merge) {
                const bf16x4 old = *reinterpret_cast<const bf16x4*>(mo + off);
                x += __builtin_convertvector(old, f32x4);
            }
            if (out.wide_out) *reinterpret_cast<f32x4*>(out.wide_out + off) = x;
            else *reinterpret_cast<bf16x4*>(mo + off) = __builtin_convertvector(x, bf16x4);
            if (zf) {
                const u32x2 z = {0u, 0u};
                *reinterpret_cast<u32x2*>(zf + off) = z;
            }
        }
    if (h == 0) {
        const size_t so = ((size_t)b * gm.Hq + head) * gm.T + pos;
        if (whole) {
            store_whole_lse(a, so, (m + __builtin_amdgcn_logf(lt)) * kLn2, routed);
            return;
        }
        out.lse_out[so] = (m + __builtin_amdgcn_logf(lt)) * kLn2;
        if (out.lse_fill) out.lse_fill[so] = -INFINITY;
    }
}

template <Kind KIND, int NW>
__device__ __forceinline__ void fwd_body(const FwdArgs& a, const Tile t, FwdLds& lds) {
    auto& lds_k = lds.k;
    auto& lds_v = lds.v;
    constexpr bool LOCAL = KIND == kLocal;
    constexpr int RW = 32;             // rows per wavefront
    constexpr int BQ = RW * NW;        // rows per workgroup: a tile, or a whole part of one
    static_assert(kBQ % BQ == 0, "a workgroup's rows lie in one tile");
    constexpr int NS = 16;             // slots (matrix instructions) per half-block: NS / 2 for S, NS / 2 for P V
    constexpr int NL = 16 / NW;        // 16-byte loads a wavefront issues per K or V block
    constexpr int kLoadSlot0 = NS - 1 - 2 * NL;  // the loads of later blocks go out in the last slots of a block's first half
    using Scores = f32x16;             // 32 keys x 32 rows

    const Geom& gm = a.gm;
    const int bh = t.bh, tile = t.tile, n_rows = t.n_rows;
    if (tile < 0) return;
    const int b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, h = lane >> 5;

    // ---- rows of this workgroup / wavefront / lane
    const int wg_r0 = tile * BQ;
    const int wg_r1 = min(wg_r0 + BQ, n_rows);  // exclusive
    const int wg_pmin = row_code(a.rs, gm, bh, wg_r0) / gm.G;
    const int wg_pmax = row_code(a.rs, gm, bh, wg_r1 - 1) / gm.G;
    const int wv_r0 = wg_r0 + wave * RW;
    const bool wave_active = wv_r0 < n_rows;

    const bool valid = wv_r0 + n < n_rows;
    // rows past the end repeat the last row: computed, never written
    const int code = row_code(a.rs, gm, bh, min(wv_r0 + n, n_rows - 1));
    const int pos = code / gm.G, head = hk * gm.G + (code - pos * gm.G);
    const bool routed = KIND == kWhole && a.routed[(size_t)bh * gm.T * gm.G + code] != 0;
    bf16x8 qreg[8];
    const __bf16* qp = a.q + (((size_t)b * gm.T + pos) * gm.Hq + head) * kD + 8 * h;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);

    // ---- block range of the workgroup, and its three runs: blocks that need the window-start
    // mask (LOCAL only), blocks no row of the tile needs a mask for, blocks on the causal diagonal.  Parts of a
    // tile start where the whole one would: a row's reference, and so its bits, are the same either way.
    const int pmin_all = BQ == kBQ ? wg_pmin : row_code(a.rs, gm, bh, wg_r0 / kBQ * kBQ) / gm.G;
    const int jb0 = LOCAL ? max(pmin_all - gm.W, 0) / kBK : 0;
    const int jb1 = wg_pmax / kBK;  // inclusive
    int j_mid = jb0;                // first block without window-start masking
    if (LOCAL) j_mid = min(jb1 + 1, max(jb0, (max(wg_pmax - gm.W, 0) + kBK - 1) / kBK));
    const int j_diag = max(j_mid, min(jb1 + 1, (wg_pmin + 1) / kBK));  // first block with a key > some row
    const int n_all = jb1 - jb0 + 1;

    // Loads: a wave-uniform base per block plus per-lane offsets fixed for the whole kernel.
    const unsigned kv_row_bytes = (unsigned)gm.Hkv * kD * 2;
    const char* kbase = (const char*)(a.k + ((size_t)b * gm.T * gm.Hkv + hk) * kD);
    const char* vtbase = (const char*)(a.vt + (size_t)bh * kD * a.vt_cap);
    const unsigned lds_k0 = lds_offset(&lds_k[0][0]), lds_v0 = lds_offset(&lds_v[0][0]);
    const RmDma<kBK, NW> k_off = rm_dma_setup<kBK, NW>(kv_row_bytes, wave);
    const TmDma<kBK, NW> v_off = tm_dma_setup<kBK, NW>((unsigned)a.vt_cap * 2u, wave);
    auto load_k = [&](int jb, int buf) __attribute__((always_inline)) {
        const char* src = kbase + (size_t)jb * kBK * kv_row_bytes;
        const unsigned dst = lds_k0 + buf * (kBK * 256);
        if ((jb + 1) * kBK <= gm.T) rm_dma_issue(k_off, src, dst, wave);
        else  // keys past the end of the sequence are clamped: always masked, never out of bounds
            rm_dma_issue_clamped<kBK, NW>(kv_row_bytes, gm.T - jb * kBK, src, dst, wave);
    };
    auto load_v = [&](int jb, int buf) __attribute__((always_inline)) {
        tm_dma_issue(v_off, vtbase + (size_t)jb * kBK * 2, lds_v0 + buf * (kD * kBK * 2), wave);
    };
    // In the main loop the 2 NL loads of a block are issued one at a time between matrix
    // instructions.  K rows are clamped to the end of the sequence on the fly (rows past it are always
    // masked), so that the ragged last block needs no code path of its own:
    // lane l of load i fetches chunk (l & 15) ^ (row & 15) of row (NW i + wave) * 4 + (l >> 4).
    const int k_lane_row = wave * 4 + (lane >> 4);
    const unsigned k_lane_chunk = (unsigned)(((lane & 15) ^ (k_lane_row & 15)) * 16);
    struct BlockLoads {
        const char* ksrc;
        const char* vsrc;
        unsigned kdst, vdst;
        int krows;  // rows of the K block that exist
    };
    auto issue_block_load = [&](const BlockLoads& L, auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i < NL) {
            const unsigned row = (unsigned)min(k_lane_row + 4 * NW * i, L.krows - 1);
            dma16_so(L.ksrc, __umul24(row, kv_row_bytes) + k_lane_chunk, L.kdst + (i * NW + wave) * 1024);
        } else {
            dma16_so(L.vsrc, v_off.voff[i - NL], L.vdst + ((i - NL) * NW + wave) * 1024);
        }
    };

    f32x16 oacc[4];
    float mref = -INFINITY, negm, l = 0.f;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] = 0.f;
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // keys of a score tile that starts at key k0 are k0 + c_row(r, h): those in reach have first <= c_row(r, 0) <= last
    auto last_row = [&](int k0) __attribute__((always_inline)) { return pos - k0 - 4 * h; };
    auto first_row = [&](int k0) __attribute__((always_inline)) { return pos - k0 - 4 * h - gm.W; };

    // One half-block (32 keys, half KB of block jb; keys k0 .. k0+31): exp of `cur` against the
    // row's fixed reference, overlapped with the scores of the next half-block into `nxt` (K rows
    // krow0.. of tile kt) and with O += P V for this half-block (tile vt).  16 matrix-core
    // instructions = 16 slots:
    //   first half of the slots   next half-block's scores | exp, row sum, pack P  (pair q in slot 3 q / 2)
    //   second half               O += P V
    auto half_block = [&](auto mask_tag, auto kb_tag, Scores& cur, Scores& nxt, const __bf16* kt, int krow0,
                          const __bf16* vt, int k0, auto&& side) __attribute__((always_inline)) {
        constexpr bool MASK = decltype(mask_tag)::value;
        constexpr int KB = decltype(kb_tag)::value;
        const float c2 = gm.scale_log2;
        bf16x8 opnd[16 + kAhead];
        uint32_t pw[2][4];  // P as packed bf16 pairs: [16-key group][dword]
        float rsum = 0.f;
        const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
        int last, first;
        if (MASK) last = last_row(k0), first = LOCAL ? first_row(k0) : 0;
        // operand o: o < 8 -> K rows of the next half-block (ks = o); else V^T (16-key group, channel block)
        auto read_operand = [&](auto oc) {
            constexpr int o = decltype(oc)::value;
            if constexpr (o < 8) opnd[o] = rm_operand(kt, krow0 + n, o, h);
            else if constexpr (o < 16) opnd[o] = tm_operand<kBK>(vt, ((o - 8) & 3) * 32 + n, 2 * KB + ((o - 8) >> 2), h);
        };
        auto issue = [&](auto mc) {
            constexpr int mm = decltype(mc)::value;
            if constexpr (mm < NS / 2) {
                nxt = mfma32(opnd[mm], qreg[mm], mm == 0 ? zero16 : nxt);
            } else {
                constexpr int x = mm - NS / 2, grp = x / 4, d = x & 3;
                const u32x4 pv = {pw[grp][0], pw[grp][1], pw[grp][2], pw[grp][3]};
                oacc[d] = mfma32(opnd[8 + x], __builtin_bit_cast(bf16x8, pv), oacc[d]);
            }
        };
        // exp of one pair of scores: pair q in 0 .. 7, in the order the P V product consumes them
        auto exp_pair = [&](auto qc) {
            constexpr int q = decltype(qc)::value;
            constexpr int grp = q / 4, i2 = (q & 3) * 2, r = grp * 8 + i2;
            float p0 = fast_exp2(fmaf(cur[r], c2, negm));
            float p1 = fast_exp2(fmaf(cur[r + 1], c2, negm));
            if (MASK) {
                constexpr int c0 = c_row(r, 0), c1 = c_row(r + 1, 0);
                p0 = c0 <= last && (!LOCAL || c0 >= first) ? p0 : 0.f;
                p1 = c1 <= last && (!LOCAL || c1 >= first) ? p1 : 0.f;
            }
            f32x2 f = {p0, p1};
            const bf16x2 pb = __builtin_convertvector(f, bf16x2);
            pw[grp][i2 >> 1] = __builtin_bit_cast(uint32_t, pb);
            // row sum of the weights as the matrix cores will see them (rounded to bf16): one
            // v_dot2 per pair, and the normalisation is exact for the weights actually used
            rsum = __builtin_amdgcn_fdot2_f32_bf16(pb, one2, rsum, false);
        };

        static_for<0, kAhead>([&](auto oc) { read_operand(oc); });
        L2A_FENCE();
        static_for<0, NS>([&](auto mc) {
            constexpr int mm = decltype(mc)::value;
            issue(mc);
            read_operand(Int<mm + kAhead>{});
            static_for<0, 8>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                if constexpr ((3 * q) / 2 == mm) exp_pair(qc);
            });
            side(mc);
            L2A_FENCE();
        });
        l += rsum;
    };

    // ---- prologue: K of the first two blocks, V of the first
    Scores Sa, Sb;
    load_k(jb0, 0);
    if (n_all > 1) load_k(jb0 + 1, 1);
    load_v(jb0, 0);
    dma_wait();
    __syncthreads();
    // Reference of every row's exponentials: the largest score among the row's own keys in the first two blocks (no masks where
    // the workgroup's rows see all of them), 0 where there is none.  It is never updated: scores that come
    // later may exceed it, which costs no accuracy in floating point; the epilogue checks that the
    // row sums stayed far from overflow and otherwise leaves the tile to running_max_body.  (Masks for every tile's two blocks took it to
    // 5200 cycles of a tile's 57000 at 1001 tokens.  Fewer keys, the first 32 or those that all rows of the tile see, would do,
    // but the weights next to a row's largest are rounded best -- error against 64 bits 1.2-1.6 % larger with 32 -- and a row
    // whose largest score is its window's first key would overflow.)
    {  // wavefronts whose rows all lie past the end compute on a repeated row and store nothing
        if ((jb0 + 2) * kBK - 1 <= wg_pmin && (!LOCAL || wg_pmax - gm.W <= jb0 * kBK)) {
#pragma unroll 1
            for (int at = 0; at < 2 * kBK; at += 32) {
                Scores S;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    const bf16x8 op = rm_operand(&lds_k[at / kBK][0], at % kBK + n, ks, h);
                    S = mfma32(op, qreg[ks], ks == 0 ? zero16 : S);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) mref = fmaxf(mref, S[r]);
            }
        } else {
            const int nb = jb0 < jb1 ? 2 : 1;
            for (int bi = 0; bi < nb; ++bi) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    Scores S;
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        const bf16x8 op = rm_operand(&lds_k[bi][0], kb * 32 + n, ks, h);
                        S = mfma32(op, qreg[ks], ks == 0 ? zero16 : S);
                    }
                    const int last = last_row((jb0 + bi) * kBK + kb * 32);
                    const int first = LOCAL ? first_row((jb0 + bi) * kBK + kb * 32) : 0;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const bool ok = c_row(r, 0) <= last && (!LOCAL || c_row(r, 0) >= first);
                        mref = fmaxf(mref, ok ? S[r] : -INFINITY);
                    }
                }
            }
        }
        mref = fmaxf(mref, __shfl_xor(mref, 32)) * gm.scale_log2;
        if (!(mref > -INFINITY)) mref = 0.f;  // no key in reach yet: any finite reference will do
        negm = -mref;
        // scores of the first half-block
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const bf16x8 op = rm_operand(&lds_k[0][0], n, ks, h);
            Sa = mfma32(op, qreg[ks], ks == 0 ? zero16 : Sa);
        }
    }

    // One block = two half-blocks; Sa holds the scores of a block's first half on entry and exit.
    // K blocks rotate through three buffers: block jb in kbuf, jb+1 in kbuf1, and the block loaded now, jb+2, in kbuf2
    int kbuf = 0, kbuf1 = 1, kbuf2 = 2;
    auto run = [&](auto mask_tag, int i_begin, int i_end) __attribute__((always_inline)) {
        for (int rel = i_begin; rel < i_end; ++rel) {
            const int jb = jb0 + rel;
            // prefetch: K of block jb+2 (its buffer held block jb-1), V of block jb+1 (held block jb-1),
            // issued in the slots of the first half-block where the VALU has nothing to do.  Past the
            // last block the last one is loaded again, into buffers nobody reads any more.
            const int jk = min(jb + 2, jb1), jv = min(jb + 1, jb1);
            BlockLoads L;
            auto stage = [&]() __attribute__((always_inline)) {
                L.ksrc = kbase + (size_t)jk * kBK * kv_row_bytes;
                L.vsrc = vtbase + (size_t)jv * kBK * 2;
                L.kdst = lds_k0 + kbuf2 * (kBK * 256);
                L.vdst = lds_v0 + ((rel + 1) & 1) * (kD * kBK * 2);
                L.krows = min(kBK, gm.T - jk * kBK);
            };
            // wavefronts whose rows all lie past the end compute on a repeated row and store nothing
            const __bf16* vt = &lds_v[rel & 1][0];
            half_block(mask_tag, Int<0>{}, Sa, Sb, &lds_k[kbuf][0], 32, vt, jb * kBK, [&](auto mc) {
                constexpr int mm = decltype(mc)::value;
                if constexpr (mm == kLoadSlot0 - 1) stage();
                if constexpr (mm >= kLoadSlot0 && mm < kLoadSlot0 + 2 * NL) issue_block_load(L, Int<mm - kLoadSlot0>{});
            });
            half_block(mask_tag, Int<1>{}, Sb, Sa, &lds_k[kbuf1][0], 0, vt, jb * kBK + 32, [](auto) {});
            dma_wait();
            __syncthreads();
            const int t = kbuf;
            kbuf = kbuf1, kbuf1 = kbuf2, kbuf2 = t;
        }
    };
    // ---- did every row sum stay in range, and every accumulator finite?  A row sum below 1e30 bounds the weights, not the
    // products with V: values beyond ~3e8 can still overflow an accumulator, so those are checked themselves
    // (x * 0 is NaN exactly when x is infinite or NaN).  A sum above 1e-30 (a reference of 0 may leave it small) still
    // holds every weight that counts beside it, none flushed to zero.
    float lt;
    bool bad = false;
    auto check_sums = [&]() __attribute__((always_inline)) {
        lt = l + __shfl_xor(l, 32);
        float chk = 0.f;
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) chk = fmaf(oacc[d][e], 0.f, chk);
        bad = bad || (wave_active && valid && !(lt > 1.0e-30f && lt < 1.0e30f && chk == 0.f));
    };
    auto row_base = [&]() __attribute__((always_inline)) { return (((size_t)b * gm.T + pos) * gm.Hq + head) * kD; };
    auto row_stat = [&]() __attribute__((always_inline)) { return ((size_t)b * gm.Hq + head) * gm.T + pos; };
    auto row_lse = [&]() __attribute__((always_inline)) { return (mref + __builtin_amdgcn_logf(lt)) * kLn2; };

    // runs of blocks: window-start masks (LOCAL), no masks, causal diagonal
    for (int seg = 0; seg < 3; ++seg) {
        const int i_begin = seg == 0 ? 0 : seg == 1 ? j_mid - jb0 : j_diag - jb0;
        const int i_end = seg == 0 ? j_mid - jb0 : seg == 1 ? j_diag - jb0 : n_all;
        if (seg == 1)
            run(std::false_type{}, i_begin, i_end);
        else
            run(std::true_type{}, i_begin, i_end);
    }

    // (workgroup-wide vote; LDS is free after the last barrier)
    check_sums();
    int* vote = reinterpret_cast<int*>(&lds_v[1][kD * kBK - 2]);
    if (threadIdx.x == 0) *vote = 0;
    __syncthreads();
    if (bad) *vote = 1;
    __syncthreads();
    if (*vote) {
        if (threadIdx.x == 0) a.redo[(size_t)bh * a.redo_stride + tile / (kBQ / BQ)] = 1;
        running_max_body<KIND == kLocal, NW>(a, t, lds, KIND == kWhole);
        return;
    }

    // ---- epilogue: normalise, log-sum-exp, merge / scatter
    if (!wave_active) return;
    if constexpr (KIND == kLocal || KIND == kWhole) {
        // Through LDS, where a lane's 8 bytes of its own row become 16 bytes of rows that sixteen lanes write whole: written
        // straight from the accumulators a store touched 32 rows, and a tile's outputs took 4700 to 9300 cycles.  A wavefront's
        // rows lie 272 bytes apart; behind a row's 256 bytes, where it goes (elements) and what it is (-1: nowhere, else routed).
        static_assert(NW * 32 * 272 < sizeof(FwdLds) - 16, "below the vote");
        char* const st = reinterpret_cast<char*>(&lds) + wave * (32 * 272);
        const float inv = 1.f / lt;
        auto put = [&](bool sum) __attribute__((always_inline)) {  // s, or o where it differs
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    f32x4 x = {oacc[d][4 * rg + 0] * inv, oacc[d][4 * rg + 1] * inv, oacc[d][4 * rg + 2] * inv,
                               oacc[d][4 * rg + 3] * inv};
                    bf16x4 y = __builtin_convertvector(x, bf16x4);
                    if (KIND == kWhole && sum && routed) y = __builtin_convertvector(x + __builtin_convertvector(y, f32x4), bf16x4);
                    *reinterpret_cast<bf16x4*>(st + n * 272 + d * 64 + rg * 16 + h * 8) = y;
                }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_wave_barrier();
        };
        if (h == 0) {
            *reinterpret_cast<size_t*>(st + n * 272 + 256) = row_base();
            *reinterpret_cast<int*>(st + n * 272 + 264) = valid ? (KIND == kWhole && routed ? 1 : 0) : -1;
        }
        auto rows_out = [&](auto f) __attribute__((always_inline)) {  // f(16 bytes, element offset, routed)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const char* row = st + (4 * i + (lane >> 4)) * 272;
                const u32x4 x = *reinterpret_cast<const u32x4*>(row + (lane & 15) * 16);
                const size_t off = *reinterpret_cast<const size_t*>(row + 256) + (lane & 15) * 8;
                const int what = *reinterpret_cast<const int*>(row + 264);
                if (what >= 0) f(x, off, what);
            }
        };
        __bf16* mo = (__bf16*)a.out.main_out;
        if constexpr (KIND == kWhole) {
            __bf16* ao = (__bf16*)a.out.copy_out;
            if (a.s_out || ao) {
                put(false);
                rows_out([&](const u32x4& x, size_t off, int r) __attribute__((always_inline)) {
                    if (a.s_out) *reinterpret_cast<u32x4*>(a.s_out + off) = x;
                    if (ao) *reinterpret_cast<u32x4*>(ao + off) = r ? x : u32x4{0u, 0u, 0u, 0u};
                });
            }
            put(true);
            rows_out([&](const u32x4& x, size_t off, int) __attribute__((always_inline)) { *reinterpret_cast<u32x4*>(mo + off) = x; });
            if (h == 0 && valid) store_whole_lse(a, row_stat(), row_lse(), routed);
        } else {
            __bf16 *co = (__bf16*)a.out.copy_out, *zf = (__bf16*)a.out.zero_fill;
            put(false);
            rows_out([&](const u32x4& x, size_t off, int) __attribute__((always_inline)) {
                *reinterpret_cast<u32x4*>(mo + off) = x;
                if (co) *reinterpret_cast<u32x4*>(co + off) = x;
                if (zf) *reinterpret_cast<u32x4*>(zf + off) = u32x4{0u, 0u, 0u, 0u};
            });
            if (h == 0 && valid) {
                a.out.lse_out[row_stat()] = row_lse();
                if (a.out.lse_fill) a.out.lse_fill[row_stat()] = -INFINITY;
            }
        }
        return;
    }
    __bf16* mo = (__bf16*)a.out.main_out;
    __bf16* co = (__bf16*)a.out.copy_out;
    __bf16* zf = (__bf16*)a.out.zero_fill;
    if (!valid) return;
    if (h == 0) {
        const size_t so = row_stat();
        a.out.lse_out[so] = row_lse();
        if (a.out.lse_fill) a.out.lse_fill[so] = -INFINITY;
    }
    const float inv = 1.f / lt;
    const size_t base = row_base() + 4 * h;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            const size_t off = base + d * 32 + 8 * rg;
            f32x4 x = {oacc[d][4 * rg + 0] * inv, oacc[d][4 * rg + 1] * inv,
                       oacc[d][4 * rg + 2] * inv, oacc[d][4 * rg + 3] * inv};
            if (co) *reinterpret_cast<bf16x4*>(co + off) = __builtin_convertvector(x, bf16x4);
            if (a.out.merge) {
                const bf16x4 old = *reinterpret_cast<const bf16x4*>(mo + off);
                x += __builtin_convertvector(old, f32x4);
            }
            if (a.out.wide_out) *reinterpret_cast<f32x4*>(a.out.wide_out + off) = x;
            else *reinterpret_cast<bf16x4*>(mo + off) = __builtin_convertvector(x, bf16x4);
            if (zf) {
                const u32x2 z = {0u, 0u};
                *reinterpret_cast<u32x2*>(zf + off) = z;
            }
        }
}

template <bool LOCAL, int NW>
__global__ __launch_bounds__(64 * NW) void fwd_kernel(FwdArgs a) {
    __shared__ __attribute__((aligned(1024))) FwdLds lds;
    const Tile t = tile_of<32 * NW>(a.gm, a.rs, LOCAL, (int)blockIdx.x, (int)blockIdx.y, (int)gridDim.x, (int)gridDim.y);
    fwd_body<LOCAL ? kLocal : kGlobal, NW>(a, t, lds);
}

// Shared inputs, the window spans the sequence: every row once, in identity order (no lists to wait for), no merge behind it.
// Whole forward, 20 % routed, 28 / 4 heads, the two branches in one launch and a merge / this, us: T = 600 35.3 / 29.0, T = 1001
// 42.3 / 33.4, T = 4096 172.8 / 138.5.
template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void fwd_whole_kernel(FwdArgs a) {
    __shared__ __attribute__((aligned(1024))) FwdLds lds;
    fwd_body<kWhole, NW>(a, tile_of<32 * NW>(a.gm, a.rs, false, (int)blockIdx.x, (int)blockIdx.y, (int)gridDim.x, (int)gridDim.y), lds);
}

// Both branches in one launch, for sequences so short that the Global rows' tiles alone leave most
// compute units idle: the first gx_global workgroups (per b, KV head) take the Global rows' tiles,
// the others the Local rows'.  The branches then must not depend on each other: the Global one
// writes its rows of A only (in fp32, besides the caller's bf16 copy), and O = S + A is formed
// afterwards (merge_rows) with the one rounding the sequential order has.
template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void fwd_pair_kernel(FwdArgs ag, FwdArgs al, int gx_global) {
    __shared__ __attribute__((aligned(1024))) FwdLds lds;
    constexpr int BQ = 32 * NW;
    if ((int)blockIdx.x < gx_global)
        fwd_body<kGlobal, NW>(ag, tile_of<BQ>(ag.gm, ag.rs, false, (int)blockIdx.x, (int)blockIdx.y, gx_global, (int)gridDim.y), lds);
    else
        fwd_body<kLocal, NW>(al, tile_of<BQ>(al.gm, al.rs, true, (int)blockIdx.x - gx_global, (int)blockIdx.y,
                                                  (int)gridDim.x - gx_global, (int)gridDim.y), lds);
}

// One launch for both branches: workgroups of 128 rows up to this many 256-row tiles of a branch.  The longest tile's
// walk sets the time of a short sequence, and half of it takes less; in longer ones every block of K and V
// passes through LDS twice as often for nothing.  Measured, whole forward, 256 / 128 rows, us (28 / 4 heads, W = 4096): T =
// 512 43.8 / 37.9, 1001 56.0 / 49.3, 2048 (224 tiles) 81.1 / 75.8, 4096 (448) 184.6 / 180.1, 8192 (896) 474.0 / 476.8, 16384
// 1192 / 1214; 32 / 8 heads, W = 1024: T = 4096 (512) 136.3 / 135.9, 16384 588 / 574.
bool half_tiles(size_t tiles) { return tiles <= 512; }

// tiles of 256 rows of a branch, per (b, KV head): a multiple of 8, see the tile order
unsigned tiles_x(const Geom& g) { return (unsigned)((((long long)g.T * g.G + kBQ - 1) / kBQ + 7) / 8 * 8); }

}  // namespace

int mfma_fwd(const Geom& g, const RowSet& rs, const void* q, const void* k, const void* v, const void* vt,
             int vt_cap, int32_t* redo, const FwdOut& out, hipStream_t st) {
    if (g.D != kD) return L2A_ERR_UNSUPPORTED;
    // per-lane load offsets are 32-bit
    if ((unsigned long long)vt_cap * 2ull * kD > 0xffffffffull) return L2A_ERR_UNSUPPORTED;
    FwdArgs a{g, rs, (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (const __bf16*)vt, vt_cap, redo,
              (int)tiles_x(g), out};
    const dim3 grid(tiles_x(g), g.B * g.Hkv);
    KernelTimer kt(rs.local ? "fwd_local" : "fwd_global", st);
    if (rs.local)
        hipLaunchKernelGGL((fwd_kernel<true, kFwdNW>), grid, dim3(64 * kFwdNW), 0, st, a);
    else
        hipLaunchKernelGGL((fwd_kernel<false, kFwdNW>), grid, dim3(64 * kFwdNW), 0, st, a);
    return launch_status();
}

// Both branches at once (fwd_pair_kernel): the Global branch's result goes to out_g.wide_out, and
// neither branch may write where the other does.  redo: 2 x mfma_fwd_redo_entries flags, set to zero.
int mfma_fwd_pair(const Geom& g, const RowSet& rs_l, const void* q_l, const void* k_l, const void* v_l,
                  const void* vt_l, const FwdOut& out_l, const RowSet& rs_g, const void* q_g, const void* k_g,
                  const void* v_g, const void* vt_g, const FwdOut& out_g, int vt_cap, int32_t* redo, hipStream_t st) {
    if (g.D != kD || out_g.merge || !out_g.wide_out || out_l.wide_out) return L2A_ERR_UNSUPPORTED;
    if ((unsigned long long)vt_cap * 2ull * kD > 0xffffffffull) return L2A_ERR_UNSUPPORTED;
    const unsigned gx = tiles_x(g);  // per branch
    const size_t entries = (size_t)gx * g.B * g.Hkv;
    FwdArgs al{g, rs_l, (const __bf16*)q_l, (const __bf16*)k_l, (const __bf16*)v_l, (const __bf16*)vt_l, vt_cap, redo, (int)gx, out_l};
    FwdArgs ag{g, rs_g, (const __bf16*)q_g, (const __bf16*)k_g, (const __bf16*)v_g, (const __bf16*)vt_g, vt_cap,
               redo + entries, (int)gx, out_g};
    {
        KernelTimer kt("fwd_pair", st);
        if (half_tiles(entries))
            hipLaunchKernelGGL((fwd_pair_kernel<4>), dim3(4 * gx, g.B * g.Hkv), dim3(256), 0, st, ag, al, (int)(2 * gx));
        else
            hipLaunchKernelGGL((fwd_pair_kernel<kFwdNW>), dim3(2 * gx, g.B * g.Hkv), dim3(64 * kFwdNW), 0, st, ag,
                               al, (int)gx);
    }
    return launch_status();
}

// Shared inputs while the window spans the sequence (fwd_whole_kernel): routed [B*Hkv][T*G] bytes by row code; out: a (main_out: o)
int mfma_fwd_whole(const Geom& g, const void* q, const void* k, const void* v, const void* vt, int vt_cap, int32_t* redo,
                   const unsigned char* routed, const FwdOut& out, void* S, float* lse_l, hipStream_t st) {
    if (g.D != kD || g.T > g.W + 1LL) return L2A_ERR_UNSUPPORTED;
    if ((unsigned long long)vt_cap * 2ull * kD > 0xffffffffull) return L2A_ERR_UNSUPPORTED;
    const unsigned gx = tiles_x(g);
    FwdArgs a{g, RowSet{nullptr, nullptr, nullptr, 0}, (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (const __bf16*)vt, vt_cap,
              redo, (int)gx, out, (__bf16*)S, lse_l, routed};
    KernelTimer kt("fwd_whole", st);
    if (half_tiles((size_t)gx * g.B * g.Hkv)) hipLaunchKernelGGL((fwd_whole_kernel<4>), dim3(2 * gx, g.B * g.Hkv), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((fwd_whole_kernel<8>), dim3(gx, g.B * g.Hkv), dim3(512), 0, st, a);
    return launch_status();
}

size_t mfma_fwd_redo_entries(const Geom& g) {
    return (size_t)tiles_x(g) * g.B * g.Hkv;
}

}  // namespace l2a
