// fp32 attention kernels on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 sums), head
// sizes 64 and 128, both branches of the layer, forward and backward (Secs. 3.1, 3.2; App. C Alg. 1).
//
// Matrix-core instruction: D[16x16] += A[16x4] B[4x16]; lane l, n = l & 15, k = l >> 4:
//   A: row n, contracted index k;  B: column n, contracted index k;  C/D register r: column n, row 4 k + r.
// The contraction only pairs slot k of A with slot k of B, so one 16-byte load per lane feeds four
// instructions wherever both operands agree on which index a slot stands for:
//   row layout     lane (n, k) holds channels 16 s + 4 k .. + 3 of row n: instruction m of load s contracts
//                  channels 16 s + 4 k + m (used for the scores and dP)
//   column layout  lane (n, k) holds channels 64 t + 4 n .. + 3 of row 4 k + r: instruction (r, m) contracts rows
//                  4 k + r -- the order in which a score tile's registers hold them, so that P and dS go
//                  from one product into the next without leaving their registers -- and its output row i is
//                  channel 64 t + 4 i + m
// Global memory is always read in the column layout, where sixteen adjacent lanes read 256 contiguous bytes; in the
// row layout adjacent lanes read different rows, and the cache served such a load one lane at a time (64 cycles
// instead of 16).  A tile that is needed in the row layout passes through its wavefront's LDS.
//
// What bounds them: the fp32 matrix rate, 157 TFLOP/s, and every vector instruction beside it -- unlike the bf16
// ones, these matrix instructions leave no room under them (microbenchmark, two wavefronts per SIMD: 13.7 ns
// alone, 19.0 with one vector instruction behind each, 24.1 with four).  So addresses are kept out of the loops and, in
// the forward and dQ, masks in code of their own (dK/dV tests every pair: a uniform branch there gained nothing).  With
// D = 128 the registers are all taken: 10 (dK/dV), 16 and 19 (forward and dQ, 32-row tiles) are spilled, 33, 20 and 23 where the
// branches share their inputs, none of them inside a matrix loop.  (dK/dV with its second computation inlined in the tile loop and a branch for each of the four stores
// of a row's data spilled 221, four of which came back from scratch on every row tile: 4096 tokens, Hq = 8, Hkv = 2, W =
// 1024, whole step 1174 us, now 1129; 3000 tokens, Hq = Hkv = 8, W = 256 942, now 870.)  A workgroup owns one small tile (16 or 32 query rows, 16 keys) and its NW
// wavefronts share the *other* axis, each with a partial result of its own, and these meet in LDS at the end:
// with 16-row tiles a sequence of a few thousand tokens gives a few hundred workgroups, and a serial walk of a
// whole prefix by one wavefront would set the kernel's time.
// Layers whose branches share q, k, v take both branches' forward in one launch, and dQ alike, the routed rows' keys in parts
// (Parts): the few routed tiles of a short sequence walked their prefixes alone on a tenth of the chip.  In dK and dV a routed row's
// window counts once for both branches (row_stats).  a and dQ do not take over the Local rows' sums: the errors of s and a are then
// one error twice, which their sum does not average out (O and dQ up to 3.4 and 2.6 % further from 64 bits at 4096 tokens).
// Training step, us, the branches one after the other / this: T = 2048, 1 head, D = 64, W = 256, 20 % routed 110.5 / 70.3 (forward
// 41 -> 23, dQ 48 -> 24); T = 3000, 1 head, D = 128, W = 1024, 5 % 290 / 148; T = 4096, Hq = 8, Hkv = 2, D = 128, W = 1024, 20 %
// 1134 / 1048 (forward 283 -> 267, dQ 363 -> 342, dK/dV 493 -> 439).
// Errors against 64 bits there, dK / dV: 7.7e-7 / 7.5e-7 -> 6.0e-7 / 5.2e-7 of the norm, because rows are walked downwards.
#include "attn_simple.hpp"


#include <algorithm>
#include <type_traits>

namespace l2a {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float sum_k(float x) {  // over the four lanes of a column
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}
__device__ __forceinline__ float max_k(float x) {
    x = fmaxf(x, __shfl_xor(x, 16));
    return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// Tiles a launch covers directly; beyond that its workgroups take several (keeps the grid within the limit of 2^32
// threads at every length), at most 2^27 / 2^20: a tile is 16 of fewer than 2^31 rows or keys.
constexpr long long kMaxTiles = 1 << 20;
constexpr int kMaxPerGroup = 128;

// code of the r-th row of one (b, KV head) (device data: clamped into the valid range)
__device__ __forceinline__ int row_code(const RowSet& rs, const Geom& gm, int bh, int r) {
    return rs.row_idx ? min(max(rs.row_idx[(size_t)bh * gm.T * gm.G + r], 0), gm.T * gm.G - 1) : r;
}

template <int D>
struct ColOperand {  // channels 64 t + 4 n .. + 3 of rows 4 k + r
    f32x4 x[4][D / 64];
    __device__ __forceinline__ void load(const float* const (&p)[4]) {  // p[r]: channel 4 n of row 4 k + r
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < D / 64; ++t) x[r][t] = ld4(p[r] + 64 * t);
    }
    __device__ __forceinline__ void load(const char* base, const unsigned (&off)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < D / 64; ++t) x[r][t] = *reinterpret_cast<const f32x4*>(base + off[r] + 256 * t);
    }
};
// Loads of 16 consecutive key rows: a wave-uniform base and per-lane 32-bit offsets fixed for the whole kernel,
// so that a load costs no vector instruction; the sequence's ragged last block, whose rows past the end repeat
// the last one (always masked), computes offsets of its own.
struct KeyRows {
    size_t row_bytes;
    int T;
    unsigned off[4];
    int n, k;
    __device__ __forceinline__ void init(int T_, size_t row_bytes_, int n_, int k_) {
        row_bytes = row_bytes_, T = T_, n = n_, k = k_;
#pragma unroll
        for (int r = 0; r < 4; ++r) off[r] = (unsigned)((4 * k + r) * row_bytes) + 16 * n;
    }
    template <int D>
    __device__ __forceinline__ void load(ColOperand<D>& o, const char* at, int k0) const {
        if (k0 + 16 <= T) {
            o.load(at + (size_t)k0 * row_bytes, off);
        } else {
            unsigned c[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) c[r] = (unsigned)(min(4 * k + r, T - 1 - k0) * row_bytes) + 16 * n;
            o.load(at + (size_t)k0 * row_bytes, c);
        }
    }
};
template <int D>
struct Acc {  // [channel, column]: register r of tile (t, m) is channel 64 t + 4 (4 k + r) + m of column n
    f32x4 x[D / 64][4];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int t = 0; t < D / 64; ++t)
#pragma unroll
            for (int m = 0; m < 4; ++m) x[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void scale(float a) {
#pragma unroll
        for (int t = 0; t < D / 64; ++t)
#pragma unroll
            for (int m = 0; m < 4; ++m) x[t][m] *= a;
    }
    // += op^T w, w[r] the weight of row 4 k + r in column n
    __device__ __forceinline__ void add(const ColOperand<D>& op, const f32x4& w) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < D / 64; ++t)
#pragma unroll
                for (int m = 0; m < 4; ++m) x[t][m] = mfma16(op.x[r][t][m], w[r], x[t][m]);
    }
    // 0 exactly when every value is finite (x * 0 is NaN otherwise)
    __device__ __forceinline__ float check() const {
        float c = 0.f;
#pragma unroll
        for (int t = 0; t < D / 64; ++t)
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) c = fmaf(x[t][m][r], 0.f, c);
        return c;
    }
    // column n's channels to p[0 .. D)
    __device__ __forceinline__ void store(float* p, int k) const {
#pragma unroll
        for (int t = 0; t < D / 64; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<f32x4*>(p + 64 * t + 16 * k + 4 * r) = f32x4{x[t][0][r], x[t][1][r], x[t][2][r], x[t][3][r]};
    }
};

// The stationary operand of the scores (Q, dO of a row tile; K, V of a key tile) is the same for all wavefronts of
// a workgroup and lies in LDS; rows are D + 4 floats apart, which keeps the 16-byte reads of sixteen rows free
// of bank conflicts.  R rows, copied by all threads of the workgroup; row(r): global address of row r.
template <int D, int R, int NT, typename RowPtr>
__device__ __forceinline__ void stage_rows(float (*dst)[D + 4], RowPtr row) {
#pragma unroll
    for (int i = threadIdx.x; i < R * (D / 4); i += NT) {
        const int r = i / (D / 4), ch = (i - r * (D / 4)) * 4;
        *reinterpret_cast<f32x4*>(&dst[r][ch]) = ld4(row(r) + ch);
    }
}
// A wavefront's own 16-row tile on its way from the column layout to the row layout (one wavefront, whose LDS
// operations execute in order: no wait beyond the compiler's own, but nothing may move across).
template <int D>
__device__ __forceinline__ void put_tile(float (*t)[D + 4], const ColOperand<D>& c, int n, int k) {
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < D / 64; ++i) *reinterpret_cast<f32x4*>(&t[4 * k + r][64 * i + 4 * n]) = c.x[r][i];
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}
// c[b][row n of the tile, column n of block b of the staged rows] = sum over channels
template <int D, int RB>
__device__ __forceinline__ void dot_tile(const float (*t)[D + 4], const float (*st)[D + 4], int n, int k, f32x4 (&c)[RB]) {
#pragma unroll
    for (int b = 0; b < RB; ++b) c[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 16; ++s) {
        const f32x4 x = ld4(&t[n][16 * s + 4 * k]);
        f32x4 y[RB];
#pragma unroll
        for (int b = 0; b < RB; ++b) y[b] = ld4(&st[16 * b + n][16 * s + 4 * k]);
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int b = 0; b < RB; ++b) c[b] = mfma16(x[m], y[b][m], c[b]);
    }
}

// the rows of one workgroup's tile of 16 RB rows
struct TileRange {
    int r0, n_rows;   // first row, rows of the (b, KV head)
    int pmin, pmax;   // positions of the tile's first and last row
    int key0, nblk;   // first key (a multiple of 16) and number of 16-key blocks any of the rows can see
};
// part z of nz of the blocks: key0 and nblk are that part's
template <int RB>
__device__ __forceinline__ TileRange tile_range(const Geom& gm, const RowSet& rs, int bh, int tile, int n_rows, int z, int nz) {
    TileRange t;
    t.r0 = tile * 16 * RB;
    t.n_rows = n_rows;
    t.pmin = __builtin_amdgcn_readfirstlane(row_code(rs, gm, bh, t.r0) / gm.G);
    t.pmax = __builtin_amdgcn_readfirstlane(row_code(rs, gm, bh, min(t.r0 + 16 * RB, n_rows) - 1) / gm.G);
    const int first = (rs.local ? max(t.pmin - gm.W, 0) : 0) & ~15, all = max(t.pmax - first, 0) / 16 + 1;
    const int b0 = all * z / nz;
    t.key0 = first + 16 * b0;
    t.nblk = all * (z + 1) / nz - b0;
    return t;
}
// Routed rows beside the Local ones, in one launch: a tile's blocks are shared between nz workgroups, and what each finds goes
// to its rows' places in x ([bh][z][row of the list][D]) and s (forward [bh][z][row][2], dQ [bh][z][row]), which the combine
// kernels add up.
struct Parts {
    float *x, *s;
    int nz;
    int groups;  // the first `groups` workgroups of the grid take these tiles (nz each), the others the Local ones
};
// Which tile a workgroup starts with, how far the next one is, and which part it takes
struct Role {
    bool part;
    int it, step, z, nz;
};
template <bool PARTS>  // false: a launch of one set's tiles
__device__ __forceinline__ Role role_of(const Parts& p) {
    const int x = blockIdx.x;
    if (!PARTS) return Role{false, x, (int)gridDim.x, 0, 1};
    if (x < p.groups) return Role{true, x / p.nz, p.groups / p.nz, x % p.nz, p.nz};
    return Role{false, x - p.groups, (int)gridDim.x - p.groups, 0, 1};
}
__device__ __forceinline__ size_t part_row(const Geom& gm, const Role& ro, int bh, int r) {
    return ((size_t)bh * ro.nz + ro.z) * gm.T * gm.G + r;
}
// which of the keys k0 + 4 k + r (r = bit) the row whose last key is pos sees
__device__ __forceinline__ unsigned keys_seen(const Geom& gm, const RowSet& rs, int first_key, int pos) {
    unsigned ok = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (first_key + r <= pos && (!rs.local || first_key + r >= pos - gm.W)) ok |= 1u << r;
    return ok;
}
__device__ __forceinline__ float exp2_(float x) { return __builtin_amdgcn_exp2f(x); }

// ---------------------------------------------------------------------------------------
// Forward.  Workgroup = 16 RB rows, wavefront w takes the 16-key blocks w, w + NW, ... of the rows' keys with
// a streaming softmax of its own (Alg. 1, running maximum per row); the partials are merged in LDS.
// ---------------------------------------------------------------------------------------
template <int D, int RB, int NW, bool PARTS>
__global__ __launch_bounds__(64 * NW, 2) void fp32_fwd_kernel(Geom gm, RowSet rs_main, RowSet rs_parts, const float* __restrict__ q,
                                                              const float* __restrict__ k, const float* __restrict__ v,
                                                              FwdOut out, Parts parts) {
    constexpr int R = 16 * RB;
    // first the Q rows and the wavefronts' K tiles, then the partial results
    constexpr int kFirst = R + 16 * NW, kRows = kFirst > R * NW ? kFirst : R * NW;
    __shared__ __attribute__((aligned(16))) float lds[kRows][D + 4];
    float(*const sq)[D + 4] = lds;
    float(*const so)[R][D + 4] = reinterpret_cast<float(*)[R][D + 4]>(lds);
    __shared__ float sm[NW][R], sl[NW][R];
    const int bh = blockIdx.y, b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kq = lane >> 4;
    const Role ro = role_of<PARTS>(parts);
    const RowSet rs = ro.part ? rs_parts : rs_main;
    const int n_rows = num_rows(rs, gm, bh), n_tiles = (n_rows + R - 1) / R;
    const size_t kv_row = (size_t)gm.Hkv * D;
    const size_t kv0 = ((size_t)b * gm.T * gm.Hkv + hk) * D;
    const char* kbase = (const char*)(k + kv0);
    const char* vbase = (const char*)(v + kv0);
    KeyRows keys;
    keys.init(gm.T, kv_row * sizeof(float), n, kq);
    const float c2 = gm.scale_log2;

    for (int it = ro.it; it < n_tiles; it += ro.step) {  // longest prefixes first
        const TileRange tr = tile_range<RB>(gm, rs, bh, n_tiles - 1 - it, n_rows, ro.z, ro.nz);
        auto q_row = [&](int r) {  // rows past the end repeat the last one
            const int code = row_code(rs, gm, bh, min(tr.r0 + r, n_rows - 1)), p = code / gm.G;
            return q + (((size_t)b * gm.T + p) * gm.Hq + hk * gm.G + (code - p * gm.G)) * D;
        };
        stage_rows<D, R, 64 * NW>(sq, q_row);
        Acc<D> o[RB];
        int pos[RB];
        float m[RB], l[RB];
#pragma unroll
        for (int c = 0; c < RB; ++c) {
            pos[c] = row_code(rs, gm, bh, min(tr.r0 + 16 * c + n, n_rows - 1)) / gm.G;
            o[c].zero();
            m[c] = -INFINITY;
            l[c] = 0.f;
        }
        float(*const sk)[D + 4] = lds + R + 16 * wave;
        ColOperand<D> kc;
        const int k_last = tr.key0 + 16 * max(tr.nblk - 1, 0);  // past the last block it is loaded again, for nobody
        keys.load(kc, kbase, min(tr.key0 + 16 * wave, k_last));
        __syncthreads();
        for (int blk = wave; blk < tr.nblk; blk += NW) {
            const int k0 = tr.key0 + 16 * blk;
            ColOperand<D> vc;
            keys.load(vc, vbase, k0);
            put_tile<D>(sk, kc, n, kq);
            keys.load(kc, kbase, min(k0 + 16 * NW, k_last));  // this wavefront's next block
            __builtin_amdgcn_sched_barrier(0);
            f32x4 s[RB];
            dot_tile<D, RB>(sk, sq, n, kq, s);
            __builtin_amdgcn_sched_barrier(0);
            auto softmax = [&](auto mask_tag) __attribute__((always_inline)) {
                constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll
                for (int c = 0; c < RB; ++c) {
                    unsigned ok = 15u;
                    if (MASK) {
                        ok = keys_seen(gm, rs, k0 + 4 * kq, pos[c]);
#pragma unroll
                        for (int r = 0; r < 4; ++r) s[c][r] = (ok >> r) & 1u ? s[c][r] : -INFINITY;
                    }
                    const float mx = max_k(fmaxf(fmaxf(s[c][0], s[c][1]), fmaxf(s[c][2], s[c][3])));
                    if (__any(mx > m[c])) {
                        const float mnew = fmaxf(m[c], mx);
                        const float alpha = mnew > m[c] ? exp2_((m[c] - mnew) * c2) : 1.f;
                        l[c] *= alpha;
                        o[c].scale(alpha);
                        m[c] = mnew;
                    }
                    const float mref = m[c] == -INFINITY ? 0.f : m[c];  // nothing in reach so far
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        s[c][r] = exp2_((s[c][r] - mref) * c2);  // masked: exp2(-inf) = 0
                        if (MASK) s[c][r] = (ok >> r) & 1u ? s[c][r] : 0.f;
                    }
                    l[c] += (s[c][0] + s[c][1]) + (s[c][2] + s[c][3]);
                }
            };
            if (k0 + 15 > tr.pmin || (rs.local && k0 < tr.pmax - gm.W)) softmax(std::true_type{});
            else softmax(std::false_type{});
#pragma unroll
            for (int c = 0; c < RB; ++c) o[c].add(vc, s[c]);
        }
        // Keys a row does not see enter the products with weight 0; if one of them holds an infinity or a NaN
        // (or a sum overflowed), the whole tile is computed again without them.  The barrier also ends the use of Q.
        float chk = 0.f;
#pragma unroll
        for (int c = 0; c < RB; ++c) chk = fmaf(l[c], 0.f, chk + o[c].check());
        if (__syncthreads_or(chk != 0.f)) {
            const int r = tr.r0 + (int)(threadIdx.x >> 2), part = threadIdx.x & 3;
            if (threadIdx.x < 4 * R && !ro.part) {
                simple_fwd_row<float, D / 4>(gm, rs, q, k, v, out, bh, r, part);
            } else if (threadIdx.x < 4 * R && r < n_rows) {
                const Row row = get_row(rs, gm, bh, r);
                float m_, l_, acc[D / 4];
                simple_fwd_keys<float, D / 4>(gm, q, k, v, b, hk, (((size_t)b * gm.T + row.pos) * gm.Hq + hk * gm.G + row.g) * D + part * (D / 4),
                                              part, tr.key0, min(tr.key0 + 16 * tr.nblk - 1, row.pos), m_, l_, acc);
                const size_t at = part_row(gm, ro, bh, r);
                for (int i = 0; i < D / 4; ++i) parts.x[at * D + part * (D / 4) + i] = acc[i];
                if (part == 0) parts.s[2 * at] = m_ / gm.scale, parts.s[2 * at + 1] = l_;
            }
            continue;
        }
#pragma unroll
        for (int c = 0; c < RB; ++c) {
            o[c].store(&so[wave][16 * c + n][0], kq);
            const float lt = sum_k(l[c]);
            if (kq == 0) {
                sm[wave][16 * c + n] = m[c];
                sl[wave][16 * c + n] = lt;
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < R * (D / 4); i += 64 * NW) {
            const int row = i / (D / 4), ch = (i - row * (D / 4)) * 4;
            if (tr.r0 + row >= n_rows) break;
            float mm = -INFINITY, lt = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) mm = fmaxf(mm, sm[w][row]);
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float mw = sm[w][row];
                const float f = mw == -INFINITY ? 0.f : exp2_((mw - mm) * c2);
                lt += f * sl[w][row];
                x += f * ld4(&so[w][row][ch]);
            }
            if (ro.part) {
                const size_t at = part_row(gm, ro, bh, tr.r0 + row);
                *reinterpret_cast<f32x4*>(parts.x + at * D + ch) = x;
                if (ch == 0) parts.s[2 * at] = mm, parts.s[2 * at + 1] = lt;
                continue;
            }
            const int code = row_code(rs, gm, bh, tr.r0 + row), p = code / gm.G, h = hk * gm.G + (code - p * gm.G);
            const size_t off = (((size_t)b * gm.T + p) * gm.Hq + h) * D + ch;
            x *= 1.f / lt;
            float* mo = (float*)out.main_out + off;
            if (out.copy_out) *reinterpret_cast<f32x4*>((float*)out.copy_out + off) = x;
            *reinterpret_cast<f32x4*>(mo) = out.merge ? ld4(mo) + x : x;
            if (out.zero_fill) *reinterpret_cast<f32x4*>((float*)out.zero_fill + off) = f32x4{0.f, 0.f, 0.f, 0.f};
            if (ch == 0) {
                const size_t st = ((size_t)b * gm.Hq + h) * gm.T + p;
                out.lse_out[st] = fmaf(mm, gm.scale, logf(lt));
                if (out.lse_fill) out.lse_fill[st] = -INFINITY;
            }
        }
        __syncthreads();
    }
}

// a of the routed rows from their parts, and o = s + a (s lies in O).  nz = 0: the window spans the sequence, a = s.  D / 4 lanes
// per row.
template <int D>
__global__ __launch_bounds__(256) void fp32_fwd_combine_kernel(Geom gm, RowSet rs, Parts parts, const float* __restrict__ lse_l, FwdOut out) {
    const int bh = blockIdx.y, b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    const int n_rows = num_rows(rs, gm, bh), ch = (threadIdx.x % (D / 4)) * 4;
    for (int r = blockIdx.x * (1024 / D) + threadIdx.x / (D / 4); r < n_rows; r += gridDim.x * (1024 / D)) {
        const int code = row_code(rs, gm, bh, r), p = code / gm.G, h = hk * gm.G + (code - p * gm.G);
        const size_t off = (((size_t)b * gm.T + p) * gm.Hq + h) * D + ch, so = ((size_t)b * gm.Hq + h) * gm.T + p;
        const f32x4 sx = ld4((const float*)out.main_out + off);
        float top = -INFINITY, sum = 0.f;
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        for (int z = 0; z < parts.nz; ++z) {
            const size_t at = ((size_t)bh * parts.nz + z) * gm.T * gm.G + r;
            const float m = parts.s[2 * at], l = parts.s[2 * at + 1];
            const f32x4 px = ld4(parts.x + at * D + ch);
            if (!(l > 0.f || l != l)) continue;  // no key in reach there
            const float up = fmaxf(top, m), f0 = exp2_((top - up) * gm.scale_log2), f1 = exp2_((m - up) * gm.scale_log2);
            x = x * f0 + px * f1;
            sum = sum * f0 + l * f1;
            top = up;
        }
        x *= 1.f / sum;
        if (parts.nz == 0) x = sx;
        if (out.copy_out) *reinterpret_cast<f32x4*>((float*)out.copy_out + off) = x;
        *reinterpret_cast<f32x4*>((float*)out.main_out + off) = sx + x;
        if (ch == 0) out.lse_out[so] = parts.nz == 0 ? lse_l[so] : fmaf(top, gm.scale, logf(sum));
    }
}

// ---------------------------------------------------------------------------------------
// dQ.  Tiles and key split as in the forward; the exact delta = sum_j p dp replaces the one from the saved output.
// ---------------------------------------------------------------------------------------
template <int D, int RB, int NW, bool PARTS>
__global__ __launch_bounds__(64 * NW, 2) void fp32_bwd_dq_kernel(Geom gm, RowSet rs_main, RowSet rs_parts,
                                                                 const float* __restrict__ q,
                                                                 const float* __restrict__ k,
                                                                 const float* __restrict__ v,
                                                                 const float* __restrict__ dO,
                                                                 const float* __restrict__ lse_main,
                                                                 const float* __restrict__ lse_parts, float* delta_main,
                                                                 const float* __restrict__ delta_parts, float* dq, int accumulate,
                                                                 Parts parts) {
    constexpr int R = 16 * RB;
    // first the Q and dO rows and the wavefronts' K, V tiles, then the partial results
    constexpr int kFirst = 2 * R + 16 * NW, kRows = kFirst > R * NW ? kFirst : R * NW;
    __shared__ __attribute__((aligned(16))) float lds[kRows][D + 4];
    float(*const sq)[D + 4] = lds;
    float(*const sg)[D + 4] = lds + R;
    float(*const so)[R][D + 4] = reinterpret_cast<float(*)[R][D + 4]>(lds);
    __shared__ float sd[NW][R];
    const int bh = blockIdx.y, b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kq = lane >> 4;
    const Role ro = role_of<PARTS>(parts);
    const RowSet rs = ro.part ? rs_parts : rs_main;
    const float *lse = ro.part ? lse_parts : lse_main, *delta = ro.part ? delta_parts : delta_main;
    const int n_rows = num_rows(rs, gm, bh), n_tiles = (n_rows + R - 1) / R;
    const size_t kv_row = (size_t)gm.Hkv * D;
    const size_t kv0 = ((size_t)b * gm.T * gm.Hkv + hk) * D;
    const char* kbase = (const char*)(k + kv0);
    const char* vbase = (const char*)(v + kv0);
    KeyRows keys;
    keys.init(gm.T, kv_row * sizeof(float), n, kq);

    for (int it = ro.it; it < n_tiles; it += ro.step) {
        const TileRange tr = tile_range<RB>(gm, rs, bh, n_tiles - 1 - it, n_rows, ro.z, ro.nz);
        auto row_at = [&](const float* base) {
            return [&, base](int r) {
                const int code = row_code(rs, gm, bh, min(tr.r0 + r, n_rows - 1)), p = code / gm.G;
                return base + (((size_t)b * gm.T + p) * gm.Hq + hk * gm.G + (code - p * gm.G)) * D;
            };
        };
        stage_rows<D, R, 64 * NW>(sq, row_at(q));
        stage_rows<D, R, 64 * NW>(sg, row_at(dO));
        Acc<D> acc[RB];
        int pos[RB];
        float L[RB], dl[RB], dx[RB];
#pragma unroll
        for (int c = 0; c < RB; ++c) {
            const int code = row_code(rs, gm, bh, min(tr.r0 + 16 * c + n, n_rows - 1));
            pos[c] = code / gm.G;
            const size_t st = ((size_t)b * gm.Hq + hk * gm.G + (code - pos[c] * gm.G)) * gm.T + pos[c];
            L[c] = lse[st];
            dl[c] = delta[st];
            dx[c] = 0.f;
            acc[c].zero();
        }
        float(*const st)[D + 4] = lds + 2 * R + 16 * wave;
        ColOperand<D> kn, vn;  // the next block's
        const int k_last = tr.key0 + 16 * max(tr.nblk - 1, 0);
        keys.load(kn, kbase, min(tr.key0 + 16 * wave, k_last));
        keys.load(vn, vbase, min(tr.key0 + 16 * wave, k_last));
        __syncthreads();
        for (int blk = wave; blk < tr.nblk; blk += NW) {
            const int k0 = tr.key0 + 16 * blk;
            const int next = min(k0 + 16 * NW, k_last);
            f32x4 s[RB], dp[RB];
            put_tile<D>(st, vn, n, kq);
            keys.load(vn, vbase, next);
            __builtin_amdgcn_sched_barrier(0);
            dot_tile<D, RB>(st, sg, n, kq, dp);
            __builtin_amdgcn_sched_barrier(0);
            const ColOperand<D> kc = kn;
            put_tile<D>(st, kc, n, kq);
            keys.load(kn, kbase, next);
            __builtin_amdgcn_sched_barrier(0);
            dot_tile<D, RB>(st, sq, n, kq, s);
            __builtin_amdgcn_sched_barrier(0);
            auto weights = [&](auto mask_tag) __attribute__((always_inline)) {
                constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll
                for (int c = 0; c < RB; ++c) {
                    const unsigned ok = MASK ? keys_seen(gm, rs, k0 + 4 * kq, pos[c]) : 15u;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool in = !MASK || ((ok >> r) & 1u);
                        // scale s - L first: a rounded product of scale and log2(e) would put its error times the score into it
                        const float p = exp2_(fmaf(s[c][r], gm.scale, -L[c]) * kLog2e);
                        dx[c] += in ? p * dp[c][r] : 0.f;
                        s[c][r] = in ? p * (dp[c][r] - dl[c]) : 0.f;  // dS
                    }
                }
            };
            if (k0 + 15 > tr.pmin || (rs.local && k0 < tr.pmax - gm.W)) weights(std::true_type{});
            else weights(std::false_type{});
#pragma unroll
            for (int c = 0; c < RB; ++c) acc[c].add(kc, s[c]);
        }
        float chk = 0.f;  // as in the forward
#pragma unroll
        for (int c = 0; c < RB; ++c) chk += acc[c].check();
        if (__syncthreads_or(chk != 0.f)) {
            const int r = tr.r0 + (int)(threadIdx.x >> 2), part = threadIdx.x & 3;
            if (threadIdx.x < 4 * R && !ro.part) {
                simple_dq_row<float, D / 4>(gm, rs, q, k, v, dO, lse, delta_main, dq, accumulate, bh, r, part);
            } else if (threadIdx.x < 4 * R && r < n_rows) {
                const Row row = get_row(rs, gm, bh, r);
                const int h = hk * gm.G + row.g;
                const size_t so = ((size_t)b * gm.Hq + h) * gm.T + row.pos;
                float dx_, acc_[D / 4];
                simple_dq_keys<float, D / 4>(gm, q, k, v, dO, b, hk, (((size_t)b * gm.T + row.pos) * gm.Hq + h) * D + part * (D / 4), part,
                                             tr.key0, min(tr.key0 + 16 * tr.nblk - 1, row.pos), lse[so], delta[so], dx_, acc_);
                const size_t at = part_row(gm, ro, bh, r);
                for (int i = 0; i < D / 4; ++i) parts.x[at * D + part * (D / 4) + i] = acc_[i];
                if (part == 0) parts.s[at] = dx_;
            }
            continue;
        }
#pragma unroll
        for (int c = 0; c < RB; ++c) {
            acc[c].store(&so[wave][16 * c + n][0], kq);
            const float d = sum_k(dx[c]);
            if (kq == 0) sd[wave][16 * c + n] = d;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < R * (D / 4); i += 64 * NW) {
            const int row = i / (D / 4), ch = (i - row * (D / 4)) * 4;
            if (tr.r0 + row >= n_rows) break;
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < NW; ++w) x += ld4(&so[w][row][ch]);
            const int code = row_code(rs, gm, bh, tr.r0 + row), p = code / gm.G, h = hk * gm.G + (code - p * gm.G);
            if (ro.part) {
                const size_t at = part_row(gm, ro, bh, tr.r0 + row);
                *reinterpret_cast<f32x4*>(parts.x + at * D + ch) = x;
                if (ch == 0) {
                    float d = 0.f;
#pragma unroll
                    for (int w = 0; w < NW; ++w) d += sd[w][row];
                    parts.s[at] = d;
                }
                continue;
            }
            float* dst = dq + (((size_t)b * gm.T + p) * gm.Hq + h) * D + ch;
            x *= gm.scale;
            *reinterpret_cast<f32x4*>(dst) = accumulate ? ld4(dst) + x : x;
            if (ch == 0) {
                float d = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) d += sd[w][row];
                delta_main[((size_t)b * gm.Hq + h) * gm.T + p] = d;
            }
        }
        __syncthreads();
    }
}

// dQ of the routed rows: their parts are added to the Local branch's.  nz = 0: the window spans the sequence, and what lies in dq is
// that of the row that the two branches make (row_stats), which counts 1 + a times.  Then the exact deltas: delta_g, and delta_l
// of the row that the branches make in the window, which the dK/dV kernel takes.
template <int D>
__global__ __launch_bounds__(256) void fp32_dq_combine_kernel(Geom gm, RowSet rs, Parts parts, const float* __restrict__ share,
                                                              float* delta_l, float* delta_g, float* dq) {
    const int bh = blockIdx.y, b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    const int n_rows = num_rows(rs, gm, bh), ch = (threadIdx.x % (D / 4)) * 4;
    for (int r = blockIdx.x * (1024 / D) + threadIdx.x / (D / 4); r < n_rows; r += gridDim.x * (1024 / D)) {
        const int code = row_code(rs, gm, bh, r), p = code / gm.G, h = hk * gm.G + (code - p * gm.G);
        const size_t off = (((size_t)b * gm.T + p) * gm.Hq + h) * D + ch, so = ((size_t)b * gm.Hq + h) * gm.T + p;
        const float a = share[so];
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
        float d = 0.f;
        for (int z = 0; z < parts.nz; ++z) {
            const size_t at = ((size_t)bh * parts.nz + z) * gm.T * gm.G + r;
            x += ld4(parts.x + at * D + ch);
            d += parts.s[at];
        }
        const f32x4 y = ld4(dq + off);
        *reinterpret_cast<f32x4*>(dq + off) = parts.nz ? y + x * gm.scale : y * (1.f + a);
        if (ch == 0) {
            const float dl = delta_l[so], dg = parts.nz ? d : a * dl;
            delta_g[so] = dg;
            delta_l[so] = (dl + a * dg) / (1.f + a);
        }
    }
}

// ---------------------------------------------------------------------------------------
// dK, dV.  Workgroup = 16 keys, wavefront w takes the 16-row tiles w, w + NW, ... of the rows that can see them.
// ---------------------------------------------------------------------------------------
template <int D, int NW, bool SHARE>
__global__ __launch_bounds__(64 * NW, 2) void fp32_bwd_dkdv_kernel(Geom gm, DkdvSets sets, const float* __restrict__ q,
                                                                   const float* __restrict__ k,
                                                                   const float* __restrict__ v,
                                                                   const float* __restrict__ dO, float* dk, float* dv) {
    // first the K and V rows and the wavefronts' row tiles, then the partial results
    constexpr int kFirst = 32 + 16 * NW, kRows = kFirst > 32 * NW ? kFirst : 32 * NW;
    __shared__ __attribute__((aligned(16))) float lds[kRows][D + 4];
    float(*const sk)[D + 4] = lds;
    float(*const sv)[D + 4] = lds + 16;
    float(*const so)[2][16][D + 4] = reinterpret_cast<float(*)[2][16][D + 4]>(lds);
    // of a wavefront's row tile: last key its row sees (-1: no row), row index within the batch, log-sum-exp, delta
    __shared__ __attribute__((aligned(16))) uint32_t row_data[NW][4][16];
    // log2 of what the row's weights count (1 + share); of this tile and the next: read where it is used, which costs
    // the matrix loop no registers
    __shared__ __attribute__((aligned(16))) float row_weight[NW][2][16];
    __shared__ uint32_t redo[kMaxPerGroup / 32];  // tiles of this workgroup to be computed again
    const int bh = blockIdx.y, b = bh / gm.Hkv, hk = bh - b * gm.Hkv;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kq = lane >> 4;
    float(*const st)[D + 4] = lds + 32 + 16 * wave;
    const int n_tiles = (gm.T + 15) / 16, nkb = (gm.T + 63) / 64;
    const float* qb = q + (size_t)b * gm.T * gm.Hq * D;
    const float* gb = dO + (size_t)b * gm.T * gm.Hq * D;

    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {  // key 0 is seen by the most rows
        const int k0 = tile * 16, key = k0 + n;
        auto key_row = [&](const float* base) {
            return [&, base](int r) { return base + (((size_t)b * gm.T + min(k0 + r, gm.T - 1)) * gm.Hkv + hk) * D; };
        };
        stage_rows<D, 16, 64 * NW>(sk, key_row(k));
        stage_rows<D, 16, 64 * NW>(sv, key_row(v));
        __syncthreads();
        Acc<D> ak, av;
        ak.zero();
        av.zero();
        // The rows that weigh most for a key are the first ones that see it, and an early large sum is what later small terms are
        // rounded against: so the last rows come first, and the keys-before-the-window rows before the Local ones.
        for (int s_i = sets.n - 1; s_i >= 0; --s_i) {
            const RowSet rs = sets.rs[s_i];
            const float* lse = sets.lse[s_i];
            const float* delta = sets.delta[s_i];
            const float* share = sets.share[s_i];
            int r0, r1;  // candidate rows [r0, r1)
            if (rs.local) {
                r0 = k0 * gm.G;
                r1 = (int)min((long long)k0 + 15 + gm.W, (long long)gm.T - 1) * gm.G + gm.G;
            } else {
                r0 = rs.kblk_first_row ? max(rs.kblk_first_row[(size_t)bh * (nkb + 1) + walk::list_bounds(k0, rs.shift, nkb).lo], 0) : k0 * gm.G;
                r1 = num_rows(rs, gm, bh);
            }
            const int rt0 = r0 + 16 * wave;
            if (rt0 >= r1) continue;
            int rt = rt0 + (r1 - 1 - rt0) / (16 * NW) * (16 * NW);
            // Of the next tile: position (-1: no row), row index within the batch and statistics of lane n's row,
            // passed through LDS to the lanes whose weights and operands are rows 4 kq + r (one wavefront, in order);
            // then those rows of dO and Q.
            typedef int i32x4 __attribute__((ext_vector_type(4)));
            i32x4 pr;
            f32x4 Lr, dr;
            int par = 0;
            ColOperand<D> gn, qn;
            int pos, idx;
            float L, dl, wt;
            auto fetch_row = [&](int t) __attribute__((always_inline)) {
                const int code = row_code(rs, gm, bh, max(min(t + n, r1 - 1), r0));
                pos = code / gm.G;
                const int h = hk * gm.G + (code - pos * gm.G);
                idx = pos * gm.Hq + h;
                const size_t so_ = ((size_t)b * gm.Hq + h) * gm.T + pos;
                L = lse[so_];
                dl = delta[so_];
                if (SHARE) wt = share ? __builtin_amdgcn_logf(1.f + share[so_]) : 0.f;
                pos = t + n >= r1 ? -1 : pos - rs.shift;  // the last key the row sees
            };
            i32x4 pn;
            f32x4 Ln, dn;
            auto fetch_tile = [&]() __attribute__((always_inline)) {
                __builtin_amdgcn_wave_barrier();
                // one store, each quarter of the wavefront its own of the four (a branch per quarter took a jump each)
                const uint32_t a = kq & 1 ? (uint32_t)idx : (uint32_t)pos;
                const uint32_t c = kq & 1 ? __builtin_bit_cast(uint32_t, dl) : __builtin_bit_cast(uint32_t, L);
                row_data[wave][kq][n] = kq & 2 ? c : a;
                if (SHARE) row_weight[wave][par][n] = wt;
                asm volatile("" ::: "memory");
                __builtin_amdgcn_wave_barrier();
                pn = *reinterpret_cast<const i32x4*>(&row_data[wave][0][4 * kq]);
                const i32x4 ir = *reinterpret_cast<const i32x4*>(&row_data[wave][1][4 * kq]);
                Ln = *reinterpret_cast<const f32x4*>(&row_data[wave][2][4 * kq]);
                dn = *reinterpret_cast<const f32x4*>(&row_data[wave][3][4 * kq]);
                asm volatile("" ::: "memory");
                __builtin_amdgcn_wave_barrier();
                const float *qrow[4], *grow[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    qrow[r] = qb + (size_t)ir[r] * D + 4 * n;
                    grow[r] = gb + (size_t)ir[r] * D + 4 * n;
                }
                gn.load(grow);
                qn.load(qrow);
            };
            fetch_row(rt);
            fetch_tile();
            fetch_row(rt - 16 * NW);
            for (; rt >= rt0; rt -= 16 * NW) {
                const ColOperand<D> gc = gn, qc = qn;
                pr = pn, Lr = Ln, dr = dn;
                f32x4 s[1], dp[1];
                put_tile<D>(st, gc, n, kq);
                dot_tile<D, 1>(st, sv, n, kq, dp);
                __builtin_amdgcn_sched_barrier(0);
                put_tile<D>(st, qc, n, kq);
                par ^= 1;
                fetch_tile();  // (past the first tile rows are fetched again, for nobody)
                fetch_row(rt - 32 * NW);
                __builtin_amdgcn_sched_barrier(0);
                dot_tile<D, 1>(st, sk, n, kq, s);
                __builtin_amdgcn_sched_barrier(0);
                f32x4 wr;
                if (SHARE) wr = ld4(&row_weight[wave][par ^ 1][4 * kq]);
                unsigned ok = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (key <= pr[r] && (!rs.local || key >= pr[r] - gm.W)) ok |= 1u << r;
                f32x4 p;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool in = (ok >> r) & 1u;
                    const float x = exp2_(SHARE ? fmaf(fmaf(s[0][r], gm.scale, -Lr[r]), kLog2e, wr[r])
                                                : fmaf(s[0][r], gm.scale, -Lr[r]) * kLog2e);
                    p[r] = in ? x : 0.f;
                    s[0][r] = in ? x * (dp[0][r] - dr[r]) : 0.f;  // dS
                }
                av.add(gc, p);
                ak.add(qc, s[0]);
            }
        }
        // As in the forward, for rows that do not see a key; but behind the loop, where the registers that the second
        // computation takes do not cost the first its own.
        const int turn = tile / (int)gridDim.x;
        const bool again = __syncthreads_or(ak.check() + av.check() != 0.f);
        if (threadIdx.x == 0 && (turn & 31) == 0) redo[turn >> 5] = 0;
        if (threadIdx.x == 0 && again) redo[turn >> 5] |= 1u << (turn & 31);
        if (again) continue;
        ak.store(&so[wave][0][n][0], kq);
        av.store(&so[wave][1][n][0], kq);
        __syncthreads();
        for (int i = threadIdx.x; i < 2 * 16 * (D / 4); i += 64 * NW) {
            const int which = i / (16 * (D / 4)), j = i - which * (16 * (D / 4));
            const int row = j / (D / 4), ch = (j - row * (D / 4)) * 4;
            if (k0 + row >= gm.T) continue;
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < NW; ++w) x += ld4(&so[w][which][row][ch]);
            if (which == 0) x *= gm.scale;
            *reinterpret_cast<f32x4*>((which ? dv : dk) + (((size_t)b * gm.T + k0 + row) * gm.Hkv + hk) * D + ch) = x;
        }
        __syncthreads();
    }
    __syncthreads();
    for (int tile = blockIdx.x, turn = 0; tile < n_tiles; tile += gridDim.x, ++turn)
        if ((redo[turn >> 5] >> (turn & 31) & 1u) && threadIdx.x < 64)
            simple_dkdv_key<float, D / 4>(gm, sets, q, k, v, dO, dk, dv, bh, tile * 16 + (threadIdx.x >> 2), threadIdx.x & 3);
}

inline dim3 tile_grid(long long tiles, const Geom& g) {
    return dim3((unsigned)(tiles < kMaxTiles ? tiles : kMaxTiles), g.B * g.Hkv);
}

const float* cf(const void* p) { return (const float*)p; }

// Tiles of 32 rows (an operand read once for two matrix instructions, two workgroups of 4 wavefronts per CU) or
// of 16 rows with the keys shared by 8 wavefronts; the second while the first would leave CUs idle or give each
// a single long walk.  How many rows are routed is device data; a routed set counts as a quarter of all rows.
// Measured, Hq = 8, Hkv = 2, D = 128, W = 1024, 20 % routed, us with 16 / 32 rows: Local rows forward T = 2048 (512
// tiles of 32) 92 / 98, T = 4096 198 / 183, T = 16384 847 / 693; Global rows T = 4096 100 / 205, T = 8192 333 / 598,
// T = 16384 (4096 tiles) 1204 / 1152; dQ alike.
bool wide_tiles(const Geom& g, const RowSet& rs) {
    const long long tiles = (long long)g.T * g.G / 32 * g.B * g.Hkv;
    return (rs.row_idx ? tiles / 4 : tiles) >= 1024;
}

// Workgroups that share a routed tile's keys.  Each part has a tile's first and last steps of its own, so that many of them cost
// most where many rows are routed, and few of them leave the longest tiles to themselves where few are.  Forward and dQ, the
// branches one after the other / this, 5 / 20 / 50 % routed, W = 256, by parts:
//   narrow tiles   1 head, D = 64, T = 2000    1: 1.13 / 1.12 / 1.13   3: 1.92 / 1.95 / 1.78   6: 2.12 / 1.90 / 1.57
//                  8 heads of their own K and V, D = 128, T = 2000     1: 1.08 / 0.93 / 1.07   2: 1.28 / 1.12 / 1.16   4: 1.35 / 1.06 / 0.99
//                  8 query, 2 KV heads, D = 128, T = 700               1: 1.46 / 1.41 / 1.21   2: 1.45 / 1.35 / 1.08
//                  ditto T = 2000      1: 1.23 / 1.15 / 0.99   2: 1.45 / 1.17 / 0.92   4: 1.39 / 1.05 / 0.78
//   wide tiles     ditto T = 4096      2: 1.15 / 0.82 / 1.04   4: 1.44 / 1.00 / 1.01   8: 1.40 / 0.92 / 0.87
//                  ditto T = 16384, W = 1024      2: 1.92 / 1.07 / 1.01   4: 1.93 / 1.06 / 1.00   8: 1.87 / 1.03 / 0.95
// Wide tiles, which are so for the Local rows' sake, take at least two: no wavefront's sums are then longer than in the routed
// set's own narrow ones.  None while the window spans the sequence and the tiles are narrow: the Local rows then hold the very
// bits that a has.
int routed_parts(const Geom& g) {
    const bool wide = wide_tiles(g, RowSet{nullptr, nullptr, nullptr, 1});
    if (g.T - 1 <= g.W && !wide) return 0;
    const long long tiles = (long long)g.T * g.G / 64 * g.B * g.Hkv;  // of 16 rows, a quarter of them routed
    if (wide) return (int)std::max(2LL, std::min(std::min((g.T + 512) / 1024LL, 4LL), 8192 / tiles));
    if (tiles <= 64) return std::min(std::max(g.T / 128, 1), 3);
    return g.G >= 4 && tiles >= 128 ? 1 : 2;
}
size_t round256(size_t n) { return (n + 255) / 256 * 256; }
size_t all_rows(const Geom& g) { return (size_t)g.B * g.Hkv * g.T * g.G; }
Parts place_parts(const Geom& g, char* ws) {
    Parts p{};
    p.nz = routed_parts(g);
    p.x = (float*)ws;
    p.s = (float*)(ws + round256(all_rows(g) * p.nz * g.D * sizeof(float)));
    return p;
}
size_t parts_bytes(const Geom& g, int stats) {  // stats: floats per row and part
    const int nz = routed_parts(g);
    return round256(all_rows(g) * nz * g.D * sizeof(float)) + round256(all_rows(g) * nz * stats * sizeof(float));
}
// The grid of tiles of 16 RB rows: those of the main set, behind parts.nz workgroups for each tile of the routed rows
dim3 role_grid(const Geom& g, int rows, Parts& parts) {
    const long long tiles = std::min(((long long)g.T * g.G + rows - 1) / rows, kMaxTiles / 16);
    parts.groups = (int)tiles * parts.nz;
    return dim3((unsigned)tiles + parts.groups, g.B * g.Hkv);
}

struct FwdCall {
    RowSet main, routed;
    const void *q, *k, *v;
    FwdOut out;
    Parts parts;
};
template <int D, int RB, int NW>
void launch_fwd(const Geom& g, FwdCall c, hipStream_t st) {
    const dim3 grid = role_grid(g, 16 * RB, c.parts);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(64 * NW), 0, st, g, c.main, c.routed, cf(c.q), cf(c.k), cf(c.v), c.out, c.parts); };
    c.parts.nz ? launch(fp32_fwd_kernel<D, RB, NW, true>) : launch(fp32_fwd_kernel<D, RB, NW, false>);
}
void run_fwd(const Geom& g, const FwdCall& c, bool wide, hipStream_t st) {
    if (g.D == 64) wide ? launch_fwd<64, 2, 4>(g, c, st) : launch_fwd<64, 1, 8>(g, c, st);
    else wide ? launch_fwd<128, 2, 4>(g, c, st) : launch_fwd<128, 1, 8>(g, c, st);
}
struct DqCall {
    RowSet main, routed;
    const void *q, *k, *v, *dO;
    const float *lse_main, *lse_parts;
    float *delta_main, *delta_parts;
    void* dq;
    int accumulate;
    Parts parts;
};
template <int D, int RB, int NW>
void launch_dq(const Geom& g, DqCall c, hipStream_t st) {
    const dim3 grid = role_grid(g, 16 * RB, c.parts);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(64 * NW), 0, st, g, c.main, c.routed, cf(c.q), cf(c.k), cf(c.v), cf(c.dO), c.lse_main, c.lse_parts,
                           c.delta_main, c.delta_parts, (float*)c.dq, c.accumulate, c.parts);
    };
    c.parts.nz ? launch(fp32_bwd_dq_kernel<D, RB, NW, true>) : launch(fp32_bwd_dq_kernel<D, RB, NW, false>);
}
void run_dq(const Geom& g, const DqCall& c, bool wide, hipStream_t st) {
    if (g.D == 64) wide ? launch_dq<64, 2, 4>(g, c, st) : launch_dq<64, 1, 8>(g, c, st);
    else wide ? launch_dq<128, 2, 4>(g, c, st) : launch_dq<128, 1, 8>(g, c, st);
}
dim3 row_grid(const Geom& g) {
    return dim3((unsigned)std::min(((long long)g.T * g.G * g.D + 1023) / 1024, 65536LL), g.B * g.Hkv);
}

}  // namespace

int fp32_fwd(const Geom& g, const RowSet& rs, const void* q, const void* k, const void* v, const FwdOut& out,
             hipStream_t st) {
    if (g.D != 64 && g.D != 128) return L2A_ERR_UNSUPPORTED;
    KernelTimer kt(rs.local ? "fp32_fwd_local" : "fp32_fwd_global", st);
    run_fwd(g, FwdCall{rs, rs, q, k, v, out, Parts{}}, wide_tiles(g, rs), st);
    return launch_status();
}

size_t fp32_fwd_shared_bytes(const Geom& g) { return parts_bytes(g, 2); }

int fp32_fwd_shared(const Geom& g, const RowSet& rs_l, const RowSet& rs_g, const void* q, const void* k, const void* v,
                    const FwdOut& out_l, const FwdOut& out_g, void* ws, hipStream_t st) {
    if (g.D != 64 && g.D != 128) return L2A_ERR_UNSUPPORTED;
    const Parts parts = place_parts(g, (char*)ws);
    {
        KernelTimer kt("fp32_fwd_shared", st);
        run_fwd(g, FwdCall{rs_l, rs_g, q, k, v, out_l, parts}, wide_tiles(g, rs_l), st);
    }
    KernelTimer kt("fp32_fwd_combine", st);
    if (g.D == 64) hipLaunchKernelGGL(fp32_fwd_combine_kernel<64>, row_grid(g), dim3(256), 0, st, g, rs_g, parts, (const float*)out_l.lse_out, out_g);
    else hipLaunchKernelGGL(fp32_fwd_combine_kernel<128>, row_grid(g), dim3(256), 0, st, g, rs_g, parts, (const float*)out_l.lse_out, out_g);
    return launch_status();
}

int fp32_bwd_dq(const Geom& g, const RowSet& rs, const void* q, const void* k, const void* v, const void* dO,
                const float* lse, float* delta, void* dq, int accumulate, hipStream_t st) {
    if (g.D != 64 && g.D != 128) return L2A_ERR_UNSUPPORTED;
    KernelTimer kt(rs.local ? "fp32_bwd_dq_local" : "fp32_bwd_dq_global", st);
    run_dq(g, DqCall{rs, rs, q, k, v, dO, lse, lse, delta, delta, dq, accumulate, Parts{}}, wide_tiles(g, rs), st);
    return launch_status();
}

size_t fp32_dq_shared_bytes(const Geom& g) { return parts_bytes(g, 1); }

bool fp32_window_is_all(const Geom& g) { return routed_parts(g) == 0; }

int fp32_bwd_dq_shared(const Geom& g, const RowSet& rs_l, const RowSet& rs_g, const void* q, const void* k, const void* v,
                       const void* dO, const float* lse_l, const float* lse_g, float* delta_l, float* delta_g, const float* share,
                       void* dq, void* ws, hipStream_t st) {
    if (g.D != 64 && g.D != 128) return L2A_ERR_UNSUPPORTED;
    const Parts parts = place_parts(g, (char*)ws);
    {
        KernelTimer kt("fp32_bwd_dq_shared", st);
        run_dq(g, DqCall{rs_l, rs_g, q, k, v, dO, lse_l, lse_g, delta_l, delta_g, dq, 0, parts}, wide_tiles(g, rs_l), st);
    }
    KernelTimer kt("fp32_dq_combine", st);
    if (g.D == 64) hipLaunchKernelGGL(fp32_dq_combine_kernel<64>, row_grid(g), dim3(256), 0, st, g, rs_g, parts, share, delta_l, delta_g, (float*)dq);
    else hipLaunchKernelGGL(fp32_dq_combine_kernel<128>, row_grid(g), dim3(256), 0, st, g, rs_g, parts, share, delta_l, delta_g, (float*)dq);
    return launch_status();
}

int fp32_bwd_dkdv(const Geom& g, const RowSet* sets, int nsets, const void* q, const void* k, const void* v,
                  const void* dO, const float* const* lse, const float* const* delta, const float* const* share, void* dk,
                  void* dv, hipStream_t st) {
    DkdvSets s;
    s.n = nsets;
    for (int i = 0; i < nsets; ++i) {
        s.rs[i] = sets[i];
        s.lse[i] = lse[i];
        s.delta[i] = delta[i];
        s.share[i] = share[i];
    }
    KernelTimer kt("fp32_bwd_dkdv", st);
    const dim3 grid = tile_grid(((long long)g.T + 15) / 16, g);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(512), 0, st, g, s, cf(q), cf(k), cf(v), cf(dO), (float*)dk, (float*)dv); };
    const bool folded = s.share[0] || s.share[1];
    if (g.D == 64) folded ? launch(fp32_bwd_dkdv_kernel<64, 8, true>) : launch(fp32_bwd_dkdv_kernel<64, 8, false>);
    else if (g.D == 128) folded ? launch(fp32_bwd_dkdv_kernel<128, 8, true>) : launch(fp32_bwd_dkdv_kernel<128, 8, false>);
    else return L2A_ERR_UNSUPPORTED;
    return launch_status();
}

}  // namespace l2a
