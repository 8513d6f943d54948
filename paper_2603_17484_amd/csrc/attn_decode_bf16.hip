// Decode step of the layer (Sec. 3.4): one new token per sequence attends to the KV cache --
// Local attention over the last W+1 keys for every token, Global attention over the whole prefix
// only if the token's router decision is 1, skipped entirely otherwise -- and the two are merged
// as o = s + d a (Sec. 3.1 Eq. 5).  HBM-bound: every cache row in reach is read once, a routed sequence's window
// for both branches together.
//
// Split-key scheme, two launches:
//   decode_partial_kernel  works through the units (decode_units.hpp): one KV head of a sequence, one chunk of 512 keys.
//       The G query heads of the KV group are the rows of one 32-row matrix tile (rows >= G are padding), so K and V
//       are read once for all of them.  The chunk is walked in sub-blocks of 32 keys: K and V rows go global -> LDS
//       with direct loads, S^T = K Q^T and O^T += V^T P^T run on the matrix cores with the streaming softmax of
//       App. C Alg. 1 in between; V^T operands are transposed on the way out of LDS (ds_read_b64_tr_b16).  One
//       partial (max, sum, O) per unit and head.
//   decode_combine_kernel  one workgroup per (batch, query head): merges the chunks of each branch, writes S, A,
//       the log-sum-exps and O = S + d A.
//
// A sequence's result depends, to the bit, on its own query, cache, position and decisions and on the cache's
// capacity, never on the sequences decoded with it.  P is rounded to bf16 against its chunk's running maximum and sums
// of floats follow their order, so chunks, the order within a chunk and the order of the merge are fixed; what varies
// with the batch is only who computes a unit, and how (two walks, same bits).
//
// Which sequences are routed and how long they are is device data, so every workgroup plans the batch, a lane per
// sequence, and takes its units from that (large batches: a wavefront for every unit there may be).  Whole step, us, a grid over all chunks with one wavefront each (the same
// bits) / chunks of a length derived from the whole call (other bits) / now: 1 x 32K tokens, routed 33 / 22 / 22; 8 x 128K, 2
// routed 135 / 114 / 118, none 40 / 24 / 22, all 411 / 378 / 389; 64 x 8K, 16 routed 203 / 133 / 135; 32 ring caches of 4K
// 126 / 108 / 113; 130 x 4K, 32 routed 324 / 350 / 195; 512 x 1K 272 / 322 / 186; 16384 x 256 312 / 469 / 278; per-head
// decisions, 28 heads, 8 x 32K 63 / 58 / 68 (the whole cache stays in the last-level cache there), 32 heads, 32 x 16K 314 / 246 / 253.
#include "decode_units.hpp"
#include "tiles.hpp"

namespace l2a {
namespace {

using units::kChunk;
using units::kSub;
using units::kWaves;
constexpr int kPart = kD + 4;  // floats per partial: max (log2 units), sum, 2 unused, O[128]
constexpr int kMostGroups = 512;  // workgroups of the first kernel: two on every CU

struct DecodeArgs {
    Geom gm;            // gm.T = capacity of the cache (tokens per sequence)
    const __bf16* q;    // [B, Hq, D]
    const __bf16* k;    // [B, T, Hkv, D]
    const __bf16* v;
    const int32_t* pos; // [B] position of the new token (keys 0..pos are valid)
    const uint8_t* mask;  // [B, mask_heads]; nullptr: every head routed
    int mask_heads;
    int do_local, do_global;
    int ring;           // the cache is a ring of gm.T slots: key j lies in slot j mod gm.T, pos is unbounded (Local only)
    float* part;        // [B, Hkv][units][G][kPart]
    int nchunks;        // chunks of the cache, = ceil(T / kChunk)
    int units;          // partials per (b, KV head): the chunks and, where a window may begin inside one, the Local one's
    int planned;        // units::planned
    __bf16* O;          // [B, Hq, D]
    __bf16* S;
    __bf16* A;
    float* lse_l;       // [B, Hq]
    float* lse_g;
};

__device__ __forceinline__ bool head_routed(const DecodeArgs& a, int b, int head) {
    if (!a.mask) return true;
    const int mh = a.mask_heads == 1 ? 0 : (a.mask_heads == a.gm.Hq ? head : head / a.gm.G);
    return a.mask[(size_t)b * a.mask_heads + mh] != 0;
}
// Sixteen decisions of sequence b from the at-th on, those past the last as zero; a bit each.
__device__ __forceinline__ unsigned decisions16(const DecodeArgs& a, int b, int at) {
    const uint8_t* p = a.mask + (size_t)b * a.mask_heads;
    unsigned bits = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i)  // the bytes' loads do not wait for one another
        bits |= (unsigned)(at + i < a.mask_heads && p[min(at + i, a.mask_heads - 1)] != 0) << i;
    return bits;
}
// Whether any of the heads of a KV group is routed (at most 16 of them).
__device__ __forceinline__ bool kv_routed(const DecodeArgs& a, int b, int hk) {
    if (!a.mask || a.mask_heads != a.gm.Hq) return head_routed(a, b, hk * a.gm.G);
    return (decisions16(a, b, hk * a.gm.G) & ((1u << a.gm.G) - 1u)) != 0;
}
struct SeqPlan {
    units::Keys keys;
    int pos;       // position of the new token, in a ring also beyond its slots
    int routed;    // KV heads whose whole prefix is needed
    unsigned long long set;  // which, a bit each, where there are at most 64 and they differ
};
__device__ __forceinline__ SeqPlan seq_plan(const DecodeArgs& a, int b) {
    SeqPlan s;
    // positions outside the cache are clamped, never followed; in a ring only negative ones are
    s.pos = max(a.pos[b], 0);
    const int t = min(s.pos, a.gm.T - 1);
    s.keys = units::Keys{t, a.ring ? 0 : max(t - a.gm.W, 0), a.do_local};  // a ring: the age of every written slot decides
    s.routed = 0, s.set = 0;
    if (!a.do_global) return s;
    const int hkv = a.gm.Hkv;
    if (!a.mask || a.mask_heads == 1) {
        s.routed = head_routed(a, b, 0) ? hkv : 0;
    } else {
        const int per = a.mask_heads / hkv;  // decisions of a KV head, at most 16
        unsigned long long bits = 0;         // those not yet assigned to a head
        for (int at = 0, have = 0, hk = 0; hk < hkv; at += 16) {
            bits |= (unsigned long long)decisions16(a, b, at) << have;
            for (have += 16; have >= per && hk < hkv; have -= per, bits >>= per, ++hk) {
                const unsigned on = (bits & ((1u << per) - 1u)) != 0;
                s.routed += on;
                s.set |= (unsigned long long)on << (hk & 63);
            }
        }
    }
    return s;
}

// A unit: the keys lo..hi of one (b, KV head).
struct Unit {
    int b, hk, slot;  // slot: where the partial goes
    int lo, hi;       // its keys
    int sb, pos;      // next sub-block to be computed; position of the new token
    __device__ __forceinline__ int ke() const { return hi / kSub; }
};
__device__ __forceinline__ Unit make_unit(const DecodeArgs& a, int b, int hk, const SeqPlan& s, int c) {
    Unit u;
    u.b = b, u.hk = hk;
    u.slot = c == units::kEdge ? a.nchunks : c;
    u.lo = units::first_key(s.keys, c);
    u.hi = units::last_key(s.keys, u.lo);
    u.sb = u.lo / kSub;
    u.pos = s.pos;
    return u;
}
// The i-th unit of sequence b on the XCD with residue r.
__device__ __forceinline__ Unit find_unit(const DecodeArgs& a, int b, const SeqPlan& s, int i, int r) {
    const int lane = threadIdx.x & 63, hkv = a.gm.Hkv;
    const units::Place at = units::place(s.keys, hkv, s.routed, i, r);
    int rank = at.rank, hk = rank;
    if (s.routed != 0 && s.routed != hkv) {
        unsigned long long set = 0;  // the heads that are routed, or not
        for (int h0 = 0; h0 < hkv; h0 += 64) {
            set = hkv <= 64 ? (at.routed ? s.set : ~s.set)
                            : __ballot(h0 + lane < hkv && kv_routed(a, b, min(h0 + lane, hkv - 1)) == (at.routed != 0));
            hk = h0;
            const int here = __popcll(set);
            if (rank < here) break;
            rank -= here;
        }
        for (; rank > 0; --rank) set &= set - 1;
        hk = min(max(hk + __ffsll((long long)set) - 1, 0), hkv - 1);  // (decisions that changed meanwhile must not lead outside)
    }
    return make_unit(a, b, __builtin_amdgcn_readfirstlane(hk), s, at.c);
}

// An address that is the same in all lanes, in scalar registers.
__device__ __forceinline__ const char* uniform(const char* p) {
    const uintptr_t x = (uintptr_t)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)x), hi = __builtin_amdgcn_readfirstlane((unsigned)(x >> 32));
    return (const char*)((uintptr_t)hi << 32 | lo);
}

// LDS of a workgroup, 77.5 KB: two of them on a CU.
struct PartialLds {
    __bf16 k[kWaves][kSub * 128];         // the wavefront's own sub-block
    __bf16 v[kWaves][kWaves * kSub * 32]; // the wavefront's own channels of the four sub-blocks
    __bf16 q[16 * 128];                   // the group's heads
    u32x4 p[kWaves][2][64];               // P of the four sub-blocks as operands
    float mx[kWaves][32], rsum[kWaves][64];
};

// Scores of one sub-block (32 keys from k0, a lane holds those of row n at c_row(r, h)) in log2 units, -inf where the
// row does not see the key.  Without a ring: lo <= key <= hi.  In a ring the token in slot `key` is age = (t_ref - key)
// mod T positions back and counts if age <= W; a ring that has not wrapped yet (position below T) must not wrap
// either: its slots behind the new token are unwritten.  (A wrapped ring has a multiple of 32 slots, so no sub-block
// reaches past its end.)  Returns the row's maximum.
template <bool RING>
__device__ __forceinline__ float masked_scores(const Geom& gm, const Unit& u, int k0, int h, f32x16& s) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] *= gm.scale_log2;
    if constexpr (RING) {
        const unsigned t_ref = u.pos % gm.T, wrap = u.pos >= gm.T ? gm.T : 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const unsigned d = t_ref - (unsigned)(k0 + c_row(r, h)), age = min(d, d + wrap);  // d < 0 reads as a huge number
            s[r] = age <= (unsigned)gm.W ? s[r] : -INFINITY;
        }
    } else if (k0 < u.lo || k0 + kSub - 1 > u.hi) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = k0 + c_row(r, h);
            s[r] = key >= u.lo && key <= u.hi ? s[r] : -INFINITY;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
    return fmaxf(mx, __shfl_xor(mx, 32));
}
// P of a sub-block against the reference `ref` as the operands of the product with V; returns this lane's sum
__device__ __forceinline__ float weights(const f32x16& s, float ref, u32x4 (&p)[2]) {
    float rsum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
        const float p0 = fast_exp2(s[r] - ref), p1 = fast_exp2(s[r + 1] - ref);
        rsum += p0 + p1;
        f32x2 f = {p0, p1};
        p[r >> 3][(r & 7) >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
    }
    return rsum;
}
// K and V of 32 keys, as a tile of 256-byte rows.  The rows behind the new token are not written yet (or past the end of
// the cache) and may hold anything, NaN patterns included, which a zero weight would not keep out of the sums: in
// the sub-block that holds it they repeat the last valid row (always masked).
typedef RmDma<kSub, 1> RowOffsets;
__device__ __forceinline__ void load_rows(const RowOffsets& off, unsigned row_bytes, const char* src, int valid, unsigned lds) {
    if (valid >= kSub) rm_dma_issue(off, src, lds, 0);
    else rm_dma_issue_clamped<kSub, 1, true>(row_bytes, valid, src, lds, 0);
}
__device__ __forceinline__ const char* rows_at(const DecodeArgs& a, const __bf16* x, const Unit& u, int sb) {
    return uniform((const char*)(x + (((size_t)u.b * a.gm.T + (size_t)sb * kSub) * a.gm.Hkv + u.hk) * kD));
}
// (LDS addresses are made anew for every use: kept, they would take the scalar registers that the loops are short of)
__device__ __forceinline__ unsigned lds_at(const void* p) { return __builtin_amdgcn_readfirstlane(lds_offset(p)); }

// One unit by one wavefront.
template <bool RING>
__device__ __forceinline__ void unit_by_wave(const DecodeArgs& a, const Unit& u, const RowOffsets& off, const __bf16* kt, const __bf16* vt) {
    const Geom& gm = a.gm;
    const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
    const unsigned row_bytes = (unsigned)gm.Hkv * kD * 2;
    bf16x8 qreg[8];  // lane n = row (head in group), rows >= G repeat the last head
    {
        const __bf16* qp = a.q + ((size_t)u.b * gm.Hq + u.hk * gm.G + min(n, gm.G - 1)) * kD + 8 * h;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
    }
    f32x16 oacc[4];
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] = 0.f;
    float m = -INFINITY, l = 0.f;
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto load = [&](const __bf16* x, int sb, const __bf16* tile) __attribute__((always_inline)) {
        load_rows(off, row_bytes, rows_at(a, x, u, sb), u.hi + 1 - sb * kSub, lds_at(tile));
    };
    load(a.k, u.sb, kt);
    load(a.v, u.sb, vt);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) asm volatile("" : "+v"(qreg[ks]));  // waited for here, and so not in the loop, behind its loads
    for (int sb = u.sb; sb <= u.ke(); ++sb) {
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // K; V, loaded after it, may be on its way still
        f32x16 s = zero16;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) s = mfma32(rm_tr_row_operand(kt, n, ks, h), qreg[ks], s);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the reads of K have returned
        if (sb < u.ke()) load(a.k, sb + 1, kt);
        const float mnew = fmaxf(m, masked_scores<RING>(gm, u, sb * kSub, h, s));
        const float ref = (RING && mnew == -INFINITY) ? 0.f : mnew, alpha = fast_exp2(m - ref);
        m = mnew;
        u32x4 p[2];
        l = fmaf(l, alpha, weights(s, ref, p));
        if (__any(alpha != 1.f)) {  // the running maximum of some row grew
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[d][r] *= alpha;
        }
        if (sb < u.ke()) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else dma_wait();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int d = 0; d < 4; ++d) oacc[d] = mfma32(rm_tr_col_operand(vt, d, i, lane), __builtin_bit_cast(bf16x8, p[i]), oacc[d]);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the reads of V have returned
        if (sb < u.ke()) load(a.v, sb + 1, vt);
    }
    l += __shfl_xor(l, 32);
    if (n < gm.G) {
        float* out = a.part + (((size_t)(u.b * gm.Hkv + u.hk) * a.units + u.slot) * gm.G + n) * kPart;
        if (h == 0) *reinterpret_cast<f32x2*>(out) = f32x2{m, l};
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int r = 0; r < 16; r += 4)
                *reinterpret_cast<f32x4*>(out + 4 + d * 32 + c_row(r, h)) = f32x4{oacc[d][r], oacc[d][r + 1], oacc[d][r + 2], oacc[d][r + 3]};
    }
}

// The XCD's units in order: full rounds of one per wavefront, then one per workgroup.
//
// A workgroup's own units come out of one stream of rounds of four sub-blocks.  Within a chunk the sub-blocks come one after
// the other, in the order and with the roundings of a single wavefront: wavefront w takes the scores of sub-block w of
// the four; the row maxima meet in LDS, and with them each wavefront knows the running maximum that its sub-block
// is to be taken against; P meets in LDS too, and wavefront w adds the four products to its quarter of O's channels.
// K of the next round, of this unit or the next, is on its way as soon as the scores are done, V as soon as the products
// are, each into the wavefront's own tiles.  What bounds a unit is its chain of 4 such rounds, 1 us each.
template <bool RING>
__global__ __launch_bounds__(64 * kWaves, 2) void decode_partial_kernel(DecodeArgs a) {
    __shared__ __attribute__((aligned(1024))) PartialLds lds;
    const Geom& gm = a.gm;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;

    // ---- the plan: 64 sequences at a time, a lane each
    const int xcd = blockIdx.x & 7, step = gridDim.x >> 3;
    int next = blockIdx.x >> 3, base = 0, total = 0, b0 = -64;  // next: number of the next unit on this XCD
    SeqPlan plan{};
    int start = 0, end = 0;  // the units of this lane's sequence, counted from base
    auto plan_next = [&]() __attribute__((always_inline)) {  // the next 64 sequences
        base += total;
        b0 += 64;
        if (b0 >= gm.B) return false;
        plan = seq_plan(a, min(b0 + lane, gm.B - 1));
        end = b0 + lane < gm.B ? units::seq_share(plan.keys, gm.Hkv, plan.routed, units::residue(xcd, b0 + lane)) : 0;
        start = -end;
        for (int o = 1; o < 64; o <<= 1) {
            const int below = __shfl_up(end, o);
            if (lane >= o) end += below;
        }
        start += end;
        total = __builtin_amdgcn_readlane(end, 63);
        return true;
    };
    auto fetch = [&](Unit& u) __attribute__((always_inline)) {
        while (next >= base + total)
            if (!plan_next()) return false;
        const int j = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(end > next - base)) - 1);
        SeqPlan s;
        s.keys = units::Keys{__builtin_amdgcn_readlane(plan.keys.t, j), __builtin_amdgcn_readlane(plan.keys.win, j), a.do_local};
        s.pos = __builtin_amdgcn_readlane(plan.pos, j);
        s.routed = __builtin_amdgcn_readlane(plan.routed, j);
        s.set = (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(plan.set >> 32), j) << 32 |
                (unsigned)__builtin_amdgcn_readlane((int)plan.set, j);
        u = find_unit(a, b0 + j, s, next - base - __builtin_amdgcn_readlane(start, j), units::residue(xcd, b0 + j));
        return true;
    };

    // ---- loads: 8 instructions for a wavefront's 8 KB of K, 8 for those of V (its 64 bytes of each row), one for its rows
    // of Q (rows past the group repeat the last head)
    const unsigned kv_row_bytes = (unsigned)gm.Hkv * kD * 2;
    const RowOffsets koff = rm_tr_dma_setup<kSub, 1>(kv_row_bytes, 0);
    const unsigned vrow = lane >> 2, vchunk = (lane & 3) * 16;
    auto load_k = [&](const Unit& u) __attribute__((always_inline)) {
        load_rows(koff, kv_row_bytes, rows_at(a, a.k, u, u.sb + wave), u.hi + 1 - (u.sb + wave) * kSub, lds_at(&lds.k[wave][0]));
    };
    auto load_v = [&](const Unit& u) __attribute__((always_inline)) {
        const char* src = rows_at(a, a.v, u, u.sb) + wave * 64;
        const int valid = u.hi + 1 - u.sb * kSub;
        const unsigned v_lds = lds_at(&lds.v[wave][0]);
        if (valid >= kWaves * kSub) {
            const unsigned off = vrow * kv_row_bytes + vchunk;
#pragma unroll
            for (int i = 0; i < 8; ++i) dma16_so(src + (size_t)(16 * i) * kv_row_bytes, off, v_lds + i * 1024);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) dma16_so(src, (unsigned)min(16 * i + (int)vrow, valid - 1) * kv_row_bytes + vchunk, v_lds + i * 1024);
        }
    };
    auto load_q = [&](const Unit& u) __attribute__((always_inline)) {
        rm_dma_issue_clamped<16, kWaves>(kD * 2, gm.G, uniform((const char*)(a.q + ((size_t)u.b * gm.Hq + u.hk * gm.G) * kD)), lds_at(&lds.q[0]), wave);
    };
    // transposed reads of a 16-key group of V: 16 lanes read 4 rows x 16 channels, the wavefront 512 contiguous bytes
    const int tr_i = lane & 15;
    const lds_cptr vread = (lds_cptr)(uintptr_t)(lds_offset(&lds.v[wave][0]) + (4 * h + (tr_i >> 2)) * 64 + (16 * ((lane >> 4) & 1) + 4 * (tr_i & 3)) * 2);

    if (!a.planned) {
        const long long at = (long long)blockIdx.x * kWaves + wave;
        const int per = gm.Hkv * a.units, b = (int)(at / per);
        if (b >= gm.B) return;
        const int i = (int)(at - (long long)b * per), hk = i / a.units, slot = i - hk * a.units;
        const SeqPlan s = seq_plan(a, b);
        const int c = slot == a.nchunks ? units::kEdge : slot;
        if (units::needed(s.keys, c, false) || (a.do_global && c != units::kEdge && kv_routed(a, b, hk) && units::needed(s.keys, c, true)))
            unit_by_wave<RING>(a, make_unit(a, b, hk, s, c), koff, &lds.k[wave][0], &lds.v[wave][0]);
        return;
    }
    // ---- the units for single wavefronts
    {
        while (plan_next()) {}
        const int all = base;
        if (gm.B > 64) b0 = -64, plan_next();
        else b0 = 0;
        base = 0;
        const int alone = units::by_wave(all, step);
        Unit u;
        for (next = (blockIdx.x >> 3) * kWaves + wave; next < min(alone, all); next += kWaves * step)
            if (fetch(u)) unit_by_wave<RING>(a, u, koff, &lds.k[wave][0], &lds.v[wave][0]);
        next = alone + (blockIdx.x >> 3);
    }
    // ---- the workgroup's own
    Unit cur;
    if (!fetch(cur)) return;
    if (cur.sb + wave <= cur.ke()) load_k(cur);
    load_q(cur);
    load_v(cur);
    bf16x8 qreg[8];
    f32x16 oacc;
    float m, l;
    bool first = true, more = true;
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    while (more) {
        const int count = min(kWaves, cur.ke() - cur.sb + 1);  // sub-blocks of this round
        const bool mine = wave < count;
        Unit nxt = cur;
        nxt.sb += kWaves;
        const bool last = nxt.sb > cur.ke();
        if (last) next += step, more = fetch(nxt);
        const bool mine_next = more && nxt.sb + wave <= nxt.ke();

        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // all but this round's V, issued last
        if (first) {
            __syncthreads();  // every wavefront's rows of Q are there
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) qreg[ks] = rm_operand(lds.q, n & 15, ks, h);
            m = -INFINITY, l = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[r] = 0.f;
        }
        // ---- S^T[key, row] = K Q^T and the row maxima of this wavefront's sub-block
        f32x16 s = zero16;
        float mx = -INFINITY;
        if (mine) {
            const __bf16* kt = &lds.k[wave][0];
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) s = mfma32(rm_tr_row_operand(kt, n, ks, h), qreg[ks], s);
            mx = masked_scores<RING>(gm, cur, (cur.sb + wave) * kSub, h, s);
        }
        if (h == 0) lds.mx[wave][n] = mx;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the reads of K have returned
        if (mine_next) load_k(nxt);
        __syncthreads();
        if (last && more) load_q(nxt);  // every wavefront has its operands of this unit's
        // ---- the running maximum after each sub-block.  A ring larger than the window has sub-blocks out of reach:
        // while no key has been seen the running maximum stays -inf and the exponentials take 0 as their reference (all
        // of them are 0); without a ring every sub-block has a valid key and it is finite.
        float alpha[kWaves], ref = 0.f;
        bool grew = false;
#pragma unroll
        for (int j = 0; j < kWaves; ++j) {
            const float mnew = fmaxf(m, lds.mx[j][n]);
            const float mref = (RING && mnew == -INFINITY) ? 0.f : mnew;
            alpha[j] = fast_exp2(m - mref);  // exp2(-inf) = 0 on the first step
            if (j == wave) ref = mref;
            if (j < count) grew = grew || alpha[j] != 1.f, m = mnew;
        }
        if (mine) {
            u32x4 p[2];
            lds.rsum[wave][lane] = weights(s, ref, p);
            lds.p[wave][0][lane] = p[0], lds.p[wave][1][lane] = p[1];
        }
        __syncthreads();
        // ---- O^T[ch, row] += V^T P^T, this wavefront's 32 channels; the next round's K and Q may be on their way still
        if (last && more) {
            if (mine_next) asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(1)" ::: "memory");
        } else if (mine_next) {
            asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        } else {
            dma_wait();
        }
        auto product = [&](int j) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                typedef s16x4 __attribute__((address_space(3)))* lds_ptr;
                const lds_cptr at = vread + (j * kSub + 16 * i) * 64;
                const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)at);
                const s16x4 v2 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + 8 * 64));
                const bf16x8 vo = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v1, v2, 0, 1, 2, 3, 4, 5, 6, 7));
                oacc = mfma32(vo, __builtin_bit_cast(bf16x8, lds.p[j][i][lane]), oacc);
            }
        };
        if (count == kWaves && !__any(grew)) {
#pragma unroll
            for (int j = 0; j < kWaves; ++j) {
                l = fmaf(l, alpha[j], lds.rsum[j][lane]);
                product(j);
            }
        } else {  // the running maximum of some row grew, or the chunk ends
#pragma unroll
            for (int j = 0; j < kWaves; ++j) {
                if (j >= count) break;
                l = fmaf(l, alpha[j], lds.rsum[j][lane]);
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[r] *= alpha[j];
                product(j);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the reads of V have returned
        if (last) {
            l += __shfl_xor(l, 32);
            if (n < gm.G) {
                float* out = a.part + (((size_t)(cur.b * gm.Hkv + cur.hk) * a.units + cur.slot) * gm.G + n) * kPart;
                if (wave == 0 && h == 0) *reinterpret_cast<f32x2*>(out) = f32x2{m, l};
#pragma unroll
                for (int r = 0; r < 16; r += 4)
                    *reinterpret_cast<f32x4*>(out + 4 + wave * 32 + c_row(r, h)) = f32x4{oacc[r], oacc[r + 1], oacc[r + 2], oacc[r + 3]};
            }
        }
        if (more) load_v(nxt);
        first = last;
        cur = nxt;
    }
}

// Thread = (branch, slice, four channels): slice i takes every nslices-th chunk of its branch with a
// running maximum; the slices meet in LDS, where a thread is a channel.  What it spends its time on is waiting for
// partials that other XCDs wrote: 16 chunks' loads in flight together, 32 with MANY (184 registers), whole step against 8,
// us: 1 x 32K 23.6 / 22.2 / 22.2, 8 x 128K, 2 routed 122.0 / 119.6 / 117.4, but 256 x 4K 374 / 374 / 389.
constexpr int kSlices = 8;
template <bool MANY>
__global__ __launch_bounds__(2 * kSlices * 32) void decode_combine_kernel(DecodeArgs a) {
    const int nslices = blockDim.x >> 6;
    __shared__ __attribute__((aligned(16))) float so[2][kSlices][kD];
    __shared__ float sm[2][kSlices], sl[2][kSlices];
    const Geom& gm = a.gm;
    const int bhq = blockIdx.x, b = bhq / gm.Hq, head = bhq - b * gm.Hq;
    const int hk = head / gm.G, g = head - hk * gm.G;
    const bool on[2] = {a.do_local != 0, a.do_global && head_routed(a, b, head)};
    const int t = min(max(a.pos[b], 0), gm.T - 1);  // ring: the last written slot while it fills up, then the last slot
    {
        const int c4 = (threadIdx.x & 31) * 4, i = threadIdx.x >> 5, branch = i >= nslices, slice = i - branch * nslices;
        const int lo = branch || a.ring ? 0 : max(t - gm.W, 0), c_lo = lo / kChunk, c_hi = t / kChunk;
        const float* base = a.part + ((size_t)(b * gm.Hkv + hk) * a.units * gm.G + g) * kPart;
        float m = -INFINITY, l = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        auto batch = [&](auto kc, int ch0) __attribute__((always_inline)) {
            constexpr int K = decltype(kc)::value;
            f32x2 ml[K];
            f32x4 x[K];
#pragma unroll
            for (int j = 0; j < K; ++j) {  // past the end the first is read again, for nobody
                const int ch = ch0 + j * nslices, at = ch <= c_hi ? ch : ch0;
                const int unit = at == c_lo && lo % kChunk ? a.nchunks : at;
                const float* part = base + (size_t)unit * gm.G * kPart;
                ml[j] = *reinterpret_cast<const f32x2*>(part);
                x[j] = *reinterpret_cast<const f32x4*>(part + 4 + c4);
            }
#pragma unroll
            for (int j = 0; j < K; ++j) {
                if (ch0 + j * nslices > c_hi) break;
                const float mn = fmaxf(m, ml[j][0]);
                // exp2(-inf) = 0 on the first chunk; a chunk of a ring may have no slot in the window (its
                // maximum is -inf): while nothing has been seen the reference is 0 and both factors are 0
                const float ref = mn == -INFINITY ? 0.f : mn;
                const float s0 = fast_exp2(m - ref), s1 = fast_exp2(ml[j][0] - ref);
                l = fmaf(l, s0, ml[j][1] * s1);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = fmaf(o[e], s0, x[j][e] * s1);
                m = mn;
            }
        };
        if (on[branch]) {
            int ch0 = c_lo + slice;
            if (MANY)
                for (; ch0 + 16 * nslices <= c_hi; ch0 += 32 * nslices) batch(std::integral_constant<int, 32>{}, ch0);
            for (; ch0 + 4 * nslices <= c_hi; ch0 += 16 * nslices) batch(std::integral_constant<int, 16>{}, ch0);
            for (; ch0 <= c_hi; ch0 += 4 * nslices) batch(std::integral_constant<int, 4>{}, ch0);
        }
        *reinterpret_cast<f32x4*>(&so[branch][slice][c4]) = o;
        if (c4 == 0) sm[branch][slice] = m, sl[branch][slice] = l;
    }
    __syncthreads();
    if (threadIdx.x >= kD) return;
    const int c = threadIdx.x;
    float out[2] = {0.f, 0.f};
    float lse[2] = {-INFINITY, -INFINITY};
#pragma unroll
    for (int branch = 0; branch < 2; ++branch) {
        if (!on[branch]) continue;
        float mn = sm[branch][0];  // slices that had no chunk hold (-inf, 0, 0); slice 0 always has one
        for (int i = 1; i < nslices; ++i) mn = fmaxf(mn, sm[branch][i]);
        float lsum = 0.f, osum = 0.f;
        for (int i = 0; i < nslices; ++i) {
            const float mi = sm[branch][i], sc = mi == -INFINITY ? 0.f : fast_exp2(mi - mn);
            lsum = fmaf(sl[branch][i], sc, lsum);
            osum = fmaf(so[branch][i][c], sc, osum);
        }
        out[branch] = osum / lsum;
        lse[branch] = (mn + __builtin_amdgcn_logf(lsum)) * kLn2;
    }
    const size_t o = (size_t)bhq * kD + c;
    a.O[o] = (__bf16)(out[0] + out[1]);
    if (a.S) a.S[o] = (__bf16)out[0];
    if (a.A) a.A[o] = (__bf16)out[1];
    if (c == 0) {
        if (a.lse_l) a.lse_l[bhq] = lse[0];
        if (a.lse_g) a.lse_g[bhq] = lse[1];
    }
}

}  // namespace

// Room for two partials per chunk and query head; the units are at most that many (a chunk more than the cache has).
size_t decode_partial_floats(const Geom& g) {
    return (size_t)g.B * g.Hq * 2 * ((g.T + kChunk - 1) / kChunk) * kPart;
}

int mfma_decode(const Geom& g, const void* q, const void* k, const void* v, const int32_t* pos, const uint8_t* mask,
                int mask_heads, int do_local, int do_global, int ring, float* part, void* O, void* S, void* A, float* lse_l,
                float* lse_g, hipStream_t st) {
    if (g.D != kD || g.G > 16) return L2A_ERR_UNSUPPORTED;
    DecodeArgs a{};
    a.gm = g;
    a.q = (const __bf16*)q;
    a.k = (const __bf16*)k;
    a.v = (const __bf16*)v;
    a.pos = pos;
    a.mask = mask;
    a.mask_heads = mask_heads;
    a.do_local = do_local;
    a.do_global = do_global;
    a.ring = ring;
    a.part = part;
    a.nchunks = (g.T + kChunk - 1) / kChunk;
    a.units = a.nchunks + (do_local && !ring ? 1 : 0);
    a.O = (__bf16*)O;
    a.S = (__bf16*)S;
    a.A = (__bf16*)A;
    a.lse_l = lse_l;
    a.lse_g = lse_g;
    {
        KernelTimer kt("decode_partial", st);
        // no more workgroups than an XCD can have units
        const long long most = 8ll * g.B * g.Hkv * ((a.units + 7) / 8);
        a.planned = units::planned(g.B, do_global && mask && mask_heads > 1);
        const long long places = (long long)g.B * g.Hkv * a.units;
        const dim3 grid((unsigned)(!a.planned ? (places + kWaves - 1) / kWaves : most < kMostGroups ? most : kMostGroups));
        if (ring)
            hipLaunchKernelGGL(decode_partial_kernel<true>, grid, dim3(64 * kWaves), 0, st, a);
        else
            hipLaunchKernelGGL(decode_partial_kernel<false>, grid, dim3(64 * kWaves), 0, st, a);
    }
    {
        KernelTimer kt("decode_combine", st);
        // from the capacity alone: the order of the merge decides the bits
        const int slices = a.nchunks >= 128 ? kSlices : (a.nchunks >= 32 ? 4 : 2);
        // long lists, and no more workgroups than two per CU
        if (slices == kSlices && g.B * g.Hq <= 512)
            hipLaunchKernelGGL(decode_combine_kernel<true>, dim3(g.B * g.Hq), dim3(2 * slices * 32), 0, st, a);
        else
            hipLaunchKernelGGL(decode_combine_kernel<false>, dim3(g.B * g.Hq), dim3(2 * slices * 32), 0, st, a);
    }
    return launch_status();
}

}  // namespace l2a
