// Decode step of the layer (Sec. 3.4): one new token per sequence attends to the KV cache --
// Local attention over the last W+1 keys for every token, Global attention over the whole prefix
// only if the token's router decision is 1, skipped entirely otherwise -- and the two are merged
// as o = s + d a (Sec. 3.1 Eq. 5).  HBM-bound: the cache is read once per branch that runs.
//
// Split-key scheme, two launches:
//   decode_partial_kernel  one wavefront per workgroup and chunk of a sequence's keys.  The G query heads of a
//       KV group are the rows of one 32-row matrix tile (rows >= G are padding), so K and V are read once
//       for all of them.  The wavefront walks its chunk in 32-key sub-blocks: K and V rows go global -> LDS
//       with direct loads, S^T = K Q^T and O^T += V^T P^T run on the matrix cores with the streaming softmax
//       of App. C Alg. 1 in between; V^T operands are transposed on the way out of LDS (ds_read_b64_tr_b16).
//       One partial (max, sum, O) per chunk and head.
//   decode_combine_kernel  one workgroup per (batch, query head): merges the chunks of each branch, writes S, A,
//       the log-sum-exps and O = S + d A.
//
// A sequence's keys fall into two segments, the window (near) and what lies before it (far): the Local branch
// is the near chunks, the Global branch all of them, so a routed sequence's window is read once for both.
//
// What bounds it: the bytes of the cache rows in reach, and for small batches the latency of a wavefront's walk.
// Which sequences are routed and how long they are is device data, so the chunk length is too: every workgroup
// sums the sub-blocks of the whole call and all take about S / kTargetChunks of them; unequal sequences and mixes
// of routed and unrouted ones then fill the chip evenly and no workgroup is launched for nothing.  The
// heads of a key range are adjacent workgroups: together they read whole rows of the cache at about the same time.
#include "tiles.hpp"

namespace l2a {
namespace {

constexpr int kSub = 32;       // keys per wavefront step
constexpr int kWaves = 4;      // wavefronts of a workgroup: they share a chunk's sub-blocks, 16 KB of LDS each
constexpr int kPart = kD + 4;  // floats per partial: max (log2 units), sum, 2 of segment_slots, O[128]
// Chunks a call is cut into (plus at most one more per segment).  Two workgroups fit a CU: 512 are at work at once,
// and twice that evens out what is left at the end.  Measured with 512 / 1024 / 2048, partial + combine kernel, us:
// 8 x 128K, 2 routed 134 / 129 / 132; 64 x 8K, 16 routed 157 / 151 / 162; 1 x 128K 67 / 73 / 81.
constexpr int kTargetChunks = 1024;
// Batches beyond this size have chunks of kFixedSub sub-blocks, found from the workgroup's index alone: summing the
// whole batch in every workgroup would cost more than an even split gains there.
constexpr int kMaxScanBatch = 128, kFixedSub = 16;

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
    float* part;        // [slot][G][kPart], one slot per chunk
    int target;      // chunks to cut the call into, 0: one per segment (there are no slots for more)
    int unit_slots;  // batches beyond kMaxScanBatch: slots of each (batch, KV head); else 0
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

// One sequence's part of a call.  near: keys lo..t, far: keys 0..lo-1 (Local alone: no far; Global alone: no near).
struct SeqPlan {
    int t, lo;            // position of the new token, first key of the window
    int n_near, n_far;    // sub-blocks of the segments
    int routed;           // KV heads whose far segment is needed
};
__device__ __forceinline__ bool kv_routed(const DecodeArgs& a, int b, int hk) {
    if (a.mask && a.mask_heads != a.gm.Hq) return head_routed(a, b, hk * a.gm.G);
    bool any = false;
    for (int g = 0; g < a.gm.G; ++g) any = any || head_routed(a, b, hk * a.gm.G + g);
    return any;
}
__device__ __forceinline__ SeqPlan seq_plan(const DecodeArgs& a, int b) {
    const Geom& gm = a.gm;
    SeqPlan s;
    // positions outside the cache are clamped, never followed; in a ring only negative ones are, and slots 0..t are
    // written: which of them lie in the window is decided per key
    s.t = min(max(a.pos[b], 0), gm.T - 1);
    s.lo = !a.do_local ? s.t + 1 : (a.ring ? 0 : max(s.t - gm.W, 0));
    s.n_near = a.do_local ? s.t / kSub - s.lo / kSub + 1 : 0;
    s.routed = 0;
    if (a.do_global && s.lo > 0) {
        if (!a.mask || a.mask_heads == 1) s.routed = head_routed(a, b, 0) ? gm.Hkv : 0;
        else
            for (int hk = 0; hk < gm.Hkv; ++hk) s.routed += kv_routed(a, b, hk) ? 1 : 0;
    }
    s.n_far = s.routed ? (s.lo - 1) / kSub + 1 : 0;
    return s;
}
__device__ __forceinline__ int ceil_div(int x, int y) { return (x + y - 1) / y; }

// Chunks in order: sequence; its near chunks, then its far ones.  Within a segment blocks of 8 chunks, head by head: the
// chunks of all heads that read the same rows of the cache then lie a multiple of 8 workgroups apart, which is
// the same XCD (8 x 128K, 2 routed: 123.5 -> 118.4 us; 8 x 128K all routed 404 -> 396).  With per-head decisions
// the far chunks are those of the routed KV heads in ascending order, key range by key range.
constexpr int kHeadBlock = 8;
struct Chunk {
    int b, hk, far;          // far: which segment
    int c, count, step;      // the chunk's number in its segment, the segment's chunks and the distance of their slots
    int sub;                 // sub-blocks per chunk
};
__device__ __forceinline__ void by_head_blocks(Chunk& k, int left, int heads) {
    const int blk = left / (kHeadBlock * heads), r = left - blk * kHeadBlock * heads;
    const int width = min(kHeadBlock, k.count - blk * kHeadBlock);  // the last block may be narrower
    k.hk = r / width;
    k.c = blk * kHeadBlock + r - k.hk * width;
}
// The slot of chunk ch of a segment of KV head hk, whose chunk 0 lies in slot first.
__device__ __forceinline__ int chunk_slot(int first, int ch, int count, int step, int hk, int heads) {
    if (step != heads) return first + ch * step;
    const int blk = ch / kHeadBlock * kHeadBlock;
    return first + hk * (min(kHeadBlock, count - blk) - min(kHeadBlock, count)) + blk * heads + ch - blk;
}
// The slot-th chunk of the call, b = -1 if there are fewer.  Wave-uniform; a lane plans the sequences b0 + lane.
__device__ __forceinline__ Chunk find_chunk(const DecodeArgs& a, int slot) {
    const Geom& gm = a.gm;
    const int lane = threadIdx.x & 63;
    Chunk k{-1, 0, 0, 0, 0, 1, kFixedSub};
    if (a.unit_slots) {
        const int unit = slot / a.unit_slots, c = slot - unit * a.unit_slots;
        const int b = unit / gm.Hkv, hk = unit - b * gm.Hkv;
        const SeqPlan s = seq_plan(a, b);
        const int near = ceil_div(s.n_near, kFixedSub), far = s.n_far && kv_routed(a, b, hk) ? ceil_div(s.n_far, kFixedSub) : 0;
        if (c < near + far) k = Chunk{b, hk, c >= near, c >= near ? c - near : c, c >= near ? far : near, 1, kFixedSub};
        return k;
    }
    SeqPlan s[kMaxScanBatch / 64];
    long long total = 0;
#pragma unroll
    for (int i = 0; i < kMaxScanBatch / 64; ++i) {
        if (64 * i >= gm.B) break;
        s[i] = seq_plan(a, min(64 * i + lane, gm.B - 1));
        const int n = gm.Hkv * s[i].n_near + s[i].routed * s[i].n_far;
        for (int j = 0; j < min(gm.B - 64 * i, 64); ++j) total += __builtin_amdgcn_readlane(n, j);
    }
    // sub-blocks per chunk; without room for more, one chunk per segment
    k.sub = a.target ? max(kWaves, (int)((total + a.target - 1) / a.target)) : gm.T / kSub + 2;
    int left = slot;
#pragma unroll
    for (int i = 0; i < kMaxScanBatch / 64; ++i) {
        if (64 * i >= gm.B) break;
        const int near = ceil_div(s[i].n_near, k.sub), far = ceil_div(s[i].n_far, k.sub);
        const int n = gm.Hkv * near + s[i].routed * far;
        for (int j = 0; j < min(gm.B - 64 * i, 64); ++j) {
            const int nj = __builtin_amdgcn_readlane(n, j);
            if (left >= nj) {
                left -= nj;
                continue;
            }
            const int nearj = __builtin_amdgcn_readlane(near, j);
            k.b = 64 * i + j;
            if (left < gm.Hkv * nearj) {
                k.count = nearj, k.step = gm.Hkv;
                by_head_blocks(k, left, gm.Hkv);
                return k;
            }
            left -= gm.Hkv * nearj;
            k.far = 1;
            k.count = __builtin_amdgcn_readlane(far, j), k.step = __builtin_amdgcn_readlane(s[i].routed, j);
            if (k.step == gm.Hkv) {
                by_head_blocks(k, left, gm.Hkv);
            } else {
                k.c = left / k.step;
                int rank = left - k.c * k.step, hk = 0;  // the rank-th of the routed heads
                for (;; ++hk)
                    if (kv_routed(a, k.b, hk) && rank-- == 0) break;
                k.hk = hk;
            }
            return k;
        }
    }
    return k;
}
// Where a segment's chunks lie (first slot, count << 16 | step): left by the workgroup of its first chunk, for the
// combine kernel, in the two unused floats of the partial in slot 2 (b Hkv + hk) + far.
__device__ __forceinline__ u32x2* segment_slots(const DecodeArgs& a, int b, int hk, int far) {
    return reinterpret_cast<u32x2*>(a.part + (size_t)(2 * (b * a.gm.Hkv + hk) + far) * a.gm.G * kPart + 2);
}

// Running (max, sum, O) of four channels; a partial with no key in reach (m = -inf) changes nothing.
struct Merge {
    float m = -INFINITY, l = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    __device__ __forceinline__ void add(float m1, float l1, f32x4 o1) {
        const float mn = fmaxf(m, m1);
        const float ref = mn == -INFINITY ? 0.f : mn;
        const float s0 = fast_exp2(m - ref), s1 = fast_exp2(m1 - ref);
        l = l * s0 + l1 * s1;
        o = o * s0 + o1 * s1;
        m = mn;
    }
    __device__ __forceinline__ void add(const float* part, int c4) {
        const f32x2 ml = *reinterpret_cast<const f32x2*>(part);
        add(ml[0], ml[1], *reinterpret_cast<const f32x4*>(part + 4 + c4));
    }
};

// A wavefront does not overlap its own loads with its arithmetic; the eight at work on a CU overlap each other's
// (a second buffer each, 2 x 32 KB per wavefront pair of the CU's 160, left room for half as many and was slower).
template <bool RING>
__global__ __launch_bounds__(64 * kWaves, 2) void decode_partial_kernel(DecodeArgs a) {
    // per wavefront: (K tile, V tile), 32 keys x 128 channels each
    __shared__ __attribute__((aligned(1024))) __bf16 lds[kWaves][2][kSub * 128];

    const Geom& gm = a.gm;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, h = lane >> 5;
    const Chunk ck = find_chunk(a, (int)blockIdx.x);
    const int b = __builtin_amdgcn_readfirstlane(ck.b), hk = __builtin_amdgcn_readfirstlane(ck.hk);
    if (b < 0) return;
    const int far = __builtin_amdgcn_readfirstlane(ck.far), c = __builtin_amdgcn_readfirstlane(ck.c);
    if (c == 0 && threadIdx.x == 0) *segment_slots(a, b, hk, far) = u32x2{blockIdx.x, (unsigned)ck.count << 16 | (unsigned)ck.step};
    const int t_abs = max(a.pos[b], 0);
    const int t = min(t_abs, gm.T - 1);
    const int lo_near = !a.do_local ? t + 1 : (RING ? 0 : max(t - gm.W, 0));
    const int lo = far ? 0 : lo_near, hi = far ? lo_near - 1 : t;  // keys lo..hi of the segment
    // A chunk is every count-th sub-block of the segment: the workgroups at work then read neighbouring rows at
    // about the same time.
    const int count = __builtin_amdgcn_readfirstlane(ck.count);
    const int ke = hi / kSub;
    // Which keys of a sub-block count is decided without branches (a basic-block boundary between
    // the score instructions and the code that reads their results costs the compiler its
    // bookkeeping of the wait between them).  Without a ring: lo <= key <= hi.  In a ring the token
    // in slot `key` is age = (t_ref - key) mod T positions back and counts if age <= W; a ring that
    // has not wrapped yet (t_abs < T) must not wrap either: its slots behind the new token are
    // unwritten.  (A wrapped ring has a multiple of 32 slots, so no sub-block reaches past its end.)
    const unsigned t_ref = RING ? t_abs % gm.T : 0;
    const unsigned wrap = (RING && t_abs >= gm.T) ? gm.T : 0;

    // Q of the group's heads as B operands: lane n = row (head in group), rows >= G repeat the last head
    const int head = hk * gm.G + min(n, gm.G - 1);
    bf16x8 qreg[8];
    {
        const __bf16* qp = a.q + ((size_t)b * gm.Hq + head) * kD + 8 * h;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
    }

    const unsigned kv_row_bytes = (unsigned)gm.Hkv * kD * 2;
    const char* kbase = (const char*)(a.k + ((size_t)b * gm.T * gm.Hkv + hk) * kD);
    const char* vbase = (const char*)(a.v + ((size_t)b * gm.T * gm.Hkv + hk) * kD);
    const RmDma<kSub, 1> off = rm_tr_dma_setup<kSub, 1>(kv_row_bytes, 0);  // one chunk permutation, and so one set of offsets, for both
    const unsigned lds0 = lds_offset(&lds[0][0][0]) + wave * (unsigned)sizeof(lds[0]);
    auto load = [&](int sb) __attribute__((always_inline)) {
        const size_t src = (size_t)sb * kSub * kv_row_bytes;
        const unsigned dst = lds0;
        if ((sb + 1) * kSub <= hi + 1) {
            rm_dma_issue(off, kbase + src, dst, 0);
            rm_dma_issue(off, vbase + src, dst + kSub * 256, 0);
        } else {  // the sub-block that holds the new token: the rows behind it are not written yet (or past
                  // the end of the cache) and may hold anything, NaN patterns included, which a zero
                  // weight would not keep out of the sums: they repeat the last valid row (always masked)
            rm_dma_issue_clamped<kSub, 1, true>(kv_row_bytes, hi + 1 - sb * kSub, kbase + src, dst, 0);
            rm_dma_issue_clamped<kSub, 1, true>(kv_row_bytes, hi + 1 - sb * kSub, vbase + src, dst + kSub * 256, 0);
        }
    };

    f32x16 oacc[4];
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] = 0.f;
    float m = -INFINITY, l = 0.f;
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    const __bf16* kt = &lds[wave][0][0];
    const __bf16* vt = &lds[wave][1][0];
    for (int sb = lo / kSub + c + wave * count; sb <= ke; sb += kWaves * count) {
        load(sb);  // the previous step's LDS reads have all returned (their MFMAs were issued)
        dma_wait();

        // S^T[key, row] = K Q^T
        f32x16 s = zero16;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) s = mfma32(rm_tr_row_operand(kt, n, ks, h), qreg[ks], s);

        // streaming softmax, one row per lane (the lane 32 apart holds the row's other 16 keys)
        const int k0 = sb * kSub;
        float mx = -INFINITY;
        const int lo_l = lo - k0 - 4 * h, hi_l = hi - k0 - 4 * h;  // the lane's keys are k0 + 4 h + cr
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int cr = 8 * (r >> 2) + (r & 3);
            bool ok;
            if constexpr (RING) {
                const unsigned d = t_ref - (unsigned)(k0 + 4 * h + cr), age = min(d, d + wrap);  // d < 0 reads as a huge number
                ok = age <= (unsigned)gm.W;
            } else {
                ok = cr >= lo_l && cr <= hi_l;
            }
            s[r] = ok ? s[r] * gm.scale_log2 : -INFINITY;
            mx = fmaxf(mx, s[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        // a ring larger than the window has sub-blocks out of reach: while no key has been seen the
        // running maximum stays -inf and the exponentials take 0 as their reference (all of them are 0)
        const float mnew = fmaxf(m, mx);  // without a ring every sub-block of the range has a valid key: mnew is finite
        const float mref = (RING && mnew == -INFINITY) ? 0.f : mnew;
        const float alpha = fast_exp2(m - mref);  // exp2(-inf) = 0 on the first step
        m = mnew;
        float rsum = 0.f;
        uint32_t pw[2][4];
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const float p0 = fast_exp2(s[r] - mref), p1 = fast_exp2(s[r + 1] - mref);
            rsum += p0 + p1;
            f32x2 f = {p0, p1};
            pw[r >> 3][(r & 7) >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
        }
        l = l * alpha + rsum;
        if (__any(alpha != 1.f)) {  // the running maximum of some row grew
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[d][r] *= alpha;
        }

        // O^T[ch, row] += V^T P^T
#pragma unroll
        for (int step = 0; step < 2; ++step) {
            const u32x4 pv = {pw[step][0], pw[step][1], pw[step][2], pw[step][3]};
#pragma unroll
            for (int d = 0; d < 4; ++d)
                oacc[d] = mfma32(rm_tr_col_operand(vt, d, step, lane), __builtin_bit_cast(bf16x8, pv), oacc[d]);
        }
    }
    l += __shfl_xor(l, 32);

    // ---- the wavefronts' partials meet in LDS (rows < G only)
    float* part = a.part + (size_t)blockIdx.x * gm.G * kPart;
    float* stage = reinterpret_cast<float*>(&lds[0][0][0]);  // [kWaves][G][kPart]
    __syncthreads();  // every wavefront is done with its tiles
    if (n < gm.G) {
        float* out = stage + (wave * gm.G + n) * kPart;
        if (h == 0) *reinterpret_cast<f32x2*>(out) = f32x2{m, l};
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int r = 0; r < 16; r += 4)
                *reinterpret_cast<f32x4*>(out + 4 + d * 32 + c_row(r, h)) = f32x4{oacc[d][r], oacc[d][r + 1], oacc[d][r + 2], oacc[d][r + 3]};
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < gm.G * (kD / 4); idx += 64 * kWaves) {
        const int g = idx / (kD / 4), c4 = (idx - g * (kD / 4)) * 4;
        Merge x;
        for (int w = 0; w < kWaves; ++w) x.add(stage + (w * gm.G + g) * kPart, c4);
        *reinterpret_cast<f32x4*>(part + g * kPart + 4 + c4) = x.o;
        if (c4 == 0) *reinterpret_cast<f32x2*>(part + g * kPart) = f32x2{x.m, x.l};
    }
}

// Thread = (four channels, slice): slice i of n (n = blockDim.x / 32) takes every n-th chunk with a running
// maximum, the loads of kInFlight chunks in flight together, also of the last few (1 x 32K, whole step 22.5 -> 21.8 us, 8 x
// 128K 115.5 -> 113.5; in a plain loop the last few waited for one another); the two slices of a wavefront
// meet by an exchange, the wavefronts in LDS.
constexpr int kInFlight = 4;
constexpr int kCombineWaves = 16;
__global__ __launch_bounds__(kCombineWaves * 64) void decode_combine_kernel(DecodeArgs a) {
    const int nwaves = blockDim.x >> 6, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __shared__ __attribute__((aligned(16))) float so[2][kCombineWaves][kD];
    __shared__ float sm[2 * kCombineWaves], sl[2 * kCombineWaves], sf[2][2 * kCombineWaves], st[2][2];
    const Geom& gm = a.gm;
    const int bhq = blockIdx.x, b = bhq / gm.Hq, head = bhq - b * gm.Hq;
    const int hk = head / gm.G, g = head - hk * gm.G;
    const int c4 = (lane & 31) * 4, slice = threadIdx.x >> 5;
    const bool routed = a.do_global && head_routed(a, b, head);
    // both segments' slots at once: a chain of dependent loads is all that the kernel spends its time on (an absent
    // segment's are whatever the workspace holds, and unused)
    const u32x2 slots[2] = {*segment_slots(a, b, hk, 0), *segment_slots(a, b, hk, 1)};
    const SeqPlan plan = seq_plan(a, b);
#pragma unroll
    for (int seg = 0; seg < 2; ++seg) {
        Merge x;
        if (seg == 0 ? plan.n_near > 0 : (routed && plan.lo > 0)) {
            const u32x2 d = slots[seg];
            const int count = d[1] >> 16, step = d[1] & 0xffff;
            for (int ch0 = slice; ch0 < count; ch0 += kInFlight * 2 * nwaves) {
                f32x2 ml[kInFlight];
                f32x4 o[kInFlight];
#pragma unroll
                for (int i = 0; i < kInFlight; ++i) {  // past the end the first is read again, for nobody
                    const int ch = ch0 + i * 2 * nwaves, at = ch < count ? ch : ch0;
                    const float* part = a.part + ((size_t)chunk_slot(d[0], at, count, step, hk, gm.Hkv) * gm.G + g) * kPart;
                    ml[i] = *reinterpret_cast<const f32x2*>(part);
                    o[i] = *reinterpret_cast<const f32x4*>(part + 4 + c4);
                }
#pragma unroll
                for (int i = 0; i < kInFlight; ++i)
                    if (ch0 + i * 2 * nwaves < count) x.add(ml[i][0], ml[i][1], o[i]);
            }
        }
        const f32x4 other = {__shfl_xor(x.o[0], 32), __shfl_xor(x.o[1], 32), __shfl_xor(x.o[2], 32), __shfl_xor(x.o[3], 32)};
        x.add(__shfl_xor(x.m, 32), __shfl_xor(x.l, 32), other);
        if (lane < 32) *reinterpret_cast<f32x4*>(&so[seg][wave][c4]) = x.o;
        if (lane == 0) sm[seg * nwaves + wave] = x.m, sl[seg * nwaves + wave] = x.l;
    }
    __syncthreads();
    if (wave == 0) {  // lane = (segment, wavefront): its weight in Local (the window) and in Global (both segments)
        const bool on = lane < 2 * nwaves;
        const float m = on ? sm[lane] : -INFINITY, l = on ? sl[lane] : 0.f;
#pragma unroll
        for (int branch = 0; branch < 2; ++branch) {
            const float mb = lane < (branch + 1) * nwaves ? m : -INFINITY;
            float mx = mb;
            for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
            const float f = mb == -INFINITY ? 0.f : fast_exp2(mb - mx);
            float sum = l * f;
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
            if (on) sf[branch][lane] = f;
            if (lane == 0) st[branch][0] = mx, st[branch][1] = sum;
        }
    }
    __syncthreads();
    if (threadIdx.x >= kD) return;
    const int c = threadIdx.x;
    float out[2] = {0.f, 0.f};
    float lse[2] = {-INFINITY, -INFINITY};
#pragma unroll
    for (int branch = 0; branch < 2; ++branch) {
        if (branch == 0 ? !a.do_local : !routed) continue;
        float osum = 0.f;
        for (int seg = 0; seg <= branch; ++seg)
            for (int i = 0; i < nwaves; ++i) osum = fmaf(so[seg][i][c], sf[branch][seg * nwaves + i], osum);
        out[branch] = osum / st[branch][1];
        lse[branch] = (st[branch][0] + __builtin_amdgcn_logf(st[branch][1])) * kLn2;
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

// Slots of the partials: two per 512 keys of capacity and (batch, KV head).  Chunks never need more: a call's
// sub-blocks / chunk length + the rounding up of two segments per (batch, KV head).
static long long unit_slots(const Geom& g) { return 2 * ((long long)(g.T + 511) / 512); }
size_t decode_partial_floats(const Geom& g) { return (size_t)(g.B * g.Hkv * unit_slots(g)) * g.G * kPart; }

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
    const long long units = (long long)g.B * g.Hkv, slots = units * unit_slots(g);
    a.target = (int)(slots - 2 * units < kTargetChunks ? slots - 2 * units : kTargetChunks);
    a.unit_slots = g.B > kMaxScanBatch ? (int)unit_slots(g) : 0;
    const long long chunks = a.unit_slots ? slots : a.target + 2 * units;
    a.O = (__bf16*)O;
    a.S = (__bf16*)S;
    a.A = (__bf16*)A;
    a.lse_l = lse_l;
    a.lse_g = lse_g;
    {
        KernelTimer kt("decode_partial", st);
        const dim3 grid((unsigned)chunks);
        if (ring)
            hipLaunchKernelGGL(decode_partial_kernel<true>, grid, dim3(64 * kWaves), 0, st, a);
        else
            hipLaunchKernelGGL(decode_partial_kernel<false>, grid, dim3(64 * kWaves), 0, st, a);
    }
    {
        KernelTimer kt("decode_combine", st);
        // many heads: the chip is full with 4 wavefronts each; few: as many loads in flight as possible
        const int waves = g.B * g.Hq >= 512 ? 4 : kCombineWaves;
        hipLaunchKernelGGL(decode_combine_kernel, dim3(g.B * g.Hq), dim3(waves * 64), 0, st, a);
    }
    return launch_status();
}

}  // namespace l2a
