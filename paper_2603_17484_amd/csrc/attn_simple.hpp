// Scalar-FMA arithmetic of the layer, one query row (forward, dQ) or one key token (dK/dV) at a time: four
// adjacent lanes share a row, each keeps DL = D/4 of its channels in registers, and partial dot products
// are combined with two cross-lane exchanges.  Keys a row does not see are never touched, so whatever
// they hold stays out of its results.  Used by the kernels of attn_simple.hip, and by those of
// attn_fp32.hip for tiles whose matrix-core result is not finite.
//
// Forward: streaming softmax over the row's keys (App. C Alg. 1, with a key tile of one);
// backward: the standard softmax-attention gradient restricted to the routed rows (Sec. 3.2).
#pragma once
#include "common.hpp"
#include "dkdv_walk.hpp"

namespace l2a {
namespace {

template <typename E>
__device__ __forceinline__ float ld(const E* p) {
    return (float)*p;
}
template <typename E>
__device__ __forceinline__ void st(E* p, float x) {
    *p = (E)x;
}

__device__ __forceinline__ float quad_sum(float x) {
    x += __shfl_xor(x, 1);
    x += __shfl_xor(x, 2);
    return x;
}

struct Row {
    int pos, g;
};

// rows of one (b, KV head): how many, and the r-th one (device data: clamped into the valid ranges)
__device__ __forceinline__ int num_rows(const RowSet& rs, const Geom& gm, int bh) {
    return rs.count ? min(max(rs.count[bh], 0), gm.T * gm.G) : gm.T * gm.G;
}
__device__ __forceinline__ Row get_row(const RowSet& rs, const Geom& gm, int bh, int r) {
    const int code = rs.row_idx ? min(max(rs.row_idx[(size_t)bh * gm.T * gm.G + r], 0), gm.T * gm.G - 1) : r;
    Row x;
    x.pos = code / gm.G;
    x.g = code - x.pos * gm.G;
    return x;
}

// Running sums of a row over the keys j0 .. j1 (inclusive; none if j1 < j0): m, l and acc as in the streaming softmax
template <typename E, int DL>
__device__ __forceinline__ void simple_fwd_keys(const Geom& gm, const E* __restrict__ q, const E* __restrict__ k,
                                                const E* __restrict__ v, int b, int hk, size_t qoff, int part, int j0, int j1,
                                                float& m, float& l, float (&acc)[DL]) {
    float qr[DL];
#pragma unroll
    for (int i = 0; i < DL; ++i) {
        qr[i] = ld(q + qoff + i);
        acc[i] = 0.f;
    }
    m = -INFINITY, l = 0.f;
    for (int j = j0; j <= j1; ++j) {
        const size_t koff = (((size_t)b * gm.T + j) * gm.Hkv + hk) * gm.D + part * DL;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < DL; ++i) s += qr[i] * ld(k + koff + i);
        s = quad_sum(s) * gm.scale;
        const float mn = fmaxf(m, s);
        const float alpha = expf(m - mn);
        const float p = expf(s - mn);
        l = l * alpha + p;
#pragma unroll
        for (int i = 0; i < DL; ++i) acc[i] = acc[i] * alpha + p * ld(v + koff + i);
        m = mn;
    }
}

// Forward of row r of (b, KV head) bh, channels part * DL ..
template <typename E, int DL>
__device__ __forceinline__ void simple_fwd_row(const Geom& gm, const RowSet& rs, const E* __restrict__ q,
                                               const E* __restrict__ k, const E* __restrict__ v, const FwdOut& out,
                                               int bh, int r, int part) {
    const int b = bh / gm.Hkv, hk = bh % gm.Hkv;
    if (r >= num_rows(rs, gm, bh)) return;
    const Row row = get_row(rs, gm, bh, r);
    const int h = hk * gm.G + row.g;
    const size_t qoff = (((size_t)b * gm.T + row.pos) * gm.Hq + h) * gm.D + part * DL;

    float acc[DL], m, l;
    simple_fwd_keys<E, DL>(gm, q, k, v, b, hk, qoff, part, rs.local ? max(row.pos - gm.W, 0) : 0, row.pos, m, l, acc);
    const float inv = 1.f / l;
    E* mo = (E*)out.main_out;
    E* co = (E*)out.copy_out;
    E* zf = (E*)out.zero_fill;
#pragma unroll
    for (int i = 0; i < DL; ++i) {
        const float x = acc[i] * inv;
        const float y = out.merge ? ld(mo + qoff + i) + x : x;
        st(mo + qoff + i, y);
        if (co) st(co + qoff + i, x);
        if (zf) st(zf + qoff + i, 0.f);
    }
    if (part == 0) {
        const size_t so = ((size_t)b * gm.Hq + h) * gm.T + row.pos;
        out.lse_out[so] = m + logf(l);
        if (out.lse_fill) out.lse_fill[so] = -INFINITY;
    }
}

// dQ (not scaled) and sum_j p_j dp_j of a row over the keys j0 .. j1
template <typename E, int DL>
__device__ __forceinline__ void simple_dq_keys(const Geom& gm, const E* __restrict__ q, const E* __restrict__ k,
                                               const E* __restrict__ v, const E* __restrict__ dO, int b, int hk, size_t qoff,
                                               int part, int j0, int j1, float L, float dl, float& dx, float (&acc)[DL]) {
    float qr[DL], gr[DL];
#pragma unroll
    for (int i = 0; i < DL; ++i) {
        qr[i] = ld(q + qoff + i);
        gr[i] = ld(dO + qoff + i);
        acc[i] = 0.f;
    }
    dx = 0.f;  // the delta of the row without the rounding of the saved output
    for (int j = j0; j <= j1; ++j) {
        const size_t koff = (((size_t)b * gm.T + j) * gm.Hkv + hk) * gm.D + part * DL;
        float s = 0.f, dp = 0.f;
#pragma unroll
        for (int i = 0; i < DL; ++i) {
            s += qr[i] * ld(k + koff + i);
            dp += gr[i] * ld(v + koff + i);
        }
        s = quad_sum(s) * gm.scale;
        dp = quad_sum(dp);
        const float p = expf(s - L);
        const float ds = p * (dp - dl);
        dx += p * dp;
#pragma unroll
        for (int i = 0; i < DL; ++i) acc[i] += ds * ld(k + koff + i);
    }
}

// dQ and the exact delta of that row
template <typename E, int DL>
__device__ __forceinline__ void simple_dq_row(const Geom& gm, const RowSet& rs, const E* __restrict__ q,
                                              const E* __restrict__ k, const E* __restrict__ v,
                                              const E* __restrict__ dO, const float* __restrict__ lse, float* delta,
                                              E* dq, int accumulate, int bh, int r, int part) {
    const int b = bh / gm.Hkv, hk = bh % gm.Hkv;
    if (r >= num_rows(rs, gm, bh)) return;
    const Row row = get_row(rs, gm, bh, r);
    const int h = hk * gm.G + row.g;
    const size_t qoff = (((size_t)b * gm.T + row.pos) * gm.Hq + h) * gm.D + part * DL;
    const size_t so = ((size_t)b * gm.Hq + h) * gm.T + row.pos;

    float acc[DL], dl_exact;
    simple_dq_keys<E, DL>(gm, q, k, v, dO, b, hk, qoff, part, rs.local ? max(row.pos - gm.W, 0) : 0, row.pos, lse[so], delta[so],
                          dl_exact, acc);
    if (part == 0) delta[so] = dl_exact;
#pragma unroll
    for (int i = 0; i < DL; ++i) {
        float x = acc[i] * gm.scale;
        if (accumulate) x += ld(dq + qoff + i);
        st(dq + qoff + i, x);
    }
}

struct DkdvSets {
    RowSet rs[2];
    const float* lse[2];
    const float* delta[2];
    const float* share[2] = {nullptr, nullptr};  // optional: the rows' weights count 1 + share times (see row_stats)
    int n;
};

// dK, dV of key token j
template <typename E, int DL>
__device__ __forceinline__ void simple_dkdv_key(const Geom& gm, const DkdvSets& sets, const E* __restrict__ q,
                                                const E* __restrict__ k, const E* __restrict__ v,
                                                const E* __restrict__ dO, E* dk, E* dv, int bh, int j, int part) {
    const int b = bh / gm.Hkv, hk = bh % gm.Hkv;
    if (j >= gm.T) return;
    const size_t koff = (((size_t)b * gm.T + j) * gm.Hkv + hk) * gm.D + part * DL;
    float kr[DL], vr[DL], ak[DL], av[DL];
#pragma unroll
    for (int i = 0; i < DL; ++i) {
        kr[i] = ld(k + koff + i);
        vr[i] = ld(v + koff + i);
        ak[i] = 0.f;
        av[i] = 0.f;
    }
    const int nkb = (gm.T + 63) / 64;
    for (int s = 0; s < sets.n; ++s) {
        const RowSet rs = sets.rs[s];
        int r0, r1;  // candidate rows [r0, r1)
        if (rs.local) {
            const int last = j + gm.W < gm.T - 1 ? j + gm.W : gm.T - 1;
            r0 = j * gm.G;
            r1 = (last + 1) * gm.G;
        } else {
            r0 = rs.kblk_first_row ? max(rs.kblk_first_row[(size_t)bh * (nkb + 1) + walk::list_bounds(j, rs.shift, nkb).lo], 0) : (j >> 6) * 64 * gm.G;
            r1 = num_rows(rs, gm, bh);
        }
        for (int r = r0; r < r1; ++r) {
            const Row row = get_row(rs, gm, bh, r);
            if (row.pos - rs.shift < j) continue;
            const int h = hk * gm.G + row.g;
            const size_t qoff = (((size_t)b * gm.T + row.pos) * gm.Hq + h) * gm.D + part * DL;
            const size_t so = ((size_t)b * gm.Hq + h) * gm.T + row.pos;
            float sc = 0.f, dp = 0.f;
#pragma unroll
            for (int i = 0; i < DL; ++i) {
                sc += ld(q + qoff + i) * kr[i];
                dp += ld(dO + qoff + i) * vr[i];
            }
            sc = quad_sum(sc) * gm.scale;
            dp = quad_sum(dp);
            const float p = expf(sc - sets.lse[s][so]) * (sets.share[s] ? 1.f + sets.share[s][so] : 1.f);
            const float ds = p * (dp - sets.delta[s][so]);
#pragma unroll
            for (int i = 0; i < DL; ++i) {
                av[i] += p * ld(dO + qoff + i);
                ak[i] += ds * ld(q + qoff + i);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < DL; ++i) {
        st(dk + koff + i, ak[i] * gm.scale);
        st(dv + koff + i, av[i]);
    }
}

}  // namespace
}  // namespace l2a
