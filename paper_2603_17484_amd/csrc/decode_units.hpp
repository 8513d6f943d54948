// Which unit of work each workgroup of the decode step's first kernel has: plain integer code, compiled for the kernel
// and for the host, where the CPU test replays every workgroup and checks that each unit is taken exactly once.
//
// A unit is the keys of one chunk that one KV head of a sequence needs.  Chunk c is keys 512 c .. 512 c + 511 of the cache,
// whatever else is in the batch.  A KV head whose prefix is needed has all chunks up to the new token's; one that needs
// the window alone those that lie in it whole; and either, for the Local branch, the chunk the window begins
// inside of, from there on (kEdge).
#pragma once

#ifdef __HIPCC__
#define L2A_UNITS_FN __host__ __device__ inline __attribute__((always_inline))
#else
#define L2A_UNITS_FN inline
#endif

namespace l2a {
namespace units {

constexpr int kChunk = 512;  // keys of a chunk
constexpr int kSub = 32;     // keys per wavefront step
constexpr int kWaves = 4;    // wavefronts of a workgroup
constexpr int kEdge = -1;

struct Keys {
    int t, win;  // last cache row that counts, first one of the window
    int local;   // whether the Local branch runs
    L2A_UNITS_FN int chunks() const { return t / kChunk + 1; }
    L2A_UNITS_FN int edge() const { return local && win % kChunk != 0 ? 1 : 0; }
    L2A_UNITS_FN int first() const { return (win + kChunk - 1) / kChunk; }  // the first chunk that lies in the window whole
    L2A_UNITS_FN int n_prefix() const { return chunks() + edge(); }
    L2A_UNITS_FN int n_window() const { return local ? chunks() - first() + edge() : 0; }
};

// With a head's units numbered v = 0, 1, ..., XCD number x takes those with v = x - b modulo 8 of every KV head of sequence
// b: the heads that read the same rows of the cache do so through one L2, and the sequence's number rotates
// the shares (8 x 128K tokens, 2 routed: 123.5 us with the heads on any XCD, 118.4 so).
L2A_UNITS_FN int residue(int xcd, int b) { return (xcd - b) & 7; }
L2A_UNITS_FN int share_of(int n, int r) { return (n - r + 7) >> 3; }  // numbers below n that are r modulo 8
L2A_UNITS_FN int seq_share(const Keys& s, int heads, int routed, int r) {
    return routed * share_of(s.n_prefix(), r) + (heads - routed) * share_of(s.n_window(), r);
}
// The i-th unit of that share: the prefix's first, all heads' v-th ones together.
struct Place {
    int routed, rank, c;  // the rank-th of the heads that are routed, or not; its chunk
};
L2A_UNITS_FN Place place(const Keys& s, int heads, int routed, int i, int r) {
    const int n = routed * share_of(s.n_prefix(), r);
    const bool prefix = i < n;
    const int j = prefix ? i : i - n, of = prefix ? routed : heads - routed;
    const int v8 = j / of, v = 8 * v8 + r;
    if (prefix) return Place{1, j - v8 * of, v < s.chunks() ? v : kEdge};
    return Place{0, j - v8 * of, v < s.edge() ? kEdge : s.first() + v - s.edge()};
}
// Whether a head needs chunk c at all.
L2A_UNITS_FN bool needed(const Keys& s, int c, bool prefix) {
    if (c == kEdge) return s.edge() != 0;
    return c < s.chunks() && (prefix || (s.local && c >= s.first()));
}
L2A_UNITS_FN int first_key(const Keys& s, int c) { return c == kEdge ? s.win : c * kChunk; }
L2A_UNITS_FN int last_key(const Keys& s, int lo) {
    const int end = lo / kChunk * kChunk + kChunk - 1;
    return end < s.t ? end : s.t;
}

// Whether the workgroups plan the batch, each going through all its sequences, 64 at a time, or a wavefront is launched for every
// place where a partial may go and finds out whether it is needed.  Whole step, us, planned / not: 8 x 128K tokens, 2 routed
// 118 / 130, none routed 22 / 32; 64 x 8K 134 / 135; 256 x 4K, W = 1024 90 / 97, 256 x 1K 37 / 34; 512 x 1K 58 / 55, 4K 198 / 192; 4096 x
// 512 194 / 138; 16384 x 256 494 / 278.  With decisions of its own for every head a sequence takes longer to plan: 65 x 1K
// 30 / 24, 128 x 1K 39 / 28, but 8 x 128K, 2 % routed 78 / 98.
inline bool planned(long long batch, bool per_head) { return batch <= (per_head ? 64 : 256); }

// How many of an XCD's units its `wgs` workgroups work on with a wavefront each (full rounds of kWaves wgs; the last one
// may be a half); the others are for whole workgroups.  A unit takes a wavefront 14 us, a workgroup 4; but while the chip
// streams, wavefronts that never wait for each other keep more loads on their way.  Whole step, us, all by workgroups /
// by this rule: 8 x 128K tokens, all routed 460 / 393, 2 routed 141 / 121, none 21 / 22 (by wavefronts alone 27); 1 x
// 32K 23 / 23 (31); 16 x 32K, 4 routed (2.9 units per workgroup) 88 / 81 (with a merge that took 2-4 us longer).
L2A_UNITS_FN int by_wave(int all, int wgs) { return (all + 2 * wgs) / (kWaves * wgs) * (kWaves * wgs); }

}  // namespace units
}  // namespace l2a
