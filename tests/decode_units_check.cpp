// Host-side check of the decode step's division of work (csrc/decode_units.hpp): all workgroups of a launch are replayed
// and every unit that a sequence needs has to be taken exactly once, by whom the two walks' loops say.  Built with
// g++ by tests/test_decode_units.py; no GPU code.
#include <cstdarg>
#include <cstdio>
#include <map>
#include <tuple>
#include <vector>

#include "../paper_2603_17484_amd/csrc/decode_units.hpp"

using namespace l2a::units;

static int fail(char* msg, int len, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(msg, len, fmt, ap);
    va_end(ap);
    return 1;
}

extern "C" {

// t, win, routed: per sequence.  wgs: workgroups per XCD.  *alone: units taken by single wavefronts.
int units_check(int B, int heads, int local, const int* t, const int* win, const int* routed, int wgs, int* alone, char* msg, int len) {
    msg[0] = 0;
    *alone = 0;
    std::map<std::tuple<int, int, int, int>, int> seen;  // (sequence, routed, rank, chunk) -> times
    for (int xcd = 0; xcd < 8; ++xcd) {
        int all = 0;
        for (int b = 0; b < B; ++b) all += seq_share(Keys{t[b], win[b], local}, heads, routed[b], residue(xcd, b));
        std::vector<int> taken(all, 0);
        const int by = by_wave(all, wgs);
        for (int w = 0; w < wgs; ++w) {
            for (int wave = 0; wave < kWaves; ++wave)
                for (int i = w * kWaves + wave; i < (by < all ? by : all); i += kWaves * wgs) ++taken[i], ++*alone;
            for (int i = by + w; i < all; i += wgs) ++taken[i];
        }
        int i0 = 0;
        for (int b = 0; b < B; ++b) {
            const Keys s{t[b], win[b], local};
            const int r = residue(xcd, b), n = seq_share(s, heads, routed[b], r);
            for (int i = 0; i < n; ++i) {
                if (taken[i0 + i] != 1) return fail(msg, len, "XCD %d: unit %d of %d taken %d times", xcd, i0 + i, all, taken[i0 + i]);
                const Place p = place(s, heads, routed[b], i, r);
                ++seen[std::make_tuple(b, p.routed, p.rank, p.c)];
            }
            i0 += n;
        }
    }
    // what the sequences need, key by key: each branch's keys covered by its chunks, every unit's keys its own
    size_t want = 0;
    for (int b = 0; b < B; ++b) {
        const Keys s{t[b], win[b], local};
        for (int kind = 0; kind < 2; ++kind)
            for (int rank = 0; rank < (kind ? routed[b] : heads - routed[b]); ++rank) {
                std::vector<int> need;  // chunks, as the merge reads them
                if (kind)
                    for (int c = 0; c <= t[b] / 512; ++c) need.push_back(c);
                else if (local)
                    for (int c = win[b] / 512 + (win[b] % 512 != 0); c <= t[b] / 512; ++c) need.push_back(c);
                if (local && win[b] % 512 != 0) need.push_back(kEdge);
                want += need.size();
                for (int c = kEdge; c < t[b] / 512 + 3; ++c) {  // without a plan: every place where a partial may go
                    int in = 0;
                    for (int x : need) in += x == c;
                    if (in != (kind || local ? needed(s, c, kind != 0) : 0)) return fail(msg, len, "sequence %d, chunk %d: needed or not?", b, c);
                }
                for (int c : need) {
                    if (seen[std::make_tuple(b, kind, rank, c)] != 1)
                        return fail(msg, len, "sequence %d, %s head %d, chunk %d: %d times", b, kind ? "routed" : "unrouted", rank, c, seen[std::make_tuple(b, kind, rank, c)]);
                    const int lo = first_key(s, c), hi = last_key(s, lo);
                    const int end = (c == kEdge ? win[b] / 512 : c) * 512 + 511;
                    if (lo != (c == kEdge ? win[b] : 512 * c) || hi != (end < t[b] ? end : t[b]) || lo > hi)
                        return fail(msg, len, "sequence %d, chunk %d: keys %d..%d", b, c, lo, hi);
                }
            }
    }
    if (seen.size() != want) return fail(msg, len, "%d units, %d wanted", (int)seen.size(), (int)want);
    return 0;
}

}  // extern "C"
