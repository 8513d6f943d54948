// Host-side check of the dK/dV kernel's launch order by heads (csrc/dkdv_walk.hpp: host_launch, head_job, walk_down):
// every (head, key block, split) is one job, every XCD gets the same number of jobs, and with the walk direction
// the kernel takes the loads and the arithmetic visit the same tiles in the same order, each tile with a pair
// that counts once, none that needs a mask unmasked.  Built with g++ by tests/test_dkdv_heads.py; no GPU code.
#include "dkdv_walk_check.cpp"

extern "C" {

void heads_launch(int T, long long nbh, int W, int* out5) {
    const Launch l = host_launch(T, nbh, W);
    out5[0] = l.nblk, out5[1] = l.groups, out5[2] = l.chunk, out5[3] = l.nsplit, out5[4] = l.jobs;
}

int heads_jobs_check(int nblk, int nbh, int groups, int nsplit, char* msg, int len) {
    msg[0] = 0;
    const int jobs = 8 * (nbh / groups) * head_jobs(nblk, groups, nsplit);
    std::vector<int> seen((size_t)nbh * nblk * nsplit, 0);
    for (int lin = 0; lin < jobs; ++lin) {
        const Job j = head_job(lin, nblk, groups, nsplit);
        if (j.bh < 0 || j.bh >= nbh || j.kblk < 0 || j.z < 0 || j.z >= nsplit) return fail(msg, len, "job %d out of range: head %d block %d split %d", lin, j.bh, j.kblk, j.z);
        if (j.kblk >= nblk) continue;  // empty
        if (seen[((size_t)j.bh * nblk + j.kblk) * nsplit + j.z]++) return fail(msg, len, "job %d: head %d block %d split %d twice", lin, j.bh, j.kblk, j.z);
        if (groups == 8 && j.bh % 8 != (lin & 7)) return fail(msg, len, "job %d: head %d on another XCD", lin, j.bh);
    }
    for (size_t i = 0; i < seen.size(); ++i)
        if (!seen[i]) return fail(msg, len, "job missing: %d", (int)i);
    return 0;
}

// the walk of every key block and split with chunk and direction as the kernel takes them
int heads_walk_check(int T, int G, int W, int chunk, int nsplit, int nsets, const int* kinds, const int* rows_pos, int nrows,
                     int* n_down, char* msg, int len) {
    msg[0] = 0;
    *n_down = 0;
    const int Wc = W < T ? W : T, nkb = (T + 63) / 64, nblk = (T + kKeysPerWg - 1) / kKeysPerWg;
    SetDesc sets[2];
    for (int s = 0; s < nsets; ++s) {
        sets[s].kind = kinds[s];
        if (kinds[s] == kListRows) {
            sets[s].pos.assign(rows_pos, rows_pos + nrows);
            sets[s].first.assign(nkb + 1, 0);
            for (int k = 0; k <= nkb; ++k)
                for (int r = 0; r < nrows; ++r) sets[s].first[k] += rows_pos[r] < 64 * k;
        } else {
            for (int r = 0; r < T * G; ++r) sets[s].pos.push_back(r / G);
        }
    }
    for (int kblk = 0; kblk < nblk; ++kblk) {
        const int k0 = kblk * kKeysPerWg;
        const bool down = walk_down(kblk, chunk, T, Wc);
        *n_down += down;
        std::vector<int> visits[2];
        for (int s = 0; s < nsets; ++s) visits[s].assign((sets[s].pos.size() + kRT - 1) / kRT + 1, 0);
        for (int z = 0; z < nsplit; ++z) {
            Runs r[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
            bool local[2] = {false, false};
            for (int s = 0; s < nsets; ++s) {
                const bool list = sets[s].kind == kListRows;
                const int e = (k0 + kKeysPerWg) >> 6;
                r[s] = tile_runs(sets[s].kind, k0, T, G, Wc, list ? sets[s].first[k0 >> 6] : 0,
                                 list ? sets[s].first[e < nkb ? e : nkb] : 0, (int)sets[s].pos.size(), nsplit, z);
                local[s] = sets[s].kind == kLocalRows && !down;
            }
            const Plan plan = make_plan(nsets, r[0], local[0], r[1], local[1], kblk, chunk, T, G, 1);
            std::vector<int> seg_set, seg_masked;
            for_each_segment(plan, [&](int s, bool masked, int count) {
                for (int i = 0; i < count; ++i) seg_set.push_back(s), seg_masked.push_back(masked);
            });
            if ((int)seg_set.size() != plan.total) return fail(msg, len, "block %d split %d: %d steps, plan %d", kblk, z, (int)seg_set.size(), plan.total);
            Cursor c = cursor_begin(plan);
            int first_tile[2] = {-1, -1};
            for (int i = 0; i < plan.total; ++i, cursor_advance(c, plan)) {
                const int s = (int)c.set;
                if (s != seg_set[i] || c.t < r[s].tb || c.t >= r[s].te) return fail(msg, len, "block %d split %d step %d: set %d tile %d", kblk, z, i, s, c.t);
                if (first_tile[s] < 0) first_tile[s] = c.t;
                ++visits[s][c.t];
                if (!seg_masked[i] && !brute(sets[s], c.t, k0, T, Wc).all) return fail(msg, len, "block %d split %d: tile %d of set %d runs unmasked", kblk, z, c.t, s);
            }
            for (int s = 0; s < nsets; ++s)  // the point of walking down: all blocks of the chunk start on the same tile
                if (down && nsplit == 1 && first_tile[s] >= 0 && first_tile[s] != ((int)sets[s].pos.size() - 1) / kRT)
                    return fail(msg, len, "block %d walked down starts on tile %d of set %d", kblk, first_tile[s], s);
        }
        for (int s = 0; s < nsets; ++s)
            for (int t = 0; t < (int)visits[s].size(); ++t)
                if (visits[s][t] > 1 || (visits[s][t] == 0 && brute(sets[s], t, k0, T, Wc).any)) return fail(msg, len, "block %d: tile %d of set %d visited %d times", kblk, t, s, visits[s][t]);
    }
    return 0;
}

}  // extern "C"
