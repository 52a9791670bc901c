// One read's pairs between two rounds of early termination (csrc/dtw_bnb.h).
#include "dtw_bnb.h"

extern "C" {

// Rounds that align every part of pair p to cost[p][row reached], or that
// give up where fails[p] == round; the final results.  max_n columns a pair.
void rounds(int n_pairs, int max_n, const int *n, const float *cost, const int *fails, int n_events, double b_match,
            int block_rows, int n_rounds, float *out_score, int *out_end, int *swept,
            int *took) {
    ra::BnbArgs b{};
    int64_t q_off[64] = {}, part_off[64];
    int read_of[64] = {}, part_len[64], part_row[64], part_end[64];
    uint8_t status[64], first[64];
    float part_score[64];
    uint64_t best = ra::order_key(-__builtin_inf());
    b.a.q_len = n;
    b.a.q_off = q_off;
    b.a.out_score = out_score;
    b.a.out_end = out_end;
    b.n_pairs = n_pairs;
    b.n_events = &n_events;
    b.b_match = b_match;
    b.s.read_of = read_of;
    b.s.status = status;
    b.s.best = &best;
    b.s.part_off = part_off;
    b.s.part_len = part_len;
    b.s.part_row = part_row;
    b.s.part_first = first;
    b.s.part_score = part_score;
    b.s.part_end = part_end;
    for (int p = 0; p < n_pairs; ++p) {
        status[p] = p == 0 ? ra::kBnbFirst : ra::kBnbWaiting;
        ra::bnb_part(b, p, 0, p == 0 || n[p] < block_rows ? n[p] : block_rows);
        swept[p] = took[p] = 0;
    }
    for (int round = 0; round < n_rounds; ++round) {
        for (int p = 0; p < n_pairs; ++p) {
            if (part_row[p] < 0) continue;
            const int to = part_row[p] + part_len[p];
            swept[p] = to;
            took[p] |= 1 << round;
            const bool lost = fails[p] == round;
            part_score[p] = lost ? __builtin_nanf("") : cost[p * max_n + to - 1];
            part_end[p] = lost ? -5 : p;
        }
        for (int p = 0; p < n_pairs; ++p) {
            uint64_t key;
            if (ra::bnb_finish(b, p, key) >= 0 && key > best) best = key;
        }
        if (round + 1 < n_rounds)
            for (int p = 0; p < n_pairs; ++p) ra::bnb_advance(b, p, block_rows, round + 2 == n_rounds);
    }
}
}
