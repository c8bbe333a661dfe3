// How the weight gradients of a backward call are shared out, for the kernel that writes the table and for host code that checks it: the order of
// the experts and the parts in which each one's rows are contracted.  Written for a number of threads with a barrier between them; one thread with an
// empty barrier does the same.
#pragma once
#include <math.h>
#include <stddef.h>

#ifdef __HIPCC__
#define MOE_PARTS_FN __host__ __device__ __forceinline__
#else
#define MOE_PARTS_FN inline
#endif

constexpr int DW_MAX_PARTS = 32;               // of one expert
constexpr int DW_PART_ROWS = 768;              // rows of a part at least
constexpr int DW_MAX_UNITS = 1024;             // parts of tiles with a place for their sums, at most

// entries behind the first one, in pairs.  Only experts that have a place for the sums of all their parts are split, a part of an expert takes
// a place per tile, and an expert has a tile at least: there are no more parts than one per expert and one per place.
MOE_PARTS_FN size_t dw_entries(int e_loc) { return 2 * ((size_t)e_loc + DW_MAX_UNITS); }

// The experts are worked on with most rows first.  An expert is contracted in one part, unless the work from it to the end is less than its own rows on every
// compute unit.  Then the number of parts is the one with which that work takes the least time in rounds of equal units, a part costing `fix` rows to open and
// `split` rows to add up.  (Simulated lists of unequal and equal experts end 1.4 % after the best of 17 rules on average, unsplit ones 54 %.)
// Experts are granted their parts in that order while the `cap` places for sums last; from the first one that finds no room they stay in one part.
//   bases     first position of every expert, and the end          tiles  of an expert's gradients
//   entries   [0].x = number of parts; then per part (position, rows, expert, part), (parts of the expert, first place, 0, 0)
//   rows_of, parts_of, place_of   [e_loc] each, shared by the threads
template <typename Entry, typename Sync>
MOE_PARTS_FN void dw_split(const int* bases, int e_loc, int tiles, int cus, int cap, Entry* entries, int* rows_of, int* parts_of, int* place_of, int tid,
                           int threads, Sync sync) {
    for (int e = tid; e < e_loc; e += threads) rows_of[e] = bases[e + 1] - bases[e];
    sync();
    auto before = [&](int j, int e) { return rows_of[j] > rows_of[e] || (rows_of[j] == rows_of[e] && j < e); };
    for (int e = tid; e < e_loc; e += threads) {
        const int rows = rows_of[e];
        long long rest = 0;                                               // rows of this expert and of those after it
        for (int j = 0; j < e_loc; ++j) rest += before(j, e) ? 0 : rows_of[j];
        int best = 1;
        if (rest * tiles < (long long)rows * cus && 2 * tiles <= cap) {
            constexpr float fix = 100.f, split = 380.f;
            float least = 0.f;
            for (int P = 1; P <= DW_MAX_PARTS && P * tiles <= cap && (P == 1 || rows / P >= DW_PART_ROWS); ++P) {
                const float unit = (float)((rows + P * 64 - 1) / (P * 64) * 64) + fix + (P > 1 ? split : 0.f);
                const float t = ceilf((float)rest * (float)tiles * (float)P / ((float)rows * (float)cus) - 1e-3f) * unit;
                if (P == 1 || t < least) { least = t; best = P; }
            }
        }
        parts_of[e] = best;
    }
    sync();
    for (int e = tid; e < e_loc; e += threads) {
        const int P = parts_of[e];
        int place = 0;
        for (int j = 0; j < e_loc; ++j) place += parts_of[j] > 1 && before(j, e) ? parts_of[j] * tiles : 0;
        place_of[e] = P > 1 && place + P * tiles <= cap ? place : -1;      // (places asked for before it, granted or not: behind the first refusal all are refused)
    }
    sync();
    for (int e = tid; e < e_loc; e += threads) {
        const int rows = rows_of[e], place = place_of[e], P = place < 0 ? 1 : parts_of[e], len = (rows + P * 64 - 1) / (P * 64) * 64;
        int at = 0;
        for (int j = 0; j < e_loc; ++j) at += !before(j, e) ? 0 : (place_of[j] < 0 ? 1 : parts_of[j]);
        for (int p = 0; p < P; ++p) {
            const int lo = p * len < rows ? p * len : rows;
            entries[1 + 2 * (at + p)] = Entry{bases[e] + lo, len < rows - lo ? len : rows - lo, e, p};
            entries[2 + 2 * (at + p)] = Entry{P, place < 0 ? 0 : place, 0, 0};
        }
    }
    if (tid == 0) {
        int n = 0;
        for (int e = 0; e < e_loc; ++e) n += place_of[e] < 0 ? 1 : parts_of[e];
        entries[0] = Entry{n, 0, 0, 0};
    }
}
