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
constexpr int DW_MAX_EXPERTS = 4096;           // of a call (a power of two)

// entries behind the first one, in pairs.  Only experts that have a place for the sums of all their parts are split, a part of an expert takes
// a place per tile, and an expert has a tile at least: there are no more parts than one per expert and one per place.
MOE_PARTS_FN size_t dw_entries(int e_loc) { return 2 * ((size_t)e_loc + DW_MAX_UNITS); }

// The experts are worked on with most rows first.  An expert is contracted in one part, unless the work from it to the end is less than its own rows on every
// compute unit.  Then the number of parts is the one with which that work takes the least time in rounds of equal units, a part costing `fix` rows to open and
// `split` rows to add up.  (Simulated lists of unequal and equal experts end 1.4 % after the best of 17 rules on average, unsplit ones 54 %.)
// Experts are granted their parts in that order while the `cap` places for sums last; from the first one that finds no room they stay in one part.
//   bases     first position of every expert, and the end          tiles  of an expert's gradients
//   entries   [0].x = number of parts; then per part (position, rows, expert, part), (parts of the expert, first place, 0, 0)
//   rows, order   [least power of two >= e_loc] each, parts [e_loc], sums [threads]: shared by the threads
// The experts are sorted by exchanges (order among any number of them in log^2 steps) and what lies before each one is a prefix sum: loops over all experts for
// each of them took 60, 256 and 3467 us with 256, 1024 and 4096 experts, this takes 18, 29 and 70.
template <typename Entry, typename Sync>
MOE_PARTS_FN void dw_split(const int* bases, int e_loc, int tiles, int cus, int cap, Entry* entries, int* rows, int* order, int* parts, int* sums, int tid,
                           int threads, Sync sync) {
    int n = 1;
    while (n < e_loc) n *= 2;
    for (int e = tid; e < n; e += threads) { rows[e] = e < e_loc ? bases[e + 1] - bases[e] : -1; order[e] = e; }
    sync();
    auto before = [&](int i, int j) { return rows[i] > rows[j] || (rows[i] == rows[j] && order[i] < order[j]); };
    for (int run = 2; run <= n; run *= 2)
        for (int step = run / 2; step > 0; step /= 2) {
            for (int pair = tid; pair < n / 2; pair += threads) {
                const int i = 2 * pair - (pair & (step - 1)), j = i + step;
                if (before(j, i) == ((i & run) == 0)) {
                    const int r = rows[i], o = order[i];
                    rows[i] = rows[j]; order[i] = order[j];
                    rows[j] = r; order[j] = o;
                }
            }
            sync();
        }
    // every thread takes `len` experts next to each other; -> the sum of `mine` over the threads before it
    const int len = (e_loc + threads - 1) / threads, used = (e_loc + len - 1) / len;
    const int lo = tid * len < e_loc ? tid * len : e_loc, hi = lo + len < e_loc ? lo + len : e_loc;
    auto sum_before = [&](int mine) {
        sync();
        if (tid < used) sums[tid] = mine;
        sync();
        int sum = 0;
        if (used <= 16) {                                                 // (a few: less than the steps' barriers)
            if (tid < used)
                for (int j = 0; j < tid; ++j) sum += sums[j];
            return sum;
        }
        for (int off = 1; off < used; off *= 2) {
            const int v = tid < used && tid >= off ? sums[tid - off] : 0;
            sync();
            if (tid < used) sums[tid] += v;
            sync();
        }
        return tid < used ? sums[tid] - mine : 0;
    };
    int mine = 0;
    for (int i = lo; i < hi; ++i) mine += rows[i];
    int at = sum_before(mine), places = 0;
    const int all = bases[e_loc] - bases[0];
    for (int i = lo; i < hi; ++i) {
        const long long rest = all - at;                                  // rows of this expert and of those after it
        int best = 1;
        if (rest * tiles < (long long)rows[i] * cus && 2 * tiles <= cap) {
            constexpr float fix = 100.f, split = 380.f;
            float least = 0.f;
            for (int P = 1; P <= DW_MAX_PARTS && P * tiles <= cap && (P == 1 || rows[i] / P >= DW_PART_ROWS); ++P) {
                const float unit = (float)((rows[i] + P * 64 - 1) / (P * 64) * 64) + fix + (P > 1 ? split : 0.f);
                const float t = ceilf((float)rest * (float)tiles * (float)P / ((float)rows[i] * (float)cus) - 1e-3f) * unit;
                if (P == 1 || t < least) { least = t; best = P; }
            }
        }
        parts[i] = best;
        places += best > 1 ? best * tiles : 0;
        at += rows[i];
    }
    // places asked for before an expert, granted or not: behind the first refusal all are refused
    const int first = sum_before(places);
    auto granted = [&](int i, int place) { return place + parts[i] * tiles <= cap ? parts[i] : 1; };
    int place = first, entry = 0;
    for (int i = lo; i < hi; ++i) {
        entry += granted(i, place);
        place += parts[i] > 1 ? parts[i] * tiles : 0;
    }
    mine = entry;
    entry = sum_before(mine);
    if (tid == used - 1) entries[0] = Entry{entry + mine, 0, 0, 0};
    place = first;
    for (int i = lo; i < hi; ++i) {
        const int P = granted(i, place), e = order[i], span = (rows[i] + P * 64 - 1) / (P * 64) * 64;
        for (int p = 0; p < P; ++p, ++entry) {
            const int from = p * span < rows[i] ? p * span : rows[i];
            entries[1 + 2 * entry] = Entry{bases[e] + from, span < rows[i] - from ? span : rows[i] - from, e, p};
            entries[2 + 2 * entry] = Entry{P, P > 1 ? place : 0, 0, 0};
        }
        place += parts[i] > 1 ? parts[i] * tiles : 0;
    }
}
