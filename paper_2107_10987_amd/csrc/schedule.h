// How a stage launch is split over workgroups: the host's rules, without HIP.
#pragma once

#include <stdint.h>

#include <initializer_list>

#include "../../include/hydro.h"

namespace hydro {

enum Kernel { KERNEL_FACE = 0, KERNEL_COLUMN = 1, KERNEL_PERSISTENT = 2 };

// Workgroups per leaf of `left` blocks that have num_cu compute units to
// themselves, so that all of them run at once; 1 where whole leaves take more
// than half of them (150 leaves as 300 halves: two rounds of 41 us against one
// of 68).
inline int leaf_parts(int left, int num_cu) {
    for (int t : {8, 4, 3, 2})
        if ((int64_t)t * left <= num_cu) return t;
    return 1;
}

// Blocks that run at one time while a launch of nleaf of a stage's nstage
// blocks does: all of them where every launch has a stream of its own; where
// `streams` take the stage's nlaunch launches in turn, four fifths of what so
// many launches hold, for they do not end together and the next one's start
// leaves gaps (60 launches of 10 leaves on 4 streams: 0.37 ms in 8 parts, which
// 32 leaves at a time would fill the chip with, 0.44 in 4).
inline int blocks_beside(int nleaf, int nstage, int nlaunch, int streams) {
    const int64_t held = nlaunch > streams ? (int64_t)nstage * streams * 4 / (5 * (int64_t)nlaunch) : nstage;
    return held > nleaf ? (int)held : nleaf;
}

// Schedule of a launch without a table: parts of leaves where whole ones, of
// all launches that run beside it, leave half the chip idle (ten launches of 32
// leaves: 164 us in halves, 245 whole).
inline int auto_schedule(int beside, int num_cu) {
    return leaf_parts(beside, num_cu) > 1 ? HYDRO_SCHED_TILED : HYDRO_SCHED_COLUMN;
}

// Autotune bucket of a launch of nleaf blocks: launch sizes [2^b, 2^(b+1)).
inline int bucket_of(int nleaf) {
    int b = 0;
    while ((2 << b) <= nleaf && b < HYDRO_NBUCKET - 1) ++b;
    return b;
}

// Schedule of a launch of nleaf blocks by an autotune table.  A bucket's
// HYDRO_SCHED_TILED stands for parts of leaves, which run at once up to half
// of the compute units; past that the column walk takes whole leaves, not the
// queue of axis items that TILED is there when a caller asks for it (128
// leaves: 41 us as halves, 68 whole; 129 leaves 79 us from the queue, 68 whole;
// 255 leaves 127 and 73; 512 leaves 226 and 145).
inline int table_schedule(const int32_t table[HYDRO_NBUCKET], int nleaf, int beside, int num_cu) {
    const int s = table[bucket_of(nleaf)];
    return s == HYDRO_SCHED_TILED ? auto_schedule(beside, num_cu) : s;
}

// A launch of the column walk: the first `whole` blocks by a workgroup each
// and the others in `tiles` parts (direct), or `tiles` items a block from the
// queue (persistent).
struct Split {
    int kernel, tiles, whole;
};

// Split of a launch of nleaf blocks by schedule sched, `beside` blocks running
// at one time (blocks_beside); alone: no other launch of the stage runs beside
// it.
inline Split split_launch(int sched, int nleaf, int beside, bool alone, int num_cu) {
    Split s{KERNEL_COLUMN, 1, nleaf};
    switch (sched) {
    case HYDRO_SCHED_FACE: s.kernel = KERNEL_FACE; break;
    case HYDRO_SCHED_PERSISTENT: s.kernel = KERNEL_PERSISTENT; break;
    case HYDRO_SCHED_TILED:
        // the parts of all launches at once; where those do not fit but this
        // launch's do, halves (ten launches of 40 leaves: 0.19 ms)
        s.tiles = leaf_parts(beside, num_cu);
        if (s.tiles == 1 && leaf_parts(nleaf, num_cu) > 1) s.tiles = 2;
        s.whole = 0;
        if (s.tiles == 1) {   // a queue of axis items
            s.kernel = KERNEL_PERSISTENT;
            s.tiles = 3;
        }
        break;
    default:
        // a last round that would leave half the chip idle runs as parts
        if (alone && nleaf > num_cu && nleaf % num_cu) {
            s.tiles = leaf_parts(nleaf % num_cu, num_cu);
            if (s.tiles > 1) s.whole = nleaf - nleaf % num_cu;
        }
    }
    return s;
}

}  // namespace hydro
