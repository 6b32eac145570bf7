// A workgroup's way through a batch: which cloud its team samples next and
// when the team splits.  One definition for the kernel and for the host tests,
// which run it with a thread per workgroup.
//
// All workgroups of an XCD start as one team of the largest level; a team
// takes the level's clouds until none is left and then splits in two for the
// next level, down to single workgroups.  Teams never join again, so a level's
// control word, once it says "no more", stays.
//
// Every posted cloud costs at least one exchange, which the leader cannot
// finish before every member has read the post, and nothing follows the post
// that ends the level, so a post is never overwritten unread.
//
// Inside a team a slot is written again two exchanges on, which the writer
// reaches only after every member has published the exchange between, and so
// has read the slot.  A split ends that: one half may run two exchanges before
// a member of the other half has read the last one of the whole team.  So a
// team splits only when all of its workgroups have arrived, each after its
// last read.
#pragma once

#if defined(__HIP__)
#include <hip/hip_runtime.h>
#endif

#include "round_layout.h"

#if defined(__HIP__)
#define RFPS_TEAM_FN __device__ __forceinline__
#else
#define RFPS_TEAM_FN inline
#endif

namespace rfps {

constexpr uint32_t kNoCloud = 0xffffffffu;  // a wait expired

// The team's next place in the order of the clouds (its level's `last` or
// beyond when there is none left and the team has split), by one thread of
// every workgroup of the team.  io:
//   next(lev)         takes a place of the level, counted from 0
//   wanted(q)         the cloud at place q needs an exchange
//   post(lev, T, v), posted(lev, T)       the team's control word
//   arrive(lev, T), arrived(lev, T)       its count of workgroups that left the level
//   kSpins            looks at a word before a wait expires
template <class Io>
RFPS_TEAM_FN uint32_t team_next(Io &io, int lev, int T, int rank, uint32_t turn, uint32_t first, uint32_t last)
{
    uint32_t q = kNoCloud;
    if (rank == 0) {
        do {
            q = first + io.next(lev);
        } while (q < last && !io.wanted(q));
        q = q < last ? q : last;
        if (T > 1)
            io.post(lev, T, ((unsigned long long)turn << 32) | q);
    } else {
        for (uint32_t spin = 0; spin < io.kSpins; ++spin) {
            const unsigned long long v = io.posted(lev, T);
            if ((uint32_t)(v >> 32) == turn) {
                q = (uint32_t)v;
                break;
            }
        }
    }
    if (q == last && T > 1) {
        io.arrive(lev, T);
        uint32_t spin = 0;
        while (io.arrived(lev, T) < (unsigned long long)T && spin < io.kSpins)
            ++spin;
        if (spin >= io.kSpins)
            q = kNoCloud;
    }
    return q;
}

// All levels, by every thread of workgroup `xrank` of the XCD.  io, besides:
//   first(lev)        first place of the level (its clouds: up to first(lev + 1))
//   one(f)            f() by one thread, for all
//   sample(lev, T, rank, q)       the cloud at place q; false ends the workgroup
// Returns false when a wait expired or a cloud failed.
template <class Io>
RFPS_TEAM_FN bool walk_levels(Io &io, int per_xcd, int xrank)
{
    uint32_t turn = 0;
    for (int lev = 0; lev < kBatchLevels && (per_xcd >> lev) > 0; ++lev) {
        const int T = per_xcd >> lev, rank = xrank & (T - 1);
        const uint32_t first = io.first(lev), last = io.first(lev + 1);
        if (first == last)
            continue;
        for (;;) {
            ++turn;
            const uint32_t q = io.one([&] { return team_next(io, lev, T, rank, turn, first, last); });
            if (q == kNoCloud)
                return false;
            if (q >= last)
                break;
            if (!io.sample(lev, T, rank, q))
                return false;
        }
    }
    return true;
}

}  // namespace rfps
