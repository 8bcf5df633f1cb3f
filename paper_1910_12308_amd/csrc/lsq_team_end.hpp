// What a workgroup of a least-squares team (lsq_team.hip) does that has waited long enough for the others.  On plain integers and
// with the accesses to the team's claim passed in, so that the model of a team on the host (tests/lsq_team_end.cpp) runs these lines.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define SWARM_TEAM_FN __host__ __device__ __forceinline__
#else
#define SWARM_TEAM_FN inline
#endif

namespace swarm {

// Of a team's part of a launch: number of its first step << 32 | how many of its steps are left to all workgroups.  The one whose
// claim is the first of the launch takes the others by itself.
typedef unsigned long long TeamClaim;

enum class TeamWait { GO_ON, END, ALONE, LOST };

// At the launch's step `done`, for a workgroup that holds columns: it has had the whole totals of every step before, so that these
// are there for all others too.  (One that adds some of the rows knows of its own totals only: it ends without a claim, and a
// workgroup that misses its next totals makes one.)  load and swap (compare and exchange, which returns what was there) reach the
// claim; it is another launch's until one of this launch is made.  The load may be late: swap says what holds.  So that no step
// falls between two workgroups, leaving and claiming are one: a workgroup that finds a claim goes on with every step that the claim
// leaves to all.  It finds the totals at its next look; `overdue`, when it has not for long, ends the wait all the same, as an error.
template <class Load, class Swap>
SWARM_TEAM_FN TeamWait out_of_patience(uint32_t first, uint32_t done, bool overdue, Load load, Swap swap) {
    TeamClaim there = load();
    if ((uint32_t)(there >> 32) != first) {
        const TeamClaim before = swap(there, (TeamClaim)first << 32 | done);
        if (before == there) return TeamWait::ALONE;
        there = before;
    }
    if (done >= (uint32_t)there) return TeamWait::END;
    return overdue ? TeamWait::LOST : TeamWait::GO_ON;
}

// Number of the next launch's first step, by the steps of this one.  A workgroup by itself numbers the steps of a node that was begun
// once more, past the others': twice the steps are more than it needs, so that no word carries a number of the next launch.
SWARM_TEAM_FN uint32_t next_number(uint32_t first, uint32_t steps) { return first + 2u * steps; }

}  // namespace swarm
