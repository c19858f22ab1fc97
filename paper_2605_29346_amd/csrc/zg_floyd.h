// Floyd's subset algorithm with every slot resolved at once (one lane per slot).
//
// As written, slot j of a vertex with deg > F neighbors draws a candidate t_j in [0, deg-F+j] and takes it
// unless an earlier slot already holds that position, in which case it takes deg-F+j: the test is sequential
// over the slots.  Before slot i the chosen set is exactly {every earlier candidate} united with
// {deg-F+a for every earlier slot a that collided}, so slot i collides iff an earlier slot drew the same
// candidate, or its candidate equals deg-F+a for an earlier slot a that itself collided.  The second clause
// refers to a strictly earlier slot, so iterating it from "collides iff an earlier slot drew the same
// candidate" reaches its fixed point in at most F rounds.
//
// The rule is written against a small interface, so that the sampling kernel (lanes of a wavefront) and a host-side lockstep
// harness (a CPU test that enumerates every candidate sequence, many groups to a wavefront) run the very same code:
//   up(x)          the value of x in the lane before this one of the wavefront, 0 in the first
//   flag_of(j, b)  the boolean b of the group's slot j
//   any(b)         true if b holds for any lane of the wavefront
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define ZG_FLOYD_FN __host__ __device__ __forceinline__
#else
#define ZG_FLOYD_FN inline
#endif

namespace zg {

// Whether an earlier slot of the lane's group holds the same candidate: groups of F consecutive lanes, `group` the number of
// the lane's; all of the wavefront's lanes take part.  The candidates travel one lane up per round, in the kernel a register move, three
// instructions a round (a look through LDS per slot, ds_bpermute, is a round trip each, and F - 1 of them one after another).  What
// comes from the group before differs in the top bit, which no candidate has (cand < a row's length < 2^31); what comes from before the
// first lane is zero, which none of them is.
template <class Wave>
ZG_FLOYD_FN bool floyd_drawn_before(Wave &wave, uint32_t cand, uint32_t group, uint32_t F)
{
    const uint32_t mine = (cand + 1u) | (group << 31);
    uint32_t x = mine, nearest = 0xFFFFFFFFu;
    auto round = [&]() {
        x = wave.up(x);
        const uint32_t t = x ^ mine;
        nearest = t < nearest ? t : nearest;
    };
    uint32_t left = F - 1u;
    for (; left >= 4u; left -= 4u) {
        round();
        round();
        round();
        round();
    }
    for (; left; --left) round();
    return nearest == 0u;
}

// Position taken by slot `slot` of a vertex with `deg` neighbors and fanout F.  `active` lanes are slots of a
// vertex with deg > F (cand = their draw, in [0, deg-F+slot]); the other lanes of the wavefront pass through with
// position = slot, and take part in the exchanges only as partners.
template <class Wave>
ZG_FLOYD_FN uint32_t floyd_position(Wave &wave, uint32_t group, uint32_t slot, uint32_t F, uint32_t deg, bool active, uint32_t cand)
{
    const uint32_t tail0 = deg - F; // candidates >= tail0 coincide with the fallback position of slot cand - tail0
    const bool dup = floyd_drawn_before(wave, cand, group, F) && active;
    if (!wave.any(dup)) return active ? cand : slot; // nobody collides
    const uint32_t a = cand - tail0; // meaningful only when cand >= tail0
    const bool chase = active && cand >= tail0 && a < slot;
    bool collide = dup;
    for (uint32_t it = 0; it < F; ++it) {
        const bool ca = wave.flag_of(chase ? a : 0u, collide);
        const bool nc = dup || (chase && ca);
        const bool changed = nc != collide;
        collide = nc;
        if (!wave.any(changed)) break;
    }
    return active ? (collide ? tail0 + slot : cand) : slot;
}

} // namespace zg
