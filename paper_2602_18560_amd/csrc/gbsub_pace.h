// gbsub_pace.h -- the progress word of a run: what the tail of a loop body tells
// the host that paces the launches, and the form the host gives each body by it.
// Plain C++ (host and device).
#pragma once

#include <stdint.h>

namespace gbs {

// `finished` bodies have ended, `done`: the loop has settled; `fits`: the dirty
// tiles of body `finished`, the next one, fit the split budget, `fitted`: so
// did those of the body before it.  All in one word, so that the host never
// sees one without the others; 0: no body has ended.
constexpr uint64_t pace_word(uint32_t finished, bool done, bool fits, bool fitted)
{
    return (uint64_t)fitted << 33 | (uint64_t)fits << 32 | (uint64_t)finished << 1 | (uint64_t)done;
}
constexpr bool pace_done(uint64_t w) { return w & 1u; }
constexpr uint32_t pace_finished(uint64_t w) { return (uint32_t)w >> 1; }

// Bodies the host keeps queued beyond the last finished one.
constexpr uint32_t AHEAD = 2;
constexpr bool pace_room(uint64_t w, uint64_t t) { return t < (uint64_t)pace_finished(w) + AHEAD; }

// Whether body t runs in two launches: if the dirty tiles of body t - 1 fit the
// budget (for the first two bodies: if all tiles do, fits0).  Those of body t
// itself may not be known yet when it is queued, and a choice by the latest
// count in sight would follow the host's timing: a body of two launches works
// in parts also where its tiles do not fit, and the sums of 1/S (and the
// running mean) round differently in parts and in whole tiles.  When body t is
// queued the word is that of body t - 1 or t, and holds the same answer.
constexpr bool pace_two(uint64_t w, uint64_t t, bool fits0)
{
    const uint32_t f = pace_finished(w);
    return f == 0 ? fits0 : t == f ? (w >> 33 & 1u) : (w >> 32 & 1u);
}

}  // namespace gbs
