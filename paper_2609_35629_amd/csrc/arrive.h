// Which of a pair's workgroups finds that all of them have arrived, without
// any of them waiting: each leaves the call's token in its own slot and then
// looks at all slots.
#pragma once

#include <stdint.h>

namespace santapp {

// True for exactly one of the workgroups, and only after every one has left
// the token; the slots are then 0 again.  `slots` gives
//   leave(token)  writes this workgroup's slot, performed before what follows
//   all(token)    whether every slot holds the token
//   take(token)   compare-and-swap of one slot from the token to 0
//   clear()       0 into every slot
// The last workgroup to leave its token sees them all, unless one that saw
// them before it has cleared some; of several that see them all one succeeds in
// take.  That one clears when no token is still to come, so none is left
// behind for a later launch that brings the same one (a replayed graph).  What
// the slots held before does not matter as long as it is not the token.
template <typename Slots>
__host__ __device__ inline bool last_to_arrive(Slots& slots, uint64_t token) {
    slots.leave(token);
    if (!slots.all(token) || !slots.take(token)) return false;
    slots.clear();
    return true;
}

}  // namespace santapp
