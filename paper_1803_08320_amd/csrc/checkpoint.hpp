// The checkpoint slots of a fixed-step integration: slot s holds the state after s K steps
// (K = checkpoint_every).  K and the step indices are at most 2^31 - 1, so the step of the next
// slot can lie beyond 32 bits and is formed in 64.  Compiled for the host by the tests.
#pragma once

#include <stdint.h>

#include "kerr_accel.hpp"

namespace malbec {

// Steps k0 .. k0 + n_steps - 1 of a call, from slot to slot.  put(s) stores the lane's present
// state in slot s; run(n, active) takes at most n >= 1 steps of the active lane, returns how many
// and clears `active` when the lane stops.  Returns the steps taken.  When it is done, the slots up to the
// end of this launch that the lane did not reach have its present state: the final one for a
// stopped lane, and for the call's last slot, last_of_call, the state after the launch (a slot
// at the end of any other launch is left to the next one).
template <class Run, class Put>
MALBEC_HD inline int32_t run_checkpointed(int32_t k0, int32_t n_steps, int32_t every,
                                          int32_t last_of_call, bool active, Run run, Put put)
{
    int64_t slot = ((int64_t)k0 + every - 1) / every;  // first slot at or after k0
    int32_t taken = 0;
    while (active && taken < n_steps) {
        const int64_t k = (int64_t)k0 + taken;
        if (k == slot * every) put((int32_t)slot++);
        const int64_t to_slot = slot * every - k;  // >= 1
        const int32_t left = n_steps - taken;
        taken += run(to_slot < left ? (int32_t)to_slot : left, active);
    }
    const int64_t end = (int64_t)k0 + n_steps;
    int64_t last = end / every;
    if (last * every == end && last != last_of_call) --last;
    for (; slot <= last; ++slot) put((int32_t)slot);
    return taken;
}

// The segments between the slots of a call of n_steps >= 1 steps, for the walk back.
MALBEC_HD inline int32_t checkpoint_segments(int32_t n_steps, int32_t every) { return (n_steps - 1) / every + 1; }

}  // namespace malbec
