// The turns of a block that advances m lanes with 256 threads: the threads of a turn are a run of
// the sequence 0, 1, .. m - 1, 0, 1, .., and a lane takes up to q steps in each of its turns.  With
// fewer than 256 lanes every thread keeps its own.  Step counts go up to 2^31 - 1, so no sum here may
// pass it.  Compiled for the host by the tests.
#pragma once

#include <stdint.h>

#include "kerr_accel.hpp"

namespace malbec {

// Turns of the block until every lane has had n_steps steps (at most
// 2^27 runs of q steps, and m < 4096, below 2^31 turns).
MALBEC_HD inline int32_t turns_of_block(int32_t n_steps, int32_t q, int32_t m)
{
    const int32_t runs = n_steps / q + (n_steps % q != 0);
    return m >= 256 ? (int32_t)(((int64_t)runs * m + 255) / 256) : runs;
}

// The steps of a lane's next turn after it has had `had` whole ones, 0 when it has had all.
MALBEC_HD inline int32_t steps_of_turn(int32_t n_steps, int32_t q, int32_t had)
{
    const int64_t left = n_steps - (int64_t)had * q;
    return left < q ? (left > 0 ? (int32_t)left : 0) : q;
}

// A thread's lane j in the next turn, and the turns that this lane has had.
MALBEC_HD inline void next_turn(int32_t m, int32_t &j, int32_t &had)
{
    if (m < 256) {
        ++had;
        return;
    }
    j += 256;
    if (j >= m) {
        j -= m;
        ++had;
    }
}

// A block whose lanes have all stopped leaves its remaining turns out, as one thread per lane would (a
// run "until every lane stops" has a step count far beyond its longest lane): it looks every kIdleTurns
// turns whether one of its threads had a lane that stepped in them, in which every lane has had its turn.
constexpr int32_t kIdleTurns = 16;
constexpr int32_t kMaxShare = kIdleTurns * 256;  // the lanes of a block are fewer
MALBEC_HD inline bool look_after(int32_t turn) { return turn % kIdleTurns == kIdleTurns - 1; }

}  // namespace malbec
