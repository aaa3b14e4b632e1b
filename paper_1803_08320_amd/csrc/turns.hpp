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

// The blocks per CU of a launch in turns (rk4_f64_turns_kernel, rk4_record_turns_kernel), 0 where one thread per
// lane is the better launch.  With n / (256 lanes per CU) = w + f, w whole, one thread per lane takes the
// time of w + 1 blocks on every CU, in turns w blocks per CU (four at most) share the lanes.  FP64 kernels,
// 1,000 steps on one MI355X, one thread per lane and in turns, ms (Christoffel; Hamiltonian form):
//   w + f   1.1            1.5            1.65           2.1            2.6            3.1
//         1.47 1.02      1.48 1.34      1.48 1.48      2.16 1.64      2.18 2.00      2.95 2.49
//         1.19 0.85      1.21 1.13      1.21 1.25      1.71 1.36      1.73 1.62      2.29 1.90
//   w + f   3.6            4.05           4.6            5.3            6.45           8.2
//         2.98 2.85      3.66 3.16      3.66 3.50      4.55 4.30      5.34 5.23      6.84 6.71
//         2.27 2.16      2.82 2.42      2.85 2.74      3.42 3.22      4.18 4.09      5.38 5.30
// The kernels' registers keep three of four blocks resident (four only at M = 1, a = 0, where it is the same);
// the fourth follows as the others end, at one wave per SIMD, which steps a lane at 0.85 of the rate of three.
// Four are nevertheless better than three (4.05: 3.16 and 3.22 ms, 2.42 and 2.46; 5.3: 4.30 and 4.34, 3.22
// and 3.25; 8.1: 6.49 and 6.58, 5.09 and 5.20): their shares take fewer turns.
// f up to 0.55 with one block per CU, 0.6 up to w = 5, 0.45 at 6 and 0.3 from 7 on: beyond, over both forms,
// a = 0, M = 2 and 16 spacetimes, turns are level or up to 3 % slower (5.6 0 to 3 % faster, 6.6 level, 7.45 1 %
// slower to 3 % faster, 7.6 3 % slower to level, 8.45 2 % slower to 2 % faster, 8.6 level to 3 % slower).
// A turn costs about 0.4 us besides its steps, and the last one is partly idle: at 100 steps the gain at
// w + f = 1.5 and 4.6 is still 8 and 2 %, at 64 steps it is within +-2 %, at 32 none, so from 100 steps on.
// Measured up to w + f = 8.6; the lanes of three blocks (531 each at 8.3) fit a CU's LDS.
MALBEC_HD inline int32_t turns_per_cu(int64_t n, int64_t n_cu, int64_t n_steps)
{
    const int64_t level = n_cu * 256, w = n / level, over = n - w * level;
    if (n_steps < 100 || w < 1 || w > 8 || over == 0) return 0;
    const double most = w == 1 ? 0.55 : w <= 5 ? 0.6 : w == 6 ? 0.45 : 0.3;
    return (double)over <= most * (double)level ? (int32_t)(w < 4 ? w : 4) : 0;
}

}  // namespace malbec
