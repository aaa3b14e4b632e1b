// The FP64 persistent kernel of the Christoffel form, in a file of its own because it is compiled
// with the default instruction schedule: the schedule for instruction-level parallelism, which the
// kernels of integrate.hip have, takes it from 128 to 144 registers and from four waves per SIMD to
// three, or, held to four, slows it down (600 steps of 16 spacetimes, medians on one MI355X: 1,048,576
// lanes 7.60 ms here, 7.83 with that schedule and 7.77 held to four waves; 524,288 lanes 3.75, 3.71 and
// 3.95).
#include "f64_prog.hpp"

namespace malbec {

int launch_queue_f64(const IntArgs &A, const StTable &T, bool multi, int block, int32_t sub,
                     bool &declined, unsigned long long *counter, hipStream_t s)
{
    return multi ? launch_persistent<true, false>(A, T, block, sub, declined, counter, s)
                 : launch_persistent<false, false>(A, T, block, sub, declined, counter, s);
}

}  // namespace malbec
