// tt_wait.h -- rules of a sweep's waits and of the end of an iteration, free of
// anything of the device, so that they can be compiled and tested on a host.
#pragma once

#if defined(__HIPCC__)
#define TT_HD __host__ __device__ __forceinline__
#else
#define TT_HD inline
#endif

namespace tt {

// Polls a wait makes before it is given up, some 10 s of them.  Polls are counted,
// not time: a clock runs on while the queue is off the chip, where neither the
// waiting wave nor the one it waits for can do anything.
constexpr unsigned kWaitPolls = 1u << 24;
constexpr unsigned kLostPolls = 1u << 10;  // ... and between two looks at whether another wave gave up

// Poll ready() until it holds.  false if the wait was given up: after `polls`
// polls (a wave was lost, and what it should have done never comes), or as soon
// as lost() says that another wave has given up on the same source.  ready() has
// the last word: a wave that was off the chip between its two calls looks again.
template <class Ready, class Lost, class Pause>
TT_HD bool poll_until(Ready ready, Lost lost, Pause pause, unsigned polls) {
    for (unsigned n = 1; !ready(); ++n) {
        if (n >= polls || (n % kLostPolls == 0 && lost())) return ready();
        pause();
    }
    return true;
}

// How a source's iteration number it ends: its status, and whether the source is
// done.  A source that lost a wave has values in its field that no sweep gives: it
// ends there, as not converged.
struct Outcome {
    int status;
    bool done;
};
TT_HD Outcome iteration_outcome(double eps, double tol, int it, int max_iter, bool lost) {
    if (lost) return {-it, true};
    if (eps < tol) return {it, true};
    return {-it, it >= max_iter};
}

}  // namespace tt
