// Host-only parts of the CG loop.  No HIP here, so that they are testable on a
// host without a GPU.
#pragma once

#include <chrono>
#include <thread>

#if defined(__x86_64__)
#include <immintrin.h>
#endif

namespace matamg {

// the part of the foreseen residual that has to be above the tolerance for
// the next V-cycle to be launched ahead
constexpr double kAheadMargin = 0.5;

// Whether the next step's V-cycle goes out before the test of step `it`, whose
// relative residual is foreseen to be last * rate.  Not on one level: there the
// V-cycle is the whole inverse and the first step as a rule the last one, so
// that a V-cycle ahead would read the inverse again for nothing, in front of
// the check of the true residual (solve of 4,900 unknowns, whose inverse is 190
// MB: 166 us with it, 138 us without; of 961 unknowns 118 and 111 us).
inline bool look_ahead(int levels, int it, int max_iter, double last, double rate, double tol) {
    return levels > 1 && it < max_iter && last * rate * kAheadMargin > tol;
}

// Waits until ready(), or until idle() says that nothing more will come (asked
// every kIdleUs); true if ready.  The steps of small systems are over within
// microseconds and are polled for.  From kPollUs on the core is offered to other
// threads at every poll: a caller's solving threads may be more than its cores.
// With `nap` the thread sleeps between polls from kSleepUs on; waking up takes
// some 70 us, which pass unseen where the GPU has the next V-cycle to go on with.
// Sixteen threads on sixteen cores, each solving a 32^3 anisotropic system, held
// 15 cores polling only and hold 5.6 (an 80^3 stack 12 and 4.6), at the same rate.
constexpr int kPollUs = 50, kSleepUs = 200, kNapUs = 20, kIdleUs = 1000;

template <class Ready, class Idle>
inline bool wait_until(bool nap, Ready ready, Idle idle) {
    using us = std::chrono::microseconds;
    const auto t0 = std::chrono::steady_clock::now();
    auto ask = t0 + us(kIdleUs);
    for (;;) {
        for (int poll = 0; poll < 32; ++poll) {
            if (ready()) return true;
#if defined(__x86_64__)
            _mm_pause();
#endif
        }
        const auto now = std::chrono::steady_clock::now();
        if (now >= ask) {
            if (idle()) return ready();
            ask = now + us(kIdleUs);
        }
        if (nap && now - t0 >= us(kSleepUs)) std::this_thread::sleep_for(us(kNapUs));
        else if (now - t0 >= us(kPollUs)) std::this_thread::yield();
    }
}

}  // namespace matamg
