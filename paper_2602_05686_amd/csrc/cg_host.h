// Host-only parts of the CG loop.  No HIP here, so that they are testable on a
// host without a GPU.
#pragma once

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

}  // namespace matamg
