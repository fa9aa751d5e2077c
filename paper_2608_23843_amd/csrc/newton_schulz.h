// When the steps L (3/2 - L^T L / 2) that make vectors orthonormal end (plain
// C++: it also compiles by itself, in the tests).
#pragma once

namespace pkv {

constexpr float kOrthMax = 0.9f;   // an entry of L^T L - 1 above this: the vectors are not independent
// A step turns an error E of L^T L into 3/4 E^2 + 1/4 E^3: from norm 0.9 eight
// steps reach rounding. Entries below kOrthMax do not bound the norm of E: three
// nearly coplanar vectors have entries of 1/2 and stay dependent. Vectors that
// have not converged after kOrthSteps are not independent either.
constexpr int kOrthSteps = 12;

enum class Orth { done, last_step, step, fail };

// After looking at E `steps` steps in: whether every entry is at most kOrthMax
// (`bounded`; false for NaN), the largest is at most `tol` (`within`), and 3/4 of
// the Frobenius norm of E squared, which bounds the entries of 3/4 E^2, is
// (`within_next`: one step more needs no look).
constexpr Orth orth_next(bool bounded, bool within, bool within_next, int steps) {
    return !bounded ? Orth::fail : within ? Orth::done : steps >= kOrthSteps ? Orth::fail
           : within_next ? Orth::last_step : Orth::step;
}

}  // namespace pkv
