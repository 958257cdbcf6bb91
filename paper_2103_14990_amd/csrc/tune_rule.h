// When a timed candidate of the autotuner takes the place of the form kept so far.
#pragma once

namespace dlmpc {

// Only when it is faster by more than the 1 % that two timings of one form differ by: the forms round
// differently, and noise should not choose between near-ties anew at every setup. `us` is 0 for a
// candidate that was not timed.
inline bool replaces(double us, double kept_us) { return us > 0.0 && us < 0.99 * kept_us; }

}  // namespace dlmpc
