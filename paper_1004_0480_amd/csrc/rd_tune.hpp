// rd_tune.hpp -- rules of the autotuner that are host arithmetic alone.
#pragma once

#include <algorithm>

namespace rdk {

// Steps for which a candidate that advances `per_launch` steps a launch is
// timed, at least `trial`: whole launches alone, an even count.  What is left
// of a count runs on other launches, which long runs hardly have: ten trial
// steps of a four-step plan were timed as 4 + 4 + 2, of a three-step plan as
// 3 + 3 + 3 + 1, and two trial steps never ran either plan's own kernel.
inline int tune_steps(int trial, int per_launch) {
    const int unit = per_launch % 2 ? 2 * per_launch : per_launch;
    return (std::max(trial, 1) + unit - 1) / unit * unit;
}

// Steps before the first timed one: the plan's own kernel once, at least two.
inline int tune_warmup(int per_launch) { return std::max(2, per_launch); }

}  // namespace rdk
