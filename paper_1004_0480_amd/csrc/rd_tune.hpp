// rd_tune.hpp -- rules of the autotuner that are host arithmetic alone.
#pragma once

#include <algorithm>
#include <cstdint>
#include <map>
#include <tuple>

#include "rd.h"

namespace rdk {

// Autotuned plans by (nx, ny, nz, species, model with stencil and integrator,
// storage), for two classes of grids: those a register march takes and those
// it does not, for their faces or rounding.  A march is mostly the fastest
// plan of the former and none of the latter, so neither class answers for the
// other: held faces would lose their own plan to a march that refuses them, and
// mirror ones would be kept on a ring by a grid with held faces.  What was timed
// of the other plans on a march's grid is kept for the latter until one of them
// is tuned itself.
class PlanCache {
public:
    using Key = std::tuple<int64_t, int64_t, int64_t, int, int, int>;
    // `general`: the fastest plan that is no march, null if there is none.
    void put(const Key& k, bool march_grid, const rd_plan& best, const rd_plan* general) {
        if (march_grid) {
            march_[k] = best;
            const auto it = general_.find(k);
            if (general && (it == general_.end() || !it->second.tuned)) general_[k] = {*general, false};
        } else {
            general_[k] = {best, true};
        }
    }
    // *own: tuned on a grid of that class itself.
    const rd_plan* get(const Key& k, bool march_grid, bool* own) const {
        *own = true;
        if (march_grid) {
            const auto it = march_.find(k);
            return it == march_.end() ? nullptr : &it->second;
        }
        const auto it = general_.find(k);
        if (it == general_.end()) return nullptr;
        *own = it->second.tuned;
        return &it->second.plan;
    }

private:
    struct General { rd_plan plan; bool tuned; };
    std::map<Key, rd_plan> march_;
    std::map<Key, General> general_;
};

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
