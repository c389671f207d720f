// rd_fmarch_impl.hpp -- instantiation and dispatch of the register-march front
// kernel for one storage type.  Included by rd_fmarch_<storage>.hip with
//   RD_MARCH_STORAGE   the storage struct (rdk::StF32, ...)
//   RD_MARCH_FN        the launcher's name
#pragma once

#include <utility>

#include "rd_fmarch.hpp"

namespace rdk {
namespace {

template <int I, bool CD>
hipError_t run_fmarch(bool sr, bool ragged, const StepArgs* d, long long blocks, hipStream_t s) {
    constexpr FmarchCfg c = kFmarchCfgs[I];
    using S = RD_MARCH_STORAGE;
    const dim3 grid((unsigned)blocks), block(64 * c.w);
    if (sr) {
        if constexpr (std::is_same_v<S, StBF16>) {
            if (ragged) return hipErrorNotSupported;
            hipLaunchKernelGGL((fmarch_kernel<S, c.ry, c.w, CD, true, false>), grid, block, 0, s, d);
        } else {
            return hipErrorNotSupported;
        }
    } else if (ragged) {
        hipLaunchKernelGGL((fmarch_kernel<S, c.ry, c.w, CD, false, true>), grid, block, 0, s, d);
    } else {
        hipLaunchKernelGGL((fmarch_kernel<S, c.ry, c.w, CD, false, false>), grid, block, 0, s, d);
    }
    return hipGetLastError();
}

template <int... I>
hipError_t run_fmarch_index(int cfg, bool cd, bool sr, bool ragged, const StepArgs* d, long long blocks, hipStream_t s,
                            std::integer_sequence<int, I...>) {
    hipError_t r = hipErrorInvalidValue;
    ((void)(cfg == I && ((r = cd ? run_fmarch<I, true>(sr, ragged, d, blocks, s)
                                 : run_fmarch<I, false>(sr, ragged, d, blocks, s)), true)), ...);
    return r;
}

}  // namespace

hipError_t RD_MARCH_FN(int cfg, bool cd, bool sr, bool ragged, const StepArgs* d, long long blocks, hipStream_t s) {
    return run_fmarch_index(cfg, cd, sr, ragged, d, blocks, s, std::make_integer_sequence<int, kNumFmarchCfgs>{});
}

}  // namespace rdk
