// rd_march_impl.hpp -- instantiation and dispatch of the register-march kernel
// for one storage type and group of models.  Included by
// rd_march_<storage>_<group>.hip with
//   RD_MARCH_STORAGE / _STORAGE_ID   the storage struct and its rdk::Storage value
//   RD_MARCH_FN                      the launcher's name
//   RD_MARCH_CASES                   one RD_MARCH_CASE(PM, model) per model
#pragma once

#include <utility>

#include "rd_march.hpp"

namespace rdk {
namespace {

template <class M, int I, int K, bool MIR>
hipError_t run_march_k(int variant, const StepArgs* d, long long blocks, hipStream_t s) {
    constexpr MarchCfg c = kMarchCfgs[I];
    using S = RD_MARCH_STORAGE;
    const dim3 grid((unsigned)blocks), block(64 * c.w);
    switch (variant & 3) {
    case MARCH_PLAIN:
        hipLaunchKernelGGL((march_kernel<M, S, c.ry, c.w, K, false, 0, MIR>), grid, block, 0, s, d);
        break;
    case MARCH_EDGES:
        hipLaunchKernelGGL((march_kernel<M, S, c.ry, c.w, K, true, 0, MIR>), grid, block, 0, s, d);
        break;
    default:
        hipLaunchKernelGGL((march_kernel<M, S, c.ry, c.w, K, true, 1, MIR>), grid, block, 0, s, d);
        break;
    }
    return hipGetLastError();
}

template <class M, int PM, int I, int K>
hipError_t run_march_faces(int variant, const StepArgs* d, long long blocks, hipStream_t s) {
    // mirror x faces on both sides have their own code where that is the
    // usual problem
    if constexpr (PM == PM_DIFF1) {
        if (variant & MARCH_MIRROR) return run_march_k<M, I, K, true>(variant, d, blocks, s);
    }
    return run_march_k<M, I, K, false>(variant, d, blocks, s);
}

template <class M, int PM, int I>
hipError_t run_march(int k, int variant, const StepArgs* d, long long blocks, hipStream_t s) {
    if constexpr (march_ok(RD_MARCH_STORAGE_ID, PM, I)) {
        if (k == 1) return run_march_faces<M, PM, I, 1>(variant, d, blocks, s);
        if constexpr (kMarchCfgs[I].k > 2) {
            if (k == 2) return run_march_faces<M, PM, I, 2>(variant, d, blocks, s);
        }
        if (k == kMarchCfgs[I].k) return run_march_faces<M, PM, I, kMarchCfgs[I].k>(variant, d, blocks, s);
    }
    return hipErrorNotSupported;
}

template <class M, int PM, int... I>
hipError_t run_march_index(int cfg, int k, int variant, const StepArgs* d, long long blocks, hipStream_t s,
                           std::integer_sequence<int, I...>) {
    hipError_t r = hipErrorInvalidValue;
    ((void)(cfg == I && ((r = run_march<M, PM, I>(k, variant, d, blocks, s)), true)), ...);
    return r;
}

}  // namespace

hipError_t RD_MARCH_FN(int pm, int cfg, int k, int variant, const StepArgs* d, long long blocks, hipStream_t s) {
    switch (pm) {
#define RD_MARCH_CASE(PM, ...) \
    case PM: return run_march_index<__VA_ARGS__, PM>(cfg, k, variant, d, blocks, s, \
                                                     std::make_integer_sequence<int, kNumMarchCfgs>{});
    RD_MARCH_CASES
#undef RD_MARCH_CASE
    default: return hipErrorNotSupported;
    }
}

}  // namespace rdk
