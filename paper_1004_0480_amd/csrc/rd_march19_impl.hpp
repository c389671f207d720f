// rd_march19_impl.hpp -- instantiation and dispatch of the 19-point register
// march for one storage type.  Included by rd_march19_<storage>.hip with
//   RD_MARCH_STORAGE   the storage struct (rdk::StF32, ...)
//   RD_MARCH_FN        the launcher's name
#pragma once

#include "rd_march19.hpp"

namespace rdk {
namespace {

template <class M, int K>
hipError_t run_march19(bool ragged, const StepArgs* d, long long blocks, hipStream_t s) {
    const dim3 grid((unsigned)blocks), block(64 * kMarch19Waves);
    if (ragged)
        hipLaunchKernelGGL((march19_kernel<M, RD_MARCH_STORAGE, kMarch19Waves, K, true>), grid, block, 0, s, d);
    else
        hipLaunchKernelGGL((march19_kernel<M, RD_MARCH_STORAGE, kMarch19Waves, K, false>), grid, block, 0, s, d);
    return hipGetLastError();
}

template <class M> hipError_t run_march19_k(int k, bool ragged, const StepArgs* d, long long blocks, hipStream_t s) {
    return k == 1 ? run_march19<M, 1>(ragged, d, blocks, s)
         : k == 2 ? run_march19<M, 2>(ragged, d, blocks, s) : hipErrorInvalidValue;
}

}  // namespace

hipError_t RD_MARCH_FN(int pm, int k, bool ragged, const StepArgs* d, long long blocks, hipStream_t s) {
    switch (pm) {
    case PM_DIFF1: return run_march19_k<Diffusion<1>>(k, ragged, d, blocks, s);
    case PM_BRUSS: return run_march19_k<Brusselator>(k, ragged, d, blocks, s);
    case PM_TURING: return run_march19_k<Turing>(k, ragged, d, blocks, s);
    default: return hipErrorNotSupported;
    }
}

}  // namespace rdk
