// rd_march_bf16_batch.hip -- bf16 storage: the batched register march.
#include "rd_march.hpp"

namespace rdk {

#define RD_KERNEL batched_march_kernel<StBF16, kBatchMarch.ry, kBatchMarch.w>

hipError_t launch_batched_march_bf16(const int* meta, const BatchEntry* ents, int launch, int blocks, hipStream_t s) {
    hipLaunchKernelGGL((RD_KERNEL), dim3(blocks), dim3(64 * kBatchMarch.w), 0, s, meta, ents, launch);
    return hipGetLastError();
}

int batched_march_blocks_per_cu_bf16() {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(&RD_KERNEL),
                                                     64 * kBatchMarch.w, 0) != hipSuccess)
        return 1;
    return n > 0 ? n : 1;
}

}  // namespace rdk
