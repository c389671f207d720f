// rd_march_bf16_diff.hip -- bf16 storage, diff model group: the register-march kernel.
#define RD_MARCH_STORAGE rdk::StBF16
#define RD_MARCH_STORAGE_ID rdk::ST_BF16
#define RD_MARCH_FN launch_march_bf16_diff
#define RD_MARCH_CASES RD_MARCH_CASE(PM_DIFF1, Diffusion<1>)
#include "rd_march_impl.hpp"
