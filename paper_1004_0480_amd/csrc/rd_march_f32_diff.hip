// rd_march_f32_diff.hip -- f32 storage, diff model group: the register-march kernel.
#define RD_MARCH_STORAGE rdk::StF32
#define RD_MARCH_STORAGE_ID rdk::ST_F32
#define RD_MARCH_FN launch_march_f32_diff
#define RD_MARCH_CASES RD_MARCH_CASE(PM_DIFF1, Diffusion<1>)
#include "rd_march_impl.hpp"
