// rd_fmarch_bf16.hip -- bf16 storage: the register-march front kernel.
#define RD_MARCH_STORAGE rdk::StBF16
#define RD_MARCH_FN launch_fmarch_bf16
#include "rd_fmarch_impl.hpp"
