// rd_fmarch_f32.hip -- f32 storage: the register-march front kernel.
#define RD_MARCH_STORAGE rdk::StF32
#define RD_MARCH_FN launch_fmarch_f32
#include "rd_fmarch_impl.hpp"
