// rd_march19_f32.hip -- f32 storage: the 19-point register march.
#define RD_MARCH_STORAGE rdk::StF32
#define RD_MARCH_FN launch_march19_f32
#include "rd_march19_impl.hpp"
