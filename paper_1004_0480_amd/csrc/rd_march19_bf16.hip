// rd_march19_bf16.hip -- bf16 storage: the 19-point register march.
#define RD_MARCH_STORAGE rdk::StBF16
#define RD_MARCH_FN launch_march19_bf16
#include "rd_march19_impl.hpp"
