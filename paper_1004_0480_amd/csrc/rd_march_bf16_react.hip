// rd_march_bf16_react.hip -- bf16 storage, react model group: the register-march kernel.
#define RD_MARCH_STORAGE rdk::StBF16
#define RD_MARCH_STORAGE_ID rdk::ST_BF16
#define RD_MARCH_FN launch_march_bf16_react
#define RD_MARCH_CASES RD_MARCH_CASE(PM_BRUSS, Brusselator)
#include "rd_march_impl.hpp"
