// rd_march_f32_react.hip -- f32 storage, react model group: the register-march kernel.
#define RD_MARCH_STORAGE rdk::StF32
#define RD_MARCH_STORAGE_ID rdk::ST_F32
#define RD_MARCH_FN launch_march_f32_react
#define RD_MARCH_CASES RD_MARCH_CASE(PM_BRUSS, Brusselator)
#include "rd_march_impl.hpp"
