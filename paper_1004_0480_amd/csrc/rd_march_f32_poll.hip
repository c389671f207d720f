// rd_march_f32_poll.hip -- f32 storage, poll model group: the register-march kernel.
#define RD_MARCH_STORAGE rdk::StF32
#define RD_MARCH_STORAGE_ID rdk::ST_F32
#define RD_MARCH_FN launch_march_f32_poll
#define RD_MARCH_CASES RD_MARCH_CASE(PM_POLL1, Pollutant<1, false>) RD_MARCH_CASE(PM_POLL2, Pollutant<2, true>) RD_MARCH_CASE(PM_POLL2U, Pollutant<2, false>)
#include "rd_march_impl.hpp"
