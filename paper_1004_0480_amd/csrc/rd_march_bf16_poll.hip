// rd_march_bf16_poll.hip -- bf16 storage, poll model group: the register-march kernel.
#define RD_MARCH_STORAGE rdk::StBF16
#define RD_MARCH_STORAGE_ID rdk::ST_BF16
#define RD_MARCH_FN launch_march_bf16_poll
#define RD_MARCH_CASES RD_MARCH_CASE(PM_POLL1, Pollutant<1, false>) RD_MARCH_CASE(PM_POLL2, Pollutant<2, true>) RD_MARCH_CASE(PM_POLL2U, Pollutant<2, false>)
#include "rd_march_impl.hpp"
