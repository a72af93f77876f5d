// lamp_fwd16_sr_d64.hip -- the pipelined forward kernel with stochastic rounding
// for d = 64 (see lamp_fwd16_sr.hip), compiled apart from the others.
#ifndef LAMP_FWD16_ONE_UNIT
#define LAMP_FWD16_PART
#include "lamp_fwd16.hip"
#endif

namespace lamp {

hipError_t dispatch_fwd16_sr_d64(int BQ, const FwdParams &p, hipStream_t s, bool *found)
{
    *found = true;
    if (BQ == 64) return launch_fwd16_sr<64, 64>(p, s);
    if (BQ == 128) return launch_fwd16_sr<64, 128>(p, s);
    *found = false;
    return hipSuccess;
}

} // namespace lamp
