// lamp_fwd16_sr_d256.hip -- the pipelined forward kernel with stochastic rounding
// for d = 256 (see lamp_fwd16_sr.hip), compiled apart from the others.
#ifndef LAMP_FWD16_ONE_UNIT
#define LAMP_FWD16_PART
#include "lamp_fwd16.hip"
#endif

namespace lamp {

hipError_t dispatch_fwd16_sr_d256(int BQ, const FwdParams &p, hipStream_t s, bool *found)
{
    *found = true;
    if (BQ == 64) return launch_fwd16_sr<256, 64>(p, s);
    if (BQ == 128) return launch_fwd16_sr<256, 128>(p, s);
    *found = false;
    return hipSuccess;
}

} // namespace lamp
