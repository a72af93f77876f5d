// lamp_fwd16_sim.hip -- the pipelined forward kernel in the SIM profile (see
// lamp_fwd16.hip), compiled apart from the others.
#ifndef LAMP_FWD16_ONE_UNIT
#define LAMP_FWD16_PART
#include "lamp_fwd16.hip"
#endif

namespace lamp {

hipError_t dispatch_fwd16_sim(int D, int BQ, const FwdParams &p, hipStream_t s, bool *found)
{
    *found = true;
    if (D == 128 && BQ == 64) return launch_fwd16<128, 64, true>(p, s);
    if (D == 128 && BQ == 128) return launch_fwd16<128, 128, true>(p, s);
    if (D == 256 && BQ == 64) return launch_fwd16<256, 64, true>(p, s);
    if (D == 256 && BQ == 128) return launch_fwd16<256, 128, true>(p, s);
    *found = false;
    return hipSuccess;
}

} // namespace lamp
