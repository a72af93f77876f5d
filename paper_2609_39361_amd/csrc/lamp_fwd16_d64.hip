// lamp_fwd16_d64.hip -- the pipelined forward kernel for d = 64 with the formats
// of Sec. 3.3 (see lamp_fwd16.hip), compiled apart from the others.
#ifndef LAMP_FWD16_ONE_UNIT
#define LAMP_FWD16_PART
#include "lamp_fwd16.hip"
#endif

namespace lamp {

hipError_t dispatch_fwd16_d64(int BQ, const FwdParams &p, hipStream_t s, bool *found)
{
    *found = true;
    if (BQ == 64) return launch_fwd16<64, 64, false>(p, s);
    if (BQ == 128) return launch_fwd16<64, 128, false>(p, s);
    *found = false;
    return hipSuccess;
}

} // namespace lamp
