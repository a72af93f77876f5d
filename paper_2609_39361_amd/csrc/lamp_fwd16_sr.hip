// lamp_fwd16_sr.hip -- the pipelined forward kernel with stochastic rounding of the
// 8-bit logits (see lamp_fwd16.hip), compiled apart from the others: d = 128 here,
// d = 64 and 256 in lamp_fwd16_sr_d64.hip and lamp_fwd16_sr_d256.hip (units of
// their own with LAMP_SPLIT_UNITS).
#define LAMP_FWD16_PART
#include "lamp_fwd16.hip"

namespace lamp {

hipError_t dispatch_fwd16_sr(int D, int BQ, const FwdParams &p, hipStream_t s, bool *found)
{
    if (D == 64) return dispatch_fwd16_sr_d64(BQ, p, s, found);
    if (D == 256) return dispatch_fwd16_sr_d256(BQ, p, s, found);
    *found = true;
    if (D == 128 && BQ == 64) return launch_fwd16_sr<128, 64>(p, s);
    if (D == 128 && BQ == 128) return launch_fwd16_sr<128, 128>(p, s);
    *found = false;
    return hipSuccess;
}

} // namespace lamp

#ifndef LAMP_SPLIT_UNITS
#define LAMP_FWD16_ONE_UNIT
#include "lamp_fwd16_sr_d64.hip"
#include "lamp_fwd16_sr_d256.hip"
#endif
