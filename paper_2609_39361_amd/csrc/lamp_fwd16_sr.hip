// lamp_fwd16_sr.hip -- the pipelined forward kernel with stochastic rounding of the
// 8-bit logits (see lamp_fwd16.hip), compiled apart from the others.
#define LAMP_FWD16_PART
#include "lamp_fwd16.hip"

namespace lamp {

template <int D, int BQ>
static hipError_t launch_fwd16_sr(const FwdParams &p, hipStream_t s)
{
    if (p.mode == MODE_PURE8) return launch_fwd16_mode<D, BQ, MODE_PURE8, false, true>(p, s);
    return launch_fwd16_mode<D, BQ, MODE_LAMP, false, true>(p, s);
}

hipError_t dispatch_fwd16_sr(int D, int BQ, const FwdParams &p, hipStream_t s, bool *found)
{
    *found = true;
    if (D == 64 && BQ == 64) return launch_fwd16_sr<64, 64>(p, s);
    if (D == 64 && BQ == 128) return launch_fwd16_sr<64, 128>(p, s);
    if (D == 128 && BQ == 64) return launch_fwd16_sr<128, 64>(p, s);
    if (D == 128 && BQ == 128) return launch_fwd16_sr<128, 128>(p, s);
    if (D == 256 && BQ == 64) return launch_fwd16_sr<256, 64>(p, s);
    if (D == 256 && BQ == 128) return launch_fwd16_sr<256, 128>(p, s);
    *found = false;
    return hipSuccess;
}

} // namespace lamp
