// aspis_ws_median.hip -- the warp-specialised median.
#include "aspis_ws.h"

namespace aspis {

MedianWsFn median_ws_fn(const WsPlan &p) {
    const int key = ws_key(p.T, p.sweeps, p.half);
#define ASPIS_MWS(TT, SWW, HH) \
    case ws_key(TT, SWW, HH): return &median_ws_kernel<TT, SWW, HH>;
    if (p.fill != kWsFill) return nullptr;
    switch (key) {
#define ASPIS_MWS_FULL(TT)               \
    ASPIS_MWS(TT, 4, false)     \
    ASPIS_MWS(TT, 8, false)     \
    ASPIS_MWS(TT, 12, false)
#define ASPIS_MWS_HALF(TT)               \
    ASPIS_MWS(TT, 16, true)     \
    ASPIS_MWS(TT, 20, true)     \
    ASPIS_MWS(TT, 24, true)     \
    ASPIS_MWS(TT, 28, true)     \
    ASPIS_MWS(TT, 32, true)
        ASPIS_MWS_FULL(64)
        ASPIS_MWS(64, 16, false)
        ASPIS_MWS_FULL(32)
        ASPIS_MWS_FULL(16)
        ASPIS_MWS_FULL(8)
        ASPIS_MWS(128, 8, true)
        ASPIS_MWS(128, 12, true)
        ASPIS_MWS(128, 30, true)
        ASPIS_MWS_HALF(128)
        ASPIS_MWS_HALF(64)
        ASPIS_MWS_HALF(32)
        ASPIS_MWS(32, 36, true)
        ASPIS_MWS(16, 16, true)
        ASPIS_MWS(16, 24, true)
        ASPIS_MWS(16, 28, true)
        ASPIS_MWS(16, 32, true)
#undef ASPIS_MWS_HALF
#undef ASPIS_MWS_FULL
    default: return nullptr;
    }
#undef ASPIS_MWS
}

}  // namespace aspis
