// aspis_ws_median.hip -- the warp-specialised median.
#include "aspis_ws.h"

namespace aspis {

MedianWsFn median_ws_fn(const WsPlan &p) {
    // even split, the plans of f = C(K,r)
    if (p.fill != kWsFill) return nullptr;
#define ASPIS_MWS(TT, SWW, HH) \
    case ws_key(TT, SWW, HH): return &median_ws_kernel<TT, SWW, HH>;
    switch (ws_key(p.T, p.sweeps, p.half)) {
        ASPIS_MWS(64, 4, false)
        ASPIS_MWS(64, 8, false)
        ASPIS_MWS(64, 12, false)
        ASPIS_MWS(64, 16, false)
        ASPIS_MWS(32, 12, false)
        ASPIS_MWS(16, 8, false)
        ASPIS_MWS(16, 12, false)
        ASPIS_MWS(8, 8, false)
        ASPIS_MWS(8, 12, false)
        ASPIS_MWS(128, 12, true)
        ASPIS_MWS(128, 16, true)
        ASPIS_MWS(128, 20, true)
        ASPIS_MWS(128, 24, true)
        ASPIS_MWS(128, 30, true)
        ASPIS_MWS(64, 20, true)
        ASPIS_MWS(64, 24, true)
        ASPIS_MWS(64, 28, true)
        ASPIS_MWS(64, 32, true)
        ASPIS_MWS(32, 20, true)
        ASPIS_MWS(32, 24, true)
        ASPIS_MWS(32, 28, true)
        ASPIS_MWS(32, 32, true)
        ASPIS_MWS(16, 24, true)
        ASPIS_MWS(16, 28, true)
        ASPIS_MWS(16, 32, true)
    default: return nullptr;
    }
#undef ASPIS_MWS
}

}  // namespace aspis
