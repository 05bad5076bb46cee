// aspis_ws_median.hip -- the warp-specialised median.
#include "aspis_ws.h"

namespace aspis {

MedianWsFn median_ws_fn(const WsPlan &p) {
    const int key = ws_key(p.T, p.sweeps, p.half);
#define ASPIS_MWS(TT, SWW, HH, FF) \
    case ws_key(TT, SWW, HH): return &median_ws_kernel<TT, SWW, HH, FF>;
    if (p.fill == kWsFillWide) {
        if (!p.half) return nullptr;
        switch (key) {
            ASPIS_MWS(64, 24, true, kWsFillWide)
            ASPIS_MWS(32, 24, true, kWsFillWide)
        default: return nullptr;
        }
    }
    if (p.fill != kWsFill) return nullptr;
    switch (key) {
#define ASPIS_MWS_FULL(TT)               \
    ASPIS_MWS(TT, 4, false, kWsFill)     \
    ASPIS_MWS(TT, 8, false, kWsFill)     \
    ASPIS_MWS(TT, 12, false, kWsFill)
#define ASPIS_MWS_HALF(TT)               \
    ASPIS_MWS(TT, 16, true, kWsFill)     \
    ASPIS_MWS(TT, 20, true, kWsFill)     \
    ASPIS_MWS(TT, 24, true, kWsFill)     \
    ASPIS_MWS(TT, 28, true, kWsFill)     \
    ASPIS_MWS(TT, 32, true, kWsFill)
        ASPIS_MWS_FULL(64)
        ASPIS_MWS(64, 16, false, kWsFill)
        ASPIS_MWS_FULL(32)
        ASPIS_MWS_FULL(16)
        ASPIS_MWS_FULL(8)
        ASPIS_MWS(128, 8, true, kWsFill)
        ASPIS_MWS(128, 12, true, kWsFill)
        ASPIS_MWS(128, 30, true, kWsFill)
        ASPIS_MWS_HALF(128)
        ASPIS_MWS_HALF(64)
        ASPIS_MWS_HALF(32)
        ASPIS_MWS(32, 36, true, kWsFill)
        ASPIS_MWS(16, 16, true, kWsFill)
        ASPIS_MWS(16, 24, true, kWsFill)
        ASPIS_MWS(16, 28, true, kWsFill)
        ASPIS_MWS(16, 32, true, kWsFill)
#undef ASPIS_MWS_HALF
#undef ASPIS_MWS_FULL
    default: return nullptr;
    }
#undef ASPIS_MWS
}

}  // namespace aspis
