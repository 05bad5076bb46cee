// aspis_ws_r5.hip -- the warp-specialised single pass at r = 5, file-major.
#include "aspis_ws.h"

namespace aspis {

FusedWsFn fused_ws_r5_fn(const WsPlan &p) {
    // half keys, even split
    if (p.r != 5 || !p.half || p.fill != kWsFill || p.rtg) return nullptr;
    switch (ws_key(p.T, p.sweeps, p.half)) {
#define ASPIS_FWS5(TT, SWW) \
    case ws_key(TT, SWW, true): return &fused_ws_kernel<TT, 5, SWW, false, true, kWsFill, false>;
        ASPIS_FWS5(128, 16)
        ASPIS_FWS5(128, 30)
        ASPIS_FWS5(128, 32)
        ASPIS_FWS5(64, 16)
        ASPIS_FWS5(64, 24)
        ASPIS_FWS5(64, 32)
        ASPIS_FWS5(32, 16)
        ASPIS_FWS5(32, 24)
        ASPIS_FWS5(32, 32)
        ASPIS_FWS5(16, 16)
        ASPIS_FWS5(16, 24)
        ASPIS_FWS5(16, 32)
#undef ASPIS_FWS5
    default: return nullptr;
    }
}

}  // namespace aspis
