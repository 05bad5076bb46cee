// aspis_ws_r3.hip -- the warp-specialised single pass at r = 3, file-major.
#include "aspis_ws.h"

namespace aspis {

FusedWsFn fused_ws_r3_fn(const WsPlan &p) {
    if (p.r != 3 || p.rtg) return nullptr;
    // wide split (half keys): 1,140 files
    if (p.fill == kWsFillWide)
        return p.half && p.T == 64 && p.sweeps == 24
                   ? ASPIS_NT(fused_ws_kernel, 64, 3, 24, false, true, kWsFillWide, false)
                   : nullptr;
    if (p.fill != kWsFill) return nullptr;
    // the plans of f = C(K,3), K = 3 to 64
#define ASPIS_FWS(TT, SWW, HH) \
    case ws_key(TT, SWW, HH): return ASPIS_NT(fused_ws_kernel, TT, 3, SWW, false, HH, kWsFill, false);
#define ASPIS_FWS_NARROW(TT, SWW, HH) \
    case ws_key(TT, SWW, HH): return &fused_ws_kernel<TT, 3, SWW, false, HH, kWsFill, false, false>;
    switch (ws_key(p.T, p.sweeps, p.half)) {
        ASPIS_FWS(64, 2, false)
        ASPIS_FWS(64, 4, false)
        ASPIS_FWS(64, 8, false)
        ASPIS_FWS(64, 12, false)
        ASPIS_FWS(64, 16, false)
        ASPIS_FWS(32, 12, false)
        ASPIS_FWS(32, 16, false)
        ASPIS_FWS_NARROW(16, 12, false)
        ASPIS_FWS_NARROW(16, 16, false)
        ASPIS_FWS_NARROW(8, 12, false)
        ASPIS_FWS_NARROW(8, 16, false)
        ASPIS_FWS(128, 4, true)
        ASPIS_FWS(128, 8, true)
        ASPIS_FWS(128, 12, true)
        ASPIS_FWS(128, 16, true)
        ASPIS_FWS(128, 20, true)
        ASPIS_FWS(128, 24, true)
        ASPIS_FWS(128, 30, true)
        ASPIS_FWS(64, 20, true)
        ASPIS_FWS(64, 24, true)
        ASPIS_FWS(64, 28, true)
        ASPIS_FWS(64, 32, true)
        ASPIS_FWS(32, 24, true)
        ASPIS_FWS(32, 28, true)
        ASPIS_FWS(32, 32, true)
        ASPIS_FWS(32, 36, true)
        ASPIS_FWS_NARROW(16, 24, true)
        ASPIS_FWS_NARROW(16, 28, true)
        ASPIS_FWS_NARROW(16, 32, true)
    default: return nullptr;
    }
#undef ASPIS_FWS
#undef ASPIS_FWS_NARROW
}

}  // namespace aspis
