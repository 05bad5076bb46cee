// aspis_ws_r3.hip -- the warp-specialised single pass at r = 3, file-major.
#include "aspis_ws.h"

namespace aspis {

FusedWsFn fused_ws_r3_fn(const WsPlan &p) {
    if (p.r != 3 || p.rtg) return nullptr;
    if (p.fill == kWsFillWide) {
        // wide split: half keys only
        if (!p.half) return nullptr;
#define W(TT, SWW) \
    case ws_key(TT, SWW, true): return ASPIS_NT(fused_ws_kernel, TT, 3, SWW, false, true, kWsFillWide, false);
        switch (ws_key(p.T, p.sweeps, p.half)) {
            W(64, 24)
            W(32, 24)
        default: return nullptr;
        }
#undef W
    }
    if (p.fill != kWsFill) return nullptr;
#define ASPIS_FWS(TT, SWW, HH) \
    case ws_key(TT, SWW, HH): return ASPIS_NT(fused_ws_kernel, TT, 3, SWW, false, HH, kWsFill, false);
#define ASPIS_FWS_NARROW(TT, SWW, HH) \
    case ws_key(TT, SWW, HH): return &fused_ws_kernel<TT, 3, SWW, false, HH, kWsFill, false, false>;
    switch (ws_key(p.T, p.sweeps, p.half)) {
        ASPIS_FWS(32, 36, true)
#define ASPIS_FWS_HALF(TT)    \
    ASPIS_FWS(TT, 20, true)   \
    ASPIS_FWS(TT, 24, true)   \
    ASPIS_FWS(TT, 28, true)   \
    ASPIS_FWS(TT, 32, true)
        ASPIS_FWS(64, 2, false)
        ASPIS_FWS(64, 4, false)
        ASPIS_FWS(64, 8, false)
        ASPIS_FWS(64, 12, false)
        ASPIS_FWS(64, 16, false)
        ASPIS_FWS(32, 8, false)
        ASPIS_FWS(32, 12, false)
        ASPIS_FWS(32, 16, false)
        ASPIS_FWS_NARROW(16, 8, false)
        ASPIS_FWS_NARROW(16, 12, false)
        ASPIS_FWS_NARROW(16, 16, false)
        ASPIS_FWS_NARROW(8, 8, false)
        ASPIS_FWS_NARROW(8, 12, false)
        ASPIS_FWS_NARROW(8, 16, false)
        ASPIS_FWS(128, 4, true)
        ASPIS_FWS(128, 8, true)
        ASPIS_FWS(128, 12, true)
        ASPIS_FWS(128, 16, true)
        ASPIS_FWS(128, 30, true)
        ASPIS_FWS_HALF(128)
        ASPIS_FWS_HALF(64)
        ASPIS_FWS_HALF(32)
        ASPIS_FWS_NARROW(16, 16, true)
        ASPIS_FWS_NARROW(16, 24, true)
        ASPIS_FWS_NARROW(16, 28, true)
        ASPIS_FWS_NARROW(16, 32, true)
#undef ASPIS_FWS_HALF
    default: return nullptr;
    }
#undef ASPIS_FWS
#undef ASPIS_FWS_NARROW
}

}  // namespace aspis
