// aspis_ws_r5.hip -- the warp-specialised single pass at r = 5, file-major.
#include "aspis_ws.h"

namespace aspis {

FusedWsFn fused_ws_r5_fn(const WsPlan &p) {
    // half keys, even split; the sweeps of f = C(K,5), K = 10 to 15
    if (p.r != 5 || !p.half || p.fill != kWsFill || p.rtg) return nullptr;
    switch (ws_key(p.T, p.sweeps, p.half)) {
#define ASPIS_FWS5(TT, SWW) \
    case ws_key(TT, SWW, true): return ASPIS_NT(fused_ws_kernel, TT, 5, SWW, false, true, kWsFill, false);
        ASPIS_FWS5(128, 16)
        ASPIS_FWS5(128, 30)
        ASPIS_FWS5(64, 28)
        ASPIS_FWS5(32, 24)
        ASPIS_FWS5(32, 32)
    case ws_key(16, 24, true): return &fused_ws_kernel<16, 5, 24, false, true, kWsFill, false, false>;
#undef ASPIS_FWS5
    default: return nullptr;
    }
}

}  // namespace aspis
