// aspis_ws_r5.hip -- the warp-specialised single pass at r = 5.
#include "aspis_ws.h"

namespace aspis {

FusedWsFn fused_ws_r5_fn(const WsPlan &p, bool ind) {
    // even split; the sweeps of f = C(K,5), K = 6 to 15
    if (p.r != 5 || p.fill != kWsFill || p.rtg) return nullptr;
#define M(TT, SWW, HH)                                                               \
    case ws_key(TT, SWW, HH):                                                        \
        return ind ? ASPIS_NT(fused_ws_kernel, TT, 5, SWW, true, HH, kWsFill, false) \
                   : ASPIS_NT(fused_ws_kernel, TT, 5, SWW, false, HH, kWsFill, false);
#define FILE_MAJOR(TT, SWW) \
    case ws_key(TT, SWW, true): \
        return ind ? nullptr : ASPIS_NT(fused_ws_kernel, TT, 5, SWW, false, true, kWsFill, false);
#define NARROW(SWW, IND)        \
    case ws_key(16, SWW, true): \
        return ind != IND ? nullptr : &fused_ws_kernel<16, 5, SWW, IND, true, kWsFill, false, false>;
    switch (ws_key(p.T, p.sweeps, p.half)) {
        M(64, 2, false)
        M(64, 4, false)
        M(128, 16, true)
        M(128, 30, true)
        M(64, 28, true)
        M(32, 24, true)
        FILE_MAJOR(32, 32)
        NARROW(24, false)
        NARROW(16, true)
    default: return nullptr;
    }
#undef M
#undef FILE_MAJOR
#undef NARROW
}

}  // namespace aspis
