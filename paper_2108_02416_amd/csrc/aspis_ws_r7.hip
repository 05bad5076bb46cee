// aspis_ws_r7.hip -- the warp-specialised single pass at r = 7.
#include "aspis_ws.h"

namespace aspis {

FusedWsFn fused_ws_r7_fn(const WsPlan &p, bool ind) {
    // even split; the sweeps of f = C(K,7), K = 8 to 14
    if (p.r != 7 || p.fill != kWsFill || p.rtg) return nullptr;
#define M(TT, SWW, HH)                                                               \
    case ws_key(TT, SWW, HH):                                                        \
        return ind ? ASPIS_NT(fused_ws_kernel, TT, 7, SWW, true, HH, kWsFill, false) \
                   : ASPIS_NT(fused_ws_kernel, TT, 7, SWW, false, HH, kWsFill, false);
#define NARROW_BOTH(SWW)                                                                    \
    case ws_key(16, SWW, true):                                                             \
        return ind ? &fused_ws_kernel<16, 7, SWW, true, true, kWsFill, false, false>        \
                   : &fused_ws_kernel<16, 7, SWW, false, true, kWsFill, false, false>;
#define FILE_MAJOR_NARROW(SWW)  \
    case ws_key(16, SWW, true): \
        return ind ? nullptr : &fused_ws_kernel<16, 7, SWW, false, true, kWsFill, false, false>;
#define FILE_MAJOR(TT, SWW)     \
    case ws_key(TT, SWW, true): \
        return ind ? nullptr : ASPIS_NT(fused_ws_kernel, TT, 7, SWW, false, true, kWsFill, false);
    switch (ws_key(p.T, p.sweeps, p.half)) {
        M(64, 2, false)
        M(64, 4, false)
        M(64, 12, true)
        M(32, 16, true)
        FILE_MAJOR(32, 28)
        NARROW_BOTH(16)
        FILE_MAJOR_NARROW(28)
    default: return nullptr;
    }
#undef M
#undef FILE_MAJOR
#undef NARROW_BOTH
#undef FILE_MAJOR_NARROW
}

}  // namespace aspis
