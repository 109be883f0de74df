// Instantiates the 32 x 32 scan kernels of one precision and filter kind:
// compiled once per (CAPS_INST_PREC, CAPS_INST_FILT) pair so that they build in
// parallel.
#include "caps_x32.h"

#if !defined(CAPS_INST_PREC) || !defined(CAPS_INST_FILT)
#error "compile with -DCAPS_INST_PREC=<CAPS_PREC_*> -DCAPS_INST_FILT=<0|1|2>"
#endif

namespace caps {

template <int NS>
static LowpFn pick_mode(int mode) {
    constexpr int F = CAPS_INST_FILT;
    if constexpr (F == 0) {
        if (mode == 1) return k_scan_x32<CAPS_INST_PREC, NS, 1, 1, 0>;
    }
    if (mode == 2) return k_scan_x32<CAPS_INST_PREC, NS, 2, 1, F>;
    if (mode == 3) return k_scan_x32<CAPS_INST_PREC, NS, 2, 4, F>;
    if (mode == 4) return k_scan_x32<CAPS_INST_PREC, NS, 3, 1, F>;
    return k_scan_x32<CAPS_INST_PREC, NS, 0, 1, F>;
}

template <>
LowpFn pick_x32<CAPS_INST_PREC, CAPS_INST_FILT>(int ns, int mode) {
    return ns == 1 ? pick_mode<1>(mode) : ns == 2 ? pick_mode<2>(mode) : pick_mode<4>(mode);
}

}  // namespace caps
