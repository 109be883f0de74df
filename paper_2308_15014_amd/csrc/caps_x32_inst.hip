// Instantiates the 32 x 32 scan kernels of one precision, with or without
// label tests: compiled once per (CAPS_INST_PREC, CAPS_INST_LAB) pair so that
// they build in parallel.
#include "caps_x32.h"

#if !defined(CAPS_INST_PREC) || !defined(CAPS_INST_LAB)
#error "compile with -DCAPS_INST_PREC=<CAPS_PREC_*> -DCAPS_INST_LAB=<0|1>"
#endif

namespace caps {

template <int NS>
static LowpFn pick_mode(int mode) {
    constexpr bool LAB = CAPS_INST_LAB;
    if constexpr (!LAB) {
        if (mode == 1) return k_scan_x32<CAPS_INST_PREC, NS, 1, 1, false>;
    }
    if (mode == 2) return k_scan_x32<CAPS_INST_PREC, NS, 2, 1, LAB>;
    if (mode == 3) return k_scan_x32<CAPS_INST_PREC, NS, 2, 4, LAB>;
    return k_scan_x32<CAPS_INST_PREC, NS, 0, 1, LAB>;
}

template <>
LowpFn pick_x32<CAPS_INST_PREC, (bool)CAPS_INST_LAB>(int ns, int mode) {
    return ns == 1 ? pick_mode<1>(mode) : ns == 2 ? pick_mode<2>(mode) : pick_mode<4>(mode);
}

}  // namespace caps
