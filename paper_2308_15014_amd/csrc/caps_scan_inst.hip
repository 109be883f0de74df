// Instantiates the matrix-core scan kernels of one precision and kind
// (0 approximate keys, 1 exact main pass, 2 exact rescue pass, 3 exact main
// pass with survivor counts, 5 approximate rescue pass): compiled once per
// (CAPS_INST_PREC, CAPS_INST_KIND), the approximate kinds once per row length
// (CAPS_INST_NS) too, so that they build in parallel.
#include "caps_mfma.h"

#if !defined(CAPS_INST_PREC) || !defined(CAPS_INST_KIND)
#error "compile with -DCAPS_INST_PREC=<CAPS_PREC_*> -DCAPS_INST_KIND=<0|1|2|3|5> [-DCAPS_INST_NS=<1|2|4|8>]"
#endif

namespace caps {

#define CAPS_PICK(N)                                                                              \
    template <>                                                                                   \
    LowpFn pick_lab<CAPS_INST_PREC, N, CAPS_INST_KIND>(bool lab, int r) {                         \
        return lab ? pick_cb<CAPS_INST_PREC, true, N, CAPS_INST_KIND>(r)                          \
                   : pick_cb<CAPS_INST_PREC, false, N, CAPS_INST_KIND>(r);                        \
    }
#ifdef CAPS_INST_NS
CAPS_PICK(CAPS_INST_NS)
#else
CAPS_PICK(1)
CAPS_PICK(2)
CAPS_PICK(4)
CAPS_PICK(8)
#endif

}  // namespace caps
