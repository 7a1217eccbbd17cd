// rows_kernel for 1-bit codes (see rows_mfma.h)
#include "rows_mfma.h"

namespace specache {
hipError_t launch_rows_b1(const LayerView& L, const RowsArgs& R, int NR, int mode, hipStream_t stream) {
    return mode == kRowsBoth    ? launch_rows_mode<1, kRowsBoth>(L, R, NR, stream)
           : mode == kRowsScore ? launch_rows_mode<1, kRowsScore>(L, R, NR, stream)
                                : launch_rows_mode<1, kRowsAttend>(L, R, NR, stream);
}
}  // namespace specache
