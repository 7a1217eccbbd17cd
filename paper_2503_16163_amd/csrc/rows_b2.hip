// rows_kernel for 2-bit codes (see rows_mfma.h)
#include "rows_mfma.h"

namespace specache {
hipError_t launch_rows_b2(const LayerView& L, const RowsArgs& R, int NR, int mode, hipStream_t stream) {
    return mode == kRowsBoth    ? launch_rows_mode<2, kRowsBoth>(L, R, NR, stream)
           : mode == kRowsScore ? launch_rows_mode<2, kRowsScore>(L, R, NR, stream)
                                : launch_rows_mode<2, kRowsAttend>(L, R, NR, stream);
}
}  // namespace specache
