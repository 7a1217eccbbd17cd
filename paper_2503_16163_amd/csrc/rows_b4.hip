// rows_kernel for 4-bit codes (see rows_mfma.h): scoring and attention as two launches
#include "rows_mfma.h"

namespace specache {
hipError_t launch_rows_b4(const LayerView& L, const RowsArgs& R, int NR, int mode, hipStream_t stream) {
    return mode == kRowsScore    ? launch_rows_mode<4, kRowsScore>(L, R, NR, stream)
           : mode == kRowsAttend ? launch_rows_mode<4, kRowsAttend>(L, R, NR, stream)
                                 : hipErrorInvalidValue;
}
}  // namespace specache
