// Row sweep (row_sweep.h) for fused bonds up to 16 (and every bond of D_k = 1).
#include "row_sweep.h"

namespace gipeps {
template hipError_t launch_row_class<16, 1>(const RowArgs&, hipStream_t);
template hipError_t launch_row_class<16, 2>(const RowArgs&, hipStream_t);
}  // namespace gipeps
