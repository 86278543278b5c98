// Row sweep (row_sweep.h) for fused bonds up to 72.
#include "row_sweep.h"

namespace gipeps {
template hipError_t launch_row_class<72, 2>(const RowArgs&, hipStream_t);
}  // namespace gipeps
