// Single-axis slice kernels for detector sizes 135, 144, 150, 160, 162, 180, 192.
#include "axis_kernels.hpp"

namespace tomo {
const AxisSize kAxisSizesE[] = {axis_size<135>(), axis_size<144>(), axis_size<150>(), axis_size<160>(), axis_size<162>(), axis_size<180>(), axis_size<192>()};
const int kAxisSizesECount = int(sizeof(kAxisSizesE) / sizeof(kAxisSizesE[0]));
}  // namespace tomo
