// Single-axis slice kernels for detector sizes 100, 108, 120, 125, 128.
#include "axis_kernels.hpp"

namespace tomo {
const AxisSize kAxisSizesD[] = {axis_size<100>(), axis_size<108>(), axis_size<120>(), axis_size<125>(), axis_size<128>()};
const int kAxisSizesDCount = int(sizeof(kAxisSizesD) / sizeof(kAxisSizesD[0]));
}  // namespace tomo
