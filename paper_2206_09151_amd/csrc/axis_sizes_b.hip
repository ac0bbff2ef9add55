// Single-axis slice kernels for detector sizes 45, 48, 50, 54, 60, 64, 72.
#include "axis_kernels.hpp"

namespace tomo {
const AxisSize kAxisSizesB[] = {axis_size<45>(), axis_size<48>(), axis_size<50>(), axis_size<54>(), axis_size<60>(), axis_size<64>(), axis_size<72>()};
const int kAxisSizesBCount = int(sizeof(kAxisSizesB) / sizeof(kAxisSizesB[0]));
}  // namespace tomo
