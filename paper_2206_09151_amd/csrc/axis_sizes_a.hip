// Single-axis slice kernels for detector sizes 16, 18, 20, 24, 25, 27, 30, 32, 36, 40.
#include "axis_kernels.hpp"

namespace tomo {
const AxisSize kAxisSizesA[] = {axis_size<16>(), axis_size<18>(), axis_size<20>(), axis_size<24>(), axis_size<25>(), axis_size<27>(), axis_size<30>(), axis_size<32>(), axis_size<36>(), axis_size<40>()};
const int kAxisSizesACount = int(sizeof(kAxisSizesA) / sizeof(kAxisSizesA[0]));
}  // namespace tomo
