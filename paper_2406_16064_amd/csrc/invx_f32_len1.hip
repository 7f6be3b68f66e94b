// Inverse-x pass of one compiled length each (float, 1 cell a thread).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_len<float, 1>(int, int, const Launch<float>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
