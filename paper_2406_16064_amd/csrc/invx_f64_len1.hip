// Inverse-x pass of one compiled length each (double, 1 cell a thread).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_len<double, 1>(int, int, const Launch<double>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
