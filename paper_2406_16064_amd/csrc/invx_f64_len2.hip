// Inverse-x pass of one compiled length each (double, 2 cells a thread).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_len<double, 2>(int, int, const Launch<double>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
