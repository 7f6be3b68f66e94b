// Inverse-x pass of one compiled length each (float, 2 cells a thread).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_len<float, 2>(int, int, const Launch<float>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
