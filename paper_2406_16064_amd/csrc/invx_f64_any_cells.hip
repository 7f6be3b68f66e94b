// Inverse-x pass of the compiled lengths, each group by its own (double, general material, 1 and 2 cells a thread).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_any<double, true, 1>(int, bool, const Launch<double>&, long long, int, size_t, hipStream_t);
template void inv_x_launch_any<double, true, 2>(int, bool, const Launch<double>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
