// Inverse-x pass of the compiled lengths, each group by its own (double, 4 cells a thread).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_any<double, false, 4>(int, bool, const Launch<double>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
