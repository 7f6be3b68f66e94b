// Inverse-x pass of the compiled lengths, each group by its own (float, 4 cells a thread).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_any<float, false, 4>(int, bool, const Launch<float>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
