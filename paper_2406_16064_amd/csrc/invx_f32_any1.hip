// Inverse-x pass of the compiled lengths, each group by its own (float, 1 cell a thread).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_any<float, false, 1>(int, bool, const Launch<float>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
