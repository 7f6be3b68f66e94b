// Inverse-x pass compiled for the powers of two from 256 (float, uniform material).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_s<float, false, true>(int, int, int, bool, const Launch<float>&, long long, int, size_t,
                                          hipStream_t);
}  // namespace mmx
