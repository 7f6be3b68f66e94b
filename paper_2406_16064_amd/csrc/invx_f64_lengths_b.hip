// Inverse-x pass compiled for the powers of two from 256 (double, uniform material).
#include "hotpath.hpp"

namespace mmx {
template void inv_x_launch_s<double, false, true>(int, int, int, bool, const Launch<double>&, long long, int, size_t,
                                          hipStream_t);
}  // namespace mmx
