// Fused y and z passes of small 3-D planes (double): a translation unit of its own,
// so that the library builds in parallel.
#include "hotpath.hpp"

namespace mmx {
template void yzy_launch<double>(int, int, const Launch<double>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
