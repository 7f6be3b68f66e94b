// Y passes of the compiled lengths beyond 1024 points (double).
#include "hotpath.hpp"

namespace mmx {
template void long_launch<double>(bool, int, const Launch<double>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
