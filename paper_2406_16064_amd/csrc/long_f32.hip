// Y passes of the compiled lengths beyond 1024 points (float).
#include "hotpath.hpp"

namespace mmx {
template void long_launch<float>(bool, int, const Launch<float>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
