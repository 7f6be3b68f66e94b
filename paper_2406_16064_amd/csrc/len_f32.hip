// Forward-x and y passes of one compiled length each (float).
#include "hotpath.hpp"

namespace mmx {
template void len_launch<float>(int, int, const Launch<float>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
