// Forward-x and y passes of one compiled length each (double).
#include "hotpath.hpp"

namespace mmx {
template void len_launch<double>(int, int, const Launch<double>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
