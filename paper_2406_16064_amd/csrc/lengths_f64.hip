// Forward-x and y passes of the compiled 3-smooth lengths (double).
#include "hotpath.hpp"

namespace mmx {
template void fwd_x_launch_m<double>(const Launch<double>&, long long, int, size_t, hipStream_t);
template void y_launch_m<double>(int, const Launch<double>&, long long, int, size_t, hipStream_t);
template void yinv_launch_m<double>(const Launch<double>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
