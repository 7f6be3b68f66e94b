// Forward-x and y passes of the compiled 3-smooth lengths (float).
#include "hotpath.hpp"

namespace mmx {
template void fwd_x_launch_m<float>(const Launch<float>&, long long, int, size_t, hipStream_t);
template void y_launch_m<float>(int, const Launch<float>&, long long, int, size_t, hipStream_t);
template void yinv_launch_m<float>(const Launch<float>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
