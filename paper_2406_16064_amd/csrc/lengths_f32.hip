// Forward-x and y passes compiled for the 3-smooth lengths (float).
#include "hotpath.hpp"

namespace mmx {
template void fwd_x_launch_m<float>(int, const Launch<float>&, long long, int, size_t, hipStream_t);
template void y_launch_m<float>(bool, int, const Launch<float>&, long long, int, size_t, hipStream_t);
}  // namespace mmx
