#include "setd_small_impl.hpp"

namespace setd {
template hipError_t launch_small2d<float>(const Geo&, const Item*, int, int, int, int, bool, const Record&, hipStream_t);
}
