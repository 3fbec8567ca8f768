// Pass launchers for radii 10..12, image type float, storage type _Float16
// (split over several files so the build compiles them in parallel).
#include "rsf_kernels.hpp"

namespace rsf {
RSF_INSTANTIATE(10, float, _Float16)
RSF_INSTANTIATE(11, float, _Float16)
RSF_INSTANTIATE(12, float, _Float16)
}  // namespace rsf
