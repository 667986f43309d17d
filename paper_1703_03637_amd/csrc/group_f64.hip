// Class-blocked sector product, FP64 storage.
#include "group_impl.h"

namespace hphi {

HVG_INSTANTIATE(double, launch_hvg_f64, launch_hvg_multi_f64)

}  // namespace hphi
