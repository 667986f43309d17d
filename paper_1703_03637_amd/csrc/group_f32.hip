// Class-blocked sector product, FP32 storage.
#include "group_impl.h"

namespace hphi {

HVG_INSTANTIATE(float, launch_hvg_f32, launch_hvg_multi_f32)

}  // namespace hphi
