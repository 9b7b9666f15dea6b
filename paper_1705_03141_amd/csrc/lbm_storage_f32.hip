// lbm_storage_f32.hip -- kernels instantiated for float population storage.
#include "lbm_scan.h"

namespace lbm {
LBM_INSTANTIATE_STORAGE(float)
LBM_INSTANTIATE_STEP(float)
LBM_INSTANTIATE_SCAN(float)
}  // namespace lbm
