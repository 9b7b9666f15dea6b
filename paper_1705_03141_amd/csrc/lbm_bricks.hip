// lbm_bricks.hip -- the brick kernels of small lattices, for every population storage.
#include "lbm_brick.h"

namespace lbm {
LBM_INSTANTIATE_BRICK(float)
LBM_INSTANTIATE_BRICK(_Float16)
LBM_INSTANTIATE_BRICK(bf16)
}  // namespace lbm
