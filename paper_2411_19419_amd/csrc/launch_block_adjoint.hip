// Launches of the block kernel over T^T.
#include "launch_block.h"

namespace convspmv {

void launch_block_adjoint(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) { launch_block_any<true>(c, plan, x, y, q); }

}  // namespace convspmv
