// Launches of the block kernel over T.
#include "launch_block.h"

namespace convspmv {

void launch_block(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) { launch_block_any<false>(c, plan, x, y, q); }

}  // namespace convspmv
