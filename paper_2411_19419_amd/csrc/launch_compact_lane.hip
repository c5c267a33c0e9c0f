// Launches of the product from row descriptors with a lane per row and chunk of batch columns (compact_lane_kernel.h).
#include "dispatch.h"

namespace convspmv {

template <int K>
static void launch_compact_lane_k(const CompactChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    const dim3 grid((unsigned)c.lane.cells_per_xcd * kXcds);
    if (c.scalar) spmm_compact_lane_kernel<K, 1><<<grid, kItemThreads, 0, q>>>(plan->desc, plan->ktab, x, y, c.lane);
    else spmm_compact_lane_kernel<K, 4><<<grid, kItemThreads, 0, q>>>(plan->desc, plan->ktab, x, y, c.lane);
}

void launch_compact_lane(const CompactChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    switch (plan->shape.k) {
        case 2: launch_compact_lane_k<2>(c, plan, x, y, q); break;
        case 3: launch_compact_lane_k<3>(c, plan, x, y, q); break;
        case 4: launch_compact_lane_k<4>(c, plan, x, y, q); break;
        case 5: launch_compact_lane_k<5>(c, plan, x, y, q); break;
        case 6: launch_compact_lane_k<6>(c, plan, x, y, q); break;
        case 7: launch_compact_lane_k<7>(c, plan, x, y, q); break;
        case 8: launch_compact_lane_k<8>(c, plan, x, y, q); break;
        case 9: launch_compact_lane_k<9>(c, plan, x, y, q); break;
        case 10: launch_compact_lane_k<10>(c, plan, x, y, q); break;
        case 11: launch_compact_lane_k<11>(c, plan, x, y, q); break;
        case 12: launch_compact_lane_k<12>(c, plan, x, y, q); break;
        default: launch_compact_lane_k<13>(c, plan, x, y, q); break;
    }
}

}  // namespace convspmv
