// Launches of the block kernel over T.
#include "dispatch.h"

namespace convspmv {

template <int K, int S>
static void launch_ks(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    if constexpr (block_compiled(K, S, false)) {
        const int columns = 4 << c.lpr_log2;
        const dim3 grid((unsigned)(c.block.cells_per_xcd * kXcds), (unsigned)((c.block.batch + columns - 1) / columns));
        auto launch = [&](auto lpr_tag) {
            spmm_block_kernel<K, S, false, decltype(lpr_tag)::value><<<grid, kBlockThreads, 0, q>>>(plan->row_ptr, plan->col_idx, plan->vals, x, y, c.block);
        };
        switch (c.lpr_log2) {
            case 4: launch(std::integral_constant<int, 4>{}); break;
            case 5: launch(std::integral_constant<int, 5>{}); break;
            default: launch(std::integral_constant<int, 6>{}); break;
        }
    }
}

template <int S>
static void launch_s(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    switch (plan->shape.k) {
        case 2: launch_ks<2, S>(c, plan, x, y, q); break;
        case 3: launch_ks<3, S>(c, plan, x, y, q); break;
        case 4: launch_ks<4, S>(c, plan, x, y, q); break;
        case 5: launch_ks<5, S>(c, plan, x, y, q); break;
    }
}

void launch_block(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    switch (plan->shape.s) {
        case 1: launch_s<1>(c, plan, x, y, q); break;
        case 2: launch_s<2>(c, plan, x, y, q); break;
        case 3: launch_s<3>(c, plan, x, y, q); break;
        case 4: launch_s<4>(c, plan, x, y, q); break;
    }
}

}  // namespace convspmv
