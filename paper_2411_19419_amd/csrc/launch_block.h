// Launches of the block kernel over T or T^T (one translation unit each: they compile side by side).
#pragma once
#include "dispatch.h"

namespace convspmv {

template <bool TR, int K, int S>
void launch_block_ks(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    if constexpr (block_compiled(K, S, TR)) {
        const int columns = 4 << c.lpr_log2;
        const dim3 grid((unsigned)(c.block.cells_per_xcd * kXcds), (unsigned)((c.block.batch + columns - 1) / columns));
        auto launch = [&](auto lpr_tag) {
            spmm_block_kernel<K, S, TR, decltype(lpr_tag)::value><<<grid, kBlockThreads, 0, q>>>(plan->row_ptr, plan->col_idx, plan->vals, x, y, c.block);
        };
        switch (c.lpr_log2) {
            case 4: launch(std::integral_constant<int, 4>{}); break;
            case 5: launch(std::integral_constant<int, 5>{}); break;
            default: launch(std::integral_constant<int, 6>{}); break;
        }
    }
}

template <bool TR, int S>
void launch_block_s(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    switch (plan->shape.k) {
        case 2: launch_block_ks<TR, 2, S>(c, plan, x, y, q); break;
        case 3: launch_block_ks<TR, 3, S>(c, plan, x, y, q); break;
        case 4: launch_block_ks<TR, 4, S>(c, plan, x, y, q); break;
        case 5: launch_block_ks<TR, 5, S>(c, plan, x, y, q); break;
        case 6: launch_block_ks<TR, 6, S>(c, plan, x, y, q); break;
        case 7: launch_block_ks<TR, 7, S>(c, plan, x, y, q); break;
        case 8: launch_block_ks<TR, 8, S>(c, plan, x, y, q); break;
        case 9: launch_block_ks<TR, 9, S>(c, plan, x, y, q); break;
        case 10: launch_block_ks<TR, 10, S>(c, plan, x, y, q); break;
        case 11: launch_block_ks<TR, 11, S>(c, plan, x, y, q); break;
        case 12: launch_block_ks<TR, 12, S>(c, plan, x, y, q); break;
        case 13: launch_block_ks<TR, 13, S>(c, plan, x, y, q); break;
    }
}

template <bool TR>
void launch_block_any(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    switch (plan->shape.s) {
        case 1: launch_block_s<TR, 1>(c, plan, x, y, q); break;
        case 2: launch_block_s<TR, 2>(c, plan, x, y, q); break;
        case 3: launch_block_s<TR, 3>(c, plan, x, y, q); break;
        case 4: launch_block_s<TR, 4>(c, plan, x, y, q); break;
    }
}

}  // namespace convspmv
