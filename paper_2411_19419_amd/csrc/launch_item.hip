// Launches of the kernel with a thread or a few per row and chunk of batch columns (apply_item_kernel.h).
#include "dispatch.h"

namespace convspmv {

template <int G, int C, int U, int NB, bool MANY>
static void launch_item_as(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    spmm_item_kernel<G, C, U, NB, MANY><<<dim3((unsigned)c.item.cells_per_xcd * kXcds), MANY ? (unsigned)c.item.ways * kWave : kItemThreads,
                                          c.lds, q>>>(plan->row_ptr, plan->col_idx, plan->vals, x, y, c.item);
}

// What U and NB fit the rows (item_choice: one lane for rows of one entry and, without channels, of 4; one or two, and up to
// four with several channels, for rows of 9).
template <int G, int C>
static void launch_item_g(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    const int most = plan->max_row_nnz;
    if (plan->channels > 1) {
        if (most == 1) {
            if constexpr (G == 1) launch_item_as<G, C, 1, 8, true>(c, plan, x, y, q);
        } else if (most == 9) {
            if constexpr (G <= 4) launch_item_as<G, C, 3, 3, true>(c, plan, x, y, q);
        } else {
            launch_item_as<G, C, 4, 2, true>(c, plan, x, y, q);
        }
    } else if constexpr (G <= 2) {
        if (most <= 4) {
            if constexpr (G == 1) {
                if (most == 1) launch_item_as<G, C, 1, 1, false>(c, plan, x, y, q);
                else launch_item_as<G, C, 4, 1, false>(c, plan, x, y, q);
            }
        } else if (most == 9) launch_item_as<G, C, G == 1 ? 9 : 5, 1, false>(c, plan, x, y, q);
        else if (most == 25) launch_item_as<G, C, 5, 2, false>(c, plan, x, y, q);
        else launch_item_as<G, C, 4, 2, false>(c, plan, x, y, q);
    } else if constexpr (G < 16 || C == 1) {
        launch_item_as<G, C, 4, 2, false>(c, plan, x, y, q);
    }
}

template <int C>
static void launch_item_c(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    switch (c.g) {
        case 1: launch_item_g<1, C>(c, plan, x, y, q); break;
        case 2: launch_item_g<2, C>(c, plan, x, y, q); break;
        case 4: launch_item_g<4, C>(c, plan, x, y, q); break;
        case 8: launch_item_g<8, C>(c, plan, x, y, q); break;
        default: launch_item_g<16, C>(c, plan, x, y, q); break;
    }
}

void launch_item(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    if (c.nv) launch_item_c<4>(c, plan, x, y, q);
    else launch_item_c<1>(c, plan, x, y, q);
}

}  // namespace convspmv
