// Launches of the product from the column-compressed arrays that sums every output where it stays.
#include "dispatch.h"

namespace convspmv {

template <int KL, int STRIDE, int TW, int LPR_LOG2, bool SCALAR, int NLD, int NX, int DEPTH>
void launch_csc_gather_inst(const CscGatherChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    spmm_csc_gather_kernel<KL, STRIDE, TW, LPR_LOG2, SCALAR, NLD, NX, DEPTH><<<c.geom.blocks_per_xcd * kXcds, kCscGatherThreads, c.lds, q>>>(
        plan->row_ptr, plan->col_idx, plan->vals, x, y, c.geom, plan->edited);
}

// stride 1: the kernels that know their strip
template <int KL, int LPR_LOG2, bool SCALAR>
void launch_csc_gather_one(const CscGatherChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    constexpr int TW = csc_gather_tw(KL, 1, LPR_LOG2, SCALAR), NLD = (csc_gather_quads(TW, KL, 1) + kCscGatherThreads - 1) / kCscGatherThreads;
    constexpr int NX = (((TW + KL - 1) << LPR_LOG2) + kCscGatherThreads - 1) / kCscGatherThreads;
    launch_csc_gather_inst<KL, 1, TW, LPR_LOG2, SCALAR, NLD, NX, NLD <= 2 ? 2 : 1>(c, plan, x, y, q);
}

template <int KL, bool SCALAR>
void launch_csc_gather_kl(const CscGatherChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    if (plan->shape.s > 1) {
        if constexpr (KL > 2) {         // (k <= 2 s: fewer than 512 pixels' entries are at most 512 accesses, NLD 2)
            if (c.nld != 2) return launch_csc_gather_inst<KL, 0, 0, 0, SCALAR, 5, 3, 1>(c, plan, x, y, q);
        }
        if (c.nx == 1) launch_csc_gather_inst<KL, 0, 0, 0, SCALAR, 2, 1, 2>(c, plan, x, y, q);
        else launch_csc_gather_inst<KL, 0, 0, 0, SCALAR, 2, 3, 2>(c, plan, x, y, q);
    } else if constexpr (SCALAR) {
        if constexpr (csc_gather_few(KL, 1)) launch_csc_gather_one<KL, 0, true>(c, plan, x, y, q);
    } else {
        if (c.geom.lpr_log2 == 0) launch_csc_gather_one<KL, 0, false>(c, plan, x, y, q);
        else if (c.geom.lpr_log2 == 1) launch_csc_gather_one<KL, 1, false>(c, plan, x, y, q);
        else launch_csc_gather_one<KL, 2, false>(c, plan, x, y, q);
    }
}

template <bool SCALAR>
void launch_csc_gather_any(const CscGatherChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    switch (c.kl) {
        case 1:
            if constexpr (!SCALAR || csc_gather_few(1, 2)) launch_csc_gather_kl<1, SCALAR>(c, plan, x, y, q);
            break;
        case 2: launch_csc_gather_kl<2, SCALAR>(c, plan, x, y, q); break;
        case 3: launch_csc_gather_kl<3, SCALAR>(c, plan, x, y, q); break;
        case 4: launch_csc_gather_kl<4, SCALAR>(c, plan, x, y, q); break;
        case 5: launch_csc_gather_kl<5, SCALAR>(c, plan, x, y, q); break;
        case 6: launch_csc_gather_kl<6, SCALAR>(c, plan, x, y, q); break;
        case 7: launch_csc_gather_kl<7, SCALAR>(c, plan, x, y, q); break;
        case 8: launch_csc_gather_kl<8, SCALAR>(c, plan, x, y, q); break;
        case 9: launch_csc_gather_kl<9, SCALAR>(c, plan, x, y, q); break;
        case 10: launch_csc_gather_kl<10, SCALAR>(c, plan, x, y, q); break;
        case 11: launch_csc_gather_kl<11, SCALAR>(c, plan, x, y, q); break;
        case 12: launch_csc_gather_kl<12, SCALAR>(c, plan, x, y, q); break;
        default: launch_csc_gather_kl<13, SCALAR>(c, plan, x, y, q); break;
    }
}

void launch_csc_gather(const CscGatherChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    if (c.scalar) launch_csc_gather_any<true>(c, plan, x, y, q);
    else launch_csc_gather_any<false>(c, plan, x, y, q);
}

}  // namespace convspmv
