// Launches of the descriptor product that pushes input lines into output lines.
#include "compact_push_kernel.h"
#include "dispatch.h"

namespace convspmv {

template <int KL>
void launch_push_kl(const CompactChoice &c, const PushGeom &g, const conv_plan *plan, const float *ktab, const float *x,
                    float *y, dim3 grid, hipStream_t q) {
#define CONV_PUSH(SCALAR, FINE) \
    spmm_compact_push_kernel<KL, SCALAR, FINE><<<grid, kPushWaves * kWave, c.lds, q>>>(plan->desc, ktab, x, y, g)
    if (c.scalar) {
        if (c.fine) CONV_PUSH(true, true);
        else CONV_PUSH(true, false);
    } else {
        if (c.fine) CONV_PUSH(false, true);
        else CONV_PUSH(false, false);
    }
#undef CONV_PUSH
}

void launch_compact_push(const CompactChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    constexpr unsigned kMaxGridY = 65535;
    PushGeom g = c.push;
    const size_t plane = (size_t)(plan->cols / plan->channels) * g.batch, kk = (size_t)g.k * g.k;
    // one launch per channel (its table, its operand plane): the first stores y, the others add to it
    for (int ch = 0; ch < plan->channels; ++ch) {
        g.accum = ch > 0;
        for (unsigned cb = 0; cb < c.col_blocks; cb += kMaxGridY) {
            g.c_base = (int)(cb * (c.scalar ? 1u : 4u * c.lpr));
            const dim3 grid((unsigned)(g.blocks_per_xcd * kXcds), std::min(kMaxGridY, c.col_blocks - cb));
            const float *ktab = plan->ktab + ch * kk, *xc = x + ch * plane;
            switch ((g.k + g.s - 1) / g.s) {
                case 1: launch_push_kl<1>(c, g, plan, ktab, xc, y, grid, q); break;
                case 2: launch_push_kl<2>(c, g, plan, ktab, xc, y, grid, q); break;
                case 3: launch_push_kl<3>(c, g, plan, ktab, xc, y, grid, q); break;
                case 4: launch_push_kl<4>(c, g, plan, ktab, xc, y, grid, q); break;
                case 5: launch_push_kl<5>(c, g, plan, ktab, xc, y, grid, q); break;
                case 6: launch_push_kl<6>(c, g, plan, ktab, xc, y, grid, q); break;
                case 7: launch_push_kl<7>(c, g, plan, ktab, xc, y, grid, q); break;
                case 8: launch_push_kl<8>(c, g, plan, ktab, xc, y, grid, q); break;
                case 9: launch_push_kl<9>(c, g, plan, ktab, xc, y, grid, q); break;
                case 10: launch_push_kl<10>(c, g, plan, ktab, xc, y, grid, q); break;
                case 11: launch_push_kl<11>(c, g, plan, ktab, xc, y, grid, q); break;
                case 12: launch_push_kl<12>(c, g, plan, ktab, xc, y, grid, q); break;
                default: launch_push_kl<13>(c, g, plan, ktab, xc, y, grid, q); break;
            }
        }
    }
}

}  // namespace convspmv
