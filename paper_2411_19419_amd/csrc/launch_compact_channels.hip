// Launches of the one-launch channel sum over row descriptors.
#include "dispatch.h"

namespace convspmv {

template <int VB, int KK, int CH>
void launch_compact_channels_k(const ChannelsChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    const int threads = c.ways * kWave;
    const int per_lane = (c.geom.phx * c.geom.phy * (VB / 4) * CH + kWave - 1) / kWave;     // patch items a lane carries
    if (per_lane <= 4)
        spmm_compact_channels_kernel<VB, 4, KK, CH><<<c.grid, threads, c.lds, q>>>(plan->desc, plan->ktab, x, y, c.geom);
    else if (per_lane <= 8)
        spmm_compact_channels_kernel<VB, 8, KK, CH><<<c.grid, threads, c.lds, q>>>(plan->desc, plan->ktab, x, y, c.geom);
    else if constexpr (CH == 1)
        spmm_compact_channels_kernel<VB, kChanItems, KK, CH><<<c.grid, threads, c.lds, q>>>(plan->desc, plan->ktab, x, y, c.geom);
}

template <int VB, int CH>
void launch_compact_channels_vb(const ChannelsChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    switch (c.geom.k) {       // the kernel sizes of the paper's layer table (Table 2) have unrolled tap loops
        case 1: launch_compact_channels_k<VB, 1, CH>(c, plan, x, y, q); break;
        case 3: launch_compact_channels_k<VB, 3, CH>(c, plan, x, y, q); break;
        case 7:           // (chunks apart: 7 taps a side overlap too much for parts of tiles)
            if constexpr (CH == 1) {
                launch_compact_channels_k<VB, 7, CH>(c, plan, x, y, q);
                break;
            }
            [[fallthrough]];
        default: launch_compact_channels_k<VB, 0, CH>(c, plan, x, y, q); break;
    }
}

void launch_compact_channels(const ChannelsChoice &c, const conv_plan *plan, const float *x, float *y, hipStream_t q) {
    if (c.vb == 16) launch_compact_channels_vb<16, 1>(c, plan, x, y, q);
    else if (c.vb == 8) launch_compact_channels_vb<8, 1>(c, plan, x, y, q);
    else if (c.chunks == 4) launch_compact_channels_vb<4, 4>(c, plan, x, y, q);
    else if (c.chunks == 2) launch_compact_channels_vb<4, 2>(c, plan, x, y, q);
    else launch_compact_channels_vb<4, 1>(c, plan, x, y, q);
}

}  // namespace convspmv
