// Product over the stored CSR arrays with the batch columns on the lanes (gfx950): small kernels, batches of a wave and more.
//
// Where a batch fills a wave, or a good part of one, an input pixel is one contiguous piece of memory per access.  So 16, 32 or 64
// lanes, 4 batch columns each, take a block of RX x RY outputs, ask for the WH x WW input pixels under it and for the entries
// of its rows all at once, and sum from registers: no barrier, no walk, no staging.  A pixel is read once per block that touches
// it, from the L1 or the L2 of its XCD for all but the first (a workgroup is 2 x 2 waves, neighbours run on one XCD).
//
// The entries of a wave are dealt to its lanes by their place in a full rectangle of taps: lane t loads tap t mod KL^2 of
// output t / KL^2, 0 where the tap lies outside the image (the pixel there is 0 too), and hands it to the others
// through LDS, from where a group reads four taps at a time.  Where an entry lies follows from its row's pointer and the
// geometry; the row's length and every stored column are compared with those of the geometry, and a wave that finds
// another (edited arrays) sums its rows entry by entry as they are stored.
//
// The same kernel applies T^T: there the operand is the window grid, the result the image, and result line i takes tap
// i + p - s x of operand line x.  Blocks then start where i + p is a multiple of s, so that which taps an output
// has is known to the compiler.
//
// Edited arrays, all rows of them (one row): 224^2, k 3, batch 256: 39 us (19), tile kernel 30; 256^2, k 5, s 2, batch 64: 17 (14) and 10;
// 224^2, k 5, batch 64: 54 (24), marching kernel 18.  The loop reads a pixel per entry and is bound by the caches; more loads
// ahead cost registers that the other path needs and did not help.
//
// Measured, fresh operands on every call: 224^2, k 3, batch 256: 17.8 us (6.0 TB/s of the bytes it cannot do without), the tile
// kernel 29.0; its T^T 18.0 and 28.7; 256^2, k 5, s 2, T^T, batch 256: 14.0 and 29.6, batch 64: 6.4 and
// 9.0.  What bounds it: memory where the plane is large, a chain of two loads (row pointer, entry) and the sums where it is small.
// Small blocks because the window's registers decide how many waves are in flight, and straight code is fetched once per
// wave: 224^2, k 3, batch 256, outputs per block 2 x 2: 18.1, 2 x 4: 18.7, 4 x 2: 21 (16 lanes; 2 x 2 19.1), 4 x 4: 22.8 (weights by
// v_readlane; 2 x 2 19.1).  Four columns per lane: one or two, with all 64 lanes on a pixel, 24 and 27 us.
#pragma once
#include <type_traits>

#include "device_util.h"
#include "apply_tile_kernel.h"

namespace convspmv {

constexpr int kBlockThreads = 256;          // 2 x 2 waves

struct BlockGeom {
    int m, n;                 // operand lines and pixels per line
    int m_out, n_out;         // result lines and pixels per line
    int p;
    int batch;
    int cells_y;              // workgroups side by side, 2 RY result pixels per group of a wave
    int cells, cells_per_xcd;
};

// taps per side that an output has at most, and operand lines under R result lines
__host__ __device__ constexpr int block_taps(int k, int s, bool tr) { return tr ? (k + s - 1) / s : k; }
__host__ __device__ constexpr int block_window(int r, int k, int s, bool tr) {
    return tr ? block_taps(k, s, tr) + (r - 1) / s : (r - 1) * s + k;
}
// taps along one axis of the result that is d-th in its block, the image's border left aside
__host__ __device__ constexpr int block_row_taps(int d, int k, int s, bool tr) { return tr ? (k - d % s + s - 1) / s : k; }
// result line (pixel) at which the first block starts
__host__ __device__ constexpr int block_first(int s, int p, bool tr) { return tr ? -(p % s) : 0; }

// Outputs of a block, and which (k, s) are compiled.  T, and T^T at stride 1: windows of at most 40 pixels (four
// registers each).  T^T above: one step of the stride, so that an operand pixel serves as many results as it has, and its taps are the
// window (at most 25 pixels).
__host__ __device__ constexpr bool block_compiled(int k, int s, bool tr) {
    if (!tr || s == 1) return (s <= 2 && k >= 2 && k <= 5) || (!tr && s <= 4 && k >= 3 && k <= 5);
    return s <= 4 && k > s && k <= (s == 2 ? 5 : 4) * s && k <= 13;
}
__host__ __device__ constexpr int block_rx(int k, int s, bool tr) {
    if (tr && s > 1) return s;
    return s == 1 ? (k == 5 ? 1 : 2) : s == 2 ? (k == 4 ? 1 : 2) : 1;
}
__host__ __device__ constexpr int block_ry(int k, int s, bool tr) {
    if (tr && s > 1) return s;
    return s == 1 ? (k == 5 ? 4 : 2) : s == 2 ? (k == 5 ? 1 : 2) : k == 5 ? 1 : 2;
}
constexpr int kBlockLprLeast = 4, kBlockLprMost = 6;        // lanes over the batch: 16 to 64 (64 to 256 columns)

// words between the weights of two outputs, and of two groups of lanes (their reads meet in different banks)
__host__ __device__ constexpr int block_tap_words(int taps) { return (taps + 3) & ~3; }
__host__ __device__ constexpr int block_group_words(int outputs, int taps) { return outputs * block_tap_words(taps) + 4; }

template <int I, int N, typename F>
__device__ __forceinline__ void block_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        block_for<I + 1, N>(f);
    }
}

// Taps of result line t along one axis: the first operand line, how many.
template <int K, int S, bool TR>
__device__ __forceinline__ void block_axis(int t, int p, int lines, int &lo, int &count) {
    if constexpr (TR) {
        const int hi = min((t + p) / S, lines - 1);
        lo = t + p < K ? 0 : (t + p - K) / S + 1;
        count = max(hi - lo + 1, 0);
    } else {
        const int a = max(p - S * t, 0), b = min(K, lines + p - S * t);
        lo = S * t - p + a;
        count = max(b - a, 0);
    }
}

template <int K, int S, bool TR, int LPR_LOG2>
__global__ __launch_bounds__(kBlockThreads, 2) void spmm_block_kernel(const int *__restrict__ row_ptr,
                                                                     const int *__restrict__ col_idx,
                                                                     const float *__restrict__ vals,
                                                                     const float *__restrict__ x, float *__restrict__ y,
                                                                     const BlockGeom g) {
    constexpr int RX = block_rx(K, S, TR), RY = block_ry(K, S, TR);
    static_assert(!TR || (RX % S == 0 && RY % S == 0), "blocks start at the same place of the stride");
    constexpr int KL = block_taps(K, S, TR), TAPS = KL * KL, OUT = RX * RY;
    constexpr int WH = block_window(RX, K, S, TR), WW = block_window(RY, K, S, TR);
    constexpr int LPR = 1 << LPR_LOG2, GROUPS = kWave / LPR;
    constexpr int NW = (GROUPS * OUT * TAPS + kWave - 1) / kWave;
    constexpr int LANES = TAPS <= 10 ? 2 : 8;               // see the sums
    constexpr int TW = block_tap_words(TAPS), GW = block_group_words(OUT, TAPS);
    __shared__ __align__(16) float weights[kBlockThreads / kWave][GROUPS * GW];

    const int at = (int)blockIdx.x / kXcds, cell = ((int)blockIdx.x % kXcds) * g.cells_per_xcd + at;
    if (at >= g.cells_per_xcd || cell >= g.cells) return;
    const int lane = (int)threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int cx = cell / g.cells_y, cy = cell - cx * g.cells_y;
    const int x0 = (2 * cx + wave / 2) * RX + block_first(S, g.p, TR);
    const int y_wave = (2 * cy + wave % 2) * (GROUPS * RY) + block_first(S, g.p, TR);
    if (x0 >= g.m_out || y_wave >= g.n_out) return;
    const int group = lane >> LPR_LOG2, y0 = y_wave + group * RY;
    // first operand line and pixel of the window
    auto window = [&](int t) { return TR ? (t + g.p) / S - (KL - 1) : S * t - g.p; };
    const int i0 = window(x0), j0 = window(y0);
    const int c = ((int)blockIdx.y * LPR + (lane & (LPR - 1))) * 4, cc = chunk_col(c, g.batch);

    // the rows of this lane's taps
    int beg[NW], len[NW];
#pragma unroll
    for (int r = 0; r < NW; ++r) {
        const int t = r * kWave + lane, o = t / TAPS % OUT, xo = x0 + o / RY, yo = y_wave + t / (TAPS * OUT) * RY + o % RY;
        const bool inside = t < GROUPS * OUT * TAPS && xo >= 0 && xo < g.m_out && yo >= 0 && yo < g.n_out;
        const int row = inside ? xo * g.n_out + yo : 0;
        beg[r] = row_ptr[row];
        len[r] = row_ptr[row + 1];
    }
    // the window (lines are the same for the whole wave, pixels are not)
    const bool interior = __all(i0 >= 0 && i0 + WH <= g.m && j0 >= 0 && j0 + WW <= g.n);
    vec4u px[WH][WW];
    if (interior) {
        const unsigned lane_off = 4u * (unsigned)((i0 * g.n + j0) * g.batch + cc);
#pragma unroll
        for (int wi = 0; wi < WH; ++wi)
#pragma unroll
            for (int wj = 0; wj < WW; ++wj)
                px[wi][wj] = *reinterpret_cast<const vec4u *>(reinterpret_cast<const char *>(x + (long long)(wi * g.n + wj) * g.batch) + lane_off);
    } else {
#pragma unroll
        for (int wi = 0; wi < WH; ++wi) {
            const float *const line = x + (long long)min(max(i0 + wi, 0), g.m - 1) * g.n * g.batch;
#pragma unroll
            for (int wj = 0; wj < WW; ++wj)
                px[wi][wj] = *reinterpret_cast<const vec4u *>(reinterpret_cast<const char *>(line) +
                                                             4u * (unsigned)(min(max(j0 + wj, 0), g.n - 1) * g.batch + cc));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // the entries: weights to LDS; is anything not as built?
    float w[NW];
    int stored[NW], want[NW];
    bool odd = false;
#pragma unroll
    for (int r = 0; r < NW; ++r) {
        const int t = r * kWave + lane, o = t / TAPS % OUT, tap = t % TAPS, dx = o / RY, dy = o % RY;
        const int y_first = y_wave + t / (TAPS * OUT) * RY, xo = x0 + dx, yo = y_first + dy;
        const bool inside = t < GROUPS * OUT * TAPS && xo >= 0 && xo < g.m_out && yo >= 0 && yo < g.n_out;
        int lo1 = 0, q1 = 0, lo2 = 0, q2 = 0;
        block_axis<K, S, TR>(xo, g.p, g.m, lo1, q1);
        block_axis<K, S, TR>(yo, g.p, g.n, lo2, q2);
        const int i = i0 + (TR ? KL - 1 + dx / S - tap / KL : dx * S + tap / KL);
        const int j = window(y_first) + (TR ? KL - 1 + dy / S - tap % KL : dy * S + tap % KL);
        const bool as_built = !inside || len[r] - beg[r] == q1 * q2;
        const bool has = inside && as_built && i >= lo1 && i < lo1 + q1 && j >= lo2 && j < lo2 + q2;
        odd |= !as_built;
        const int e = has ? beg[r] + (i - lo1) * q2 + (j - lo2) : 0;
        want[r] = has ? i * g.n + j : -1;
        stored[r] = col_idx[e];
        w[r] = vals[e];
    }
    float *const mine = weights[wave];
#pragma unroll
    for (int r = 0; r < NW; ++r) {
        const int t = r * kWave + lane;
        odd |= want[r] >= 0 && stored[r] != want[r];
        if (t < GROUPS * OUT * TAPS)
            mine[t / (OUT * TAPS) * GW + t / TAPS % OUT * TW + t % TAPS] = want[r] >= 0 ? w[r] : 0.0f;
    }
    const bool live = c < g.batch;
    const unsigned out_off = 4u * (unsigned)((x0 * g.n_out + y0) * g.batch + cc);       // (of an output outside: not used)
    auto outside = [&](int dx, int dy) { return x0 + dx < 0 || x0 + dx >= g.m_out || y0 + dy < 0 || y0 + dy >= g.n_out; };
    auto store = [&](int dx, int dy, const vec4u &sum) {
        if (live && !outside(dx, dy)) {
            const unsigned off = out_off + 4u * (unsigned)((dx * g.n_out + dy) * g.batch);
            __builtin_nontemporal_store(sum, reinterpret_cast<vec4u *>(reinterpret_cast<char *>(y) + off));
        }
    };
    if (__builtin_expect(__ballot(odd) != 0, 0)) {           // (uniform) whatever the rows hold
        for (int o = 0; o < OUT; ++o) {
            const int dx = o / RY, dy = o % RY;
            if (outside(dx, dy)) continue;
            const int row = (x0 + dx) * g.n_out + y0 + dy;
            vec4u sum = vec4u(0.0f);
            for (int e = row_ptr[row], end = row_ptr[row + 1]; e < end; ++e)
                sum += vals[e] * *reinterpret_cast<const vec4u *>(x + (long long)col_idx[e] * g.batch + cc);
            store(dx, dy, sum);
        }
        return;
    }
    if (!interior) {
#pragma unroll
        for (int wi = 0; wi < WH; ++wi)
#pragma unroll
            for (int wj = 0; wj < WW; ++wj)
                if (i0 + wi < 0 || i0 + wi >= g.m || j0 + wj < 0 || j0 + wj >= g.n) px[wi][wj] = vec4u(0.0f);
    }
    wave_lds_order();

    const float *const group_weights = mine + group * GW;
    block_for<0, OUT>([&](auto out_tag) {
        constexpr int O = decltype(out_tag)::value, DX = O / RY, DY = O % RY;
        constexpr int N2 = block_row_taps(DY, K, S, TR), N = block_row_taps(DX, K, S, TR) * N2;
        float wt[TW];
#pragma unroll
        for (int q = 0; q < TW; q += 4) *reinterpret_cast<float4 *>(wt + q) = *reinterpret_cast<const float4 *>(group_weights + O * TW + q);
        // One chain for entries l, l + LANES, ... of the row, the chains added as a tree: the order of the tile kernel, whose
        // LANES lanes share a row, so that results are as far from exact ones as its are (away from the border they are the same).
        auto chain = [&](int l) -> vec4u {
            vec4u sum = vec4u(0.0f);
#pragma unroll
            for (int e = l; e < N; e += LANES) {
                const int q = TR ? N - 1 - e : e, u = q / N2, v = q % N2;
                const vec4u pixel = px[TR ? KL - 1 + DX / S - u : DX * S + u][TR ? KL - 1 + DY / S - v : DY * S + v];
                const float f = wt[u * KL + v];
#pragma unroll
                for (int h = 0; h < 4; ++h) sum[h] = e == l ? f * pixel[h] : fmaf(f, pixel[h], sum[h]);
            }
            return sum;
        };
        if constexpr (N == 1) {
            store(DX, DY, chain(0));
        } else if constexpr (LANES == 2) {
            const vec4u even = chain(0);
            store(DX, DY, even + chain(1));
        } else {
            vec4u a = chain(0);
            a += chain(7);
            vec4u b = chain(2);
            b += chain(5);
            a += b;
            b = chain(1);
            b += chain(6);
            vec4u c = chain(3);
            c += chain(4);
            b += c;
            store(DX, DY, a + b);
        }
    });
}

}  // namespace convspmv
