// Product from the row descriptors, a lane per row and chunk of batch columns, x from global memory (gfx950).
//
// The row groups of compact_kernels.h deal the taps of a row out to lanes: every lane looks its kernel number up and reads a pixel of
// its own.  Here, as in apply_item_kernel.h, the chunks of columns of a row lie side by side on the lanes, then those of the next
// row, and all lanes of a wave take the same tap at a time: the kernel number is the same for all, a scalar operand,
// and the pixels of neighbouring rows and columns come in whole memory lines.  The taps of a line, of two or of
// all for small kernels, are asked for at once.  Which taps a row has is what its descriptor says, whatever that is: a wave
// whose rows all have all taps reads without a test, else each lane tests every tap against its rectangle (and neither reads nor adds
// where it has none: a pixel that is not the row's may be infinite, and so may a number).
// Sums: one to four chains per line, the sums of lines added in 64 bits (K 2: one chain of all taps).  Error against 64 bits over that
// of the kernels it takes products from, in the mean of 535: 0.71 (K 2 1.00, K 3 0.79, K 5 0.63, K 7 0.77, K 11 0.77).  With up to four
// 32-bit sums of lines in turn, in the same time: 0.83, but K 5 from row groups of 8 lanes 1.02, one kernel of K 3 up to 1.18.
//
// Measured, two sets of operands in turn, before -> after (us):
//   row groups        85 x 92, k 4, p 2, batch 204      13.3 -> 6.6      360 x 306, k 8, p 7, batch 3     18.5 -> 8.4
//                     530 x 621, k 3, s 2, batch 92     87.6 -> 30.4     1161 x 1222, k 9, s 2, batch 1   38.2 -> 18.7
//   described         350 x 322, k 6, s 3, batch 40     13.7 -> 6.9      1628 x 1808, k 4, s 2, batch 2   23.0 -> 15.0
//   rectangles        2108 x 1652, k 2, s 2, batch 3    24.4 -> 11.5     1612 x 2501, k 3, s 2, batch 1   11.7 -> 7.9
// What bounds it: the L1 where the taps are many (a pixel per tap and lane: 208 x 277, k 11, batch 16 takes 22 us of arithmetic and
// reads that memory would give in 2.8), the memory where they are few (530 x 621 above: 22 us at the rate of a large copy).
#pragma once
#include "apply_item_kernel.h"
#include "compact_kernels.h"

namespace convspmv {

struct LaneGeom {
    int n, batch;
    int chunks;                        // chunks of C columns per row
    float inv_chunks;
    unsigned items;                    // rows * chunks
    int cells, cells_per_xcd;          // workgroups
};

template <int K, int C>
__global__ __launch_bounds__(kItemThreads) void spmm_compact_lane_kernel(
    const int2 *__restrict__ desc, const float *__restrict__ ktab, const float *__restrict__ x, float *__restrict__ y, const LaneGeom g) {
    typedef float part __attribute__((ext_vector_type(C)));
    typedef float part_at __attribute__((ext_vector_type(C), aligned(4)));
    typedef double sum_t __attribute__((ext_vector_type(C)));
    // tap lines asked for at a time: a dozen pixels at least in flight
    constexpr int LINES = K >= 7 ? 1 : K >= 4 ? 2 : K;
    // chains of a line's sum; the sums of lines are added in 64 bits (K 2: one chain of all taps)
    constexpr int CHAINS = K >= 11 ? 4 : K >= 5 ? 2 : 1;
    constexpr bool WIDE = K > 2;
    const int at = (int)blockIdx.x / kXcds, cell = ((int)blockIdx.x % kXcds) * g.cells_per_xcd + at;
    if (at >= g.cells_per_xcd || cell >= g.cells) return;
    const int lane = (int)threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const unsigned first = ((unsigned)cell * (kItemThreads / kWave) + wave) * kWave;
    const unsigned row0 = first / (unsigned)g.chunks;
    const int t = (int)(first - row0 * (unsigned)g.chunks) + lane, q = div_small(t, g.inv_chunks);
    const int row = (int)row0 + q, chunk = t - q * g.chunks;
    const int c = C == 4 ? chunk_col(4 * chunk, g.batch) : chunk;
    const bool live = first + (unsigned)lane < g.items;
    const int2 d = live ? desc[row] : make_int2(0, 0);
    const unsigned w = (unsigned)d.y;
    const int a_lo = w & 255u, r1 = (w >> 8) & 255u, b_lo = (w >> 16) & 255u, r2 = w >> 24;
    // byte offset of the pixel under tap (0, 0), whether there is one or not (modulo 2^32, as all sums of it)
    const unsigned pitch = 4u * (unsigned)g.batch;
    const unsigned origin = ((unsigned)d.x - (unsigned)(a_lo * g.n + b_lo)) * pitch + 4u * (unsigned)c;
    auto pixel = [&](unsigned tap_off) -> part {
        return *reinterpret_cast<const part_at *>(reinterpret_cast<const char *>(x) + (origin + tap_off));
    };
    auto fma_part = [&](float f, part p, part s) -> part {
        part r;
#pragma unroll
        for (int h = 0; h < C; ++h) r[h] = fmaf(f, p[h], s[h]);
        return r;
    };
    const bool whole = __builtin_amdgcn_ballot_w64(live && (b_lo != 0 || r2 != K || a_lo != 0 || r1 != K)) == 0;
    part acc = part(0.0f);
    sum_t wide = sum_t(0.0);
    auto add = [&](part (&sum)[CHAINS]) {
#pragma unroll
        for (int half = CHAINS / 2; half > 0; half /= 2) {
#pragma unroll
            for (int i = 0; i < half; ++i) sum[i] = sum[2 * i] + sum[2 * i + 1];
        }
        if constexpr (WIDE) wide += __builtin_convertvector(sum[0], sum_t);
        else acc = sum[0];
    };
    auto tap_lines = [&](int a, auto count_tag) {
        constexpr int N = decltype(count_tag)::value;
        part px[N][K];
        if (whole && live) {
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int b = 0; b < K; ++b) px[i][b] = pixel((unsigned)((a + i) * g.n + b) * pitch);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                part sum[CHAINS];
#pragma unroll
                for (int j = 0; j < CHAINS; ++j) sum[j] = WIDE ? part(0.0f) : acc;
#pragma unroll
                for (int b = 0; b < K; ++b) sum[b % CHAINS] = fma_part(ktab[(a + i) * K + b], px[i][b], sum[b % CHAINS]);
                add(sum);
            }
        } else {
            auto has = [&](int i, int b) { return a + i >= a_lo && a + i < a_lo + r1 && b >= b_lo && b < b_lo + r2; };
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int b = 0; b < K; ++b)
                    if (has(i, b)) px[i][b] = pixel((unsigned)((a + i) * g.n + b) * pitch);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                part sum[CHAINS];
#pragma unroll
                for (int j = 0; j < CHAINS; ++j) sum[j] = WIDE ? part(0.0f) : acc;
#pragma unroll
                for (int b = 0; b < K; ++b)
                    if (has(i, b)) sum[b % CHAINS] = fma_part(ktab[(a + i) * K + b], px[i][b], sum[b % CHAINS]);
                add(sum);
            }
        }
    };
    int a = 0;
    for (; a + LINES <= K; a += LINES) tap_lines(a, std::integral_constant<int, LINES>{});
    if constexpr (LINES > 1)
        for (; a < K; ++a) tap_lines(a, std::integral_constant<int, 1>{});
    if constexpr (WIDE) acc = __builtin_convertvector(wide, part);
    if (live) *reinterpret_cast<part_at *>(reinterpret_cast<char *>(y) + ((unsigned)row * pitch + 4u * (unsigned)c)) = part_at(acc);
}

}  // namespace convspmv
