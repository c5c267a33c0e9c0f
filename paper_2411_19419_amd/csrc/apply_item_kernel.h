// Product over the stored CSR arrays, a thread or a few per item: a row and a chunk of its batch columns (gfx950).
//
// The row groups of apply_kernels.h give a lane up to 16 batch columns, and a wave as many rows: its accesses are pieces of 16
// bytes at as many places as it has rows, and a batch that does not fill the blocks of 16 columns leaves lanes idle (so do tiles
// and marches).  Here the chunks of four columns of a row lie side by side on the lanes (one column each below a batch of 4), then
// those of the next row: x and y move in whole memory lines whatever the batch, the lanes of a row ask for the same entries with
// one access, and no lane is idle but the launch's last.  No staging and no barrier: neighbouring rows share their pixels through
// the L1 and the L2 (workgroups of neighbouring rows run on one XCD).
//
// G lanes share an item where the launch has few waves; lane l takes U consecutive entries at a time, U l, U l + U G, ...,
// NB such accesses are asked for together with their pixels after them.  U fits the rows: 25 entries in fives, others in fours;
// rows of 1, 4 and 9 at once (a tail of one entry would cost four pixels).
// Sums: each access is a chain of its own; the accesses of a row, its lanes and its channels are added in 64 bits, which this
// chip adds as fast as 32 (1384 products: 0.99 of the time of sums in 32 bits).  Rows at once are one chain, of 9 entries two
// of every other entry, the order of the tile kernel.  Error against 64 bits over that of the kernels it takes products
// from, in the geometric mean: rows of 1, 4 and 9 entries 1.00, 0.99 and 1.00; 16: 0.85; 25: 0.84; 36: 0.72; 49 and 64: 0.69;
// 81: 0.68; 100: 0.65; 121 and 144: 0.62; 169: 0.59; channels 0.31 of the row groups', 0.51 of the others'.  (In 32 bits, two sums in
// turn and the tail of a row on top of one of them: 25 entries 1.07, up to 1.24; 36: 1.05; 64: 1.07; three channels of 25 up to 1.18.)
//
// MANY: several channels that share the indices.  The waves of a workgroup hold the same items and deal the channels out; a lane
// keeps its entries' columns while NB of its channels pass, and the partial sums meet in LDS.
//
// Measured, two sets of operands in turn, before -> after: 1362 x 1644, k 1, s 2, batch 100: 654 -> 105 us (tiles); 909 x 1348, k 6, s 3,
// batch 132: 1148 -> 229 (march); 70 x 91, k 6, T^T, batch 85: 32 -> 7.2 (staged march); 755 x 1134, k 7, s 4, batch 116: 438 -> 125
// (row groups); 2388 x 1551, k 3, s 3, T^T, batch 64: 684 -> 379; 36 x 52, k 7, s 4, 206 channels, batch 8: 300 -> 26; 30 x 31, k 9, s 3,
// 136 channels, batch 2: 140 -> 23.  What bounds it: large products the L2, which delivers every pixel once per entry but for what
// the L1 catches (733 x 667, k 6, s 3, batch 204: 12.9 M requests of 128 bytes in 142 us, 11.6 TB/s, a quarter of the L1's accesses);
// small ones a round trip for the row's bounds and two for every NB U G entries.  Not kept: blocks of 4 to 32 chunks at a time
// instead of all of a row's (1.03 to 1.27 of the time); the next entries asked for ahead of the sums (0.97 of the time in small
// products, 1.06 in large ones, which lose waves to the registers); entries and values of channels by accesses of 16 bytes with
// a masked tail (1.08).
#pragma once
#include "apply_kernels.h"

namespace convspmv {

constexpr int kItemThreads = 256;
constexpr int kItemWaysMost = 16;

struct ItemGeom {
    int batch;
    int chunks;                        // chunks of columns per row
    float inv_chunks;
    unsigned items;                    // rows * chunks
    int cells, cells_per_xcd;          // workgroups
    int channels, ways;                // MANY: waves of a workgroup, which deal the channels out
    long long vals_stride, x_stride;   // from a channel's values and plane to the next one's
};

// C: columns of a chunk.  x and y are addressed by 32-bit byte offsets, columns are below 2^24 (item_geometry).
template <int G, int C, int U, int NB, bool MANY>
__global__ __launch_bounds__(MANY ? kItemWaysMost * kWave : kItemThreads) void spmm_item_kernel(
    const int *__restrict__ row_ptr, const int *__restrict__ col_idx, const float *__restrict__ vals,
    const float *__restrict__ x, float *__restrict__ y, const ItemGeom g) {
    typedef float part __attribute__((ext_vector_type(C)));
    typedef float part_at __attribute__((ext_vector_type(C), aligned(4)));
    typedef double sum_t __attribute__((ext_vector_type(C)));
    constexpr int ITEMS = kWave / G;                 // of a wave
    const int at = (int)blockIdx.x / kXcds, cell = ((int)blockIdx.x % kXcds) * g.cells_per_xcd + at;
    if (at >= g.cells_per_xcd || cell >= g.cells) return;
    const int lane = (int)threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const unsigned first = MANY ? (unsigned)cell * ITEMS : ((unsigned)cell * (kItemThreads / kWave) + wave) * ITEMS;
    const unsigned row0 = first / (unsigned)g.chunks;
    const int t = (int)(first - row0 * (unsigned)g.chunks) + lane / G, sub = lane % G;
    const int q = div_small(t, g.inv_chunks);
    const int row = (int)row0 + q, chunk = t - q * g.chunks;
    const int c = C == 4 ? chunk_col(4 * chunk, g.batch) : chunk;
    const bool live = first + (unsigned)(lane / G) < g.items;
    unsigned beg = 0, end = 0;
    if (live) {
        beg = row_ptr[row];
        end = row_ptr[row + 1];
    }
    auto pixel = [&](const float *xc, int col) -> part {
        return *reinterpret_cast<const part_at *>(reinterpret_cast<const char *>(xc) + (__umul24(col, 4 * g.batch) + 4u * (unsigned)c));
    };
    auto mul_part = [&](float w, part p) -> part {
        part r;
#pragma unroll
        for (int h = 0; h < C; ++h) r[h] = w * p[h];
        return r;
    };
    auto fma_part = [&](float w, part p, part s) -> part {
        part r;
#pragma unroll
        for (int h = 0; h < C; ++h) r[h] = fmaf(w, p[h], s[h]);
        return r;
    };
    sum_t sum = sum_t(0.0);
    if constexpr (!MANY && NB == 1) {
        // a row at once (the loop is for edited rows that are longer)
        static_assert(G <= 2, "the chains of two lanes per row");
        part acc = part(0.0f), odd = part(0.0f);
        for (unsigned e = beg + sub; e < end; e += U * G) {
            int col[U];
            float val[U];
            part px[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned i = min(e + u * G, end - 1);
                col[u] = col_idx[i];
                val[u] = vals[i];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u == 0 || e + u * G < end) px[u] = pixel(x, col[u]);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u == 0 || e + u * G < end) {
                    if (G == 1 && U > 4 && u % 2) odd = fma_part(val[u], px[u], odd);
                    else acc = fma_part(val[u], px[u], acc);
                }
        }
        sum = __builtin_convertvector(acc, sum_t) + __builtin_convertvector(odd, sum_t);
    } else if constexpr (!MANY) {
        unsigned e = beg + U * sub;
#pragma unroll 1
        for (; e + (NB - 1) * U * G + U <= end; e += NB * U * G) {
            int col[NB][U];
            float val[NB][U];
            part px[NB][U];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int *const cs = col_idx + (e + b * U * G);
                const float *const vs = vals + (e + b * U * G);
#pragma unroll
                for (int u = 0; u < U; ++u) { col[b][u] = cs[u]; val[b][u] = vs[u]; }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int u = 0; u < U; ++u) px[b][u] = pixel(x, col[b][u]);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                part s = mul_part(val[b][0], px[b][0]);
#pragma unroll
                for (int u = 1; u < U; ++u) s = fma_part(val[b][u], px[b][u], s);
                sum += __builtin_convertvector(s, sum_t);
            }
        }
        for (; e < end; e += U * G) {
            int col[U];
            float val[U];
            part px[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned i = min(e + u, end - 1);
                col[u] = col_idx[i];
                val[u] = vals[i];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u == 0 || e + u < end) px[u] = pixel(x, col[u]);
            part s = mul_part(val[0], px[0]);
#pragma unroll
            for (int u = 1; u < U; ++u)
                if (e + u < end) s = fma_part(val[u], px[u], s);
            sum += __builtin_convertvector(s, sum_t);
        }
    } else {
        for (unsigned e = beg + U * sub; e < end; e += U * G) {
            int col[U];
            unsigned i[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                i[u] = min(e + u, end - 1);
                col[u] = col_idx[i[u]];
            }
            for (int ch = wave; ch < g.channels; ch += NB * g.ways) {
                float val[NB][U];
                part px[NB][U];
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (b == 0 || ch + b * g.ways < g.channels) {
                        const int cb = ch + b * g.ways;
                        const float *const vc = vals + cb * g.vals_stride, *const xc = x + cb * g.x_stride;
#pragma unroll
                        for (int u = 0; u < U; ++u) val[b][u] = vc[i[u]];
#pragma unroll
                        for (int u = 0; u < U; ++u) px[b][u] = pixel(xc, col[u]);
                    }
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (b == 0 || ch + b * g.ways < g.channels) {
                        if constexpr (U == 1) {
#pragma unroll
                            for (int h = 0; h < C; ++h) sum[h] = fma((double)val[b][0], (double)px[b][0][h], sum[h]);
                        } else {
                            part s = mul_part(val[b][0], px[b][0]);
#pragma unroll
                            for (int u = 1; u < U; ++u) s = e + u < end ? fma_part(val[b][u], px[b][u], s) : s;
                            sum += __builtin_convertvector(s, sum_t);
                        }
                    }
            }
        }
    }
#pragma unroll
    for (int h = 0; h < C; ++h) sum[h] = group_sum<G>(sum[h]);
    if constexpr (MANY) {
        extern __shared__ double item_lds[];      // [ways][ITEMS][C]
        if (g.ways > 1) {
            if (sub == 0) {
#pragma unroll
                for (int h = 0; h < C; ++h) item_lds[(wave * ITEMS + lane / G) * C + h] = sum[h];
            }
            __syncthreads();
            if (wave > 0) return;
            for (int i = 1; i < g.ways; ++i) {
#pragma unroll
                for (int h = 0; h < C; ++h) sum[h] += item_lds[(i * ITEMS + lane / G) * C + h];
            }
        }
    }
    if (live && sub == 0)
        *reinterpret_cast<part_at *>(reinterpret_cast<char *>(y) + 4u * ((unsigned)row * (unsigned)g.batch + (unsigned)c)) =
            part_at(__builtin_convertvector(sum, part));
}

}  // namespace convspmv
