// y = T x from the column-compressed arrays of T, every output summed where it stays (gfx950).
//
// By columns the product is a scatter, and a scatter pays per entry: a read, an add and a write of a sum in LDS
// (spmm_csc_tile_kernel, apply_kernels.h).  But an entry's place in the column-compressed arrays is as regular as in
// the rows: column (i, j), the input pixel, holds the windows (x, y) that cover it, x ascending, then y (Section 2),
// q1(i) x q2(j) of them, so the entry of window (x, y) is number (x - x_lo(i)) q2(j) + y - y_lo(j) of its column.
// Here a workgroup owns a strip of output columns and walks down the input lines of a segment of output lines; a lane
// keeps the sums of the KL = ceil(k/s) output lines that one input line reaches in registers, for one output column
// and one batch column or four.
//   - The entries of an input line over the strip are one contiguous span of both arrays.  It travels from memory to
//     registers DEPTH lines ahead of its use, 16 bytes per lane and access, and from there to LDS entry by entry,
//     each to the slot (tap column b, output column, l) of the output line xtop - l it belongs to.  Where entry e of
//     the span goes does not change from line to line as long as the line is covered by the same windows, so these
//     places are found once (by `place_entries`) and kept.  Slots of taps that fall outside the image are never
//     written and stay zero, as do the pixels around the image.
//   - The row index an entry must have is kept beside its place and compared with the stored one when the entry
//     lands, so the indices need no room in LDS, and an entry is compared once, not once per batch column.
//   - The taps of an input line are summed before the lines are, so that a sum rounds about 2 k times and not k * k
//     times (1024^2, k 7, batch 16: 7.5e-8 from 64 bits, the scatter 1.0e-7).
// y is written once, in a fixed order of sums, and never read.
//
// Measured with the two launches behind it (below), 1024^2, k 7, batch 16: 113 us where every call brings another matrix (4.9 TB/s of the
// bytes it cannot do without), the scatter 359; one matrix, other operands on every call: 102, the scatter 358; batch 1: 80 and
// 157.  What bounds it: memory where the kernel is large, the time
// of a line (about 0.7 us, LDS round trips, one barrier) where it is small (1000 x 900, k 3, batch 16: 39 us;
// the scatter 217).  Hence the strips of 64 columns, the walk without branches at stride 1 (51 -> 36 us at k 3) and two
// lines in flight only where they cost few registers (k 11, batch 16: 106 us with two, 72 with one).
//
// The arrays decide, not the geometry: a workgroup that meets a row index which is not the one its place asks for, or a
// column pointer which is not the one of the closed form (edited arrays), notes it in the plan's EditedWord, and the two
// launches behind this one, which otherwise return at once, zero y and scatter.  The note stays: later products of the
// plan leave this kernel as they enter it, and cost what the scatter costs, whatever the arrays hold.  Nothing is
// remembered in the other direction: arrays not noted are checked whole by every product, so products that run side by
// side on a plan come to one answer.  One row index edited or all of them, 1024^2, k 7, batch 16: 540 and 690 us the first
// time, 410 then, the scatter by itself 358 (the outputs concerned summed again, one workgroup for each of the
// gather's: 7300 and 15600).  What the two launches cost where nothing is edited: 3 us (one: 1.5).
#pragma once
#include <type_traits>

#include "build_kernels.h"
#include "apply_march_kernel.h"
#include "edited_word.h"

namespace convspmv {

constexpr int kCscGatherThreads = 256, kCscGatherWaves = kCscGatherThreads / kWave;
constexpr int kCscGatherBlocks = 1 << 18;                   // workgroups at most (a launch has fewer than 2^32 threads)

// words between the slots of two output columns: odd, so that the lanes of a tap meet in no bank
__host__ __device__ constexpr int csc_gather_pitch(int kl) { return kl | 1; }

struct CscGatherGeom {
    ConvShape sh;
    long long zero1, zero2;   // where the entries of a column lie (see AxisScan): the sums at line 0 and at pixel 0,
    long long row_entries;    // entries of a fully covered line, all its pixels together
    unsigned nnz;
    int batch;
    int lpr_log2;             // log2 of the lanes per output column, four batch columns each (scalar: 0, one column)
    int opw_log2;             // log2 of the output columns per wave; the lanes beyond deal out the tap columns
    int tw;                   // output columns per strip
    int groups, ways;         // waves side by side over the strip; shares a tap sum is dealt out in
    int strips, segs, seg;    // segments of seg output lines
    int blocks, blocks_per_xcd, col_blocks;
    int iw, pw;               // input pixels of a full strip, (tw - 1) s + k; places per column phase
    int slots, line_elems;    // words of an image of slots; elements of an input line in LDS
    int quads;                // 16-byte accesses per array that a line's span takes, at most
    int sets;                 // sets of places kept: inner lines are covered alike (s divides k) or in two ways
};

// Output columns per wave and shares of a tap sum for strips of tw columns.
__host__ __device__ constexpr int csc_gather_opw_log2(int tw, int lpr_log2) {
    int o = 0;
    while ((2 << o) <= tw && o + 1 + lpr_log2 <= 6) ++o;
    return o;
}
__host__ __device__ constexpr int csc_gather_groups(int tw, int lpr_log2) { return tw >> csc_gather_opw_log2(tw, lpr_log2); }
__host__ __device__ constexpr int csc_gather_ways(int tw, int lpr_log2) {
    return kCscGatherWaves / csc_gather_groups(tw, lpr_log2) << (6 - lpr_log2 - csc_gather_opw_log2(tw, lpr_log2));
}
// Places per column phase (the last strip's pixels may reach s - 1 past its windows), elements of a line, words of an image
// of slots with a dump behind the slots, 16-byte accesses per array for a line's span.
__host__ __device__ constexpr int csc_gather_places(int tw, int k, int s) { return ((tw - 1) * s + k + 2 * (s - 1)) / s; }
__host__ __device__ constexpr int csc_gather_line(int tw, int k, int s, int lpr_log2) {
    return ((s * csc_gather_places(tw, k, s) << lpr_log2) + 3) & ~3;
}
__host__ __device__ constexpr int csc_gather_slots(int tw, int k, int s) {
    return (k * tw * csc_gather_pitch((k + s - 1) / s) + kWave + 3) & ~3;
}
__host__ __device__ constexpr int csc_gather_quads(int tw, int k, int s) {
    return ((((tw - 1) * s + k + s - 1) / s * k * ((k + s - 1) / s) + 3) / 4 + 1) & ~1;
}
__host__ __device__ constexpr int csc_gather_lds(int tw, int k, int s, int lpr_log2, bool scalar) {
    const int elem = scalar ? 4 : 16, pixels = (tw - 1) * s + k + s - 1;
    const int meet = csc_gather_ways(tw, lpr_log2) > 1 ? 2 * kCscGatherThreads : 0;
    return (2 * csc_gather_line(tw, k, s, lpr_log2) + meet) * elem + 2 * csc_gather_slots(tw, k, s) * 4 +
           (k % s == 0 ? 1 : 2) * csc_gather_quads(tw, k, s) * 24 + (pixels + 1 + 3) / 4 * 16;
}
// The widest strip whose lines take at most five accesses per thread, with at most 64 KiB (two workgroups per compute
// unit, and nothing to be allowed before a launch); 0: none.
constexpr int kCscGatherQuadsMax = 5 * kCscGatherThreads, kCscGatherLds = 64 * 1024;
__host__ __device__ constexpr int csc_gather_tw(int k, int s, int lpr_log2, bool scalar, int widest = 64) {
    for (int tw = widest; tw >= 16; tw /= 2) {
        const int pixels = (tw - 1) * s + k + s - 1;      // of a strip, at most: two column pointers and three elements per thread
        if (csc_gather_quads(tw, k, s) <= kCscGatherQuadsMax && csc_gather_lds(tw, k, s, lpr_log2, scalar) <= kCscGatherLds &&
            pixels < 2 * kCscGatherThreads && pixels << lpr_log2 <= 3 * kCscGatherThreads)
            return tw;
    }
    return 0;
}

// Do batches below 4 columns gather, somewhere?  (Columns of one entry, and of four at stride 1, are added to y directly.)
__host__ __device__ constexpr bool csc_gather_few(int kl, int s) { return kl > (s == 1 ? 2 : 1); }

// Entries along one axis before line (pixel) t, T^T.
__device__ __forceinline__ long long csc_gather_prefix(long long zero, int t, int count_out, const ConvShape &sh) {
    return started_sum((long long)t + sh.p, sh.s, count_out) - started_sum((long long)t + sh.p - sh.k, sh.s, count_out) - zero;
}

// The value is in its register from here on.
template <typename T>
__device__ __forceinline__ void arrived(T &v) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(v));
#endif
}

// Which part of the product a workgroup has.
struct CscGatherJob {
    int y0, own;              // first output column of the strip and first that is its own: the last strip is moved to
                              // the left to be full (no line of it has fewer than four entries)
    int xa, xb, c0;           // output lines [xa, xb), first batch column
    int j0, npix;             // pixels its columns touch (the last strip: to the end of the line)
    int i_a, i_b;             // input lines it reads (the last segment: to the end of the image)
    bool any;
};
__device__ __forceinline__ CscGatherJob csc_gather_job(const CscGatherGeom &g, int block, int columns) {
    CscGatherJob b{};
    const int at = block / kXcds;
    const int job = (block % kXcds) * g.blocks_per_xcd + at;
    if (at >= g.blocks_per_xcd || job >= g.blocks) return b;
    const int cell = job / g.col_blocks, sg = cell / g.strips, strip = cell - sg * g.strips;
    b.any = true;
    b.c0 = (job - cell * g.col_blocks) * columns;
    b.own = strip * g.tw;
    b.y0 = min(b.own, max(g.sh.n_out - g.tw, 0));
    b.xa = sg * g.seg;
    b.xb = min(b.xa + g.seg, g.sh.m_out);
    const int j_lo = g.sh.s * b.y0 - g.sh.p;
    b.j0 = max(j_lo, 0);
    b.npix = (strip + 1 == g.strips ? g.sh.n : min(j_lo + g.iw, g.sh.n)) - b.j0;
    b.i_a = max(g.sh.s * b.xa - g.sh.p, 0);
    b.i_b = sg + 1 == g.segs ? g.sh.m : min(g.sh.s * (b.xb - 1) - g.sh.p + g.sh.k, g.sh.m);
    return b;
}

// NLD: 16-byte accesses per thread and array for a line's span; NX: elements of the line per thread.  Every line takes the
// same accesses, at clamped places, so that a wait for one line leaves the next one's in flight.
// STRIDE 1: strips of TW columns, 1 << LPR_LOG2 lanes per output column, k = KL, all known to the compiler, which takes
// the branches and the arithmetic of addresses out of the walk; STRIDE 0: any stride, everything from the geometry.
template <int KL, int STRIDE, int TW, int LPR_LOG2, bool SCALAR, int NLD, int NX, int DEPTH>
__global__ __launch_bounds__(kCscGatherThreads, 2) void spmm_csc_gather_kernel(const int *__restrict__ col_ptr,
                                                                              const int *__restrict__ row_idx,
                                                                              const float *__restrict__ vals,
                                                                              const float *__restrict__ x,
                                                                              float *__restrict__ y, const CscGatherGeom g,
                                                                              const EditedWord edited) {
    using elem_t = typename std::conditional<SCALAR, float, vec4>::type;
    typedef int vec4i __attribute__((ext_vector_type(4)));
    typedef int vec4iu __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int NT = kCscGatherThreads, EB = SCALAR ? 1 : 4, PITCH = csc_gather_pitch(KL), NP = NX > 1 ? 2 : 1;
    // Row indices past the caches, values through them: this memory system moves more when a stream is split between the
    // two (k 7, batch 16: 123 us all through, 111 all past, 103 like this; batch 1: 90, 91, 78).  Short lines and narrow strips,
    // whose spans overlap more, lose with it (k 3: 36 -> 38, k 11: 72 -> 74).
    constexpr bool ROWS_ONCE = STRIDE != 0 && KL >= 5 && KL <= 8;
    extern __shared__ __align__(16) float csc_lds[];
    const ConvShape &sh = g.sh;
    const int s = STRIDE ? STRIDE : sh.s, k = STRIDE ? KL : sh.k, p = sh.p, n = sh.n;
    const int lpr_log2 = SCALAR ? 0 : (STRIDE ? LPR_LOG2 : g.lpr_log2), lpr = 1 << lpr_log2;
    const int tw = STRIDE ? TW : g.tw, opw_log2 = STRIDE ? csc_gather_opw_log2(TW, LPR_LOG2) : g.opw_log2;
    const int groups = STRIDE ? csc_gather_groups(TW, LPR_LOG2) : g.groups, ways = STRIDE ? csc_gather_ways(TW, LPR_LOG2) : g.ways;
    const int pw = STRIDE ? csc_gather_places(TW, KL, 1) : g.pw, line_elems = STRIDE ? csc_gather_line(TW, KL, 1, LPR_LOG2) : g.line_elems;
    const int image_words = STRIDE ? csc_gather_slots(TW, KL, 1) : g.slots, quads = STRIDE ? csc_gather_quads(TW, KL, 1) : g.quads;
    const int sets = STRIDE ? 1 : g.sets;
    const CscGatherJob job = csc_gather_job(g, (int)blockIdx.x, EB << lpr_log2);
    if (!job.any) return;
    unsigned noted = *const_cast<const volatile unsigned *>(edited.word);       // (on its way while the rest is prepared)
    const int tid = (int)threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);

    // LDS: two input lines, sums that meet, where entries go, two images of slots, column ends
    elem_t *const lines = reinterpret_cast<elem_t *>(csc_lds);
    elem_t *const meet = lines + 2 * line_elems;                                      // [2][NT]
    vec4i *const want_row = reinterpret_cast<vec4i *>(meet + (ways > 1 ? 2 * NT : 0));  // [sets][quads]
    int2 *const want_slot = reinterpret_cast<int2 *>(want_row + sets * quads);      // [sets][quads], four of 16 bits
    float *const images = reinterpret_cast<float *>(want_slot + sets * quads);      // [2][slots], a dump behind the slots
    int *const p2 = reinterpret_cast<int *>(images + 2 * image_words);                  // [npix + 1] entries before a pixel, per covering line

    for (int t = tid; t < 2 * line_elems; t += NT) lines[t] = elem_t(0.0f);
    for (int t = tid; t < 2 * image_words; t += NT) images[t] = 0.0f;
    // One thread's reading for the whole workgroup (others may note the plan meanwhile, and places that waves deal out
    // among them have to be found by all): in the last word of the second image's dump, which is not written before the barrier of
    // the first line, by the thread that has cleared it.
    unsigned *const told = reinterpret_cast<unsigned *>(images + 2 * image_words - 1);
    if (tid == (2 * image_words - 1) % NT) {
        arrived(noted);
        *told = noted;
    }
    const long long p2a = csc_gather_prefix(g.zero2, job.j0, sh.n_out, sh);
    for (int t = tid; t <= job.npix; t += NT) p2[t] = (int)(csc_gather_prefix(g.zero2, job.j0 + t, sh.n_out, sh) - p2a);
    __syncthreads();
    if ((unsigned)__builtin_amdgcn_readfirstlane((int)*told) == edited.stamp) return;                       // (y is written by the launches behind this one)
    const int taps = __builtin_amdgcn_readfirstlane(p2[job.npix]);

    // this lane: batch columns, output column, share of the tap columns
    const int v = lane & (lpr - 1), way_lanes = kWave >> (lpr_log2 + opw_log2);
    const int yl = ((wave % groups) << opw_log2) + ((lane >> lpr_log2) & ((1 << opw_log2) - 1));
    const int way_first = wave / groups * way_lanes, way = way_first + (lane >> (lpr_log2 + opw_log2));
    // tap columns of every lane of this wave, and whether this lane has one more
    const int nb = STRIDE ? KL / csc_gather_ways(TW, LPR_LOG2) : max((k - (way_first + way_lanes - 1) + ways - 1) / ways, 0);
    const bool one_more = way + nb * ways < k;
    const bool live = job.y0 + yl >= job.own && job.y0 + yl < sh.n_out && (SCALAR || job.c0 + 4 * v < g.batch);
    auto column = [&](int v_) { return SCALAR ? job.c0 : chunk_col(job.c0 + 4 * v_, g.batch); };
    const int out_off = yl * g.batch + column(v);
    float *const y_strip = y + (long long)job.y0 * g.batch;

    // this thread: its elements of an input line and its column pointers
    int x_off[NX], x_dst[NX], ptr_at[NP], ptr_p2[NP];
#pragma unroll
    for (int r = 0; r < NX; ++r) {
        const int item = min(tid + r * NT, (job.npix << lpr_log2) - 1), q = item >> lpr_log2, vv = item & (lpr - 1);
        x_off[r] = q * g.batch + column(vv);
        const int at = q + job.j0 - (s * job.y0 - p);
        x_dst[r] = (((at % s) * pw + at / s) << lpr_log2) + vv;
    }
#pragma unroll
    for (int r = 0; r < NP; ++r) {
        ptr_at[r] = min(tid + r * NT, job.npix);
        ptr_p2[r] = p2[ptr_at[r]];
    }

    struct Line {                 // a line on its way
        vec4i rows[NLD];
        vec4 vals[NLD];
        elem_t px[NX];
        int ptr[NP];
        unsigned beg;             // (uniform from here) first entry of the span
        int count, q1, off, x_lo; // entries; windows over the line, x_lo ... ; place of x_lo (l = off)
    };
    // state of the line that is asked for next
    int f_i = job.i_a, f_top = (job.i_a + p) / s, f_r0 = (job.i_a + p) - f_top * s, f_lo = axis_first_window(job.i_a, k, s, p);
    long long f_p1 = csc_gather_prefix(g.zero1, job.i_a, sh.m_out, sh);
    int f_left = job.i_b - job.i_a;
    auto fetch = [&](Line &f) {
        f.q1 = max(min(f_top, sh.m_out - 1) - f_lo + 1, 0);
        f.off = f_top - f_lo;
        f.x_lo = f_lo;
        f.beg = (unsigned)(f_p1 * g.row_entries + f.q1 * p2a);
        f.count = f_left > 0 ? f.q1 * taps : 0;              // (past the last line: that line once more, for nobody)
        const long long first = (long long)f_i * n + job.j0;
        const float *const xp = x + first * g.batch;
        const int *const cp = col_ptr + first;
#pragma unroll
        for (int r = 0; r < NX; ++r) {
            if constexpr (SCALAR) f.px[r] = xp[x_off[r]];
            else f.px[r] = *reinterpret_cast<const vec4u *>(xp + x_off[r]);
        }
#pragma unroll
        for (int r = 0; r < NP; ++r) f.ptr[r] = cp[ptr_at[r]];
        const unsigned base = min(f.beg, g.nnz - 4);         // (a line without entries may begin behind the last)
        const int last = max(f.count - 4, 0);
        const int *const rp = row_idx + base;
        const float *const vp = vals + base;
#pragma unroll
        for (int r = 0; r < NLD; ++r) {
            const int e = min((r * NT + tid) * 4, last);
            if constexpr (ROWS_ONCE) f.rows[r] = __builtin_nontemporal_load(reinterpret_cast<const vec4iu *>(rp + e));
            else f.rows[r] = *reinterpret_cast<const vec4iu *>(rp + e);
            f.vals[r] = *reinterpret_cast<const vec4u *>(vp + e);
        }
        // the next line (numbers chosen, not branched around: every line's accesses have to stay the same for the waits to count)
        const int more = --f_left > 0 ? 1 : 0;
        f_p1 += more ? f.q1 : 0;
        f_i += more;
        f_r0 += more;
        const int wrap = f_r0 == s ? 1 : 0;
        f_r0 = wrap ? 0 : f_r0;
        f_top += wrap;
        f_lo += f_i + p - k + 1 > s * f_lo ? 1 : 0;
    };

    // Rows (of line x_lo = 0) and slots of the entries of a line with q1 windows, the first at place `off`.  The entries
    // that close the span are the last four once more, wherever they lie.
    int key0 = -1, key1 = -1;                                // what the two sets hold
    auto place_entries = [&](int set, int q1, int off, int count) {
        int *const rows = reinterpret_cast<int *>(want_row + set * quads);
        unsigned short *const slots = reinterpret_cast<unsigned short *>(want_slot + set * quads);
        const int whole = count & ~3, tail = (count - 1) & ~3;
        for (int t = tid; t < job.npix * q1; t += NT) {
            const int c = div_small(t, 1.0f / (float)q1), dx = t - c * q1;
            const int before = p2[c], q2 = p2[c + 1] - before, j = job.j0 + c;
            int e = q1 * before + dx * q2, yy = axis_first_window(j, k, s, p), b = j + p - s * yy;
            for (const int end = e + q2; e < end; ++e, ++yy, b -= s) {
                const int row = dx * sh.n_out + yy, at = yy - job.y0;
                const int slot = (unsigned)at < (unsigned)tw ? (b * tw + at) * PITCH + off - dx : image_words - kWave + lane;
                if (e < whole) {
                    rows[e] = row;
                    slots[e] = (unsigned short)slot;
                }
                if (e >= count - 4) {
                    rows[tail + e - (count - 4)] = row;
                    slots[tail + e - (count - 4)] = (unsigned short)slot;
                }
            }
        }
    };
    int differs = 0;
    auto land = [&](const Line &f, int buf) {
        float *const image = images + buf * image_words;
        elem_t *const line = lines + buf * line_elems;
        // this line is here, the lines asked for after it need not be (a store lies before their loads)
        constexpr int kLater = (DEPTH - 1) * (2 * NLD + NX + NP);
        __builtin_amdgcn_s_waitcnt((kLater & 15) | kLater >> 4 << 14 | 0x0f70);
#pragma unroll
        for (int r = 0; r < NX; ++r) line[x_dst[r]] = f.px[r];
#pragma unroll
        for (int r = 0; r < NP; ++r) differs |= f.ptr[r] ^ (int)(f.beg + (unsigned)(f.q1 * ptr_p2[r]));
        const int set = f.q1 == KL ? 0 : sets - 1;
        const int key = f.q1 << 8 | f.off;
        if (f.count > 0 && __builtin_expect((set ? key1 : key0) != key, 0)) {       // (uniform)
            place_entries(set, f.q1, f.off, f.count);
            (set ? key1 : key0) = key;
            __syncthreads();
        }
        const int first_row = f.x_lo * sh.n_out;
        if (f.count > 0) {
            const int tail = (f.count - 1) >> 2;
#pragma unroll
            for (int r = 0; r < NLD; ++r) {
                const int q = set * quads + min(r * NT + tid, tail);
                const vec4i rows = want_row[q];
                const int2 slot = want_slot[q];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    differs |= (f.rows[r][u] - rows[u]) ^ first_row;
                    const unsigned w = u < 2 ? slot.x : slot.y;
                    image[u % 2 ? w >> 16 : w & 0xffff] = f.vals[r][u];
                }
            }
        }
    };

    auto fma_elem = [](elem_t &a, float wt, const elem_t &e) {
        if constexpr (SCALAR) {
            a = fmaf(wt, e, a);
        } else {
            a.x = fmaf(wt, e.x, a.x);
            a.y = fmaf(wt, e.y, a.y);
            a.z = fmaf(wt, e.z, a.z);
            a.w = fmaf(wt, e.w, a.w);
        }
    };
    // The sums of this line's taps: part[l] for output line xtop - l, l < KN
    const int step_ph = ways % s, step_at = (step_ph * pw + ways / s) << lpr_log2, wrap_at = (1 - s * pw) * (1 << lpr_log2);
    const int way_ph = way % s, way_at = ((way_ph * pw + way / s + yl) << lpr_log2) + v;
    const int way_slot = (way * tw + yl) * PITCH, step_slot = ways * tw * PITCH;
    auto push = [&](auto kn_tag, int buf, elem_t (&part)[KL]) {
        constexpr int KN = decltype(kn_tag)::value;
        if constexpr (KN > 0) {
            const float *wb = images + buf * image_words + way_slot;
            const elem_t *const line = lines + buf * line_elems;
            int ph = way_ph, at = way_at;                     // tap column b: phase b mod s, place yl + b / s
            struct Tap {
                elem_t e;
                float w[KN];
            };
            auto read = [&](Tap &t) {
                t.e = line[at];
#pragma unroll
                for (int l = 0; l < KN; ++l) t.w[l] = wb[l];
                wb += step_slot;
                ph += step_ph;
                at += step_at;
                if (ph >= s) {
                    ph -= s;
                    at += wrap_at;
                }
            };
            auto sum = [&](const Tap &t) {
#pragma unroll
                for (int l = 0; l < KN; ++l) fma_elem(part[l], t.w[l], t.e);
            };
            // two tap columns at a time: their pixels and entries first, then the sums
            auto two = [&](auto first_tag) {
                Tap t0, t1;
                read(t0);
                read(t1);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (decltype(first_tag)::value) {
#pragma unroll
                    for (int l = 0; l < KN; ++l) part[l] = t0.w[l] * t0.e;
                } else {
                    sum(t0);
                }
                sum(t1);
            };
            auto one = [&] {
                Tap t0;
                read(t0);
                __builtin_amdgcn_sched_barrier(0);
                sum(t0);
            };
            if constexpr (STRIDE != 0) {
                constexpr int NB = KL / csc_gather_ways(TW, LPR_LOG2);
                if constexpr (NB >= 2) two(std::true_type{});
#pragma unroll
                for (int b = 2; b + 2 <= NB; b += 2) two(std::false_type{});
                if constexpr (NB % 2 != 0) one();
                if constexpr (KL % csc_gather_ways(TW, LPR_LOG2) != 0)
                    if (one_more) one();
            } else {
                int b = 0;
                if (nb >= 2) {
                    two(std::true_type{});
                    b = 2;
                }
                for (; b + 2 <= nb; b += 2) two(std::false_type{});
                if (b < nb) one();
                if (one_more) one();
            }
        }
    };

    // A finished output line waits for the next barrier: the shares of its ways meet in LDS, one way stays in its register.
    const int meet_at = (yl << lpr_log2) + v, meet_way = tw << lpr_log2;
    int waits = -1, parity = 0;
    elem_t finished = elem_t(0.0f);
    auto store = [&] {
        if (waits < 0) return;
        if (live && way == 0) {
            elem_t sum = finished;
            const elem_t *const sums = meet + (parity ^ 1) * NT + meet_at;
            for (int w = 1; w < ways; ++w) sum += sums[w * meet_way];
            float *const out = y_strip + (long long)waits * sh.n_out * g.batch + out_off;
            if constexpr (SCALAR) __builtin_nontemporal_store(sum, out);
            else __builtin_nontemporal_store((vec4u)sum, reinterpret_cast<vec4u *>(out));
        }
        waits = -1;
    };

    elem_t acc[KL];                                          // acc[l]: output line xtop - l
#pragma unroll
    for (int l = 0; l < KL; ++l) acc[l] = elem_t(0.0f);
    int r0 = (job.i_a + p) % s, x_next = job.xa;
    auto one_line = [&](int i, Line &f) {
        const int buf = (i - job.i_a) & 1;
        const bool has = f.count > 0;
        land(f, buf);
        __syncthreads();                                     // line i has landed, and line i - 1 is done with
        store();
        fetch(f);
        elem_t part[KL];
#pragma unroll
        for (int l = 0; l < KL; ++l) part[l] = elem_t(0.0f);
        if (has) {
            if (s == 1 || r0 + s * (KL - 1) < k) push(std::integral_constant<int, KL>{}, buf, part);
            else push(std::integral_constant<int, KL - 1>{}, buf, part);
        }
        finished = acc[KL - 1] + part[KL - 1];
        if (i == s * x_next - p + k - 1 && x_next < job.xb) {           // the last tap line of x_next: place KL - 1 holds it
            if (ways > 1) {
                meet[parity * NT + way * meet_way + meet_at] = finished;
                parity ^= 1;
            }
            waits = x_next++;
        }
        if (++r0 == s) {
            r0 = 0;
#pragma unroll
            for (int l = KL - 1; l > 0; --l) acc[l] = acc[l - 1] + part[l - 1];
            acc[0] = elem_t(0.0f);
        } else {
#pragma unroll
            for (int l = 0; l < KL; ++l) acc[l] += part[l];
        }
    };
    // to the last output line's last tap line, which may lie below the image (nothing lands there)
    const int i_end = max(s * (job.xb - 1) - p + k, job.i_b);
    Line f[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) fetch(f[d]);
    // The first lines are waited for here: they are not asked for in the order that the waits inside the loop count on.
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
#pragma unroll
        for (int r = 0; r < NLD; ++r) {
            arrived(f[d].rows[r]);
            arrived(f[d].vals[r]);
        }
#pragma unroll
        for (int r = 0; r < NX; ++r) arrived(f[d].px[r]);
#pragma unroll
        for (int r = 0; r < NP; ++r) arrived(f[d].ptr[r]);
    }
    // (always DEPTH of them: a line more than there is finds nothing to do)
    for (int i = job.i_a; i < i_end; i += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) one_line(i + d, f[d]);
    }
    if (__any(differs) && lane == 0) *const_cast<volatile unsigned *>(edited.word) = edited.stamp;
    __syncthreads();
    store();
}

}  // namespace convspmv
