// The second launch of the product from the column-compressed arrays (csc_gather_kernel.h): arrays that hold something
// other than conv_csc_build wrote.
#pragma once
#include "csc_gather_kernel.h"

namespace convspmv {

// The outputs that the gathering kernel marked, one workgroup per workgroup of it, from whatever the arrays hold.  An
// output that still holds the mark takes the first sum that arrives in place of it, every later one is added, so
// the workgroups need no order among themselves.  An entry whose row is the one its place asks for belongs to that
// output; an entry that names another row is added there by the workgroup that has its place, and the entries of a column
// whose pointers are not those of the closed form by the workgroup that has the column's first window.
// A workgroup of the gathering kernel was `odd` where its first output holds the mark, so whoever is the first to replace the
// mark there takes that workgroup's outputs over: the workgroup itself as it starts, or another one that
// has a sum for that output earlier.  Nothing to do where no mark is.
static __global__ __launch_bounds__(kCscGatherThreads) void csc_gather_mend_kernel(const int *__restrict__ col_ptr,
                                                                                   const int *__restrict__ row_idx,
                                                                                   const float *__restrict__ vals,
                                                                                   const float *__restrict__ x, float *y,
                                                                                   const CscGatherGeom g, int columns) {
    const ConvShape &sh = g.sh;
    const CscGatherJob mine = csc_gather_job(g, (int)blockIdx.x, columns);
    if (!mine.any) return;
    extern __shared__ unsigned taken[];                      // a bit for every workgroup of the gathering kernel
    __shared__ int next;
    unsigned *const out = reinterpret_cast<unsigned *>(y);
    auto first_output = [&](const CscGatherJob &b) { return ((long long)b.xa * sh.n_out + b.own) * g.batch + b.c0; };
    auto swap = [&](long long at, unsigned &old, unsigned now) {
        return __hip_atomic_compare_exchange_strong(out + at, &old, now, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (threadIdx.x == 0) {
        unsigned old = kCscGatherMark;
        next = swap(first_output(mine), old, kCscGatherTaken) ? (int)blockIdx.x : -1;
    }
    __syncthreads();
    if (next < 0) return;
    const int blocks = g.blocks_per_xcd * kXcds;
    for (int t = threadIdx.x; t < (blocks + 31) / 32; t += kCscGatherThreads) taken[t] = 0;
    __syncthreads();
    auto add = [&](long long row, int c, float value) {
        const long long at = row * g.batch + c;
        unsigned old = __hip_atomic_load(out + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (;;) {
            const int xo = (int)(row / sh.n_out), yo = (int)(row - (long long)xo * sh.n_out);
            const int sg = xo / g.seg, strip = yo / g.tw, cb = c / columns;
            unsigned now = __float_as_uint(__uint_as_float(old) + value);
            bool take = false;
            if (old == (unsigned)kCscGatherMark || old == (unsigned)kCscGatherTaken) {
                take = old == (unsigned)kCscGatherMark && xo == sg * g.seg && yo == strip * g.tw && c == cb * columns;
                now = __float_as_uint(value);
            }
            if (!swap(at, old, now)) continue;
            if (take) {
                const int job = (sg * g.strips + strip) * g.col_blocks + cb;
                const int block = job / g.blocks_per_xcd + job % g.blocks_per_xcd * kXcds;
                atomicOr(taken + block / 32, 1u << block % 32);
            }
            return;
        }
    };
    const int s = sh.s, k = sh.k, p = sh.p;
    struct Column {
        long long beg;
        int x_lo, y_lo, q2;
        bool as_built;
    };
    auto column_of = [&](int i, int j) {
        Column c;
        c.x_lo = axis_first_window(i, k, s, p);
        c.y_lo = axis_first_window(j, k, s, p);
        const long long q1 = axis_cover(i, sh.m_out, k, s, p);
        c.q2 = axis_cover(j, sh.n_out, k, s, p);
        c.beg = csc_gather_prefix(g.zero1, i, sh.m_out, sh) * g.row_entries +
                q1 * csc_gather_prefix(g.zero2, j, sh.n_out, sh);
        const long long at = (long long)i * sh.n + j;
        c.as_built = col_ptr[at] == (int)c.beg && col_ptr[at + 1] == (int)(c.beg + q1 * c.q2);
        return c;
    };
    auto mend = [&](const CscGatherJob &b) {
        const int y0 = b.own, y1 = min(y0 + g.tw, sh.n_out), width = min(columns, g.batch - b.c0);
        // every output: the entries that are its own, and those in their places that name another row
        const long long outputs = (long long)(b.xb - b.xa) * (y1 - y0) * width;
        for (long long t = threadIdx.x; t < outputs; t += kCscGatherThreads) {
            const long long cell = t / width;
            const int c = b.c0 + (int)(t - cell * width);
            const int xo = b.xa + (int)(cell / (y1 - y0)), yo = y0 + (int)(cell % (y1 - y0));
            const long long row = (long long)xo * sh.n_out + yo;
            float sum = 0.0f;
            for (int a = 0; a < k; ++a) {
                const int i = s * xo + a - p;
                if (i < 0 || i >= sh.m) continue;
                float part = 0.0f;
                for (int d = 0; d < k; ++d) {
                    const int j = s * yo + d - p;
                    if (j < 0 || j >= sh.n) continue;
                    const Column q = column_of(i, j);
                    if (!q.as_built) continue;
                    const long long e = q.beg + (long long)(xo - q.x_lo) * q.q2 + yo - q.y_lo;
                    const float pixel = x[((long long)i * sh.n + j) * g.batch + c];
                    if (row_idx[e] == (int)row) part = fmaf(vals[e], pixel, part);
                    else add(row_idx[e], c, vals[e] * pixel);
                }
                sum += part;
            }
            add(row, c, sum);
        }
        // columns that lie elsewhere than they were built
        const long long pixels = (long long)(b.i_b - b.i_a) * b.npix;
        for (long long t = threadIdx.x; t < pixels; t += kCscGatherThreads) {
            const int i = b.i_a + (int)(t / b.npix), j = b.j0 + (int)(t % b.npix);
            const Column q = column_of(i, j);
            const int xo = min(q.x_lo, sh.m_out - 1), yo = min(q.y_lo, sh.n_out - 1);
            if (q.as_built || xo < b.xa || xo >= b.xb || yo < y0 || yo >= y1) continue;
            const long long at = (long long)i * sh.n + j;
            for (unsigned e = col_ptr[at]; e < (unsigned)col_ptr[at + 1]; ++e)
                for (int c = b.c0; c < b.c0 + width; ++c) add(row_idx[e], c, vals[e] * x[at * g.batch + c]);
        }
    };
    mend(mine);
    for (;;) {                                               // workgroups taken over on the way: each once
        __syncthreads();
        if (threadIdx.x == 0) {
            next = -1;
            for (int t = 0; t < (blocks + 31) / 32 && next < 0; ++t)
                if (taken[t]) {
                    const int bit = __ffs((int)taken[t]) - 1;
                    next = t * 32 + bit;
                    taken[t] &= ~(1u << bit);
                }
        }
        __syncthreads();
        if (next < 0) return;
        mend(csc_gather_job(g, next, columns));
    }
}

}  // namespace convspmv
