// Structure-aware product for any (k, s): input lines pushed into the output lines they reach.
//
// The marching kernel (compact_kernels.h) keeps every input line that a step of output lines needs
// in LDS and lets each row pull its k x k pixels out of them.  At stride 4 neighbouring lanes then
// read 64 bytes apart, four lanes to a bank, the ring of 15 lines leaves room for one workgroup
// per CU, and every pixel is read k/s times: 4096^2, k 11, s 4, batch 4 took 147 us (1.8 TB/s),
// bound by those reads.  Here a wave has one input line in LDS at a time, and a lane keeps the sums
// of the KL = ceil(k/s) output lines that this input line reaches in registers:
//   - a pixel is read from LDS once per tap column and used for KL rows; the kernel numbers are the
//     same for every lane (LDS broadcasts, four taps at a time);
//   - a line lies in LDS by column phase (pixel j at place j / s of plane j mod s), so the lanes of
//     a tap read consecutive 16-byte words at any stride, free of bank conflicts;
//   - waves share nothing (a workgroup is four waves, each with its own lines of a segment), so
//     there is no barrier; three input lines are on their way from memory to registers while one
//     is computed.
// 4096^2, k 11, s 4, batch 4: 66 us (4.4 TB/s); 2000^2, k 4, s 4, batch 8: 45 -> 24 us;
// 3000 x 2000, k 8, batch 1: 187 -> 79 us.
//
// The sum over a row's window on the zero-padded plane is the row's sum only if the row is
// described exactly as the window at its position must be (checked on the descriptor when the row
// is finished) and the kernel numbers that meet padding are finite; any other row is summed again
// from its descriptor, out of global memory.
#pragma once
#include "compact_channels_kernel.h"

namespace convspmv {

constexpr int kPushWaves = 4;         // waves per workgroup
constexpr int kPushItems = 5;         // elements of an input line per lane, at most
constexpr int kPushDepth = 3;         // input lines in flight

__host__ __device__ constexpr int push_k_pitch(int k) { return (k + 3) & ~3; }

// floats of LDS per wave: the table, then a line of `places` elements (a multiple of 16 bytes)
__host__ __device__ constexpr int push_wave_floats(int k, int places, bool scalar) {
    return push_k_pitch(k) * k + ((places * (scalar ? 1 : 4) + 3) & ~3);
}

struct PushGeom {
    int m, n, m_out, n_out, s, p, k;
    int batch;
    int lpr_log2;         // log2 of the lanes per output column (4 batch columns each)
    int tw;               // output columns per strip: 64 >> lpr_log2
    int strips, segs;     // segments of seg output lines; a wave walks seg / kPushWaves of them
    int seg;
    int blocks, blocks_per_xcd;
    int iw, pw;           // input pixels of a strip, (tw - 1) * s + k; places per phase, ceil(iw / s)
    int c_base;           // first batch column of this launch
    int accum;            // 1: y += T x
};

// FINE: the sum over an input line's taps is added to the output line's sum as one number (see spmm_compact_kernel).
template <int KL, bool SCALAR, bool FINE>
__global__ __launch_bounds__(kPushWaves *kWave) void spmm_compact_push_kernel(const int2 *__restrict__ desc,
                                                                             const float *__restrict__ ktab,
                                                                             const float *__restrict__ x,
                                                                             float *__restrict__ y, const PushGeom g) {
    using elem_t = typename std::conditional<SCALAR, float, vec4>::type;
    extern __shared__ float4 push_lds[];
    const int tid = (int)threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int sh = SCALAR ? 0 : g.lpr_log2, lpr = 1 << sh;
    const int s = g.s, k = g.k;
    const int places = g.pw * s * lpr;                        // elements of a line in LDS
    const int kp = push_k_pitch(k);                           // the wave's own copy of the table: 16-byte rows
    float *const kt = reinterpret_cast<float *>(push_lds) + wave * push_wave_floats(k, places, SCALAR);
    elem_t *const line = reinterpret_cast<elem_t *>(kt + kp * k);

    // a band of neighbouring segments to each XCD, strips next to each other
    const int job = ((int)blockIdx.x % kXcds) * g.blocks_per_xcd + (int)blockIdx.x / kXcds;
    if ((int)blockIdx.x / kXcds >= g.blocks_per_xcd || job >= g.blocks) return;
    const int sg = job / g.strips, strip = job - sg * g.strips;
    const int part = g.seg / kPushWaves;
    const int xa = sg * g.seg + wave * part, xb = min(xa + part, g.m_out);
    if (xa >= xb) return;                                     // (uniform over the wave; there is no barrier)
    const int y0 = strip * g.tw, v = lane & (lpr - 1), yo = y0 + (lane >> sh);
    const bool live = yo < g.n_out;
    const int c0 = g.c_base + (int)blockIdx.y * (SCALAR ? 1 : 4 << sh);
    auto column = [&](int v_) { return SCALAR ? c0 : chunk_col(c0 + 4 * v_, g.batch); };
    auto load = [](const float *q) -> elem_t {
        if constexpr (SCALAR) return *q;
        else return *reinterpret_cast<const vec4u *>(q);
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

    // this lane's elements of an input line: offset in the line (floats), place in LDS; a place whose
    // pixel is outside the image is never written and stays zero
    const int j_lo = s * y0 - g.p, items = g.iw << sh;
    int off[kPushItems], dst[kPushItems];
#pragma unroll
    for (int r = 0; r < kPushItems; ++r) {
        const int item = lane + r * kWave, q = item >> sh, vv = item & (lpr - 1);
        const int j = j_lo + q, jc = min(max(j, 0), g.n - 1);
        off[r] = jc * g.batch + column(vv);
        dst[r] = (item < items && j == jc) ? (((q % s) * g.pw + q / s) << sh) + vv : -1;
    }
    for (int t = lane; t < places; t += kWave) line[t] = elem_t(0.0f);
    const int i_a = max(s * xa - g.p, 0), i_b = min(s * (xb - 1) - g.p + k, g.m);   // not empty: p < k
    auto load_line = [&](int i, elem_t (&e)[kPushItems]) {
        const float *base = x + (long long)min(i, g.m - 1) * g.n * g.batch;
#pragma unroll
        for (int r = 0; r < kPushItems; ++r)
            if (r * kWave < items) e[r] = load(base + off[r]);
    };
    auto store_line = [&](const elem_t (&e)[kPushItems]) {
        wave_lds_order();
#pragma unroll
        for (int r = 0; r < kPushItems; ++r)
            if (r * kWave < items && dst[r] >= 0) line[dst[r]] = e[r];
        wave_lds_order();
    };

    // what Theorem 2.1 says about this lane's column
    const int b_lo_e = max(g.p - s * yo, 0), r2_e = k - b_lo_e - max(s * yo + k - g.n - g.p, 0);
    const int lane_word = b_lo_e << 16 | r2_e << 24, lane_col = s * yo + b_lo_e - g.p;
    bool finite = true;
    for (int t = lane; t < k * k; t += kWave) {
        const float kv = ktab[t];
        const int a = div_small(t, 1.0f / (float)k);
        kt[a * kp + t - a * k] = kv;
        finite = finite && __builtin_isfinite(kv);
    }
    const bool plain = __all(finite) || r2_e == k;            // no infinite kernel number meets a zero of the padding
    const long long yc = min(yo, g.n_out - 1);
    auto load_desc = [&](int xo) { return desc[(long long)min(xo, g.m_out - 1) * g.n_out + yc]; };

    elem_t acc[KL];                                           // acc[l]: output line xtop - l
#pragma unroll
    for (int l = 0; l < KL; ++l) acc[l] = elem_t(0.0f);
    int2 d = load_desc(xa);
    auto finish = [&](int xo, elem_t sum) {                   // store output line xo; its descriptor is in d
        const int a_lo_e = max(g.p - s * xo, 0), r1_e = k - a_lo_e - max(s * xo + k - g.m - g.p, 0);
        const int word_e = a_lo_e | r1_e << 8 | lane_word, base_e = (s * xo + a_lo_e - g.p) * g.n + lane_col;
        const int2 dd = d;
        d = load_desc(xo + 1);
        const bool ok = plain && dd.x == base_e && dd.y == word_e;
        if (live && !ok) {
            const unsigned w = (unsigned)dd.y;
            const int a_lo = w & 255u, r1 = (w >> 8) & 255u, b_lo = (w >> 16) & 255u, r2 = w >> 24;
            sum = elem_t(0.0f);
            for (int da = 0; da < r1; ++da)
                for (int db = 0; db < r2; ++db)
                    fma_elem(sum, ktab[(a_lo + da) * k + b_lo + db],
                             load(x + ((long long)dd.x + (long long)da * g.n + db) * g.batch + column(v)));
        }
        if (live && (SCALAR || c0 + 4 * v < g.batch)) {
            float *out = y + ((long long)xo * g.n_out + yo) * g.batch + column(v);
            if (g.accum) sum += load(out);
            if constexpr (SCALAR) __builtin_nontemporal_store(sum, out);
            else __builtin_nontemporal_store((vec4u)sum, reinterpret_cast<vec4u *>(out));
        }
    };

    int xtop = (i_a + g.p) / s, r0 = (i_a + g.p) - xtop * s, x_next = xa;     // r0: tap line of xtop; x_next: first line not stored
    const int lane_place = ((lane >> sh) << sh) + v;          // (the lane itself: place yy of plane 0)
    // KN output lines take line i: tap lines r0, r0 + s, ...
    auto push = [&](auto kn_tag) {
        constexpr int KN = decltype(kn_tag)::value;
        elem_t part[FINE && KN > 0 ? KN : 1];                 // FINE: the sums over this line's taps
        if constexpr (FINE) {
#pragma unroll
            for (int l = 0; l < KN; ++l) part[l] = elem_t(0.0f);
        }
        auto sum = [&](int l) -> elem_t & {
            if constexpr (FINE) return part[l];
            else return acc[l];
        };
        const float *kr = kt + r0 * kp;                       // tap line of slot l: kr + l * s * kp
        const int line_step = s * kp;
        int ph = 0, place = lane_place;                       // of tap column b: phase b mod s, place yy + b / s
        auto next_place = [&] {
            const int at = place + ((ph * g.pw) << sh);
            if (++ph == s) {
                ph = 0;
                place += lpr;
            }
            return at;
        };
        int b = 0;
        for (; b + 4 <= k; b += 4) {                          // four taps: their pixels and numbers first, then the sums
            elem_t e[4];
            vec4 kv[KN > 0 ? KN : 1];
#pragma unroll
            for (int t = 0; t < 4; ++t) e[t] = line[next_place()];
#pragma unroll
            for (int l = 0; l < KN; ++l) kv[l] = *reinterpret_cast<const vec4 *>(kr + l * line_step + b);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int l = 0; l < KN; ++l) fma_elem(sum(l), kv[l][t], e[t]);
        }
        for (; b < k; ++b) {
            const elem_t e = line[next_place()];
#pragma unroll
            for (int l = 0; l < KN; ++l) fma_elem(sum(l), kr[l * line_step + b], e);
        }
        if constexpr (FINE) {
#pragma unroll
            for (int l = 0; l < KN; ++l) acc[l] += part[l];
        }
    };
    auto one_line = [&](int i, elem_t (&e)[kPushItems]) {
        store_line(e);
        load_line(i + kPushDepth, e);
        if (r0 + s * (KL - 1) < k) push(std::integral_constant<int, KL>{});
        else push(std::integral_constant<int, (KL > 1 ? KL - 1 : 0)>{});
        // the output line whose last tap line this was
        const int done = i + g.p - k + 1;
        if (done >= s * x_next && x_next < xb) {
            finish(x_next, acc[KL - 1]);                      // done = s * x_next: place KL - 1 holds it
            ++x_next;
        }
        if (++r0 == s) {
            r0 = 0;
            ++xtop;
#pragma unroll
            for (int l = KL - 1; l > 0; --l) acc[l] = acc[l - 1];
            acc[0] = elem_t(0.0f);
        }
    };
    elem_t ea[kPushItems], eb[kPushItems], ec[kPushItems];
    load_line(i_a, ea);
    load_line(i_a + 1, eb);
    load_line(i_a + 2, ec);
    for (int i = i_a; i < i_b; i += kPushDepth) {
        one_line(i, ea);
        if (i + 1 < i_b) one_line(i + 1, eb);
        if (i + 2 < i_b) one_line(i + 2, ec);
    }
    // output lines that the image's end cuts short
    if (r0 == 0) {                                            // (undo the last step to a line without input)
        --xtop;
#pragma unroll
        for (int l = 0; l + 1 < KL; ++l) acc[l] = acc[l + 1];
    }
#pragma unroll
    for (int l = KL - 1; l >= 0; --l)
        if (xtop - l == x_next && x_next < xb) {
            finish(x_next, acc[l]);
            ++x_next;
        }
}

}  // namespace convspmv
