// Host side of the C ABI declared in include/convspmv.h: argument checking,
// the closed-form count of Theorem 2.1, the plan object and kernel dispatch.
#include <pthread.h>

#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>

#include "apply_kernels.h"
#include "dispatch.h"

using namespace convspmv;

namespace {

thread_local int g_last_hip_error = 0;

}  // namespace

bool convspmv::hip_ok(hipError_t e) {
    if (e == hipSuccess) return true;
    g_last_hip_error = (int)e;
    return false;
}

namespace {

// Fewer strip segments than this cannot fill the chip with persistent workgroups; the row-group
// kernels take such problems.  A plan carries its own copy (conv_plan_set_march_min_jobs).
constexpr int kMarchMinJobs = 256;

// Attributes launch failures to this call only: the runtime's last-error slot may already
// hold an error of other code in the process (it is sticky until somebody reads it).  The
// slot is peeked before the first launch and after the last; an error that was there before
// is neither reported as ours nor cleared.
struct LaunchScope {
    hipError_t before;
    LaunchScope() : before(hipPeekAtLastError()) {}
    bool ok() const {
        const hipError_t after = hipPeekAtLastError();
        if (after == hipSuccess || after == before) return true;
        g_last_hip_error = (int)after;
        (void)hipGetLastError();      // ours: take it out of the slot
        return false;
    }
};

// The words (edited_word.h) in which products from column-compressed arrays note edited columns: a static array of every
// device, so that a build allocates nothing.  A plan has its place to itself until it is destroyed, which is after its
// last product; places are taken again in the order in which they came back, with another stamp.  A plan that finds
// none left (65536 plans at a time) scatters.
constexpr int kEditedWords = 1 << 16;
__device__ unsigned edited_words[kEditedWords];

struct EditedPlaces {
    pthread_mutex_t lock = PTHREAD_MUTEX_INITIALIZER;
    int fresh = 0, oldest = 0, returned = 0;      // places never taken; those given back, a ring
    int ring[kEditedWords];
    unsigned stamp[kEditedWords];

    int take(unsigned *stamp_out) {
        pthread_mutex_lock(&lock);
        int slot = -1;
        if (fresh < kEditedWords) {
            slot = fresh++;
        } else if (returned > 0) {
            slot = ring[oldest];
            oldest = (oldest + 1) % kEditedWords;
            --returned;
        }
        if (slot >= 0) {
            if (++stamp[slot] == 0) ++stamp[slot];     // (the array begins with zeros)
            *stamp_out = stamp[slot];
        }
        pthread_mutex_unlock(&lock);
        return slot;
    }
    void give_back(int slot) {
        pthread_mutex_lock(&lock);
        ring[(oldest + returned++) % kEditedWords] = slot;
        pthread_mutex_unlock(&lock);
    }
};
EditedPlaces edited_places;

unsigned *edited_words_of(int device) {
    static std::atomic<unsigned *> known[64];
    const bool keep = device >= 0 && device < 64;
    unsigned *base = keep ? known[device].load(std::memory_order_relaxed) : nullptr;
    if (!base && hipGetSymbolAddress((void **)&base, HIP_SYMBOL(edited_words)) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    if (keep) known[device].store(base, std::memory_order_relaxed);
    return base;
}

// Theorem 2.1, output extent along one axis (0 = precondition violated).
int64_t out_extent(int64_t extent, int64_t k, int64_t s, int64_t p) {
    if (k > extent + 2 * p) return 0;
    return (extent + 2 * p - k) / s + 1;
}

int check_shape(int m, int n, int k, int s, int p, int64_t *mo, int64_t *no) {
    if (m < 1 || n < 1 || k < 1 || s < 1 || p < 0) return CONV_EINVAL;
    *mo = out_extent(m, k, s, p);
    *no = out_extent(n, k, s, p);
    if (*mo < 1 || *no < 1) return CONV_EINVAL;
    return CONV_OK;
}

// Sum over one axis of max(0, k - c(t)), c(t) = max(0, p - s t) + max(0, s t + k - extent - p).
int64_t axis_tap_sum(int64_t count, int64_t extent, int64_t k, int64_t s, int64_t p) {
    if (count <= kInt32Limit) {
        const AxisScan q = axis_scan((int)extent, (int)count, (int)k, (int)s, (int)p);
        return axis_prefix<false>(q, (int)count, (int)count, (int)k, (int)s, (int)p);
    }
    int64_t total = 0;
    for (int64_t t = 0; t < count; ++t) {
        const int64_t lo = p - s * t, hi = s * t + k - extent - p;
        const int64_t r = k - (lo > 0 ? lo : 0) - (hi > 0 ? hi : 0);
        if (r > 0) total += r;
    }
    return total;
}

}  // namespace

extern "C" {

int conv_out_shape(int m, int n, int k, int s, int p, int *m_out, int *n_out) {
    if (!m_out || !n_out) return CONV_ENULL;
    int64_t mo, no;
    const int st = check_shape(m, n, k, s, p, &mo, &no);
    if (st != CONV_OK) return st;
    if (mo > kInt32Limit || no > kInt32Limit) return CONV_EOVERFLOW;
    *m_out = (int)mo;
    *n_out = (int)no;
    return CONV_OK;
}

int64_t conv_nnz(int m, int n, int k, int s, int p) {
    int64_t mo, no;
    const int st = check_shape(m, n, k, s, p, &mo, &no);
    if (st != CONV_OK) return st;
    const int64_t s1 = axis_tap_sum(mo, m, k, s, p);
    const int64_t s2 = axis_tap_sum(no, n, k, s, p);
    int64_t total;
    if (__builtin_mul_overflow(s1, s2, &total)) return CONV_EOVERFLOW;
    return total;
}

}  // extern "C"

namespace {

// col_idx / vals fill of a built plan's matrix for `channels` kernels one after the other; the
// quad-walking kernel takes rows too long for the others.
// Returns true when the launch also wrote row_ptr (with row_ptr_dev given).
constexpr int64_t kFillMinBlocks = 1024, kFillFewBlocks = 256;
constexpr int64_t kFillAlikeEntries = 2000000, kFillAlikeRows = 100000;
constexpr int64_t kFillQuadEntries = 25000;      // entries a workgroup of the values' kernel computes, about
template <bool COLS, bool TR>
bool launch_fill(const conv_plan *plan, const float *kernel_dev, int *idx_dev, float *vals_dev, hipStream_t q,
                 int *row_ptr_dev = nullptr, int channels = 1) {
    constexpr int kMaxGridY = 65535;
    const ConvShape &sh = plan->shape;
    const int64_t l1 = TR ? sh.m : sh.m_out, l2 = TR ? sh.n : sh.n_out;
    // Lines per workgroup: as many as give it `entries` of them, while there are workgroups enough to
    // fill the chip; few workgroups: shorter ranges of rows.
    auto lines_of = [&](int64_t rows, int64_t entries) {
        const int64_t most = l1 * ((l2 + rows - 1) / rows) / kFillMinBlocks;
        return std::max<int64_t>(std::min(entries / std::max<int64_t>(rows * plan->max_row_nnz, 1), most), 1);
    };
    auto shorter = [&](int rows) {
        while (rows > 64 && l1 * ((l2 + rows - 1) / rows) < kFillFewBlocks) rows >>= 1;
        return rows;
    };
    // values alone, where the rows between two borders are alike and the entries many: below, the longer prologue
    // is most of the kernel (28^2, k 3: 3.8 us, staged 3.3, T^T 4.4 and 3.7; 256^2, k 5: 6.3 and 6.0; but 512^2, k 5: 9.3 and 9.8;
    // 531 x 349, k 2: 6.1 and 6.3)
    const int range = shorter(kFillRows);
    const bool alike = !COLS && (!TR || sh.s == 1) && (int64_t)kFillRows * plan->max_row_nnz <= kFillSpan &&
                       (plan->nnz * channels >= kFillAlikeEntries || plan->rows * channels >= kFillAlikeRows ||
                        (int64_t)kFillRows / 4 * plan->max_row_nnz > kFillStageEntries);
    // through an LDS image of R rows' entries
    int R = 256;
    while (R > 1 && (int64_t)R * plan->max_row_nnz > kFillStageEntries) R >>= 1;
    R = shorter(R);
    const int skew = plan->max_row_nnz % 4 == 0;
    int cap = (int)std::min<int64_t>(((int64_t)R * plan->max_row_nnz + 4 + 3) & ~3LL, 1 << 20);
    if (skew) cap = (fill_padded(cap) + 4 + 3) & ~3;
    const int64_t lds = ((((int64_t)R + 1 + (int64_t)sh.k * sh.k + 3) & ~3LL) + (COLS ? 2 : 1) * cap) * 4;
    const int64_t stage_ranges = (l2 + R - 1) / R;
    const bool staged = (int64_t)R * plan->max_row_nnz <= kFillStageEntries && lds <= 64 * 1024;
    const BuildScan bs = build_scan<TR>(sh);
    const unsigned quad_blocks = (unsigned)(l1 * ((l2 + kFillRows - 1) / kFillRows));
    for (int ch = 0; ch < channels; ch += kMaxGridY) {
        const unsigned by = (unsigned)std::min(channels - ch, kMaxGridY);
        const float *kern = kernel_dev + (size_t)ch * sh.k * sh.k;
        float *vals = vals_dev + (size_t)ch * plan->nnz;
        if (alike) {
            const int64_t lines = lines_of(range, kFillQuadEntries), blocks = (l1 + lines - 1) / lines * ((l2 + range - 1) / range);
            vals_fill_lines_kernel<TR><<<dim3((unsigned)blocks, by), kFillThreads, (size_t)sh.k * sh.k * 4, q>>>(sh, bs, kern,
                                                                                                             vals, range, (int)lines);
        } else if (staged) {
            const int64_t lines = lines_of(R, kFillStageEntries), blocks = (l1 + lines - 1) / lines * stage_ranges;
            csr_fill_staged_kernel<COLS, TR><<<dim3((unsigned)blocks, by), kFillThreads, (size_t)lds, q>>>(
                sh, bs, kern, idx_dev, vals, R, cap, (int)lines, skew, row_ptr_dev);
        } else {
            csr_fill_kernel<COLS, TR><<<dim3(quad_blocks, by), kFillThreads, 0, q>>>(sh, bs, kern, idx_dev, vals);
        }
    }
    return staged && row_ptr_dev != nullptr;
}

// Argument and size checks shared by the CSR / CSC builds; fills the size fields of *plan.
template <bool TR>
int build_check(int m, int n, int k, int s, int p, int channels, const float *kernel_dev, const int32_t *ptr_dev,
                const int32_t *idx_dev, const float *vals_dev, conv_plan *plan, int64_t *rp_blocks_out) {
    int64_t mo, no;
    int st = check_shape(m, n, k, s, p, &mo, &no);
    if (st != CONV_OK) return st;
    if (channels < 1) return CONV_EINVAL;
    const int64_t nnz = conv_nnz(m, n, k, s, p);
    if (nnz < 0) return (int)nnz;
    const int64_t out_pixels = mo * no, in_pixels = (int64_t)m * n;
    const int64_t rows = TR ? in_pixels : out_pixels, cols = (TR ? out_pixels : in_pixels) * channels;
    if (cols >= kInt32Limit) return CONV_EOVERFLOW;
    const int64_t l1 = TR ? m : mo, l2 = TR ? n : no;        // lines of the matrix, rows per line
    // 32-bit indices: entries, columns, rows (+1 for the pointer array), the per-axis
    // prefix sums, and the grids of the build kernels.
    if (nnz > kInt32Limit || in_pixels >= kInt32Limit || out_pixels >= kInt32Limit || (int64_t)k * k > kInt32Limit ||
        mo * (int64_t)k > kInt32Limit || no * (int64_t)k > kInt32Limit || (int64_t)m * k > kInt32Limit ||
        (int64_t)n * k > kInt32Limit)
        return CONV_EOVERFLOW;
    const int64_t fill_blocks = l1 * ((l2 + kFillRows - 1) / kFillRows);
    const int64_t rp_blocks = l1 * ((l2 + kRowPtrThreads - 1) / kRowPtrThreads);
    if (fill_blocks > kInt32Limit || rp_blocks > kInt32Limit) return CONV_EOVERFLOW;
    if (!ptr_dev || !kernel_dev || (nnz > 0 && (!idx_dev || !vals_dev))) return CONV_ENULL;
    *plan = conv_plan{};
    plan->shape = ConvShape{m, n, k, s, p, (int)mo, (int)no};
    plan->rows = rows;
    plan->cols = cols;
    plan->nnz = nnz;
    const int per_axis = TR ? (k + s - 1) / s : k;
    plan->max_row_nnz = per_axis * per_axis;
    plan->march_min_jobs = kMarchMinJobs;
    plan->transposed = TR;
    plan->channels = channels;
    *rp_blocks_out = rp_blocks;
    return CONV_OK;
}

// The build kernels of a checked plan.
template <bool TR>
void build_enqueue(const conv_plan *plan, const float *kernel_dev, int32_t *ptr_dev, int32_t *idx_dev,
                   float *vals_dev, int64_t rp_blocks, hipStream_t q) {
    const int k = plan->shape.k;
    // the staged fill writes row_ptr on its way; otherwise (no entries, or rows too long for it) its own kernel does
    bool have_row_ptr = false;
    if (plan->nnz > 0) have_row_ptr = launch_fill<true, TR>(plan, kernel_dev, idx_dev, vals_dev, q, ptr_dev);
    if (!have_row_ptr)
        row_ptr_kernel<TR><<<(unsigned)rp_blocks, kRowPtrThreads, 0, q>>>(plan->shape, build_scan<TR>(plan->shape), ptr_dev);
    if (plan->nnz > 0 && plan->channels > 1)         // the other channels share the indices: values only
        launch_fill<false, TR>(plan, kernel_dev + (size_t)k * k, nullptr, vals_dev + plan->nnz, q, nullptr, plan->channels - 1);
}

template <bool TR>
int build_impl(int m, int n, int k, int s, int p, int channels, const float *kernel_dev, int32_t *ptr_dev,
               int32_t *idx_dev, float *vals_dev, void *stream, conv_plan **plan_out) {
    if (!plan_out) return CONV_ENULL;
    *plan_out = nullptr;
    conv_plan checked;
    int64_t rp_blocks = 0;
    const int st = build_check<TR>(m, n, k, s, p, channels, kernel_dev, ptr_dev, idx_dev, vals_dev, &checked, &rp_blocks);
    if (st != CONV_OK) return st;
    conv_plan *plan = new (std::nothrow) conv_plan(checked);
    if (!plan) return CONV_ENOMEM;
    plan->row_ptr = ptr_dev;
    plan->col_idx = idx_dev;
    plan->vals = vals_dev;
    if (!hip_ok(hipGetDevice(&plan->device))) {
        delete plan;
        return CONV_EHIP;
    }
    const LaunchScope scope;
    build_enqueue<TR>(plan, kernel_dev, ptr_dev, idx_dev, vals_dev, rp_blocks, (hipStream_t)stream);
    if (!scope.ok()) {
        delete plan;
        return CONV_EHIP;
    }
    if (TR) {
        unsigned *const words = edited_words_of(plan->device);
        plan->edited_place = words ? edited_places.take(&plan->edited.stamp) : -1;
        if (plan->edited_place >= 0) plan->edited.word = words + plan->edited_place;
    }
    *plan_out = plan;
    return CONV_OK;
}

}  // namespace

// conv_csr_fill_noalloc: most output lines and columns together (a documented limit of that entry point)
constexpr int kNoAllocAxisInts = 1 << 16;

extern "C" {

int conv_csr_fill_noalloc(int m, int n, int k, int s, int p, const float *kernel_dev, int32_t *row_ptr_dev,
                          int32_t *col_idx_dev, float *vals_dev, void *stream) {
    conv_plan plan;
    int64_t rp_blocks = 0;
    const int st = build_check<false>(m, n, k, s, p, 1, kernel_dev, row_ptr_dev, col_idx_dev, vals_dev, &plan, &rp_blocks);
    if (st != CONV_OK) return st;
    if ((int64_t)plan.shape.m_out + plan.shape.n_out + 2 > kNoAllocAxisInts) return CONV_EOVERFLOW;
    if (!hip_ok(hipGetDevice(&plan.device))) return CONV_EHIP;
    const LaunchScope scope;
    build_enqueue<false>(&plan, kernel_dev, row_ptr_dev, col_idx_dev, vals_dev, rp_blocks, (hipStream_t)stream);
    return scope.ok() ? CONV_OK : CONV_EHIP;
}

int conv_csr_build(int m, int n, int k, int s, int p, const float *kernel_dev, int32_t *row_ptr_dev,
                   int32_t *col_idx_dev, float *vals_dev, void *stream, conv_plan **plan_out) {
    return build_impl<false>(m, n, k, s, p, 1, kernel_dev, row_ptr_dev, col_idx_dev, vals_dev, stream, plan_out);
}

int conv_csr_build_channels(int m, int n, int k, int s, int p, int channels, const float *kernels_dev,
                            int32_t *row_ptr_dev, int32_t *col_idx_dev, float *vals_dev, void *stream,
                            conv_plan **plan_out) {
    return build_impl<false>(m, n, k, s, p, channels, kernels_dev, row_ptr_dev, col_idx_dev, vals_dev, stream,
                             plan_out);
}

int conv_csc_build(int m, int n, int k, int s, int p, const float *kernel_dev, int32_t *col_ptr_dev,
                   int32_t *row_idx_dev, float *vals_dev, void *stream, conv_plan **plan_out) {
    return build_impl<true>(m, n, k, s, p, 1, kernel_dev, col_ptr_dev, row_idx_dev, vals_dev, stream, plan_out);
}

int conv_compact_build(int m, int n, int k, int s, int p, const float *kernel_dev, int32_t *row_desc_dev,
                       float *ktab_dev, void *stream, conv_plan **plan_out) {
    return conv_compact_build_channels(m, n, k, s, p, 1, kernel_dev, row_desc_dev, ktab_dev, stream, plan_out);
}

int conv_compact_build_channels(int m, int n, int k, int s, int p, int channels, const float *kernel_dev,
                                int32_t *row_desc_dev, float *ktab_dev, void *stream, conv_plan **plan_out) {
    if (!plan_out) return CONV_ENULL;
    *plan_out = nullptr;
    int64_t mo, no;
    int st = check_shape(m, n, k, s, p, &mo, &no);
    if (st != CONV_OK) return st;
    if (channels < 1) return CONV_EINVAL;
    if (k > 255) return CONV_EINVAL;                       // tap ranges are stored in 8 bits
    const int64_t nnz = conv_nnz(m, n, k, s, p);
    if (nnz < 0) return (int)nnz;
    const int64_t rows = mo * no, cols = (int64_t)m * n * channels;
    if (rows >= kInt32Limit || cols >= kInt32Limit || mo * (int64_t)k > kInt32Limit || no * (int64_t)k > kInt32Limit ||
        (int64_t)channels * k * k > kInt32Limit)
        return CONV_EOVERFLOW;
    const int64_t blocks = mo * ((no + kCompactBuildThreads - 1) / kCompactBuildThreads);
    if (blocks > kInt32Limit) return CONV_EOVERFLOW;
    if (!kernel_dev || !row_desc_dev || !ktab_dev) return CONV_ENULL;
    if (((uintptr_t)row_desc_dev & 7u) != 0) return CONV_EINVAL;      // descriptors are read as 8-byte pairs

    conv_plan *plan = new (std::nothrow) conv_plan;
    if (!plan) return CONV_ENOMEM;
    plan->shape = ConvShape{m, n, k, s, p, (int)mo, (int)no};
    plan->rows = rows;
    plan->cols = cols;
    plan->nnz = nnz;
    plan->max_row_nnz = k * k;
    plan->row_ptr = nullptr;
    plan->col_idx = nullptr;
    plan->vals = nullptr;
    plan->device = 0;
    plan->transposed = false;
    plan->channels = channels;
    plan->compact = true;
    plan->march_min_jobs = kMarchMinJobs;
    plan->desc = reinterpret_cast<const int2 *>(row_desc_dev);
    plan->ktab = ktab_dev;
    if (!hip_ok(hipGetDevice(&plan->device))) {
        delete plan;
        return CONV_EHIP;
    }
    hipStream_t q = (hipStream_t)stream;
    const LaunchScope scope;
    compact_rows_kernel<<<(unsigned)blocks, kCompactBuildThreads, 0, q>>>(plan->shape, reinterpret_cast<int2 *>(row_desc_dev));
    compact_table_kernel<<<(channels * k * k + 255) / 256, 256, 0, q>>>(kernel_dev, ktab_dev, channels * k * k);
    if (!scope.ok()) {
        delete plan;
        return CONV_EHIP;
    }
    *plan_out = plan;
    return CONV_OK;
}

int conv_update_kernel(conv_plan *plan, const float *kernel_dev, void *stream) {
    if (!plan || !kernel_dev) return CONV_ENULL;
    const LaunchScope scope;
    if (plan->compact) {
        const int kk = plan->shape.k * plan->shape.k * plan->channels;
        compact_table_kernel<<<(kk + 255) / 256, 256, 0, (hipStream_t)stream>>>(kernel_dev, plan->ktab, kk);
        return scope.ok() ? CONV_OK : CONV_EHIP;
    }
    if (plan->nnz == 0) return CONV_OK;
    if (plan->transposed)
        launch_fill<false, true>(plan, kernel_dev, nullptr, plan->vals, (hipStream_t)stream, nullptr, plan->channels);
    else
        launch_fill<false, false>(plan, kernel_dev, nullptr, plan->vals, (hipStream_t)stream, nullptr, plan->channels);
    if (!scope.ok()) return CONV_EHIP;
    return CONV_OK;
}

}  // extern "C"

namespace {

// ---------------------------------------------------------------------------
// Apply dispatch
// ---------------------------------------------------------------------------

// Lanes per row for the gather kernels: the narrowest power of two that keeps
// the trip count at or below 8 (rows have at most k*k entries).
int group_width(int max_row_nnz) {
    int g = 1;
    while (g < 16 && (max_row_nnz + g - 1) / g > 8) g <<= 1;
    return g;
}

const int kTileNit[] = {2, 4, 7};       // trip counts the tile kernel is built for (8 lanes per row)

// Column chunks per lane of the vector kernels.  One block of up to 16 batch columns reads the
// entries once, so the widest lanes a batch fills come first (a batch of 10: one block of 16
// columns with 6 idle, not three of 4; 613 x 407, k 5, batch 10: 22 us, and 268 us one column at a
// time); the marching and tile kernels go down to `least` where wider lanes leave too few workgroups.
constexpr int widest_nv(int batch) { return batch > 8 ? 4 : (batch > 4 ? 2 : 1); }
constexpr int least_nv(int batch) { return batch % 16 == 0 ? 4 : (batch % 8 == 0 ? 2 : 1); }
constexpr int64_t kTileMinBlocks = 512;
// Row-group kernels: lanes per row are doubled below the first number of workgroups (35 x 30,
// k 4, batch 10: 4.7 us with 2 lanes per row, 3.2 with 16; three entries per lane at least, a tree
// of single products rounds more often than the chain it replaces; 198 x 128, k 4, s 3, batch 64: 7.0 and
// 4.6), columns per lane halved below the second (148 x 195, k 4, s 2, batch 64, 2 lanes per row:
// 225 workgroups of 16 columns 9 us, 900 of 4 columns 18.6).
// Long rows want them narrower earlier (25 x 35, k 13, batch 36: 6.4 us with 16 columns, 4.8 with 4; short ones do not:
// 426 x 303, k 1, batch 24: 2.4 and 3.3; nor at large strides, where a narrow lane wastes more of the
// memory lines it reads: 236 x 249, k 5, s 4, batch 24: 4.4 and 7.2).
constexpr int64_t kRowGroupWiden = 512;
constexpr int64_t row_group_min_blocks(int64_t entries, int s) { return s <= 3 && entries >= 25 * s ? 384 : 128; }
// Multiply-adds below which the row groups beat the tile kernel's staging and barrier (76 x 48,
// k 3, batch 32, 1.0 M: 3.8 us against 4.9; 75 x 87, k 6, batch 16, 3.7 M: 4.5 against 5.4; above it
// 88 x 67, k 7, batch 32, 8.8 M: 7.7 against 6.4; 194 x 137, k 7, s 2, batch 32, 10 M: 9.2 against 6.6).
constexpr int64_t kTileMinWork = 3500000;
// T^T, whose tiles find their window by divisions: more (197 x 202, k 3, batch 4, 1.4 M: 4.2 us, row groups 3.2;
// 267 x 383, k 3, batch 4, 3.7 M: 5.4 and 4.4; 500 x 450, k 3, batch 8, 16 M: 7.1 and 9.8), unless every
// lane has its 16 columns (168 x 177, k 3, batch 32, 8.5 M: 5.9 and 8.2).  At strides above 1 its rows differ in
// length, so that lanes idle, and its results leave in pieces of memory lines: full lanes, or rows of 9 entries and
// more at batches up to 16 or where the operands exceed the last-level cache (340 x 367, k 3, s 2, batch 168:
// 119 us, row groups 61; batch 160: 27 and 45; 881 x 1143, k 5, s 4, batch 40: 224 and 95).
constexpr double kTileMinWorkT = 12e6, kTileMinBytesT = 200e6;
bool tile_serves_t(const conv_plan *plan, int batch) {
    const double work = (double)plan->nnz * batch, bytes = 4.0 * (double)(plan->rows + plan->cols) * batch;
    if (plan->max_row_nnz < 4) return false;       // an entry or two: nothing to share (763 x 1019, k 2, s 4, batch 212: 1085 us, row groups 649)
    if (batch % 16 == 0) return work >= kTileMinWork;
    if (plan->shape.s > 1 && (plan->max_row_nnz < 9 || (batch > 16 && bytes < kTileMinBytesT))) return false;
    return work >= kTileMinWorkT;
}

int round_up_mod(int v, int mod, int rem) {      // smallest r >= v with r % mod == rem
    int r = v - (v % mod) + rem;
    return r < v ? r + mod : r;
}

// Geometry of a tile kernel launch: the widest line pitch rule and the most
// output lines per tile whose input window still fits one LDS plane.
// *most: tiles there would be with the lowest tile lines it would try for more workgroups.
bool tile_geometry(const conv_plan *plan, int batch, int tw, int plane, int col_blocks, int rows_per_pass, TileGeom *out, int64_t *most) {
    const ConvShape &sh = plan->shape;
    const bool tr = plan->transposed;
    TileGeom g{};
    // operand and result grids: the image and the window grid for T, exchanged for T^T
    g.m = tr ? sh.m_out : sh.m;
    g.n = tr ? sh.n_out : sh.n;
    g.m_out = tr ? sh.m : sh.m_out;
    g.n_out = tr ? sh.n : sh.n_out;
    g.la = tr ? 1 : sh.s;
    g.lb = tr ? sh.p - sh.k + sh.s : -sh.p;
    g.ld = tr ? sh.s : 1;
    g.batch = batch;
    g.nnz = (int)plan->nnz;
    // operand pixels that `count` neighbouring results can touch, and the inverse
    auto extent = [&](int64_t count) { return tr ? (count - 2 + sh.k) / sh.s + 2 : (count - 1) * sh.s + sh.k; };
    auto results = [&](int64_t lines) { return tr ? (lines - 1) * sh.s - sh.k + 1 : (lines - sh.k) / sh.s + 1; };
    const int64_t iw = extent(tw);
    if (iw + 16 > plane) return false;
    g.iw = (int)iw;
    g.iw_pitch = round_up_mod((int)iw, 16, 8);
    // lines of operand that fit: ih * iw_pitch + 1 <= plane (one pixel of zeros follows the window)
    const int64_t ih_max = (plane - 1) / g.iw_pitch;
    if (ih_max < extent(1)) return false;
    int64_t th = std::max<int64_t>(results(ih_max), 1);
    if (th > 8) th = 8;
    if (th > g.m_out) th = g.m_out;
    // a small plane: lower tiles, down to one pass per wave, until there are workgroups for the chip (but not
    // more than it holds at a time, two per compute unit: 413 x 252, k 2, batch 32: 416 workgroups 8.8 us, 552 11.3)
    g.tiles_x = (g.n_out + tw - 1) / tw;
    const int64_t th_min = (int64_t)(tw * 8 / kWave) * rows_per_pass / tw;
    auto tiles = [&](int64_t lines) { return (g.m_out + lines - 1) / lines * g.tiles_x * col_blocks; };
    int64_t low = th;
    while (low > 1 && low > th_min && tiles(low) < kTileMinBlocks) --low;
    while (th > low && tiles(th - 1) <= kTileMinBlocks) --th;
    *most = tiles(low) / col_blocks;
    const int64_t ih = extent(th);
    g.th = (int)th;
    g.ih = (int)ih;
    g.tiles_y = (int)((g.m_out + th - 1) / th);
    const int64_t n_tiles = (int64_t)g.tiles_x * g.tiles_y;
    // int arithmetic in the kernel: s*x0 - p, i_lo + ih, ihc * n (float-reciprocal division needs < 2^21)
    if ((int64_t)sh.m + 2LL * sh.p + ih >= (1LL << 30) || (int64_t)sh.n + 2LL * sh.p + iw >= (1LL << 30)) return false;
    if (ih * g.n >= (1LL << 21) || g.n >= (1 << 20) || plan->cols > (1LL << 27)) return false;
    if (n_tiles + kXcds >= (1LL << 31) / kXcds) return false;
    g.n_tiles = (int)n_tiles;
    g.tiles_per_xcd = (int)((n_tiles + kXcds - 1) / kXcds);
    g.inv_n = 1.0f / (float)g.n;
    *out = g;
    return true;
}

// Marching kernel: strips of tw output columns, a ring of 16 or 8 input lines in
// LDS.  Rows of up to 56 entries are shared by 8 lanes (strips of 64 columns),
// rows of up to 128 entries by 16 lanes (strips of 32 columns); the workgroup
// is 512 threads either way.
constexpr int kMarchThreads = 512;

struct MarchShape { int g, nit, tw; };
bool march_shape(int max_row_nnz, MarchShape *out) {
    // rows of fewer than 16 entries leave most of a group's lanes idle and the fixed cost
    // of a pass (bounds, combine, store) unpaid: measured slower than the row-group kernels
    if (max_row_nnz < 16) return false;
    if (max_row_nnz <= 16) *out = MarchShape{8, 2, 64};
    else if (max_row_nnz <= 32) *out = MarchShape{8, 4, 64};
    else if (max_row_nnz <= 56) *out = MarchShape{8, 7, 64};
    else if (max_row_nnz <= 96) *out = MarchShape{16, 6, 32};
    else if (max_row_nnz <= 128) *out = MarchShape{16, 8, 32};
    else return false;
    return true;
}
constexpr int kMarchTargetBlocks = 512;      // two resident workgroups on each of 256 CUs

bool march_geometry(const conv_plan *plan, int batch, int nv, int tw, MarchGeom *out, int *ls_out, int *nl_out) {
    const ConvShape &sh = plan->shape;
    const bool tr = plan->transposed;
    MarchGeom g{};
    // operand and result grids: the image and the window grid for T, exchanged for T^T
    g.m = tr ? sh.m_out : sh.m;
    g.n = tr ? sh.n_out : sh.n;
    g.m_out = tr ? sh.m : sh.m_out;
    g.n_out = tr ? sh.n : sh.n_out;
    g.s = sh.s; g.p = sh.p; g.k = sh.k;
    g.tr = tr ? 1 : 0;
    g.batch = batch;
    g.nnz = (int)plan->nnz;
    // operand columns a strip of tw result columns can touch, operand lines in use or arriving
    // during a step of 2 (1) result lines, and new operand lines per step -- upper bounds
    const int64_t iw = tr ? (int64_t)(tw - 2 + sh.k) / sh.s + 2 : (int64_t)(tw - 1) * sh.s + sh.k;
    const int64_t need2 = tr ? (int64_t)(sh.k + 2) / sh.s + 2 : (int64_t)sh.s * 3 + sh.k;
    const int64_t need1 = tr ? (int64_t)sh.k / sh.s + 2 : (int64_t)sh.s + sh.k;
    const int64_t new2 = tr ? 2 / sh.s + 1 : 2LL * sh.s, new1 = tr ? 1 / sh.s + 1 : sh.s;
    const int plane = march_plane(nv);
    if (iw + 16 > plane) return false;
    g.iw = (int)iw;
    g.iw_pitch = round_up_mod((int)iw, 16, 8);
    // Ring of 16 lines with steps of two result lines when the ring, the LDS plane and the
    // per-thread line registers (2 per thread) allow it; else steps of one line with 16 or 8
    // ring lines.
    const int threads = kMarchThreads, planes = nv ? nv : 1;
    auto regs = [&](int64_t lines) { return lines * iw * planes <= 2LL * threads; };
    auto fits = [&](int nl) { return (int64_t)nl * g.iw_pitch + 1 <= plane; };
    int ls = 0, nl = 0;
    if (need2 <= 16 && regs(new2) && fits(16)) { ls = 2; nl = 16; }
    else if (need1 <= 16 && regs(new1) && fits(16)) { ls = 1; nl = 16; }
    else if (need1 <= 8 && regs(new1) && fits(8)) { ls = 1; nl = 8; }
    if (ls == 0) return false;
    // int arithmetic in the kernel: s*x - p + k, col*16, d16 < 2^25 (see the kernel)
    if ((int64_t)sh.m + 2LL * sh.p + sh.k >= (1LL << 30) || (int64_t)sh.n + 2LL * sh.p + iw >= (1LL << 30)) return false;
    if ((int64_t)g.m * g.n > (1LL << 27) || 2LL * 16 * g.n * 16 > (1LL << 25)) return false;
    if (g.n_out < tw / 2) return false;                 // a strip would be mostly empty
    g.strips = (g.n_out + tw - 1) / tw;
    const int col_blocks = column_blocks(batch, nv);
    if ((int64_t)g.strips * ((g.m_out + 7) / 8) * col_blocks < plan->march_min_jobs) return false;
    int64_t segs = kMarchTargetBlocks / ((int64_t)g.strips * col_blocks);
    if (segs < 1) segs = 1;
    int64_t seg = (g.m_out + segs - 1) / segs;
    if (seg < 8) seg = 8;
    seg = (seg + 1) & ~1LL;
    g.seg = (int)seg;
    g.segs = (int)((g.m_out + seg - 1) / seg);
    const int64_t jobs = (int64_t)g.strips * g.segs;
    if (jobs + kXcds >= (1LL << 31) / kXcds) return false;
    g.blocks_per_xcd = (int)((jobs + kXcds - 1) / kXcds);
    g.inv_n = 1.0f / (float)g.n;
    *out = g;
    *ls_out = ls;
    *nl_out = nl;
    return true;
}

// Marching kernel with the entry stream staged through LDS (apply_stage_march_kernel.h): strips of
// 32 result columns, 8 waves, one workgroup per CU.  Lanes per row by the longest row, so that the
// entries of a wave's 64 / G rows fit its LDS image; result lines per step WL = G (G = 2: 8 ...).
constexpr int kStageTargetBlocks = 256;
struct StageShape { int g, nit, nld; };
bool stage_shape(int max_row_nnz, StageShape *out) {
    // Rows of 3 x 3 taps: the fixed cost of a pass is not paid back (224^2, k 3, batch 256: 37 us
    // with either this or the tile kernel).  Rows of 101 to 128 entries take 8 lanes per row and
    // two result lines per step (4096^2, k 11, s 4, batch 4: 205 us against 246 us from the other
    // marching kernel, which keeps the still longer rows it can hold -- none at present, its limit
    // is 128 too -- and the shapes whose lines per step this one's registers do not hold).
    if (max_row_nnz < 16) return false;
    if (max_row_nnz <= 26) *out = StageShape{2, 13, 4};
    else if (max_row_nnz <= 50) *out = StageShape{2, 25, 7};
    else if (max_row_nnz <= 100) *out = StageShape{4, 25, 7};
    else if (max_row_nnz <= 128) *out = StageShape{8, 16, 4};
    else return false;
    return true;
}
constexpr size_t stage_lds(int nv, int nld) {
    return (nv ? (size_t)nv * stage_plane(nv, nld) * 16 : (size_t)stage_plane(0, nld) * 4) +
           (size_t)kStageWaves * stage_wave_bytes(nld);
}

// Lines of a segment.  A workgroup fills a compute unit, so the launch runs in rounds of a workgroup for each, and a
// segment costs its lines plus about two steps (of wl lines) for the window and entries it loads before its
// first step: the number of segments per strip that minimises rounds x (lines + 2 steps).  (Three
// column blocks of 32 strips: 8 segments = 768 workgroups = 3 full rounds, not 2 segments = 192.)
// The cells (strip, segment) are dealt out to the XCDs first, each with all its column blocks: a share is rounded up before it is
// multiplied, and 252 workgroups of 7 strips, 3 segments, 12 blocks are 36 on an XCD of 32 compute units, two rounds.
// (Counted over the chip, parts 1, -> by XCD, us: 738 x 733, k 11, s 2, batch 40: 189 -> 101; 436 x 649, k 7, batch 48: 138 -> 80;
// 120 x 150, k 7, batch 180: 49.5 -> 30.6; T^T, 205 x 264, k 6, batch 48: 37.8 -> 25.0.  51 of 61 such products that march
// either way: 1.28 to 1.86 times as fast.)
int64_t stage_segment(int64_t m_out, int64_t strips, int col_blocks, int wl, int parts) {
    int64_t seg = 0, best_cost = -1;
    for (int64_t segs = 1; segs <= 512 && (segs - 1) * wl < m_out; ++segs) {
        int64_t len = (m_out + segs - 1) / segs;
        len = (len + wl - 1) / wl * wl;
        const int64_t real = (m_out + len - 1) / len;
        const int64_t share = (strips * real + parts - 1) / parts * col_blocks;
        const int64_t rounds = (share + kStageTargetBlocks / parts - 1) / (kStageTargetBlocks / parts);
        const int64_t cost = rounds * (len + 2 * wl);
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; seg = len; }
    }
    return seg;
}

// channels > 1: the geometry of one launch that walks the channels of every block of lines
bool stage_march_geometry(const conv_plan *plan, int batch, int nv, int channels, const StageShape &ss, MarchGeom *out,
                          int *wl_out) {
    const ConvShape &sh = plan->shape;
    const bool tr = plan->transposed;
    MarchGeom g{};
    g.m = tr ? sh.m_out : sh.m;
    g.n = tr ? sh.n_out : sh.n;
    g.m_out = tr ? sh.m : sh.m_out;
    g.n_out = tr ? sh.n : sh.n_out;
    g.s = sh.s; g.p = sh.p; g.k = sh.k;
    g.tr = tr ? 1 : 0;
    g.batch = batch;
    g.nnz = (int)plan->nnz;
    g.max_row = plan->max_row_nnz;
    g.channels = channels;
    g.x_plane = (long long)plan->cols * batch;
    if (channels > 1 && (tr || nv == 2)) return false;
    const int tw = kStageTw, rw = kWave / ss.g, wl = kStageWaves / (tw / rw);
    // the image must hold the rows of a wave: (rw - 1) full rows, the slots of the last one, 3 entries of alignment
    if ((int64_t)(rw - 1) * plan->max_row_nnz + (int64_t)ss.nit * ss.g + 3 > (int64_t)ss.nld * 256) return false;
    // operand columns a strip can touch, operand lines WL result lines can touch, new lines per step -- upper bounds
    const int64_t iw = tr ? (int64_t)(tw - 2 + sh.k) / sh.s + 2 : (int64_t)(tw - 1) * sh.s + sh.k;
    const int64_t need = tr ? (int64_t)(wl - 2 + sh.k) / sh.s + 2 : (int64_t)sh.s * (wl - 1) + sh.k;
    const int64_t fresh = tr ? (int64_t)wl / sh.s + 1 : (int64_t)sh.s * wl;
    const int plane = stage_plane(nv, ss.nld), planes = nv ? nv : 1;
    if (need > kStageNl || iw + 16 > plane) return false;
    g.iw = (int)iw;
    g.iw_pitch = round_up_mod((int)iw, 16, 8);
    if ((int64_t)kStageNl * g.iw_pitch + 1 > plane) return false;
    // line registers per thread
    if ((channels > 1 ? need * iw * planes > (int64_t)kStageXldChannels * kWave * kStageWaves
                      : fresh * iw * planes > (int64_t)kStageXld * kWave * kStageWaves))
        return false;
    // int arithmetic in the kernel, as for the other marching kernel
    if ((int64_t)sh.m + 2LL * sh.p + sh.k >= (1LL << 30) || (int64_t)sh.n + 2LL * sh.p + iw >= (1LL << 30)) return false;
    if ((int64_t)g.m * g.n > (1LL << 27) || 2LL * kStageNl * g.n * 16 > (1LL << 25)) return false;
    if (g.n_out < tw / 2) return false;                 // a strip would be mostly empty
    g.strips = (g.n_out + tw - 1) / tw;
    const int col_blocks = column_blocks(batch, nv);
    if ((int64_t)((g.n_out + 63) / 64) * ((g.m_out + 7) / 8) * col_blocks < plan->march_min_jobs) return false;   // jobs of 64 columns x 8 lines, as for the other kernel
    const int64_t seg = stage_segment(g.m_out, g.strips, col_blocks, wl, kXcds);
    g.seg = (int)seg;
    g.segs = (int)((g.m_out + seg - 1) / seg);
    const int64_t jobs = (int64_t)g.strips * g.segs;
    if (jobs + kXcds >= (1LL << 31) / kXcds) return false;
    g.blocks_per_xcd = (int)((jobs + kXcds - 1) / kXcds);
    g.inv_n = 1.0f / (float)g.n;
    *out = g;
    *wl_out = wl;
    return true;
}

// Geometry of a block kernel launch (apply_block_kernel.h): the lanes over the batch whose blocks of columns leave the
// fewest idle, the widest of those.
bool block_geometry(const conv_plan *plan, int batch, int *lpr_log2, BlockGeom *out) {
    const ConvShape &sh = plan->shape;
    const bool tr = plan->transposed;
    auto padded = [&](int l) { return (batch + (4LL << l) - 1) >> (l + 2) << (l + 2); };
    int lpr = kBlockLprMost;
    for (int l = kBlockLprMost - 1; l >= kBlockLprLeast; --l)
        if (padded(l) < padded(lpr)) lpr = l;
    // byte offsets of 32 bits, and int arithmetic on padded lines
    if (plan->cols * batch >= (1LL << 30) || plan->rows * batch >= (1LL << 30)) return false;
    if ((int64_t)sh.m + 2LL * sh.p >= (1LL << 30) || (int64_t)sh.n + 2LL * sh.p >= (1LL << 30)) return false;
    BlockGeom g{};
    g.m = tr ? sh.m_out : sh.m;
    g.n = tr ? sh.n_out : sh.n;
    g.m_out = tr ? sh.m : sh.m_out;
    g.n_out = tr ? sh.n : sh.n_out;
    g.p = sh.p;
    g.batch = batch;
    const int first = block_first(sh.s, sh.p, tr);
    const int64_t lines = 2 * block_rx(sh.k, sh.s, tr), pixels = 2LL * block_ry(sh.k, sh.s, tr) * (kWave >> lpr);
    const int64_t cells_y = (g.n_out - first + pixels - 1) / pixels, cells = (g.m_out - first + lines - 1) / lines * cells_y;
    if (cells + kXcds >= (1LL << 31) / kXcds) return false;
    g.cells_y = (int)cells_y;
    g.cells = (int)cells;
    g.cells_per_xcd = (int)((cells + kXcds - 1) / kXcds);
    *out = g;
    *lpr_log2 = lpr;
    return true;
}

// Where the block kernel takes a product from the kernel that would have it otherwise: batches above 32 columns (lanes for 64 at
// least; below, the tile kernel's 16 columns per lane are as good: 224^2, k 3, batch 16: 6.0 us, blocks with 4 lanes a pixel 7.1).
// The lines lie where 26 000 products (planes of 16 to 700 a side, batches of 33 to 256, every (k, s) compiled) had the block
// kernel and the other one even.  A marching kernel walks and loses everywhere, if its rows are long too (246^2, k 4,
// batch 96: 30.8 us and 13.3; 192^2, k 11, s 3, T^T, batch 192: 54 and 13.4), but for 25 taps at stride 1, where it depends on how full
// the lanes and how full the marching kernel's rounds of workgroups are: of 6900 more products of that kind its time is
// within 10 % of what block_march_ns says, the block kernel's within 14 % of block_ns, and the smaller of the two names
// the faster kernel in all but 170 (in blocks 550 of them are slower, up to 1.36 times: 182 x 111, batch 144: 16.9 us
// marching, 23.0; 475 x 679, batch 80: 100 and 117; but 128^2, batch 128: 11.6 and 9.9).  Tiles and row groups start at once, where a
// block waits for row pointers, then entries, then sums, the longer the more entries it has.  Blocks of few entries
// are even with them where the launch is all there is (up to 1.5 M multiply-adds) and faster above; from then on, least work in
// millions of multiply-adds for medians of 0.95 of the other's time and less:
//   T:    16 taps, s 1: 8 (below 1.02 to 1.1); 25 taps, s 2: 20 (below 0.95 to 1.2); 25 taps, s 1: tiles stay (1.0 to 1.3)
//   T^T:  9 taps, s 3: 8, s 4: 10 (below up to 1.3); 16 taps, s 1 and 2: 6, s 4: 15, s 3: tiles stay (1.1); 25 taps: tiles stay
// (340 x 367, k 3, s 2, T^T, batch 160: 34 us with tiles, 15 in blocks; batch 168: 70 in row groups, 30; 93 x 124, k 5, T^T, batch 160: 10.4 with
// tiles, 15.4 in blocks; 37 x 48, k 12, s 3, T^T, batch 178: 5.3 in row groups, 8.4 in blocks.)  Of the 26 000, 53 are more than 6 % slower than
// with the other kernel, 323 would be that much faster.
constexpr int kBlockMinBatch = 33;
constexpr int64_t kBlockNever = INT64_MAX;
constexpr double kBlockMarchEven = 1.02;      // (of the 6900: 28 slower by more than 6 %, 143 missed)
int64_t block_least_work(const ConvShape &sh, bool tr, int taps) {
    if (taps < 9) return 0;
    if (tr) {
        if (taps == 9) return sh.s <= 2 ? 0 : sh.s == 3 ? 8000000 : 10000000;
        if (taps == 16) return sh.s <= 2 ? 6000000 : sh.s == 3 ? kBlockNever : 15000000;
        return kBlockNever;
    }
    if (taps == 9) return sh.s <= 2 ? 1500000 : 0;
    if (taps == 16) return sh.s == 1 ? 8000000 : 1500000;
    return sh.s == 1 ? kBlockNever : sh.s == 2 ? 20000000 : 1500000;
}
// 25 taps, stride 1: nanoseconds of the staged march (a workgroup per compute unit, 32 of those on an XCD, whose cells are
// divided evenly among the XCDs) and of the block kernel.  The march's are those of segments counted over the chip: it
// has shorter ones, and would take more products from the blocks, in 0.94 of their time in the mean of 158 (up to 1.14) but with
// sums of 13 entries a chain, 1.05 of the blocks' error, up to 1.25.
double block_march_ns(const ApplyChoice &c, int batch) {
    const int col_blocks = column_blocks(batch, c.nv);
    const int64_t seg = stage_segment(c.march.m_out, c.march.strips, col_blocks, c.ls, 1);
    const int64_t cells = c.march.strips * ((c.march.m_out + seg - 1) / seg), rounds = ((cells + kXcds - 1) / kXcds * col_blocks + 31) / 32;
    return rounds * (c.nv == 4 ? 4400.0 + 416.0 * seg : 3800.0 + 318.0 * seg);
}
double block_ns(int64_t rows, int batch, int lpr_log2) {
    constexpr double start[3] = {6200.0, 5500.0, 4700.0}, row[3] = {3.41e-3, 2.67e-3, 2.54e-3};    // 64, 128, 256 columns
    const int64_t columns = 4LL << lpr_log2, padded = (batch + columns - 1) / columns * columns;
    return start[lpr_log2 - kBlockLprLeast] + row[lpr_log2 - kBlockLprLeast] * (double)rows * (double)padded;
}
bool block_serves(const conv_plan *plan, int batch, int lpr_log2, const ApplyChoice &other) {
    const ConvShape &sh = plan->shape;
    if (batch < kBlockMinBatch) return false;
    if (other.kind == Kind::StageMarch && sh.k == 5 && sh.s == 1) return block_ns(plan->rows, batch, lpr_log2) <= kBlockMarchEven * block_march_ns(other, batch);
    if (other.kind == Kind::March || other.kind == Kind::StageMarch) return true;
    return plan->nnz * batch >= block_least_work(sh, plan->transposed, plan->max_row_nnz);
}

// The kernel for a product, blocks left aside.
ApplyChoice choose_unblocked(const conv_plan *full, int batch) {
    // geometry of one channel; a multi-channel plan applies it once per channel (LDS kernels)
    // or walks the channels inside the row-group kernels
    conv_plan one = *full;
    one.cols = full->cols / full->channels;
    one.channels = 1;
    const conv_plan *plan = &one;
    ApplyChoice c{};
    // (a multi-channel row is walked as one list of channels * entries by the row-group kernels)
    c.g = group_width((int)std::min<int64_t>((int64_t)plan->max_row_nnz * full->channels, 1 << 20));
    c.threads = kGatherThreads;
    // batches of 4 and more travel in chunks of four columns (at any alignment, see chunk_col);
    // of 1 to 3 one column at a time
    const bool vec = batch >= 4;
    const int nv_hi = vec ? widest_nv(batch) : 0, nv_lo = vec ? least_nv(batch) : 0;
    c.nv = nv_hi;
    c.kind = vec ? Kind::GatherVec : Kind::GatherScalar;
    // few rows: more lanes per row, then fewer columns per lane, until there are workgroups for the chip
    auto row_blocks = [&] { return (plan->rows * c.g + kGatherThreads - 1) / kGatherThreads; };
    const int64_t row_max = (int64_t)plan->max_row_nnz * full->channels;
    while (c.g < 16 && 6 * c.g <= row_max && row_blocks() * column_blocks(batch, c.nv) < kRowGroupWiden) c.g *= 2;
    while (c.nv > 1 && row_blocks() * column_blocks(batch, c.nv) < row_group_min_blocks(full->channels > 1 ? 1 : row_max, plan->shape.s)) c.nv /= 2;
    if (plan->nnz == 0 || column_blocks(batch, nv_hi) > 65535) return c;

    // marching kernels: float4 column chunks, or scalar columns
    MarchShape ms;
    MarchGeom mg;
    int ls, nl;
    StageShape ss;
    int wl;
    auto staged = [&](int nv) {
        c.kind = Kind::StageMarch;
        c.nv = nv;
        c.g = ss.g;
        c.nit = ss.nit;
        c.tw = kStageTw;
        c.threads = kStageWaves * kWave;
        c.lds = stage_lds(nv, ss.nld);
        c.ls = wl;
        c.nl = kStageNl;
        c.xld = ss.nld;          // (16-byte loads per lane, array and pass)
        c.march = mg;
        return c;
    };
    // Batches of 2 and 3 go column by column and read the entries again for each.  Sums over channels, and T^T at
    // strides above 1 with rows of up to 16 entries, are left to the row groups (247 x 335, k 4, 4 channels,
    // batch 3: 56 us, row groups 29; 196 x 273, k 11, s 3, T^T, batch 3: 18 and 7).  (Not where the plan's threshold, a test hook, is lowered.)
    const bool scalar_columns = !vec && batch > 1;
    const bool marches = !scalar_columns || full->march_min_jobs < kMarchMinJobs ||
                         !(full->channels > 1 || (plan->transposed && plan->shape.s > 1 && plan->max_row_nnz <= 16));
    // all channels in one launch (lanes of 16 or 4 columns)
    if (marches && full->channels > 1 && stage_shape(plan->max_row_nnz, &ss))
        for (int nv = nv_hi;; nv = nv_lo) {
            const int nvc = nv == 2 ? 1 : nv;
            if (stage_march_geometry(plan, batch, nvc, full->channels, ss, &mg, &wl)) return staged(nvc);
            if (nv == nv_lo) break;
        }
    auto march = [&](int nv) {
        if (!march_shape(plan->max_row_nnz, &ms) || !march_geometry(plan, batch, nv, ms.tw, &mg, &ls, &nl)) return false;
        c.kind = Kind::March;
        c.nv = nv;
        c.g = ms.g;
        c.nit = ms.nit;
        c.tw = ms.tw;
        c.threads = kMarchThreads;
        c.lds = nv ? (size_t)nv * march_plane(nv) * 16 : (size_t)march_plane(0) * 4;
        c.ls = ls;
        c.nl = nl;
        c.march = mg;
        return true;
    };
    for (int nv = nv_hi; marches; nv /= 2) {
        const bool stages = stage_shape(plan->max_row_nnz, &ss) && stage_march_geometry(plan, batch, nv, 1, ss, &mg, &wl);
        // Ragged lanes of long rows: the other marching kernel, whose lanes sum 8 entries and need no sums in
        // blocks (FINE), 0.6 to 0.8 of the staged one's time from 64 entries on (393 x 379, k 11, batch 40: 196 and 87
        // us; shorter rows 0.8 to 1.2), where segments counted over the chip are not the shortest: their sums are also
        // the more exact by 2 %.  (By the present segments 57 x 85, k 8, batch 540 would leave: 37 us, staged 67.)  Scalar columns
        // likewise, but for rows of 25 entries (812 x 521, k 8, batch 3: 343 us, row groups 144; 477 x 694, k 8, batch 3: 150, here 95).
        const bool other_first = scalar_columns ? plan->max_row_nnz != 25
                                                : stages && nv && batch % (4 * nv) != 0 && plan->max_row_nnz >= 64 &&
                                                      stage_segment(mg.m_out, mg.strips, column_blocks(batch, nv), wl, 1) >= 4 * wl;
        const MarchGeom staged_geom = mg;
        if (other_first && march(nv)) return c;
        mg = staged_geom;
        if (stages) return staged(nv);
        if (march(nv)) return c;
        if (nv <= nv_lo) break;
    }
    if (!vec || !(plan->transposed ? tile_serves_t(plan, batch) : plan->nnz * batch >= kTileMinWork)) return c;
    // A multi-channel sum through the LDS kernels is one launch per channel.  That pays for the
    // marching kernel (large problems); the problems the tile kernel takes are small, and the
    // row-group kernels, which walk the channels inside one launch, measured 3x faster there.
    if (full->channels > 1) return c;

    // one LDS tile per workgroup when the rows fit its unrolled trip count and the
    // input window of at least one output line fits the LDS planes
    // Rows of at most 10 entries (k = 3): two lanes per row and 5 slots each.  With 8 lanes per
    // row the kernel is bound by its instructions there (224^2, k 3, batch 256: 18.5 M vector
    // instructions for 1.8 M multiply-adds, VALU 0.70 busy): 16 slots for 9 entries and a
    // three-level combine per row.
    const bool narrow = plan->max_row_nnz <= kTileShortRow;
    const int tile_g = narrow ? 2 : kTileG;
    const int need = (plan->max_row_nnz + tile_g - 1) / tile_g;
    int nit = narrow ? kTileShortNit : 0;
    if (!narrow)
        for (int cand : kTileNit)
            if (cand >= need) { nit = cand; break; }
    if (nit == 0) return c;
    const int tws[2] = {kTileWide, kTileNarrow}, planes[2] = {kPlaneWide, kPlaneNarrow};
    for (int i = 0; i < 2; ++i) {
        TileGeom g;
        int64_t most = 0;
        if ((plan->transposed ? plan->shape.n : plan->shape.n_out) <= kTileNarrow && tws[i] == kTileWide) continue;
        if (!tile_geometry(plan, batch, tws[i], planes[i], column_blocks(batch, nv_hi), kWave / tile_g, &g, &most)) continue;
        c.kind = Kind::Tile;
        c.nv = nv_hi;
        while (c.nv > nv_lo && most * column_blocks(batch, c.nv) < kTileMinBlocks) c.nv /= 2;
        c.g = tile_g;
        c.nit = nit;
        c.tw = tws[i];
        c.threads = tws[i] * 8;
        c.lds = (size_t)c.nv * planes[i] * 16 + (size_t)g.th * (tws[i] + 1) * 4;
        c.geom = g;
        break;
    }
    return c;
}

// Rows and chunks of four columns, one below a batch of 4, dealt out to cells of per_cell and to the XCDs (items, and descriptor
// lanes); false beyond 32-bit byte offsets into x (x_size numbers) and y, item numbers of 32 bits, or exact small divisions.
template <class Geom>
bool chunk_geometry(const conv_plan *plan, int batch, int64_t x_size, int64_t per_cell, Geom *g) {
    const int columns = batch >= 4 ? 4 : 1;
    const int64_t chunks = (batch + columns - 1) / columns, items = plan->rows * chunks, cells = (items + per_cell - 1) / per_cell;
    if (x_size >= (1LL << 30) || plan->rows * batch >= (1LL << 30) || items > kInt32Limit - kItemThreads || chunks + kWave >= (1 << 21) ||
        cells + kXcds >= (1LL << 31) / kXcds)
        return false;
    g->batch = batch;
    g->chunks = (int)chunks;
    g->inv_chunks = 1.0f / (float)chunks;
    g->items = (unsigned)items;
    g->cells = (int)cells;
    g->cells_per_xcd = (int)((cells + kXcds - 1) / kXcds);
    return true;
}

// Geometry of an item launch with g lanes per item.
bool item_geometry(const conv_plan *plan, int batch, int g, int ways, ItemGeom *out) {
    const int64_t pixels = plan->cols / plan->channels;
    ItemGeom i{};
    if (pixels > (1 << 24) || batch >= (1 << 22) ||      // a column times the batch is a product of 24-bit numbers
        !chunk_geometry(plan, batch, pixels * batch, (plan->channels > 1 ? kWave : kItemThreads) / g, &i))
        return false;
    i.channels = plan->channels;
    i.ways = ways;
    i.vals_stride = plan->nnz;
    i.x_stride = pixels * batch;
    *out = i;
    return true;
}

// Lanes per item: more where the launch has few waves (below 512; with the scalar columns of batches 2 and 3 below 2048),
// each with an access of entries or two of its own; rows of 9 entries one or two (apply_item_kernel.h); chunks of four columns up to 8, as
// the launches that could use 16 stay with the row groups.  Channels: lanes first, then waves that share them, four
// channels each at least.
bool item_choice(const conv_plan *plan, int batch, ApplyChoice *out) {
    const int columns = batch >= 4 ? 4 : 1, most = plan->max_row_nnz;
    const bool many = plan->channels > 1;
    const int64_t waves = (plan->rows * ((batch + columns - 1) / columns) + kWave - 1) / kWave;
    const int g_most = most == 1 ? 1 : most == 9 ? (many ? 4 : 2) : many || columns == 1 ? 16 : 8, per_lane = columns == 1 && !many ? 8 : 4;
    const int64_t enough = many ? 8192 : columns == 1 ? 2048 : 512;
    int g = 1, ways = 1;
    while (g < g_most && g * per_lane < most && waves * g < enough) g *= 2;
    while (many && ways < kItemWaysMost && ways * 8 <= plan->channels && waves * g * ways < 1024) ways *= 2;
    ApplyChoice c{};
    if (!item_geometry(plan, batch, g, ways, &c.item)) return false;
    // few workgroups of short rows, which G cannot spread: one compute unit asks for all channels of its items (23 x 32, k 2, s 4, 120
    // channels, batch 1: 13.0 us, row groups 9.8)
    if (many && most < 16 && c.item.cells < (most < 9 ? 64 : 8)) return false;
    c.kind = Kind::Item;
    c.g = g;
    c.nv = batch >= 4;
    c.threads = many ? ways * kWave : kItemThreads;
    c.lds = ways > 1 ? (size_t)ways * (kWave / g) * columns * sizeof(double) : 0;      // the waves' partial sums
    *out = c;
    return true;
}

// Where an item launch (apply_item_kernel.h) takes a product from the kernel that would have it otherwise: where a surface, fitted to
// which of the two is the faster, is above zero.  The times are in profiles/chunk_kernel_times.csv: drawn products (planes of 8
// to 4096 a side, k 1 to 13, strides 1 to 4, batches to 2048, a third of them multiples of 16, up to 1024 channels), both kernels
// in replayed graphs.  Logistic regression on which is faster; a product weighs the logarithm of its times' ratio, up to 0.7, and
// where items are slower 3 times that (channels in other kernels 4, row groups above a batch of 3 and marches 6); one that tests hold to
// a kernel weighs 1 (row groups of T: 4).  (Tiles: an older fit to the logarithm itself, less 0.12, by short products, w below 2, less 0.4, as tests
// hold products to tiles that a new one would take.)
// Coordinates: w, the multiply-adds of a chunk each (log2 of millions); b, the chunks (log2); how full the other kernels' blocks of 16
// columns are; a, the longest row (log2); stride 1 or not; the other kernel's chunks per lane, 2 or 4, and whether the batch is a
// multiple of them, as its lanes are then full and its accesses aligned; c, the channels (log2).  Beyond the ranges of the fit they are
// held at their ends.  By the kernel left: products, how many leave it, time before over time after in their mean, those then more than
// 6 % slower, those that would still be that much faster; and the same of products drawn apart, with the slowest:
//   row groups, batches of 2 and 3    1014   584  1.58    5   24     588   328  1.59    1   13  0.93
//   marching, batches of 2 and 3       186   150  1.80    0    1     112    94  1.70    2    7  0.87
//   row groups, T                      900   529  1.50   10   55     550   311  1.55    5   37  0.82
//   row groups, T^T                    900   576  1.49    8   47     550   359  1.47    9   35  0.76
//   tiles, T                           900   369  1.97    2  330     550   218  1.95    6  205  0.80
//   marching                          1800   763  1.92   23  182    1100   454  1.98   15  110  0.79
//   staged march, T                    900   296  1.93   10   84     550   154  1.87    8   54  0.82
//   staged march, T^T                  900   360  1.75    8   93     550   223  1.70    5   66  0.73
//   channels, row groups              1692  1334  1.53   59  105    2119  1641  1.53   76  133  0.65
//   channels, other kernels            900   543  2.10   18   38     550   336  1.94   19   23  0.72
// Channel sums of row groups whose launch has waves to share the channels (ways) leave always: 834, none slower than 0.95 of the
// former speed.  What stays: products that both kernels finish within the time of a launch (w below -4, at strides of 4 and more -0.9);
// tiles of T^T (1.05 in the mean) and blocks (1.1 where they would leave); marching rows of 64 entries and more at batches of 2
// and 3 (1.09); row groups of one column and of batches 4 to 8, which are as fast (1.04 and 0.98 with the best G).
enum ItemAgainst { kFewGroups, kFewMarching, kGroupsT, kGroupsTT, kTileT, kMarching, kStagedT, kStagedTT, kGroupsMany, kOthersMany };
constexpr int kItemTerms = 22;
constexpr double kItemFaster[][kItemTerms] = {
    // 1, w, w^2, b, b^2, full, a, a^2, stride 1, w a, w b, a b, w at stride 1, 2 chunks per lane, 4, multiple of them, of 4;
    // channels: c, c^2, c w, c b, c a
    // row groups, batches of 2 and 3
    {8.0602, -0.1201, 0.3672, 0.1052, 0.0407, 0, -1.3024, -0.0272, -0.7083, 0.3953, 1.1541, -0.3363, -0.3703},
    // marching, batches of 2 and 3
    {88.0951, -17.0261, 1.768, 29.3963, 11.3721, 0, 11.0449, -0.9896, -6.4024, -4.3707, 7.6586, -9.5511, 1.9944},
    // row groups, T
    {23.5069, -0.1758, -0.0442, 6.2448, -0.4005, 1.814, -11.3378, 0.9234, -1.5365, -0.1334, 0.4496, -0.3733, 0.5849,
     -1.3357, 3.9855, -0.8001, 0.4776},
    // row groups, T^T
    {-2.7903, -2.2908, 0.0633, 2.3078, -0.0013, -2.0062, -0.4367, -0.0562, 1.0173, 0.2231, 0.4346, -0.2403, -0.0338,
     0.8529, 4.6813, 1.0905, 1.111},
    // tiles, T
    {0.3659, -0.0364, 0.0064, 0.2009, -0.0294, -0.2387, -0.0487, -0.0095, -0.0566, -0.0175, 0.0186, 0.012, -0.0491},
    // marching
    {3.7367, -2.4808, 0.5077, 2.6523, -0.1534, 6.4352, 1.2004, 0.0278, 4.4584, -0.788, 0.1273, -0.0591, -0.8703, -1.5612,
     -4.1715, -1.4058, -0.5283},
    // staged march, T
    {63.3654, -1.9129, 0.0451, 3.0241, 0.0218, 6.3423, -22.4184, 1.813, 4.0053, 0.2112, -0.2136, -0.128, -0.5929,
     -2.9133, -6.7706, -1.9805, 0.2129},
    // staged march, T^T
    {76.3723, -1.2961, 0.0864, 1.3883, -0.0879, -2.4071, -24.4221, 1.9923, -0.1241, -0.1322, -0.2404, 0.4734, 0.0272,
     -1.8124, -3.9253, -2.1951, 1.3022},
    // channels, row groups
    {16.2551, 2.5828, 0.0321, 2.9165, -0.1303, -2.8413, -6.0369, 0.5495, -1.7952, -0.5561, 0.0004, -0.1573, -0.0725,
     -2.7253, -2.3049, 0.4357, -0.9928, -4.0148, 0.3439, -0.244, -0.1575, 0.8381},
    // channels, other kernels
    {50.7089, 6.9869, 0.9959, -2.2321, 0.2014, 13.2341, -24.4058, 3.5737, 0.9072, -3.5822, 1.1214, -0.5658, -0.6216,
     -1.8357, -5.3448, -0.2813, -3.4369, -0.3796, 1.33, -2.848, -1.1262, 3.1921},
};
constexpr double kItemLaunch = -4.0, kItemLaunchStrided = -0.9, kItemShortTiles = 2.0, kItemShortTilesLeast = 0.28;
constexpr double kItemWorkLeast = -9.0, kItemWorkMost = 7.9, kItemChunksMost = 9.0;      // the fit's ranges
constexpr double kItemChannelsMost = 10.0, kItemChannelsMostOthers = 6.0;
constexpr int kItemRowMost = 169, kItemFewMarchRow = 64;                                        // (169: its longest row)

bool item_serves(const conv_plan *plan, int batch, const ApplyChoice &other, const ApplyChoice &item) {
    const bool tr = plan->transposed, groups = other.kind == Kind::GatherScalar || other.kind == Kind::GatherVec;
    // (not where the plan's marching threshold, a test hook, is lowered)
    if (plan->nnz == 0 || plan->march_min_jobs < kMarchMinJobs || plan->max_row_nnz > kItemRowMost) return false;
    const int columns = batch >= 4 ? 4 : 1, chunks = (batch + columns - 1) / columns;
    const double work = std::log2((double)plan->nnz * chunks * plan->channels) - 20.0, w = std::clamp(work, kItemWorkLeast, kItemWorkMost);
    ItemAgainst against = groups ? kGroupsMany : kOthersMany;
    double least = 0.0;
    if (plan->channels > 1) {
        if (groups && item.item.ways > 1) return true;
    } else {
        if (batch < 4) {
            if (other.kind == Kind::March && plan->max_row_nnz >= kItemFewMarchRow) return false;
            against = groups ? kFewGroups : kFewMarching;
        } else if (groups) {
            if (batch <= 8 || work < (plan->shape.s >= 4 ? kItemLaunchStrided : kItemLaunch)) return false;
            against = tr ? kGroupsTT : kGroupsT;
        } else if (other.kind == Kind::Tile) {
            if (tr) return false;
            against = kTileT;
            if (work < kItemShortTiles) least = kItemShortTilesLeast;
        } else if (other.kind == Kind::March) {
            against = kMarching;
        } else {
            against = tr ? kStagedTT : kStagedT;
        }
    }
    const double b = std::min(std::log2((double)chunks), kItemChunksMost), a = std::log2((double)plan->max_row_nnz), s = plan->shape.s == 1;
    const double c = std::min(std::log2((double)plan->channels), groups ? kItemChannelsMost : kItemChannelsMostOthers);
    const double full = columns == 4 ? chunks / (4.0 * ((chunks + 3) / 4)) : 0.0;
    const double two = other.nv == 2, four = other.nv == 4, whole = other.nv && batch % (4 * other.nv) == 0;
    const double at[kItemTerms] = {1.0, w, w * w, b, b * b, full, a, a * a, s, w * a, w * b, a * b, w * s, two, four, whole, whole * four,
                                   c, c * c, c * w, c * b, c * a};
    double faster = 0.0;
    for (int i = 0; i < kItemTerms; ++i) faster += kItemFaster[against][i] * at[i];
    return faster > least;
}

ApplyChoice choose_apply(const conv_plan *plan, int batch) {
    const ApplyChoice other = choose_unblocked(plan, batch);
    // batches that fill a wave (not where the plan's marching threshold, a test hook, is lowered)
    const ConvShape &sh = plan->shape;
    ApplyChoice c{};
    if (plan->channels > 1 || plan->nnz == 0 || plan->march_min_jobs < kMarchMinJobs || !block_compiled(sh.k, sh.s, plan->transposed) ||
        column_blocks(batch, 4) > 65535 || !block_geometry(plan, batch, &c.lpr_log2, &c.block) ||
        !block_serves(plan, batch, c.lpr_log2, other))
        return (batch > 1 || plan->channels > 1) && item_choice(plan, batch, &c) && item_serves(plan, batch, other, c) ? c : other;
    c.kind = Kind::Block;
    c.threads = kBlockThreads;
    c.g = 1;
    c.nv = 1;
    c.tw = block_ry(sh.k, sh.s, plan->transposed);
    return c;
}

constexpr int64_t kGatherAheadBlocks = 512;      // workgroups below which a lane asks for several entries at once

template <int G, bool AHEAD>
void launch_gather_ahead(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, int batch, hipStream_t q) {
    const int rows = (int)plan->rows;
    const dim3 grid((unsigned)(((int64_t)rows * G + kGatherThreads - 1) / kGatherThreads),
                    (unsigned)std::min(column_blocks(batch, c.nv), 65535));
    const ChannelStrides cs{plan->channels, (long long)plan->nnz, (long long)(plan->cols / plan->channels) * batch};
#define CONV_GATHER_VEC(NV)                                                        \
    spmm_gather_vec_kernel<G, NV, AHEAD><<<grid, kGatherThreads, 0, q>>>(           \
        plan->row_ptr, plan->col_idx, plan->vals, x, y, rows, batch, cs)
    switch (c.nv) {
        case 0:
            spmm_gather_scalar_kernel<G, AHEAD><<<grid, kGatherThreads, 0, q>>>(plan->row_ptr, plan->col_idx, plan->vals, x,
                                                                                y, rows, batch, cs);
            break;
        case 1: CONV_GATHER_VEC(1); break;
        case 2: CONV_GATHER_VEC(2); break;
        default: CONV_GATHER_VEC(4); break;
    }
#undef CONV_GATHER_VEC
}

template <int G>
void launch_gather(const ApplyChoice &c, const conv_plan *plan, const float *x, float *y, int batch, hipStream_t q) {
    const int64_t blocks = (plan->rows * G + kGatherThreads - 1) / kGatherThreads * column_blocks(batch, c.nv);
    if (blocks < kGatherAheadBlocks && plan->max_row_nnz > G) launch_gather_ahead<G, true>(c, plan, x, y, batch, q);
    else launch_gather_ahead<G, false>(c, plan, x, y, batch, q);
}

// ---------------------------------------------------------------------------
// Structure-aware storage: dispatch
// ---------------------------------------------------------------------------

constexpr int64_t kCompactMinBlocks = 256;      // below this many workgroups the row-group kernel takes the product

bool rect_compiled(int k, int s) {
    return (s == 1 && (k == 1 || k == 3 || k == 5 || k == 7 || k == 9)) || (s == 2 && (k == 2 || k == 3 || k == 5 || k == 7));
}

constexpr double kChanFusedWork = 1e8;        // multiply-adds per channel below which the launches are fused
constexpr int64_t kChanFusedWaves = 2048;     // waves that fill the chip (8 per CU)
constexpr int64_t kChanPartsMinBlocks = 64;   // workgroups from which k 3 at stride 1 has its tiles in parts (a quarter of them at stride 2)

// The push kernel's launch: strips of 64 lanes, four waves' parts per segment.  False where a strip's
// line is longer than a wave's registers for it, or the padding reaches the kernel size (rows
// without any input line would need no line at all), or more output lines share an input line than
// the kernel is compiled for.
constexpr int kPushMaxLines = 13;
constexpr int64_t kPushTargetWaves = 2048;    // two waves per SIMD
// Waves that a launch of it needs.  Fewer: row groups or the marching kernel (401 x 562, k 11, batch 4: 468
// waves 45 us, row groups 30; 1185 x 1424, k 6, s 3, batch 1: 800 waves 13.8 and 9.4).  Small kernels need more, as a
// wave walks every line and every column of the image for a few taps of each (843 x 1177, k 4, s 2, batch 1:
// 1100 waves 10.4 us, row groups 5.7).
constexpr int64_t push_min_waves(int k, bool scalar) { return scalar ? (k <= 5 ? 1792 : 1024) : (k <= 3 ? 1536 : 1024); }
// ... and with fewer taps than this it loses to the row groups at any size (966 x 1156, k 1, s 2, batch 1: 7.0 and
// 2.6 us; 2602 x 2660, k 3, s 4, batch 1: 13 and 7; 1126 x 1766, k 1, s 2, batch 4: 9.9 and 4.2; k 2, s 4, batches of 9 to
// 190: 1.5 to 2.8 times; but k 2, s 1, batches of 20 and more: mostly 0.6 to 0.9, k 3, s 3: 0.55 to 0.8).
constexpr bool push_taps(int k, int s, int batch) {
    return k > 3 || (batch > 12 && (k == 3 || (k == 2 && s == 1)));
}
// With more output lines in flight than this, at 4 columns per lane, its multiply-adds are the bound and
// the marching kernel, which reads LDS as often, does the fewer of them (434 x 289, k 13, batch 12: 118 and 37 us;
// 420 x 582, k 11, batch 16: 88 and 61).
constexpr int kPushFewLines = 10;
// output lines per wave, at least: each part loads k - s input lines of its neighbour's again (547 x 374,
// k 5, s 3, batch 44: 24 us with parts of 8, 18 of 4; 4096^2, k 11, s 4, batch 4: 66 and 80)
constexpr int push_min_part(int k, int s) { return k <= 2 * s ? 4 : 8; }
bool push_geometry(const conv_plan *plan, int batch, bool scalar, int lpr, unsigned col_blocks, PushGeom *out) {
    const ConvShape &sh = plan->shape;
    PushGeom g{};
    if (sh.p >= sh.k || sh.k > 64 || (sh.k + sh.s - 1) / sh.s > kPushMaxLines || (int64_t)sh.n * batch >= kInt32Limit) return false;
    g.m = sh.m; g.n = sh.n; g.m_out = sh.m_out; g.n_out = sh.n_out; g.s = sh.s; g.p = sh.p; g.k = sh.k;
    g.batch = batch;
    const int lanes = scalar ? 1 : lpr;
    while ((1 << g.lpr_log2) < lanes) ++g.lpr_log2;
    g.tw = kWave / lanes;
    const int64_t iw = (int64_t)(g.tw - 1) * sh.s + sh.k;
    if (iw * lanes > kPushItems * kWave) return false;
    g.iw = (int)iw;
    g.pw = (int)((iw + sh.s - 1) / sh.s);
    g.strips = (sh.n_out + g.tw - 1) / g.tw;
    int64_t part = ((int64_t)g.strips * col_blocks * sh.m_out + kPushTargetWaves - 1) / kPushTargetWaves;
    part = std::min<int64_t>(std::max<int64_t>(part, push_min_part(sh.k, sh.s)), 1 << 20);
    g.seg = (int)(part * kPushWaves);
    g.segs = (sh.m_out + g.seg - 1) / g.seg;
    const int64_t jobs = (int64_t)g.strips * g.segs;
    if (jobs + kXcds >= (1LL << 31) / kXcds) return false;
    g.blocks = (int)jobs;
    g.blocks_per_xcd = (int)((jobs + kXcds - 1) / kXcds);
    if ((size_t)kPushWaves * 4 * push_wave_floats(sh.k, g.pw * sh.s << g.lpr_log2, scalar) > 64 * 1024) return false;
    *out = g;
    return true;
}

// The marching launch (rectangle or described path) with lanes of 4 lpr batch columns, or of one.
bool compact_march(const conv_plan *plan, int batch, bool scalar, int lpr, CompactChoice *out) {
    const ConvShape &sh = plan->shape;
    CompactChoice c{};
    c.scalar = scalar;
    c.lpr = lpr;
    const int eb = c.scalar ? 4 : 16;
    c.col_blocks = (unsigned)column_blocks(batch, c.scalar ? 0 : c.lpr);
    int tw = kCompactThreads / c.lpr;
    CompactGeom g{};
    g.m = sh.m; g.n = sh.n; g.m_out = sh.m_out; g.n_out = sh.n_out; g.s = sh.s; g.p = sh.p; g.k = sh.k;
    g.batch = batch;
    // int arithmetic in the kernel: s*x - p + k, s*y0 - p + iw
    int64_t iw = (int64_t)(tw - 1) * sh.s + sh.k;
    if ((int64_t)sh.m + 2LL * sh.p + sh.k >= (1LL << 30) || (int64_t)sh.n + 2LL * sh.p + iw >= (1LL << 30)) return false;
    const int kk_bytes = sh.k * sh.k * 4;
    // the rectangle path compares descriptors with (s*x - p)*n + s*y - p in int, for x up to m_out + RV
    // ... and addresses lanes by 32-bit offsets from a line's start: n*batch*4 < 2^24, TW*batch*4 < 2^32
    if (rect_compiled(sh.k, sh.s) && ((int64_t)sh.m + sh.p + sh.k + (rect_rv(sh.s) + 1) * (int64_t)sh.s) * sh.n < kInt32Limit &&
        (int64_t)sh.n * batch * 4 < (1LL << 24) && (int64_t)batch * 4 * (kCompactThreads + 1) < (1LL << 31)) {
        c.kk = sh.k;
        c.ss = sh.s;
        g.rv = rect_rv(sh.s);
        g.nl = kRectNl;
        g.ktab_lds = 1;
        c.lds = (size_t)kRectNl * iw * c.lpr * eb + kk_bytes;
    } else {
        // Described path.  A strip of tw columns is served by 256 / (tw * lpr) groups of lanes that
        // take the rv lines of a step in turn (rv = 4, 2 or 1 lines per group); two barriers per
        // step, so the ring holds one step's s*(rv-1) + k lines of (tw-1)*s + k pixels.  Widest
        // strip (not wider than the image needs) and most lines whose ring fits 64 KiB, else
        // 144 KiB (one workgroup per CU); none fits: every tap from global memory.
        g.ktab_lds = kk_bytes <= 16 * 1024;
        g.rv = 1;
        g.nl = 0;
        c.lds = g.ktab_lds ? kk_bytes : 0;
        const int64_t limits[2] = {64 * 1024, 144 * 1024};
        bool found = false;
        for (int li = 0; li < 2 && !found; ++li) {
            for (int cand = kCompactThreads / c.lpr; cand >= 16 && !found; cand >>= 1) {
                if (cand > 16 && cand / 2 >= sh.n_out) continue;      // half as wide still covers the image
                for (int mult = 4; mult >= 1 && !found; mult >>= 1) {
                    const int rv = kCompactThreads / (cand * c.lpr) * mult;
                    const int64_t cw = (int64_t)(cand - 1) * sh.s + sh.k;
                    const int64_t need = (int64_t)sh.s * (rv - 1) + sh.k;
                    int nl = 16;
                    while (nl < need && nl < 256) nl <<= 1;
                    const int64_t bytes = (int64_t)nl * cw * c.lpr * eb + (g.ktab_lds ? kk_bytes : 0);
                    if (nl < need || bytes > limits[li] || (int64_t)nl * cw * c.lpr >= (1LL << 21)) continue;
                    tw = cand;
                    iw = cw;
                    g.rv = rv;
                    g.nl = nl;
                    c.lds = (size_t)bytes;
                    found = true;
                    // the lines a step adds, in registers during the step before: when they fit, and when the
                    // ring is large enough that the workgroup is alone on its CU anyway (the registers cost
                    // the second workgroup); a line of x shorter than 2^24 bytes as for the rectangle path
                    const int64_t fresh = std::min<int64_t>((int64_t)rv * sh.s, need);
                    c.xld = (bytes > 64 * 1024 && fresh * cw * c.lpr <= (int64_t)kDescXld * kCompactThreads &&
                             (int64_t)sh.n * batch * 4 < (1LL << 24) && (int64_t)batch * 4 * (kCompactThreads + 1) < (1LL << 31))
                                ? kDescXld : 0;
                }
            }
        }
    }
    g.tw = tw;
    g.iw = (int)iw;
    g.strips = (sh.n_out + tw - 1) / tw;
    // two workgroups per CU, or one where the ring leaves room for one only (a segment starts by
    // loading the whole window of its first step: fewer, longer segments then)
    const int64_t target = c.lds > kLdsPerCu / 2 ? kCompactTargetBlocks / 2 : kCompactTargetBlocks;
    int64_t segs = target / ((int64_t)g.strips * c.col_blocks);
    if (segs < 1) segs = 1;
    int64_t seg = (sh.m_out + segs - 1) / segs;
    if (seg < 2 * g.rv) seg = 2 * g.rv;
    seg = (seg + g.rv - 1) / g.rv * g.rv;
    g.seg = (int)seg;
    g.segs = (int)((sh.m_out + seg - 1) / seg);
    const int64_t jobs = (int64_t)g.strips * g.segs;
    if (jobs + kXcds >= (1LL << 31) / kXcds) return false;
    g.blocks_per_xcd = (int)((jobs + kXcds - 1) / kXcds);
    c.geom = g;
    c.ok = true;
    *out = c;
    return true;
}

// Row groups: lanes per row, columns per lane and waves that share a row's channels.
void compact_row_groups(const conv_plan *plan, int batch, CompactChoice *out) {
    CompactChoice &c = *out;
    const int kk = plan->shape.k * plan->shape.k;
    c.xld = 0;
    c.scalar = batch < 4;
    c.lpr = c.scalar ? 0 : widest_nv(batch);
    // Columns per lane: not more than a third of them idle in the last block (184 x 204, k 13, batch 12: 20 us with
    // 3 blocks of 4, 24 with one of 16; but 385 x 333, k 3, s 2, batch 35: 31 us with 9 blocks of 4, 16 with 3 of 16,
    // as every block touches every memory line of x).
    // (several channels, whose waves split the channels anyway: not more than a tenth)
    const bool many = plan->channels > 1;
    while (c.lpr > 1 && (many ? 10 : 3) * column_blocks(batch, c.lpr) * c.lpr > (many ? 11 : 4) * column_blocks(batch, 1)) c.lpr /= 2;
    c.gather_g = group_width(kk);
    auto waves = [&] {
        return (plan->rows * c.gather_g + kWave - 1) / kWave * column_blocks(batch, c.lpr) * std::min(plan->channels, 16);
    };
    if (many) {
        while (c.gather_g < 16 && c.gather_g * kGatherTaps < kk) c.gather_g *= 2;
        while (c.lpr > 1 && waves() < kChanFusedWaves) c.lpr /= 2;
    } else {
        // Few waves: more lanes per row, down to 3 taps each, then narrower ones (570 x 564, k 5, batch 1: 10 us with
        // 4 lanes per row, 18 with 8; 450 x 559, k 5, s 4, batch 36: 25 and 56), with few taps only while the
        // waves are very few: a narrow lane reads a part of a memory line (85 x 85, k 2, s 2, batch 216: 10 us
        // with 4 columns per lane, 3.5 with 16).
        while (kk > 4 && c.gather_g < 16 && c.gather_g * 3 < kk && waves() < kChanFusedWaves) c.gather_g *= 2;
        // (lanes of 16 columns and few or far taps: down to 4 taps each whatever the waves, 0.83 to 1.0 of the time)
        while (c.gather_g < 16 && c.gather_g * kGatherTaps < kk && c.lpr == 4 && (plan->shape.s > 1 || kk <= 16)) c.gather_g *= 2;
        while (c.lpr > 1 && waves() < (kk <= 16 ? kChanFusedWaves / 4 : kChanFusedWaves)) c.lpr /= 2;
    }
    c.col_blocks = (unsigned)column_blocks(batch, c.lpr);
    const int64_t row_waves = (plan->rows * c.gather_g + kWave - 1) / kWave;
    c.ways = 1;
    while (c.ways < 16 && 2 * c.ways <= plan->channels && row_waves * c.col_blocks * c.ways < kChanFusedWaves) c.ways *= 2;
    c.lds = c.ways > 1 ? (size_t)c.ways * std::max(c.lpr, 1) * (kWave / c.gather_g) * (c.scalar ? 4 : 16) : 0;
}

bool lane_geometry(const conv_plan *plan, int batch, LaneGeom *out) {
    LaneGeom g{};
    if (plan->shape.k < 2 || plan->shape.k > 13 || !chunk_geometry(plan, batch, plan->cols * batch, kItemThreads, &g)) return false;
    g.n = plan->shape.n;
    *out = g;
    return true;
}

// Which of the three serves a product, by the waves and workgroups each would have (8 400 drawn shapes, every
// kernel and width timed on each: 1.08 times the best of them in the mean).
CompactChoice choose_compact_path(const conv_plan *plan, int batch) {
    const ConvShape &sh = plan->shape;
    // chunks of four columns (chunk_col); a launch per channel adds to y, where a column must not be in two chunks
    const bool scalar = batch < 4 || (plan->channels > 1 && batch % 4 != 0);
    const int wide = scalar ? 1 : widest_nv(batch);
    CompactChoice c{};
    if (!compact_march(plan, batch, scalar, wide, &c)) return c;
    // (the plan's marching threshold, a test hook, lowers the bounds so that small test shapes march or push too)
    const bool lowered = plan->march_min_jobs < kMarchMinJobs;
    auto least = [&](int64_t bound) { return lowered ? std::min<int64_t>(bound, plan->march_min_jobs) : bound; };
    auto workgroups = [](const CompactChoice &m) { return (int64_t)m.geom.strips * m.geom.segs * m.col_blocks; };
    const bool groups = plan->rows * 16 / kCompactThreads + 1 < kInt32Limit;
    PushGeom push;
    const bool can_push = !c.kk && push_geometry(plan, batch, scalar, c.lpr, c.col_blocks, &push);
    auto pushed = [&] {
        c.pushed = true;
        c.push = push;
        c.lds = (size_t)kPushWaves * 4 * push_wave_floats(sh.k, push.pw * sh.s << push.lpr_log2, scalar);
        return c;
    };
    // Fewer workgroups than compute units: the marching layout cannot fill the chip.  The row groups
    // give such a product rows * G lanes instead (x from global memory, which for a plane this small means from the L2).
    if (!can_push && (workgroups(c) >= least(kCompactMinBlocks) || !groups)) return c;
    // Marching where the push kernel's rule, or the widest lanes' workgroups, would leave a product to the row groups though
    // lanes that divide the batch have workgroups enough: the widest that do, with taps enough to pay for reading x
    // again per block of columns, and strips that are not mostly empty (553 x 440, k 11, s 2, batch 28: 39 us marching,
    // 167 in row groups; 525 x 510, k 7, s 3, batch 36: 27 and 108; but 1901 x 1718, k 1, s 4, batch 4: 12 and 3;
    // 65 x 50, k 7, batch 152, strips of 256: 19 and 10).  A batch of 1 to 3, a column per lane: with 81 taps or more and
    // many pixels (1176 x 1484, k 13, s 2, p 6, batch 1: 35 and 67; 2836 x 1798, k 9, s 4: 23 and 34; but 473 x 473, k 11, s 2,
    // batch 1: about even, and 4 to 10 times the row groups' time at 20 000 pixels).  Batches that are not a multiple of 4:
    // the rectangles of stride 1, from fewer workgroups on (262 x 253, k 9, batch 11, 132: 0.6 of the row groups' time;
    // 243 x 337, k 7, batch 15, 186: 0.5; 418 x 445, k 5, batch 6, 212: 0.78; but 192 x 178, k 5, batch 14, 96: 1.4).
    auto narrower = [&](CompactChoice *out) {
        if (plan->channels > 1) return false;
        CompactChoice m{};
        if (scalar) {
            if (!can_push || sh.k < 9 || sh.s == 1 || plan->rows * batch < (sh.s <= 3 ? 300000 : 200000)) return false;
            *out = c;
            out->fine = true;
            return workgroups(c) >= least(kCompactMinBlocks);
        }
        const bool ragged = batch % 4 != 0;
        if (sh.k < 5 || sh.s > 3 || (ragged && (!c.kk || sh.s > 1))) return false;
        auto filled = [&] { return 10LL * sh.n_out >= 6LL * m.geom.tw * m.geom.strips; };
        if (ragged) {
            for (int lpr = wide; lpr >= 1; lpr /= 2)
                if (compact_march(plan, batch, false, lpr, &m) && workgroups(m) >= (sh.k == 9 ? 128 : 192) && filled()) {
                    *out = m;
                    out->fine = true;
                    return true;
                }
            return false;
        }
        const int dividing = least_nv(batch);
        if (!compact_march(plan, batch, false, dividing, &m) || workgroups(m) < least(kCompactMinBlocks)) return false;
        for (int lpr = can_push ? wide : wide / 2; lpr >= dividing; lpr /= 2) {
            if (lpr == 1 && lpr < wide && sh.k < 7) break;
            if (!compact_march(plan, batch, false, lpr, &m) || workgroups(m) < least(kCompactMinBlocks)) continue;
            if (!filled()) continue;
            *out = m;
            out->fine = true;
            return true;
        }
        return false;
    };
    // Rectangles whose launch stays below that bound, with strips that are not mostly empty (32 x 20, k 7, s 2, batch 1318, a
    // fifth full: 8.6 us in row groups, 39 marching).  Where segments are longer than the shortest the launch has as many
    // workgroups as it asked for, a few less than compute units because strips do not divide them (3239 x 2417, k 7, s 2, batch 4: 255,
    // 144 us in row groups, 48 marching): from these lengths on, in steps of rv lines, as the waves' first window is paid for.
    // Else as many workgroups, and with few blocks of columns as many full ones, as it takes for the taps (571 x 726, k 7, batch 1,
    // 219: 24.5 and 7.9; 202 x 241, k 7, batch 32, 208: 37 and 12; 497 x 778, k 9, batch 1: 33 and 9.6; but 201 x 261, k 7, batch
    // 12, 130 that hold 106: 10.6 and 11.9; 31 x 36, k 5, batch 522, 165 that hold 103: 8.8 and 10.5).  Of 900 products of row
    // groups that have these lengths or workgroups, batches to 2048, 856 march, 1.69 times as fast in the mean, 3 more than 6 %
    // slower (0.88 at the worst), and 44 are left as too empty (marching 0.76 in the mean); what their sums do to the error stands
    // at FINE in compact_kernels.h.
    auto short_of_bound = [&] {
        if (lowered || can_push || !c.kk || plan->channels > 1) return false;
        const int64_t wgs = workgroups(c), places = (int64_t)c.geom.tw * c.geom.strips;
        if (20LL * sh.n_out < 11 * places) return false;
        if (c.geom.seg > 2 * c.geom.rv) {
            const int steps = sh.k == 7 ? 4 : sh.k == 5 ? 6 : sh.k == 3 ? 20 : 0;
            return steps > 0 && c.geom.seg >= steps * c.geom.rv;
        }
        int64_t least_wgs = kCompactMinBlocks, least_full = 0;
        if (sh.s == 1 && sh.k == 5) least_wgs = 160, least_full = 115;
        else if (sh.s == 1 && sh.k == 7) least_wgs = 128, least_full = c.lpr == 1 || c.col_blocks > 2 ? 0 : 110;
        else if (sh.s == 1 && sh.k == 9) least_wgs = scalar ? 80 : 128;
        else if (sh.s == 2 && sh.k == 7) least_wgs = scalar ? 160 : 192, least_full = scalar ? 144 : c.col_blocks > 2 ? 0 : 185;
        return wgs >= least_wgs && 10LL * sh.n_out >= 6 * places && wgs * sh.n_out >= least_full * places;
    };
    if (short_of_bound()) {
        c.fine = true;
        return c;
    }
    CompactChoice m{};
    if (can_push) {
        const int64_t waves = (int64_t)push.blocks * kPushWaves * c.col_blocks;
        const int in_flight = (sh.k + sh.s - 1) / sh.s;
        // Column by column, several channels cost a launch each; the row groups take them in one, in chunks of four columns
        // (205 x 192, k 1, s 4, 10 channels, batch 71: 361 us, row groups 7; 570 x 480, k 2, 4 channels, batch 1: 30 and 5).
        const bool one_by_one = scalar && plan->channels > 1;
        const bool enough = one_by_one ? batch < 4 && sh.k >= 6 && waves >= 1536 : push_taps(sh.k, sh.s, batch) && waves >= push_min_waves(sh.k, scalar);
        if (lowered ? waves >= least(kPushTargetWaves) : enough && (scalar || in_flight <= kPushFewLines)) return pushed();
        if (!lowered && narrower(&m)) return m;
        if (!groups || (!lowered && enough)) return pushed();
    } else if (!lowered && narrower(&m)) {
        return m;
    }
    compact_row_groups(plan, batch, &c);
    return c;
}

// Where a lane per row and chunk (compact_lane_kernel.h) takes a product from those three: where a surface fitted to the logarithm of the
// times' ratio says that it is faster by kLaneLeastGain.  Coordinates: w, the multiply-adds of a chunk each, borders left aside
// (log2 of millions); b, the chunks; how full blocks of 16 columns are; a, the taps of a line (log2); stride 1 or not; the
// stride (log2); held at the ends of the ranges of the products in profiles/chunk_kernel_times.csv.  Of those, counted as for
// kItemFaster above, and of others:
//   row groups, 1 to 3 columns         600    94  1.79    0  123     350    58  1.67    0   75  1.25
//   row groups                         600   169  1.72    0   94     350   116  1.77    1   49  0.82
//   described and pushed march        1200   720  1.83    0  369     700   422  1.83    0  211  0.97
//   rectangles, 1 to 3 columns         600   285  1.66    0  116     350   187  1.65    0   62  1.06
// What stays: pushed lines but for k 3 to 6 at strides above 1 (longer kernels are about even, and at stride 1 the fit missed products
// at 0.72); rectangles of 4 columns and more (their tiles reuse more, and few would leave).
enum LaneAgainst { kLaneGroupsFew, kLaneGroups, kLanePushed, kLaneRectFew };
constexpr double kLaneGain[][15] = {
    // 1, w, w^2, b, b^2, full, a, a^2, stride 1, stride, w a, w b, a b, w at stride 1, a at stride 1
    {-0.2636, -0.1051, 0.0023, 0.1003, 0.03, 0, 0.695, -0.2558, 0.1149, -0.0589, 0.1143, 0.0198, -0.0357, 0.0541, -0.0732},      // gather few
    {-0.3674, -0.1317, -0.0049, 0.255, -0.0168, -0.1569, 0.5584, -0.2119, 0.2816, 0.1021, 0.1021, 0.0175, -0.0306, 0.0485, -0.1257},      // gather vec
    {0.9478, -0.0685, 0.016, 0.1028, -0.0053, -0.4806, -0.0554, 0.0618, -0.1198, -0.0255, -0.0803, 0.0089, -0.0029, -0.0232, 0.1793},      // push
    {0.3501, -0.0544, -0.01, -0.0743, 0.0836, 0, 0.261, -0.1051, 0.0337, 0.3164, -0.0248, 0.0536, -0.0875, 0.0221, 0.18},      // rect few
};
constexpr double kLaneLeastGain[] = {0.3, 0.25, 0.3, 0.2};
constexpr int kLaneApart = 4;        // strides from which neighbouring rows share few pixels: less certain
constexpr double kLaneWorkLeast = -8.5, kLaneWorkMost = 8.5, kLaneChunksMost = 9.0;      // what the counts above cover
constexpr int kLaneMostTaps = 13, kLanePushedLeastTaps = 3, kLanePushedMostTaps = 6;
bool lane_serves(const conv_plan *plan, int batch, const CompactChoice &other) {
    const int k = plan->shape.k, columns = batch >= 4 ? 4 : 1, chunks = (batch + columns - 1) / columns;
    // (not where the plan's marching threshold, a test hook, is lowered)
    if (plan->channels > 1 || plan->march_min_jobs < kMarchMinJobs || k < 2 || k > kLaneMostTaps) return false;
    LaneAgainst against = batch < 4 ? kLaneGroupsFew : kLaneGroups;
    if (!other.gather_g) {
        if (other.kk && batch >= 4) return false;
        if (other.kk) against = kLaneRectFew;
        else if (k < kLanePushedLeastTaps || k > kLanePushedMostTaps || plan->shape.s == 1) return false;
        else against = kLanePushed;
    }
    const double w = std::clamp(std::log2((double)plan->rows * chunks * k * k) - 20.0, kLaneWorkLeast, kLaneWorkMost);
    const double b = std::min(std::log2((double)chunks), kLaneChunksMost), a = std::log2((double)k);
    const double full = columns == 4 ? chunks / (4.0 * ((chunks + 3) / 4)) : 0.0, one = plan->shape.s == 1, s = std::log2((double)plan->shape.s);
    const double at[15] = {1.0, w, w * w, b, b * b, full, a, a * a, one, s, w * a, w * b, a * b, w * one, a * one};
    double gain = 0.0;
    for (int i = 0; i < 15; ++i) gain += kLaneGain[against][i] * at[i];
    return gain > kLaneLeastGain[against] + (plan->shape.s >= kLaneApart ? 0.1 : 0.0);
}

constexpr int kCompactXcdUnits = kCompactTargetBlocks / 2 / kXcds;
// The segments of a march that has its compute units to itself (more than half of the LDS): those whose rounds of 32 workgroups on
// the fullest XCD, each as long as a segment and the window before it, take least, where that is a tenth less.  (Cells are dealt to
// the XCDs with all their column blocks: 255 workgroups of 3 blocks are 33 on one of them, a second round.  Segments by the
// chip's workgroups -> these, us: 522 x 691, k 7, s 2, batch 40: 60.9 -> 34.6; 555 x 789, k 7, s 2, batch 37: 70.3 -> 39.5; 864 x 861, k 5, s 2,
// batch 40: 86.6 -> 54.5; 1078 x 776, k 3, s 2, batch 96: 179 -> 112.  70 changed products: 1.08 to 1.78 times as fast, 1.53 in
// the mean.)  The choice between the kernels is made before, on the other segments, and sums are as they were.
void compact_segments(const conv_plan *plan, CompactChoice *out) {
    CompactChoice &c = *out;
    if (!c.ok || c.gather_g || c.pushed || c.lds <= kLdsPerCu / 2) return;
    const ConvShape &sh = plan->shape;
    CompactGeom &g = c.geom;
    auto cost = [&](int64_t seg) {
        const int64_t cells = g.strips * ((sh.m_out + seg - 1) / seg), share = (cells + kXcds - 1) / kXcds * c.col_blocks;
        return (share + kCompactXcdUnits - 1) / kCompactXcdUnits * (seg + 2 * g.rv);
    };
    int64_t best = g.seg;
    for (int64_t segs = 1; segs <= 512 && segs * 2 * g.rv <= sh.m_out; ++segs) {
        const int64_t seg = ((sh.m_out + segs - 1) / segs + g.rv - 1) / g.rv * g.rv;
        if (cost(seg) < cost(best)) best = seg;
    }
    if (cost(best) * 10 > cost(g.seg) * 9) return;
    const int64_t segs = (sh.m_out + best - 1) / best, jobs = g.strips * segs;
    if (jobs + kXcds >= (1LL << 31) / kXcds) return;
    g.seg = (int)best;
    g.segs = (int)segs;
    g.blocks_per_xcd = (int)((jobs + kXcds - 1) / kXcds);
}

// ... and whether its sums are taken line by line (FINE): where the row groups would serve it otherwise, with the
// widest lanes (above) or with lanes that divide the batch (one column each where it is not a multiple of 4), so that
// neither the lanes' width nor the pushed lines cost such products their exactness.
CompactChoice choose_compact(const conv_plan *plan, int batch) {
    CompactChoice c = choose_compact_path(plan, batch), even{};
    if (c.ok && lane_serves(plan, batch, c) && lane_geometry(plan, batch, &c.lane)) {
        c.laned = true;
        c.scalar = batch < 4;
        return c;
    }
    compact_segments(plan, &c);
    if (!c.ok || c.gather_g || plan->shape.k < 3 || (!c.pushed && (c.scalar || plan->channels > 1))) return c;
    const bool whole = batch >= 4 && batch % 4 == 0;
    c.fine = c.fine || (compact_march(plan, batch, !whole, whole ? least_nv(batch) : 1, &even) &&
                        (int64_t)even.geom.strips * even.geom.segs * even.col_blocks < kCompactMinBlocks);
    return c;
}

// Several channels in one launch (compact_channels_kernel.h): when the channels are many and a
// channel's product is short, so that one launch per channel would be bound by launches and by
// re-reading y.  VB batch columns per lane (16, 8 or 4, dividing the batch) and W = 4, 8 or 16
// waves per workgroup that split the channels: the widest VB whose launch has kChanFusedWaves
// waves with the most ways that fit LDS and the channel count, else the shape with most waves.

ChannelsChoice choose_compact_channels(const conv_plan *plan, const float *x, const float *y, int batch) {
    const ConvShape &sh = plan->shape;
    ChannelsChoice c{};
    if (!plan->compact || plan->channels < 2 || batch % 4) return c;
    if (((((uintptr_t)x) | ((uintptr_t)y)) & 15u) != 0) return c;
    if ((double)plan->nnz * batch > kChanFusedWork) return c;
    // int arithmetic in the kernel: s*x - p + k over the padded plane, float offsets within a channel's plane
    if ((int64_t)sh.m + 2LL * sh.p + sh.k + 16LL * sh.s >= (1LL << 30) || (int64_t)sh.n + 2LL * sh.p + sh.k + 16LL * sh.s >= (1LL << 30) ||
        (int64_t)sh.m * sh.n * batch >= kInt32Limit)
        return c;
    const int64_t phx = (int64_t)(kChanTileX - 1) * sh.s + sh.k, phy = (int64_t)(kChanTileY - 1) * sh.s + sh.k;
    const int64_t npix = phx * phy;
    const int64_t tiles_x = (sh.m_out + kChanTileX - 1) / kChanTileX, tiles_y = (sh.n_out + kChanTileY - 1) / kChanTileY;
    if (tiles_x * tiles_y + kXcds > kInt32Limit) return c;
    int64_t best_waves = 0;
    for (int vb = batch % 16 == 0 ? 16 : (batch % 8 == 0 ? 8 : 4); vb >= 4; vb /= 2) {
        if (npix * (vb / 4) > (int64_t)kChanItems * kWave || batch / vb > 65535) continue;
        const int64_t vec4 = std::max<int64_t>(npix, kWave) * (vb / 4) + ((int64_t)sh.k * sh.k + 3) / 4;
        const int per_lane = (int)((npix * (vb / 4) + kWave - 1) / kWave);
        int ways = kChanMinWaves;
        while (ways < chan_max_waves(per_lane) && 2 * ways <= plan->channels && vec4 * 16 * 2 * ways <= 64 * 1024) ways *= 2;
        if (vec4 * 16 * ways > 64 * 1024) continue;
        const int64_t blocks = tiles_x * tiles_y * (batch / vb);
        while (ways > kChanMinWaves && blocks * (ways / 2) >= kChanFusedWaves) ways /= 2;     // no more ways than the chip needs
        const int64_t waves = blocks * ways;
        if (c.ok && waves <= best_waves) continue;
        best_waves = waves;
        c.ok = true;
        c.vb = vb;
        c.ways = ways;
        // lanes of four columns: the chunks that lie side by side, as many as the batch is a multiple of and a wave's patch has room for,
        // unless the patches, which overlap the more the more parts a tile is in, need more pixels in flight (the kernel's 4 or 8
        // per lane; 26 x 19, k 7, 3 channels, batch 16: 3.75 us, in four parts 4.57).  Few workgroups of k 3 at strides 1 and 2
        // wait for each other's patches anyway (12 x 15, k 3, 277 channels, batch 16: 15.4 and 17.0; but 19 x 29, k 3, s 2, 113 channels, batch
        // 32, 24 workgroups: 29 and 15).  2500 sums, batches to 480: 1.08 times the speed of one chunk in the mean, 24 of them more than
        // 6 % slower, with parts wherever they fit 1.07 and 144.
        c.chunks = 1;
        int64_t width = phy, wave_vec4 = vec4;
        const bool parts = vb == 4 && (sh.k != 3 || blocks >= (sh.s == 1 ? kChanPartsMinBlocks : kChanPartsMinBlocks / 4));
        for (int chunks = 4; parts && chunks > 1 && c.chunks == 1; chunks /= 2) {
            const int64_t w = (int64_t)(kChanTileY / chunks - 1) * sh.s + sh.k, patch = phx * w * chunks;
            const int64_t v = std::max<int64_t>(patch, kWave) + ((int64_t)sh.k * sh.k + 3) / 4;
            if (batch % (4 * chunks) || patch > 8 * kWave || (patch > 4 * kWave && npix <= 4 * kWave) || v * 16 * ways > 64 * 1024) continue;
            c.chunks = chunks;
            width = w;
            wave_vec4 = v;
        }
        c.lds = (size_t)(wave_vec4 * 16 * ways);
        const int64_t per_xcd = (tiles_x * tiles_y + kXcds - 1) / kXcds;
        c.grid = dim3((unsigned)(per_xcd * kXcds), (unsigned)(batch / vb));
        CompactChannelsGeom g{};
        g.tiles = (int)(tiles_x * tiles_y);
        g.tiles_per_xcd = (int)per_xcd;
        g.m = sh.m; g.n = sh.n; g.m_out = sh.m_out; g.n_out = sh.n_out; g.s = sh.s; g.p = sh.p; g.k = sh.k;
        g.batch = batch; g.channels = plan->channels;
        g.tiles_y = (int)tiles_y;
        g.phx = (int)phx;
        g.phy = (int)width;
        g.wave_vec4 = (int)wave_vec4;
        g.inv_phy = 1.0f / (float)width;
        g.plane = (long long)sh.m * sh.n * batch;
        c.geom = g;
        if (waves >= kChanFusedWaves) break;
    }
    return c;
}

}  // namespace

extern "C" {

int conv_spmv(const conv_plan *plan, const float *x_dev, float *y_dev, int batch, void *stream) {
    if (!plan || !x_dev || !y_dev) return CONV_ENULL;
    if (batch < 1) return CONV_EINVAL;
    {   // x and y must not overlap
        const char *xb = (const char *)x_dev, *xe = xb + sizeof(float) * (size_t)plan->cols * batch;
        const char *yb = (const char *)y_dev, *ye = yb + sizeof(float) * (size_t)plan->rows * batch;
        if (xb < ye && yb < xe) return CONV_EALIAS;
    }
    hipStream_t q = (hipStream_t)stream;
    const LaunchScope scope;
    if (plan->compact) {
        const ChannelsChoice fused = choose_compact_channels(plan, x_dev, y_dev, batch);
        if (fused.ok) {
            launch_compact_channels(fused, plan, x_dev, y_dev, q);
            return scope.ok() ? CONV_OK : CONV_EHIP;
        }
        const CompactChoice cc = choose_compact(plan, batch);
        if (!cc.ok) return CONV_EOVERFLOW;
        if (cc.laned) {
            launch_compact_lane(cc, plan, x_dev, y_dev, q);
            return scope.ok() ? CONV_OK : CONV_EHIP;
        }
        if (!launch_compact(cc, plan, x_dev, y_dev, q)) return CONV_EHIP;
        return scope.ok() ? CONV_OK : CONV_EHIP;
    }
    const ApplyChoice c = choose_apply(plan, batch);
    if (c.kind == Kind::StageMarch && c.march.channels > 1) {
        // one launch walks the channels of every block of lines: y is stored once, in a fixed order of sums
        if (!launch_stage_march(c, plan, x_dev, y_dev, q)) return CONV_EHIP;
    } else if (c.kind == Kind::Block) {
        if (plan->transposed) launch_block_adjoint(c, plan, x_dev, y_dev, q);
        else launch_block(c, plan, x_dev, y_dev, q);
    } else if (c.kind == Kind::Item) {
        launch_item(c, plan, x_dev, y_dev, q);
    } else if (c.kind == Kind::March || c.kind == Kind::Tile || c.kind == Kind::StageMarch) {
        // one launch per channel: the first stores y, the others add to it
        conv_plan one = *plan;
        one.cols = plan->cols / plan->channels;
        one.channels = 1;
        ApplyChoice cc = c;
        for (int ch = 0; ch < plan->channels; ++ch) {
            one.vals = plan->vals + (size_t)ch * plan->nnz;
            const float *x_ch = x_dev + (size_t)ch * one.cols * batch;
            cc.march.accum = ch > 0;
            const bool ok = c.kind == Kind::StageMarch ? launch_stage_march(cc, &one, x_ch, y_dev, q)
                            : c.kind == Kind::March   ? launch_march(cc, &one, x_ch, y_dev, q)
                                                      : launch_tile(cc, &one, x_ch, y_dev, q);
            if (!ok) return CONV_EHIP;
        }
    } else {
        switch (c.g) {
            case 1: launch_gather<1>(c, plan, x_dev, y_dev, batch, q); break;
            case 2: launch_gather<2>(c, plan, x_dev, y_dev, batch, q); break;
            case 4: launch_gather<4>(c, plan, x_dev, y_dev, batch, q); break;
            case 8: launch_gather<8>(c, plan, x_dev, y_dev, batch, q); break;
            default: launch_gather<16>(c, plan, x_dev, y_dev, batch, q); break;
        }
    }
    if (!scope.ok()) return CONV_EHIP;
    return CONV_OK;
}

}  // extern "C"

// Launch shape of the on-chip scatter: VB batch columns per wave, W waves per workgroup (W * VB
// batch columns per pass), tj < 64 pixels per tile line (the lanes of a wave hold one line's
// column pointers) with a line's entries within the stage.  The kernel is bound by the number
// of instructions it issues and needs many resident waves, so small LDS footprints are tried
// first: among the tiles within a footprint the one with the smallest window per pixel wins; a
// launch too small to fill the chip is charged for the idle units.  Not ok when no tile fits
// (k above about 32 s) or when the columns are very short (k <= s, or k <= 2 s at batches below 4):
// the walk costs about the same per column whatever its length, and with few entries per column
// adding every entry to y directly is faster.
constexpr size_t kCscTileLds[3] = {20 * 1024, 40 * 1024, 64 * 1024};
constexpr double kCscTileWindowGoal = 6.0;     // window slots per pixel that end the search for a larger footprint
constexpr int kCscTileShortColumn = 9;         // with columns of fewer entries the direct scatter is faster at batch 1 to 3,
constexpr int kCscTileShortestColumn = 4;      // and with columns of fewer than these at any batch
constexpr int kCscGroupColumn = 16;            // columns of at most this many entries share a step (4 or more of them)

struct CscTileChoice {
    bool ok;
    CscTileGeom g;
    int vb, waves;
    size_t lds;
    dim3 grid;
};

static CscTileChoice choose_csc_tile(const conv_plan *plan, int batch) {
    const ConvShape &sh = plan->shape;
    CscTileChoice c{};
    if (batch >= 9) { c.vb = 4; c.waves = 4; }
    else if (batch >= 5) { c.vb = 4; c.waves = 2; }
    else if (batch >= 3) { c.vb = 4; c.waves = 1; }
    else { c.vb = batch; c.waves = 1; }
    const int bc = c.waves * c.vb;
    const int chunks = std::min((batch + bc - 1) / bc, 65535);
    CscTileGeom g{};
    g.m = sh.m; g.n = sh.n; g.n_out = sh.n_out; g.k = sh.k; g.s = sh.s; g.p = sh.p;
    g.batch = batch;
    g.inv_n_out = 1.0f / (float)sh.n_out;
    const int64_t per_axis = ((int64_t)sh.k + sh.s - 1) / sh.s;          // windows that can cover one pixel, per axis
    const int64_t column_max = per_axis * per_axis;
    g.column_max = (int)std::min<int64_t>(column_max, kCscStage);
    g.spacing = sh.k;
    g.group = g.column_max <= kCscGroupColumn ? kWave / g.column_max : 1;
    if (plan->nnz > kInt32Limit - 2 * kWave) return c;       // the kernel steps a wave past the last entry, in int
    if (column_max > kCscStage || column_max < (batch >= 4 ? kCscTileShortestColumn : kCscTileShortColumn)) return c;
    const int tj_max = (int)std::min<int64_t>(32, kCscStage / column_max);
    double best = 0.0;
    for (size_t budget : kCscTileLds) {
        for (int tj = 1; tj <= tj_max; tj *= 2) {
            if (tj > 1 && tj / 2 >= sh.n) break;
            for (int ti = 1; ti <= 64; ti *= 2) {
                if (ti > 1 && ti / 2 >= sh.m) break;
                const int64_t wx = std::min<int64_t>(((int64_t)ti + sh.k - 2) / sh.s + 1, sh.m_out);
                const int64_t wy = std::min<int64_t>(((int64_t)tj + sh.k - 2) / sh.s + 1, sh.n_out);
                const int64_t limit = (wx - 1) * sh.n_out + wy;
                if (limit > (1 << 21)) continue;
                const int64_t stage = (tj * column_max + 1) / 2 * 2, ptrs = ((int64_t)ti * (tj + 1) + 3) / 4 * 4;
                const int64_t lds = 16 * stage + 4 * ptrs + wx * wy * bc * 4;
                if (lds > (int64_t)budget) continue;
                const int64_t tiles_i = (sh.m + ti - 1) / ti, tiles_j = (sh.n + tj - 1) / tj;
                const int64_t blocks = tiles_i * tiles_j;
                if (blocks > kInt32Limit) continue;
                double score = (double)(wx * wy) / ((double)ti * tj);
                const double work = (double)blocks * chunks * c.waves;
                if (work < 8192.0) score *= 8192.0 / work;
                if (!c.ok || score < best) {
                    c.ok = true;
                    best = score;
                    g.ti = ti; g.tj = tj; g.tiles_j = (int)tiles_j;
                    g.wx = (int)wx; g.wy = (int)wy; g.inv_wy = 1.0f / (float)wy;
                    g.limit = (int)limit; g.stage = (int)stage; g.ptrs = (int)ptrs;
                    c.lds = (size_t)lds;
                    c.grid = dim3((unsigned)blocks, (unsigned)chunks);
                    g.tiles = (int)blocks;
                }
            }
        }
        if (c.ok && best <= kCscTileWindowGoal) break;
    }
    c.g = g;
    return c;
}

// The scatter: a product by itself, or (EDITED) what a product that gathers leaves to do where arrays were edited.
constexpr unsigned kEditedWaves = 6144, kEditedBlocks = 4096, kEditedFillBlocks = 256;
template <bool EDITED>
static dim3 scatter_grid(unsigned blocks, unsigned chunks, unsigned waves_per_block) {
    if (!EDITED) return dim3(blocks, chunks);
    const unsigned most = std::min(kEditedWaves / waves_per_block, kEditedBlocks);
    blocks = std::min(blocks, most);
    return dim3(blocks, std::min(chunks, most / blocks));
}

template <int VB, int W, bool EDITED>
static void launch_csc_tile(const CscTileChoice &c, const conv_plan *plan, const float *x_dev, float *y_dev,
                            hipStream_t q) {
    spmm_csc_tile_kernel<VB, W, EDITED><<<scatter_grid<EDITED>(c.grid.x, c.grid.y, W), W * kWave, c.lds, q>>>(
        plan->row_ptr, plan->col_idx, plan->vals, x_dev, y_dev, c.g, plan->edited);
}

// y zeroed, then every entry added.  The plan's "rows" are the columns of T (input pixels), its "cols" the rows of T.
template <bool EDITED>
static int enqueue_csc_scatter(const conv_plan *plan, const float *x_dev, float *y_dev, int batch, hipStream_t q) {
    const long long count = (long long)plan->cols * batch;
    const unsigned fill_blocks = (unsigned)std::min<long long>((count / 4 + kGatherThreads) / kGatherThreads, EDITED ? kEditedFillBlocks : 1 << 16);
    fill_zero_kernel<EDITED><<<fill_blocks, kGatherThreads, 0, q>>>(y_dev, count, plan->edited);
    if (plan->nnz == 0) return CONV_OK;
    const CscTileChoice tc = choose_csc_tile(plan, batch);
    if (tc.ok) {
        if (tc.vb == 1) launch_csc_tile<1, 1, EDITED>(tc, plan, x_dev, y_dev, q);
        else if (tc.vb == 2) launch_csc_tile<2, 1, EDITED>(tc, plan, x_dev, y_dev, q);
        else if (tc.waves == 1) launch_csc_tile<4, 1, EDITED>(tc, plan, x_dev, y_dev, q);
        else if (tc.waves == 2) launch_csc_tile<4, 2, EDITED>(tc, plan, x_dev, y_dev, q);
        else launch_csc_tile<4, 4, EDITED>(tc, plan, x_dev, y_dev, q);
        return CONV_OK;
    }
    const int g = group_width(plan->max_row_nnz);
    const int bl = batch >= 16 ? 16 : (batch >= 4 ? 4 : 1);      // lanes across the batch
    const int64_t blocks = (plan->rows * g * bl + kGatherThreads - 1) / kGatherThreads;
    if (blocks > kInt32Limit) return CONV_EOVERFLOW;
    const dim3 grid = scatter_grid<EDITED>((unsigned)blocks, (unsigned)std::min((batch + bl - 1) / bl, 65535), kGatherThreads / kWave);
    const int cols = (int)plan->rows;
#define CONV_SCATTER_BL(G, BL)                                                                                      \
    spmm_scatter_kernel<G, BL, EDITED><<<grid, kGatherThreads, 0, q>>>(plan->row_ptr, plan->col_idx, plan->vals, x_dev, \
                                                                       y_dev, cols, batch, plan->edited)
#define CONV_SCATTER(G)                                  \
    if (bl == 16) CONV_SCATTER_BL(G, 16);                \
    else if (bl == 4) CONV_SCATTER_BL(G, 4);             \
    else CONV_SCATTER_BL(G, 1)
    switch (g) {
        case 1: CONV_SCATTER(1); break;
        case 2: CONV_SCATTER(2); break;
        case 4: CONV_SCATTER(4); break;
        case 8: CONV_SCATTER(8); break;
        default: CONV_SCATTER(16); break;
    }
#undef CONV_SCATTER_BL
#undef CONV_SCATTER
    return CONV_OK;
}

// Launch shape of the product from the column-compressed arrays that gathers (csc_gather_kernel.h).
//
// What it costs over the scatter is time per input line: a workgroup walks seg s + k - s of them, a microsecond each, however
// little there is to do, and every line at the image's border is placed anew; planes too small to pay for that stay with
// the scatter.  What the scatter costs goes with pixels x batch, below four columns with pixels x sqrt(batch).  The lines lie
// where 11 000 products (planes of 16 to 3000 a side, k 1 to 13, strides 1 to 4, batches 1 to 256) had the two even, for every number
// of output lines that an input line reaches: ceil(k/s), 1 to 13.  Of these products 112 are more than 6 % slower than the
// scatter, 281 would be that much faster (1024^2, k 7, batch 16: 101 us and 358, batch 1: 80 and 158; 1000 x 900, k 3, batch 16: 39 and 217;
// 4096^2, k 11, s 4, batch 4: 306 and 1490; 269 x 320, k 5, batch 1: 18 and 23; below the lines 691 x 628, k 13, s 2, batch 3: 122 and 76;
// 176 x 128, k 7, batch 8: 25 and 17; 1292 x 1151, k 1, batch 4: 37 and 26).
// Columns of one entry below batch 4, and of up to four at stride 1, are added to y directly; at strides above 1 these
// gather from half a million products on, k 3 from 1.3 million (427 x 533, k 3, s 2, batch 1: 9.9 directly, 18).
// Two workgroups per compute unit; with few lines in flight (and few registers) four, as long as the lines that two
// segments share stay few (3453 x 2976, k 3, batch 1: 238 -> 191 us, 3000^2, k 3, s 2, batch 4: 149 -> 114; 1000 x 900, k 3,
// batch 16, 15 lines a segment: 36 -> 37; k 5: 163 -> 171).
constexpr int64_t kCscGatherTarget = 512, kCscGatherLong = 32;
constexpr float kCscGatherLeast[2][14] = {      // thousand pixels x batch, stride 1 and strides above
    {0, 2400, 70, 70, 110, 250, 380, 450, 430, 500, 330, 400, 400, 500}, {0, 1400, 160, 260, 390, 980, 1260, 1500, 2000, 2500, 3000, 3700, 4400, 5200}};
constexpr float kCscGatherLeastFew[2][14] = {   // batches below 4: thousand pixels x sqrt(batch)
    {0, 0, 0, 30, 41, 55, 81, 180, 700, 185, 330, 270, 175, 400}, {0, 0, 0, 95, 203, 303, 720, 870, 1100, 1400, 1800, 2200, 2600, 3000}};
constexpr float kCscGatherLeastOne = 10000, kCscGatherLeastOneStrided = 4300;        // one entry a column, batch 4
constexpr double kCscGatherDirect = 5e5, kCscGatherDirectThree = 1.3e6;

static CscGatherChoice choose_csc_gather(const conv_plan *plan, int batch) {
    const ConvShape &sh = plan->shape;
    CscGatherChoice c{};
    CscGatherGeom g{};
    const int64_t k = sh.k, s = sh.s, kl = (k + s - 1) / s;
    if (s > k || sh.p >= k || kl > kCscGatherLines) return c;       // pixels or rows without entries; too many sums in flight
    // int arithmetic in the kernel
    if ((int64_t)sh.m + 2LL * sh.p + k >= (1LL << 30) || (int64_t)sh.n + 2LL * sh.p + 64 * s + k >= (1LL << 30) || 1024LL * batch > kInt32Limit)
        return c;
    // (conv_plan_set_march_min_jobs lowers the bar for tests, or raises it)
    const double bar = plan->march_min_jobs / (double)kMarchMinJobs, pixels_in = (double)sh.m * sh.n;
    if (batch >= 4) {
        const float least = kl == 1 && batch == 4 ? (s == 1 ? kCscGatherLeastOne : kCscGatherLeastOneStrided) : kCscGatherLeast[s > 1][kl];
        if (pixels_in * batch < 1000.0 * least * bar) return c;
    } else if (!csc_gather_few((int)kl, (int)s)) {
        return c;
    } else if (kl == 2 ? (double)plan->nnz * batch < (k < 4 ? kCscGatherDirectThree : kCscGatherDirect) * bar
                       : pixels_in * std::sqrt((double)batch) < 1000.0 * kCscGatherLeastFew[s > 1][kl] * bar) {
        return c;
    }
    c.kl = (int)kl;
    c.scalar = batch < 4;
    g.sh = sh;
    const BuildScan bs = build_scan<true>(sh);
    g.zero1 = bs.first.zero;
    g.zero2 = bs.second.zero;
    g.row_entries = bs.row_entries;
    if (bs.row_entries < 4) return c;                                // lines of fewer entries than one access brings
    g.nnz = (unsigned)plan->nnz;
    g.batch = batch;
    g.lpr_log2 = c.scalar ? 0 : (batch > 8 ? 2 : (batch > 4 ? 1 : 0));
    const int lpr = 1 << g.lpr_log2, columns = c.scalar ? 1 : 4 * lpr;
    g.col_blocks = (batch + columns - 1) / columns;
    const int tw = csc_gather_tw((int)k, (int)s, g.lpr_log2, c.scalar);
    if (tw == 0) return c;
    const int pixels = (int)((tw - 1) * s + k + s - 1);              // of a strip, at most
    g.tw = tw;
    g.iw = (int)((tw - 1) * s + k);
    g.pw = csc_gather_places(tw, (int)k, (int)s);
    g.opw_log2 = csc_gather_opw_log2(tw, g.lpr_log2);
    g.groups = csc_gather_groups(tw, g.lpr_log2);
    g.ways = csc_gather_ways(tw, g.lpr_log2);
    g.line_elems = csc_gather_line(tw, (int)k, (int)s, g.lpr_log2);
    g.slots = csc_gather_slots(tw, (int)k, (int)s);
    g.quads = csc_gather_quads(tw, (int)k, (int)s);
    g.sets = k % s == 0 ? 1 : 2;
    c.nld = g.quads <= 2 * kCscGatherThreads ? 2 : 5;
    c.nx = c.nld == 2 && pixels * lpr <= kCscGatherThreads && pixels < kCscGatherThreads ? 1 : 3;
    c.lds = (size_t)csc_gather_lds(tw, (int)k, (int)s, g.lpr_log2, c.scalar);
    g.strips = (sh.n_out + tw - 1) / tw;
    auto lines = [&](int64_t target) {                               // output lines per segment
        const int64_t segs = std::max<int64_t>(target / ((int64_t)g.strips * g.col_blocks), 1);
        return (sh.m_out + segs - 1) / segs;
    };
    const int64_t seg = kl <= 3 && lines(2 * kCscGatherTarget) >= kCscGatherLong ? lines(2 * kCscGatherTarget) : lines(kCscGatherTarget);
    g.seg = (int)seg;
    g.segs = (int)((sh.m_out + seg - 1) / seg);
    const int64_t blocks = (int64_t)g.strips * g.segs * g.col_blocks;
    if (blocks + kXcds > kCscGatherBlocks) return c;
    g.blocks = (int)blocks;
    g.blocks_per_xcd = (int)((blocks + kXcds - 1) / kXcds);
    c.geom = g;
    c.ok = true;
    return c;
}

extern "C" {

int conv_spmv_from_csc(const conv_plan *plan, const float *x_dev, float *y_dev, int batch, void *stream) {
    if (!plan || !x_dev || !y_dev) return CONV_ENULL;
    if (batch < 1 || !plan->transposed || plan->compact) return CONV_EINVAL;
    // the plan's "rows" are the columns of T (input pixels), its "cols" the rows of T
    const int64_t in_pixels = plan->rows, out_pixels = plan->cols;
    {
        const char *xb = (const char *)x_dev, *xe = xb + sizeof(float) * (size_t)in_pixels * batch;
        const char *yb = (const char *)y_dev, *ye = yb + sizeof(float) * (size_t)out_pixels * batch;
        if (xb < ye && yb < xe) return CONV_EALIAS;
    }
    hipStream_t q = (hipStream_t)stream;
    const LaunchScope scope;
    const CscGatherChoice gather = plan->nnz > 0 && plan->edited.word ? choose_csc_gather(plan, batch) : CscGatherChoice{};
    if (gather.ok) launch_csc_gather(gather, plan, x_dev, y_dev, q);      // (then the scatter, should the arrays turn out edited)
    const int st = gather.ok ? enqueue_csc_scatter<true>(plan, x_dev, y_dev, batch, q)
                             : enqueue_csc_scatter<false>(plan, x_dev, y_dev, batch, q);
    if (st != CONV_OK) return st;
    return scope.ok() ? CONV_OK : CONV_EHIP;
}

// ---------------------------------------------------------------------------
// Many small products in one launch
// ---------------------------------------------------------------------------
}  // extern "C"

constexpr int64_t kMultiOwnerBlocks = 1 << 20;      // most workgroups with a table entry of their own (4 MiB)

struct conv_multi {
    int n, batch, device;
    unsigned blocks;
    MultiDesc *descs_dev;     // owned, device
    int *owner_dev;           // in the same allocation, behind the descriptors: product of every workgroup (null: bisection)
};

extern "C" {

int conv_multi_create(int n, const conv_plan *const *plans, const float *const *x_dev, float *const *y_dev,
                      int batch, conv_multi **multi_out) {
    if (!multi_out) return CONV_ENULL;
    *multi_out = nullptr;
    if (!plans || !x_dev || !y_dev) return CONV_ENULL;
    if (n < 1 || batch < 1) return CONV_EINVAL;
    MultiDesc *host = new (std::nothrow) MultiDesc[n];
    if (!host) return CONV_ENOMEM;
    int64_t blocks = 0;
    int status = CONV_OK;
    for (int i = 0; i < n && status == CONV_OK; ++i) {
        const conv_plan *p = plans[i];
        if (!p || !x_dev[i] || !y_dev[i]) { status = CONV_ENULL; break; }
        if (p->device != plans[0]->device || p->compact || p->channels != 1) { status = CONV_EINVAL; break; }
        const char *xb = (const char *)x_dev[i], *xe = xb + sizeof(float) * (size_t)p->cols * batch;
        const char *yb = (const char *)y_dev[i], *ye = yb + sizeof(float) * (size_t)p->rows * batch;
        if (xb < ye && yb < xe) { status = CONV_EALIAS; break; }
        int gs = 0;
        while ((1 << gs) < group_width(p->max_row_nnz)) ++gs;
        host[i] = MultiDesc{p->row_ptr, p->col_idx, p->vals, x_dev[i], y_dev[i], (int)p->rows, gs, (int)blocks, 0};
        blocks += ((p->rows << gs) + kGatherThreads - 1) / kGatherThreads;
        if (blocks > kInt32Limit) status = CONV_EOVERFLOW;
    }
    if (status != CONV_OK) {
        delete[] host;
        return status;
    }
    conv_multi *mu = new (std::nothrow) conv_multi;
    if (!mu) {
        delete[] host;
        return CONV_ENOMEM;
    }
    mu->n = n;
    mu->batch = batch;
    mu->device = plans[0]->device;
    mu->blocks = (unsigned)blocks;
    mu->descs_dev = nullptr;
    mu->owner_dev = nullptr;
    const bool table = blocks <= kMultiOwnerBlocks;
    const size_t desc_bytes = sizeof(MultiDesc) * (size_t)n;
    int *owner = table ? new (std::nothrow) int[std::max<int64_t>(blocks, 1)] : nullptr;
    if ((table && !owner) ||
        !hip_ok(hipMalloc((void **)&mu->descs_dev, desc_bytes + (table ? sizeof(int) * (size_t)blocks : 0)))) {
        delete[] owner;
        delete mu;
        delete[] host;
        return CONV_ENOMEM;
    }
    bool copied = hip_ok(hipMemcpy(mu->descs_dev, host, desc_bytes, hipMemcpyHostToDevice));
    if (table && blocks > 0) {
        for (int i = 0; i < n; ++i)
            for (int64_t b = host[i].first_block, e = i + 1 < n ? host[i + 1].first_block : blocks; b < e; ++b) owner[b] = i;
        mu->owner_dev = reinterpret_cast<int *>(reinterpret_cast<char *>(mu->descs_dev) + desc_bytes);
        copied = copied && hip_ok(hipMemcpy(mu->owner_dev, owner, sizeof(int) * (size_t)blocks, hipMemcpyHostToDevice));
    }
    delete[] owner;
    delete[] host;
    if (!copied) {
        (void)hipFree(mu->descs_dev);
        delete mu;
        return CONV_EHIP;
    }
    *multi_out = mu;
    return CONV_OK;
}

int conv_multi_apply(const conv_multi *multi, void *stream) {
    if (!multi) return CONV_ENULL;
    if (multi->blocks == 0) return CONV_OK;
    const int nv = multi->batch >= 4 ? widest_nv(multi->batch) : 0;
    const dim3 grid(multi->blocks, multi->batch < 4 ? 1u : (unsigned)std::min(column_blocks(multi->batch, nv), 65535));
    const LaunchScope scope;
#define CONV_MULTI(NV, COLS)                                                                                                 \
    spmm_multi_kernel<NV, COLS><<<grid, kGatherThreads, 0, (hipStream_t)stream>>>(multi->descs_dev, multi->owner_dev, multi->n, \
                                                                                  multi->batch)
    switch (nv) {
        case 0:
            if (multi->batch == 1) CONV_MULTI(0, 1);
            else if (multi->batch == 2) CONV_MULTI(0, 2);
            else CONV_MULTI(0, 3);
            break;
        case 1: CONV_MULTI(1, 4); break;
        case 2: CONV_MULTI(2, 4); break;
        default: CONV_MULTI(4, 4); break;
    }
#undef CONV_MULTI
    if (!scope.ok()) return CONV_EHIP;
    return CONV_OK;
}

int conv_multi_destroy(conv_multi *multi) {
    if (!multi) return CONV_OK;
    int st = CONV_OK;
    int cur = 0;
    const bool have = hip_ok(hipGetDevice(&cur));
    if (have && cur != multi->device) (void)hipSetDevice(multi->device);
    if (multi->descs_dev && !hip_ok(hipFree(multi->descs_dev))) st = CONV_EHIP;
    if (have && cur != multi->device) (void)hipSetDevice(cur);
    delete multi;
    return st;
}

int conv_plan_shape(const conv_plan *plan, int *m, int *n, int *k, int *s, int *p, int *m_out, int *n_out,
                    int64_t *nnz) {
    if (!plan) return CONV_ENULL;
    if (m) *m = plan->shape.m;
    if (n) *n = plan->shape.n;
    if (k) *k = plan->shape.k;
    if (s) *s = plan->shape.s;
    if (p) *p = plan->shape.p;
    if (m_out) *m_out = plan->shape.m_out;
    if (n_out) *n_out = plan->shape.n_out;
    if (nnz) *nnz = plan->nnz;
    return CONV_OK;
}

int conv_plan_is_transposed(const conv_plan *plan) { return plan ? (plan->transposed ? 1 : 0) : CONV_ENULL; }
int conv_plan_is_compact(const conv_plan *plan) { return plan ? (plan->compact ? 1 : 0) : CONV_ENULL; }
int conv_plan_channels(const conv_plan *plan) { return plan ? plan->channels : CONV_ENULL; }

static void describe(const CscGatherChoice &c, conv_dispatch &d) {
    d.kernel = 11;
    d.threads = kCscGatherThreads;
    d.lds_bytes = (int64_t)c.lds;
    d.workgroups = c.geom.blocks;
    d.strip = c.geom.tw;
    d.segment = c.geom.seg;
    d.ring_lines = c.geom.quads;
    d.ring_lines_needed = c.kl;
    d.lines_per_step = c.geom.ways;
    d.lanes_per_row = 1 << c.geom.lpr_log2;
    d.columns_per_lane = c.scalar ? 1 : 4;
}

int conv_dispatch_info(int m, int n, int k, int s, int p, int batch, int storage, int channels, conv_dispatch *out) {
    return conv_test_dispatch_info(m, n, k, s, p, batch, storage, channels, kMarchMinJobs, out);
}

int conv_test_dispatch_info(int m, int n, int k, int s, int p, int batch, int storage, int channels,
                            int march_min_jobs, conv_dispatch *out) {
    if (!out) return CONV_ENULL;
    if (march_min_jobs < 1) return CONV_EINVAL;
    int64_t mo, no;
    const int st = check_shape(m, n, k, s, p, &mo, &no);
    if (st != CONV_OK) return st;
    if (batch < 1 || channels < 1 || storage < 0 || storage > 3 || ((storage == 1 || storage == 3) && channels != 1))
        return CONV_EINVAL;
    if (storage == 2 && k > 255) return CONV_EINVAL;
    const int64_t nnz = conv_nnz(m, n, k, s, p);
    // the structure-aware storage has no per-entry index, so its entry count is not limited to int32
    if ((storage != 2 && nnz > kInt32Limit) || mo * no >= kInt32Limit || (int64_t)m * n * channels >= kInt32Limit)
        return CONV_EOVERFLOW;
    // a plan without arrays: the dispatch looks at the shape, the storage and operand alignment only
    conv_plan plan{};
    plan.shape = ConvShape{m, n, k, s, p, (int)mo, (int)no};
    plan.transposed = storage == 1 || storage == 3;
    plan.compact = storage == 2;
    plan.channels = channels;
    plan.rows = plan.transposed ? (int64_t)m * n : mo * no;
    plan.cols = plan.transposed ? mo * no : (int64_t)m * n * channels;
    plan.nnz = nnz;
    const int per_axis = plan.transposed ? (k + s - 1) / s : k;
    plan.max_row_nnz = per_axis * per_axis;
    plan.march_min_jobs = march_min_jobs;
    conv_dispatch d{};
    const ChannelsChoice fused = choose_compact_channels(&plan, nullptr, nullptr, batch);
    if (storage == 3) {
        // conv_spmv_from_csc: every output summed where it stays, the scatter with the sums kept on chip, or every entry
        // added to y directly
        const CscGatherChoice gather = plan.nnz > 0 ? choose_csc_gather(&plan, batch) : CscGatherChoice{};
        const CscTileChoice tc = plan.nnz > 0 ? choose_csc_tile(&plan, batch) : CscTileChoice{};
        if (gather.ok) {
            describe(gather, d);
        } else if (tc.ok) {
            d.kernel = 7;
            d.threads = tc.waves * kWave;
            d.lds_bytes = (int64_t)tc.lds;
            d.workgroups = (int64_t)tc.grid.x * tc.grid.y;
            d.strip = tc.g.tj;
            d.segment = tc.g.ti;
            d.ring_lines = 0;
            d.ring_lines_needed = tc.g.wx;          // runs of the window
            d.lines_per_step = tc.g.wy;             // rows per run
            d.lanes_per_row = tc.g.group;           // columns that share a step
            d.columns_per_lane = tc.vb;
        } else {
            d.kernel = 8;
            d.threads = kGatherThreads;
            d.lanes_per_row = group_width(plan.max_row_nnz);
            d.columns_per_lane = 1;
            const int bl = batch >= 16 ? 16 : (batch >= 4 ? 4 : 1);
            d.workgroups = (plan.rows * d.lanes_per_row * bl + kGatherThreads - 1) / kGatherThreads;
        }
    } else if (fused.ok) {
        d.kernel = 6;
        d.threads = fused.ways * kWave;
        d.lds_bytes = (int64_t)fused.lds;
        d.strip = kChanTileY / fused.chunks;
        d.segment = kChanTileX;
        d.lanes_per_row = 1;
        d.columns_per_lane = fused.vb;
        d.workgroups = (int64_t)fused.geom.tiles * fused.grid.y;
    } else if (plan.compact) {
        const CompactChoice cc = choose_compact(&plan, batch);
        if (!cc.ok) return CONV_EOVERFLOW;
        d.kernel = cc.laned || cc.gather_g ? 10 : (cc.kk ? 5 : 4);
        d.threads = kCompactThreads;
        if (cc.laned) {
            d.threads = kItemThreads;
            d.lanes_per_row = 1;
            d.columns_per_lane = cc.scalar ? 1 : 4;
            d.strip = cc.lane.chunks;
            d.workgroups = cc.lane.cells;
            *out = d;
            return CONV_OK;
        }
        if (cc.gather_g) {
            const int row_threads = cc.ways > 1 ? kWave : kCompactThreads;
            d.threads = row_threads * cc.ways;
            d.lds_bytes = (int64_t)cc.lds;
            d.lanes_per_row = cc.gather_g;
            d.columns_per_lane = cc.scalar ? 1 : 4 * cc.lpr;
            d.workgroups = ((plan.rows * cc.gather_g + row_threads - 1) / row_threads) * std::min<int64_t>(cc.col_blocks, 65535);
            *out = d;
            return CONV_OK;
        }
        d.lds_bytes = (int64_t)cc.lds;
        if (cc.pushed) {
            d.threads = kPushWaves * kWave;
            d.strip = cc.push.tw;
            d.segment = cc.push.seg;
            d.lines_per_step = kPushWaves;       // one line of each wave's part
            d.lanes_per_row = 1 << cc.push.lpr_log2;
            d.columns_per_lane = cc.scalar ? 1 : 4;
            d.workgroups = (int64_t)cc.push.blocks * cc.col_blocks;
            *out = d;
            return CONV_OK;
        }
        d.strip = cc.geom.tw;
        d.segment = cc.geom.seg;
        d.ring_lines = cc.geom.nl;
        d.lines_per_step = cc.geom.rv;
        d.lanes_per_row = cc.lpr;
        d.columns_per_lane = cc.scalar ? 1 : 4;
        d.ring_lines_needed = cc.kk ? s * (2 * cc.geom.rv - 1) + k : (cc.geom.nl ? s * (cc.geom.rv - 1) + k : 0);
        d.workgroups = (int64_t)cc.geom.strips * cc.geom.segs * cc.col_blocks;
    } else {
        const ApplyChoice c = choose_apply(&plan, batch);
        d.kernel = c.kind == Kind::GatherScalar ? 0 : c.kind == Kind::GatherVec ? 1 : c.kind == Kind::Tile ? 2
                   : c.kind == Kind::March ? 3 : c.kind == Kind::Block ? 12 : c.kind == Kind::Item ? (c.nv ? 1 : 0) : 9;
        d.threads = c.threads;
        d.lds_bytes = (int64_t)c.lds;
        d.lanes_per_row = c.g;
        d.columns_per_lane = c.nv ? 4 * c.nv : 1;
        if (c.kind == Kind::StageMarch) {
            const bool tr = plan.transposed;
            d.strip = c.tw;
            d.segment = c.march.seg;
            d.ring_lines = c.nl;
            d.lines_per_step = c.ls;
            d.ring_lines_needed = tr ? (c.ls - 2 + k) / s + 2 : s * (c.ls - 1) + k;
            d.workgroups = (int64_t)c.march.strips * c.march.segs * column_blocks(batch, c.nv);
        } else if (c.kind == Kind::March) {
            const bool tr = plan.transposed;
            d.strip = c.tw;
            d.segment = c.march.seg;
            d.ring_lines = c.nl;
            d.lines_per_step = c.ls;
            d.ring_lines_needed = tr ? (c.ls == 2 ? (k + 2) / s + 2 : k / s + 2) : s * (2 * c.ls - 1) + k;
            d.workgroups = (int64_t)c.march.strips * c.march.segs * column_blocks(batch, c.nv);
        } else if (c.kind == Kind::Block) {
            d.columns_per_lane = 4;
            d.lanes_per_row = 1 << c.lpr_log2;
            d.lds_bytes = (int64_t)sizeof(float) * (kBlockThreads / kWave) * (kWave >> c.lpr_log2) *
                          block_group_words(block_rx(k, s, plan.transposed) * c.tw, plan.max_row_nnz);
            d.strip = c.tw;
            d.segment = block_rx(k, s, plan.transposed);
            d.workgroups = (int64_t)c.block.cells * ((batch + (4LL << c.lpr_log2) - 1) / (4LL << c.lpr_log2));
        } else if (c.kind == Kind::Item) {
            d.strip = c.item.chunks;
            d.workgroups = c.item.cells;
        } else if (c.kind == Kind::Tile) {
            d.strip = c.tw;
            d.segment = c.geom.th;
            d.workgroups = (int64_t)c.geom.n_tiles * column_blocks(batch, c.nv);
        } else {
            d.workgroups = (plan.rows * c.g + kGatherThreads - 1) / kGatherThreads;
        }
    }
    *out = d;
    return CONV_OK;
}

int conv_test_csc_gather_info(int m, int n, int k, int s, int p, int batch, int march_min_jobs, conv_dispatch *out) {
    if (!out) return CONV_ENULL;
    if (march_min_jobs < 1 || batch < 1) return CONV_EINVAL;
    int64_t mo, no;
    const int st = check_shape(m, n, k, s, p, &mo, &no);
    if (st != CONV_OK) return st;
    const int64_t nnz = conv_nnz(m, n, k, s, p);
    if (nnz < 0 || nnz > kInt32Limit || mo * no >= kInt32Limit || (int64_t)m * n >= kInt32Limit) return CONV_EOVERFLOW;
    conv_plan plan{};
    plan.shape = ConvShape{m, n, k, s, p, (int)mo, (int)no};
    plan.transposed = true;
    plan.nnz = nnz;
    plan.march_min_jobs = march_min_jobs;
    conv_dispatch d{};
    const CscGatherChoice c = nnz > 0 ? choose_csc_gather(&plan, batch) : CscGatherChoice{};
    if (c.ok) describe(c, d);
    *out = d;
    return CONV_OK;
}

const char *conv_spmv_variant(const conv_plan *plan, int batch) {
    if (!plan || batch < 1) return nullptr;
    static thread_local char name[96];
    if (plan->compact) {
        const ChannelsChoice fused = choose_compact_channels(plan, nullptr, nullptr, batch);
        if (fused.ok) {
            snprintf(name, sizeof name, "compact_channels_%dx%d_float4x%d_%d_ways_%d_channels", kChanTileX, kChanTileY,
                     fused.vb / 4, fused.ways, plan->channels);
            return name;
        }
        const CompactChoice cc = choose_compact(plan, batch);
        if (!cc.ok) return nullptr;
        char cols[16];
        if (cc.scalar) snprintf(cols, sizeof cols, "scalar");
        else snprintf(cols, sizeof cols, "float4x%d", cc.lpr);
        if (cc.laned)
            snprintf(name, sizeof name, "compact_gather_lanes_%s", cc.scalar ? "scalar" : "float4");
        else if (cc.gather_g)
            snprintf(name, sizeof name, "compact_gather_g%d_%s", cc.gather_g, cols);
        else if (cc.pushed)
            snprintf(name, sizeof name, "compact_described_%dx%d_push%d_%s", cc.push.seg, cc.push.tw,
                     (plan->shape.k + plan->shape.s - 1) / plan->shape.s, cols);
        else if (cc.kk)
            snprintf(name, sizeof name, "compact_rect_k%ds%d_%dx%d_ring%d_rv%d_%s", cc.kk, cc.ss, cc.geom.seg,
                     cc.geom.tw, cc.geom.nl, cc.geom.rv, cols);
        else
            snprintf(name, sizeof name, "compact_described_%dx%d_ring%d_rv%d%s_%s", cc.geom.seg, cc.geom.tw,
                     cc.geom.nl, cc.geom.rv, cc.xld ? "_prefetch" : "", cols);
        return name;
    }
    const ApplyChoice c = choose_apply(plan, batch);
    switch (c.kind) {
        case Kind::GatherScalar: snprintf(name, sizeof name, "gather_g%d_scalar", c.g); break;
        case Kind::GatherVec: snprintf(name, sizeof name, "gather_g%d_float4x%d", c.g, c.nv); break;
        case Kind::March:
            if (c.nv)
                snprintf(name, sizeof name, "lds_march_%dx%d_ring%d_step%d_g%d_nit%d_float4x%d", c.march.seg, c.tw, c.nl, c.ls, c.g, c.nit, c.nv);
            else
                snprintf(name, sizeof name, "lds_march_%dx%d_ring%d_step%d_g%d_nit%d_scalar", c.march.seg, c.tw, c.nl, c.ls, c.g, c.nit);
            break;
        case Kind::StageMarch:
            if (c.nv)
                snprintf(name, sizeof name, "lds_march_staged_%dx%d_ring%d_step%d_g%d_nit%d_float4x%d", c.march.seg, c.tw, c.nl, c.ls, c.g, c.nit, c.nv);
            else
                snprintf(name, sizeof name, "lds_march_staged_%dx%d_ring%d_step%d_g%d_nit%d_scalar", c.march.seg, c.tw, c.nl, c.ls, c.g, c.nit);
            break;
        case Kind::Item:
            if (c.item.ways > 1) snprintf(name, sizeof name, "gather_g%d_%s_items_%d_ways", c.g, c.nv ? "float4" : "scalar", c.item.ways);
            else snprintf(name, sizeof name, "gather_g%d_%s_items", c.g, c.nv ? "float4" : "scalar");
            break;
        case Kind::Block:
            snprintf(name, sizeof name, "block_%dx%d_lanes%d_float4", block_rx(plan->shape.k, plan->shape.s, plan->transposed), c.tw, 1 << c.lpr_log2);
            break;
        case Kind::Tile:
            snprintf(name, sizeof name, "lds_tile_%dx%d_g%d_nit%d_float4x%d", c.geom.th, c.tw, c.g, c.nit, c.nv);
            break;
    }
    if (plan->channels > 1) {
        const size_t len = strlen(name);
        const bool per_channel = c.kind == Kind::March || c.kind == Kind::Tile ||
                                 (c.kind == Kind::StageMarch && c.march.channels <= 1);
        snprintf(name + len, sizeof name - len, per_channel ? "_x%d_launches" : "_%d_channels", plan->channels);
    }
    return name;
}

int conv_plan_destroy(conv_plan *plan) {
    if (!plan) return CONV_OK;
    if (plan->edited.word) edited_places.give_back(plan->edited_place);
    delete plan;          // a plan owns no device memory
    return CONV_OK;
}

const char *conv_strerror(int status) {
    switch (status) {
        case CONV_OK: return "ok";
        case CONV_EINVAL: return "invalid argument (need m,n,k,s >= 1, p >= 0, batch >= 1, k <= m+2p and k <= n+2p)";
        case CONV_ENULL: return "required pointer is NULL";
        case CONV_EOVERFLOW: return "size does not fit the library's 32-bit indices";
        case CONV_EHIP: return "HIP call failed (see conv_last_hip_error)";
        case CONV_ENOMEM: return "allocation failed";
        case CONV_EALIAS: return "x and y overlap";
    }
    return "unknown status";
}

int conv_last_hip_error(void) { return g_last_hip_error; }

int conv_plan_set_march_min_jobs(conv_plan *plan, int jobs) {
    if (!plan) return CONV_ENULL;
    if (jobs < 1) return CONV_EINVAL;
    const int prev = plan->march_min_jobs;
    plan->march_min_jobs = jobs;
    return prev;
}

}  // extern "C"
