// Sizes that the host works out for a launch: plain C++, no HIP, so that they can be checked over their whole range
// without a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace dq {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t packed_words(int64_t d, int b) { return (d * b + 31) / 32; }
inline int64_t pad4(int64_t d) { return (d + 3) / 4 * 4; }

// ------------------------------------------------------------------ full gradient on dense features (grad_dense.hip)
// Threads per block and float4 columns per thread on rows of more than 1024 floats: of 256 to 512 threads in whole
// wavefronts, as few as cover the row with 1, 2, 4 or 8 columns each.
struct FullShape {
    int threads, cols;
};

inline FullShape full_shape(int64_t d)
{
    const int64_t quads = ceil_div(d, 4);
    const int cols = quads <= 512 ? 1 : quads <= 1024 ? 2 : quads <= 2048 ? 4 : 8;
    const int64_t threads = ceil_div(ceil_div(quads, cols), 64) * 64;
    return FullShape{static_cast<int>(threads < 256 ? 256 : threads), cols};
}

// Of a thread's `cols` columns the first so many lie inside the row for every thread and need no mask, in any shape that
// full_shape gives: threads * full_whole_cols(cols) <= d / 4.  Rounding up to whole wavefronts adds up to 63 quads per
// column; with eight columns those can pass the end by more than the last column (8197 floats: 320 threads, seven
// columns of them 2240 quads of 2050).
constexpr int full_whole_cols(int cols) { return cols >= 8 ? cols - 2 : cols - 1; }

// ------------------------------------------------------------------ worker step on CSR features (grad_csr.hip)
constexpr int kColBits = 20;                     // staged entries carry column | row << kColBits
constexpr int kCsrMaxRows = 256;                 // rows a block handles per pass (LDS metadata)
constexpr int kMaxStage = 8192;                  // most entries the staging buffer is given
constexpr int64_t kMinStage = 4096;              // least entries it is given beside one of several windows
constexpr int64_t kLdsBudget = 152 * 1024;       // of the 160 KB per compute unit
constexpr int64_t kCsrFixedLds = 10 * 1024;      // static arrays, rounded up

// LDS plan for a d-vector plus the staging buffer.  When both fit, the vector is one window; otherwise it is built
// in several equal windows (multiples of 4 columns) that leave room for at least kMinStage staged entries.
// Columns carry the row number in the bits above kColBits while staged, hence the limit on d.
struct CsrPlan {
    int win;        // columns per window
    int cap;        // staged (column, value) entries
    int nwin;
    size_t lds;     // bytes of dynamic LDS: window + staging
};

// A staged entry takes 12 bytes of LDS, 16 when the caller needs two sums per row (no cached margins).
inline bool csr_plan(int64_t d, bool second, CsrPlan &p)
{
    if (d >= (1ll << kColBits)) return false;
    const int64_t budget = kLdsBudget - kCsrFixedLds;                     // bytes for window + staging
    const int64_t each = second ? 16 : 12;
    int64_t nwin = 1;
    if (pad4(d) * 4 + each * 512 > budget) nwin = ceil_div(pad4(d) * 4, budget - each * kMinStage);
    const int64_t win = pad4(ceil_div(pad4(d), nwin));
    int64_t cap = (budget - win * 4) / each;
    if (cap > kMaxStage) cap = kMaxStage;
    p.lds = static_cast<size_t>(win * 4 + cap * each);
    p.win = static_cast<int>(win);
    p.cap = static_cast<int>(cap);
    p.nwin = static_cast<int>(ceil_div(pad4(d), win));
    return true;
}

// A mini-batch prepared ahead of its round: layout in 32-bit words (see grad_csr.hip), for `cap` entries.
constexpr int kPrepRow = 4, kPrepLen = kPrepRow + kCsrMaxRows, kPrepPre = kPrepLen + kCsrMaxRows,
              kPrepY = kPrepPre + kCsrMaxRows + 4, kPrepZ = kPrepY + kCsrMaxRows, kPrepEntries = kPrepZ + kCsrMaxRows;
constexpr int64_t kPrepInts(int64_t cap) { return kPrepEntries + (2 * cap + 3) / 4 * 4; }

// Words per worker that the workspace holds for one: room for what the plan for one sum per row stages.
inline int64_t csr_prep_stride(int64_t d)
{
    CsrPlan one_sum;
    return csr_plan(d, false, one_sum) ? kPrepInts(one_sum.cap) : 0;
}

// Most entries of a mini-batch that is prepared ahead for a step with this plan.  Not the plan's capacity: without cached
// margins the vector may take more windows than with them, narrower ones, which leave MORE entries for staging than the
// workspace has room for (47,236 columns: 5151 against 4244; 34,400: 4788 against 650).
inline int csr_prep_cap(int64_t d, const CsrPlan &plan)
{
    CsrPlan one_sum;
    if (!csr_plan(d, false, one_sum)) return 0;
    return plan.cap < one_sum.cap ? plan.cap : one_sum.cap;
}

}  // namespace dq
