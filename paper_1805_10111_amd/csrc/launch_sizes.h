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

// A mini-batch prepared ahead of its round: layout in 32-bit words (see grad_csr.hip) of its tables for B rows, for `cap`
// entries.  The kernels with cached margins lay it out for the rows of the batch, those without for kCsrMaxRows; the master,
// which does not know which of them reads next, writes one word of it, so that word lies in the same place in every
// layout: the row starts come first, as many as a block takes, and it is the last behind them.
struct PrepLayout {
    int pre, dev_max;  // (see WorkerArgs::dev_max)
    int row, len, y, z, entries;
    constexpr explicit PrepLayout(int B)
        : pre(4), dev_max(pre + kCsrMaxRows + 3), row(dev_max + 1), len(row + (B + 3) / 4 * 4), y(len + (B + 3) / 4 * 4),
          z(y + (B + 3) / 4 * 4), entries(z + (B + 3) / 4 * 4) {}
};
constexpr int kPrepEntries = PrepLayout(kCsrMaxRows).entries;
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

// A step's workspace: M rows of the gradient, then kMaxSlices maxima and as many counts per worker.  A run's has its own behind
// them: pad4(d) words and twice M times csr_prep_stride(d).
constexpr int kMaxSlices = 8;                    // blocks that share a worker's step
inline int64_t csr_run_offset(int64_t d, int64_t M) { return M * pad4(d) * 4 + M * kMaxSlices * 8; }
inline int64_t csr_run_bytes(int64_t d, int64_t M) { return csr_run_offset(d, M) + pad4(d) * 4 + 2 * M * csr_prep_stride(d) * 4; }

// What a run's workspace holds behind its M rows and slice results.
// Either the difference of model and snapshot, a word per column, and the two sets of prepared mini-batches; or, where the
// worker kernel quantizes the model and has no use for that row, two sets of mini-batches in all of it, whose entries
// can have the snapshot at their column beside them.
struct PrepRoom {
    int64_t stride;     // words per worker
    int cap;            // most entries of a mini-batch
    int snap_cap;       // most entries that have the snapshot value beside them
};

inline PrepRoom csr_prep_room(int64_t d, int64_t M, int64_t B, const CsrPlan &plan, bool snaps)
{
    if (!snaps) return PrepRoom{csr_prep_stride(d), csr_prep_cap(d, plan), 0};
    PrepRoom r{};
    r.stride = (pad4(d) + 2 * M * csr_prep_stride(d)) / (2 * M) / 4 * 4;
    const int64_t room = r.stride - PrepLayout(static_cast<int>(B)).entries;
    r.cap = static_cast<int>(room / 2 < plan.cap ? room / 2 : plan.cap);
    r.snap_cap = static_cast<int>(room / 3 < r.cap ? room / 3 : r.cap);
    return r;
}

// Whether mini-batches of B of the n rows are light enough for what the worker kernel does entry by entry instead of column by
// column elsewhere: quantizing the model, in every block, instead of a launch of its own; and, in Alg. 2, finding ||alpha||_inf
// (see csr_run_layout): on average little more entries than a block keeps in its registers
// (`in_flight`), and no more than it can prepare ahead (`cap`, with an eighth to spare for batches above the average).
// `entries` is what the caller says the matrix holds; unknown (0), rows of 100 are assumed.
// Measured, Alg. 1, eight workers, us a round with a launch for the model and without: 4200 columns, 485 entries 11.7 and 9.7,
// 4757 entries 13.3 and 13.0, 6627 entries 15.1 and 15.8, 9515 (not prepared) 24.5 and 27.2; 20,958 columns, 1656 entries 13.0 and
// 11.5, 9518 (not prepared) 27.6 and 31.8; 32,000 columns, 1656 (not prepared) 19.9 and 21.0, 12,693 (not prepared) 60.2 and 74.0.
// 25 workers: 4200 columns, 4757 entries 16.4 both; 14,000 columns, 4759 entries 17.9 and 18.1, 3838 entries 17.4 and 17.0.
inline bool csr_light_batches(int64_t B, int64_t n, int64_t entries, int in_flight, int cap)
{
    const double mean = static_cast<double>(B) * (entries > 0 ? static_cast<double>(entries) / static_cast<double>(n) : 100.0);
    return mean <= 1.2 * in_flight && mean * 1.125 <= cap;
}

// ------------------------------------------------------------------ blocks that work together on one die (die.h)
constexpr uint32_t kDies = 16;                   // (numbers that a die may have; the part has eight)

// The die where a launch has most blocks (count_of a number), `own` where it has none; of several with as many the first from number
// lot % 8 on: launches that hold equal parts of all dies pick different ones, seven times of eight.
template <typename CountOf>
constexpr uint32_t die_pick(CountOf count_of, uint32_t own, uint32_t lot)
{
    uint32_t best = own, most = 0;
    for (uint32_t i = 0; i < kDies; ++i) {
        const uint32_t at = (i + lot % 8) % kDies, c = count_of(at);
        if (c > most) {
            most = c;
            best = at;
        }
    }
    return best;
}

// ------------------------------------------------------------------ rounds on one die, CSR features (csr_rounds.hip)
constexpr int kDieUnits = 32;                    // compute units of a die
constexpr int kRoundsRows = 128;                 // rows of a mini-batch: two a lane of the wavefront that lays them out
constexpr int kBusyWaves = 15, kBusy = kBusyWaves * 64;       // all but the wavefront that waits at exchanges
constexpr int kUnitWaves = kBusyWaves - 1;       // (not the one that lays out mini-batches)
constexpr int kEntriesEach = 8;                  // entries a thread holds; with more of them the rows are read in the round
constexpr int kChunk = 256;                      // columns of a chunk: a quad a lane
constexpr int kMostChunks = 7, kColumns = 2;     // of a member, and columns a thread
constexpr int kPasses = 2;                       // chunks of all workers that a wavefront takes in turn
constexpr int64_t kFewRounds = 8;                // calls of fewer are not for one die
constexpr int64_t kRoundsFixedLds = 13360;       // static arrays
constexpr int64_t kRoundsLds = 160 * 1024 - kRoundsFixedLds;  // for the dynamic part
constexpr int64_t kRoundsControl = 848;          // bytes of a run's workspace, from csr_run_offset on, for what the members share

static_assert(kMostChunks * kChunk <= kColumns * kBusy, "every column has a thread");

struct CsrRoundsShape {
    int S, win;                                  // slices of a worker, columns of one
    int want, chunks;                            // members, chunks of one
    int cap;                                     // entries of a group of rows (CsrPlan::cap)
    int room;                                    // entries that LDS has room for
    int64_t lds;                                 // bytes of dynamic LDS
};

// false: these rounds are not for one die.  They are where measured faster than launches (us a round, 30 rounds a call unless
// said; launches, then this):
//  - the snapshot has room in LDS: d 26,323, M 12, read from L2 instead: 13.1, 18.2; d 38,834, M 8: 16.1, 19.1.
//  - no wavefront has more than two chunks of gradients to quantize, which stay in registers: M 8, d 20,958 (24 chunks a
//    member) 11.4, 9.9; M 4, d 28,409 12.6, 11.3; M 28, d 5000 12.7, 10.7; M 21, d 4340 12.2, 10.1; M 1, d 300 9.0, 7.7; M 8,
//    d 20,000, b_x 12 16.4, 11.5; M 20, d 6385, batches of 128 17.2, 14.5.  With four: M 10, d 20,958 12.0, 12.7; M 16, d
//    12,000 11.6, 12.7; M 32, d 6400 13.3, 14.0.
//  - calls of eight rounds or more: the launches around it, and finding together, are 10 us a call.  M 8, d 20,958: two rounds
//    12.5, 15.2; five 11.8, 12.0; eight 11.6, 11.2.
//  - mini-batches that the busy threads hold in registers, as far as the caller's count of entries can tell.  It cannot tell uneven
//    rows, nor any where it is not given; larger batches are read in the round.  M 8, d 20,958, 64 rows of 50 entries in the mean,
//    lognormal with sigma 1, 1.5 and 2: 14.8, 12.4; 20.7, 15.6; 29.5, 20.2; no count, 32 rows of 200 and of 1000: 26.6, 18.1; 87, 51.
inline bool csr_rounds_shape(int64_t d, int64_t n, int64_t entries, int64_t M, int64_t B, int b_x, int64_t rounds, CsrRoundsShape &s)
{
    const auto least = [](int64_t a, int64_t b) { return a < b ? a : b; };
    const auto most = [](int64_t a, int64_t b) { return a > b ? a : b; };
    CsrPlan plan;
    if (b_x < 2 || b_x > 16 || B > kRoundsRows || M > kDieUnits || rounds < kFewRounds || !csr_plan(d, false, plan)) return false;
    const int64_t S = least(least(kDieUnits / M, 16), ceil_div(d, 256));
    s.win = static_cast<int>(ceil_div(ceil_div(d, S), 256) * 256);
    s.S = static_cast<int>(ceil_div(d, s.win));
    s.want = static_cast<int>(most(M * s.S, least(kDieUnits, ceil_div(d, kChunk))));
    const int64_t chunks = ceil_div(ceil_div(d, kChunk), s.want);
    if (chunks > kMostChunks || M * chunks > kPasses * kUnitWaves) return false;
    s.chunks = static_cast<int>(chunks);
    const double mean = static_cast<double>(B) * (entries > 0 ? static_cast<double>(entries) / static_cast<double>(n) : 100.0);
    s.cap = plan.cap;
    const int64_t held = least(plan.cap, kEntriesEach * kBusy);
    if (mean * 1.25 > static_cast<double>(held)) return false;
    const int64_t room = most(M * chunks * (kChunk / 4), least(held, static_cast<int64_t>(1.5 * mean) + 256));
    s.room = static_cast<int>(ceil_div(room, 64) * 64);
    const int64_t message = pad4((d * b_x + 31) / 32 + 1);
    int64_t bytes = (s.win + message + s.room + pad4(d)) * 4;
    if (bytes > kRoundsLds) return false;
    // (what is left is for larger mini-batches than the mean's, as far as the threads hold them)
    const int64_t more = least((kRoundsLds - bytes) / 256 * 64, most(0, held / 64 * 64 - s.room));
    s.room += static_cast<int>(more);
    bytes += more * 4;
    // (what makes up more than half of a compute unit's LDS: no two blocks on one)
    s.lds = most(bytes, 72 * 1024);
    return true;
}

}  // namespace dq
