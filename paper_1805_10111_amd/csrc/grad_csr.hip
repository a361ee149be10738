// CSR-feature gradient kernels: epoch prologue (full gradient, Alg. 1) and the worker step
// (Alg. 1 worker (i)-(ii), Alg. 2 worker (i)-(iii)) for bag-of-words shaped data.
//
// A mini-batch of such rows touches a few thousand entries, far too few to be bandwidth
// bound; what matters is that one launch does the whole worker step and that the result
// is reproducible.  One block of 1024 threads owns a worker: the gradient alpha (d floats)
// lives in LDS for the whole step and never goes to memory.
//   1. stage: the (column, value) pairs of the mini-batch rows are copied into LDS as one flat run, spread evenly
//      over the threads whatever the row lengths (the row of an entry comes from a table of the rows at every 64th
//      entry plus the starts of the next few rows, and is kept in the bits above the column); the thread that copies an
//      entry also gathers the model and the snapshot at its column and leaves value * operand next to it -- two
//      trips to memory for the whole mini-batch, however long its longest row;
//   2. margins: one wavefront per row, four rows in flight, adds up the products of its row from LDS; one lane per
//      row forms its coefficient;
//   3. scatter: every thread adds coefficient*value of the entries it staged to the columns' accumulators in LDS --
//      integer atomic adds of fixed-point terms (see FixedAcc), whose sum does not depend on the order of the adds:
//      the result is reproducible whichever wavefront gets there first;
//   4. the accumulators become float32 in place, the dense part l2*(q - snapshot) added, and the tail of the worker
//      step (sparsify, scale, quantize, pack) runs from LDS.
// Between the rounds of one dq_run_rounds call, everything of step 1 that does not depend on the model (which rows,
// their extents and labels, the flat run itself) is laid out one round ahead by an extra block per worker of the
// previous round's launch (see PrepLayout).
// The full gradient takes its rows straight from memory in many blocks, each leaving a partial d-vector of fixed-point
// sums that a second kernel adds up in a fixed order.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include <hip/hip_ext.h>

#include "csr_rows.h"
#include "dq_common.h"
#include "elementwise.h"
#include "grad_common.h"
#include "grad_launch.h"

namespace dq {

// The staging buffer in LDS: `cap` entries of (column | row << kColBits, value), and per entry value * first operand
// (prod_a) and, for callers that need a second sum, value * second operand (prod_b, else null).
struct CsrStage {
    int2 *entry;
    float *prod_a, *prod_b;
    int cap;
};

__device__ __forceinline__ CsrStage csr_stage_in(float *after_window, int cap, bool second)
{
    CsrStage sg;
    sg.entry = reinterpret_cast<int2 *>(after_window);
    sg.prod_a = after_window + 2 * static_cast<int64_t>(cap);
    sg.prod_b = second ? sg.prod_a + cap : nullptr;
    sg.cap = cap;
    return sg;
}

// Where the entry of staged position P + lane lies in the matrix, and its row number shifted above the column bits.
// A wavefront whose 64 positions all lie past the end (P >= total) gets `inside`, the source of a position that
// does exist, so that no load sits behind a test.
__device__ __forceinline__ int64_t csr_stage_source(const RowMeta &meta, int g0, int g1, int base, int total, int P,
                                                    int lane, int64_t inside, int &tag)
{
    const int p = min(P + lane, total - 1);
    const int r = P >= total ? g1 - 1
                  : g0 == 0  ? csr_row_in_chunk(meta, g1, P, p)
                             : csr_row_of(meta, g0, g1, base, p);
    tag = r << kColBits;
    return P < total ? meta.start[r] + (p - (meta.pre[r] - base)) : inside;
}

// Margins and scatter for the staged group of rows [g0, g1) (`total` entries; base = pre[g0]); vmax = the largest
// |value| among the entries this thread staged, as bits.
template <bool SECOND, typename CoefFn>
__device__ __forceinline__ void csr_reduce_group(RowMeta &meta, int g0, int g1, int base, int total, uint32_t vmax,
                                                 int *acc, int c0, int c1, const CsrStage &sg, FixedAcc &fx, uint32_t *su,
                                                 int *poison, CoefFn coef_of)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int2 *stage = sg.entry;
    vmax = block_max_u32(vmax, su);            // (its barriers also publish the staged entries)
    // ---- margins and coefficients: four rows per wavefront in flight; lane u evaluates row u's scalar
    for (int r = g0 + wave; r < g1; r += kFlight * kCsrWaves) {
        int len[kFlight], off[kFlight], maxlen = 0;
        float sa[kFlight], sb[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int ru = r + u * kCsrWaves;
            len[u] = ru < g1 ? meta.len[ru] : 0;
            off[u] = ru < g1 ? meta.pre[ru] - base : 0;
            maxlen = max(maxlen, len[u]);
            sa[u] = sb[u] = 0.0f;
        }
        for (int k = lane; k < maxlen; k += kWave) {           // (maxlen > 0 implies total > 0)
            float pa[kFlight], pb[kFlight];
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                const int at = min(off[u] + k, total - 1);
                pa[u] = sg.prod_a[at];
                pb[u] = SECOND ? sg.prod_b[at] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                sa[u] += k < len[u] ? pa[u] : 0.0f;
                if (SECOND) sb[u] += k < len[u] ? pb[u] : 0.0f;
            }
        }
        float mine_a = 0.0f, mine_b = 0.0f;
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const float ta = wave_sum_f32(sa[u]);
            const float tb = SECOND ? wave_sum_f32(sb[u]) : 0.0f;
            if (lane == u) {
                mine_a = ta;
                mine_b = tb;
            }
        }
        const int rl = r + lane * kCsrWaves;
        if (lane < kFlight && rl < g1) {
            const float cf = coef_of(rl, mine_a, mine_b);
            meta.coef[rl] = cf;
        }
    }
    __syncthreads();
    // ---- scatter: fixed-point terms, integer atomic adds
    fixed_admit(fx, coef_abs_sum(meta.coef, g0, g1) * __uint_as_float(vmax), acc, c1 - c0, poison);
    const float two_k = ldexpf(1.0f, fx.k);
    for (int p0 = threadIdx.x; p0 < total; p0 += kStageFlight * kCsrThreads) {
        int2 e[kStageFlight];
        float cf[kStageFlight];
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u) e[u] = stage[min(p0 + u * kCsrThreads, total - 1)];
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u) cf[u] = meta.coef[(e[u].x >> kColBits) & (kCsrMaxRows - 1)];
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u) {
            const int c = e[u].x & kColMask;
            if (p0 + u * kCsrThreads < total && c >= c0 && c < c1)
                atomicAdd(&acc[c - c0], fixed_term(cf[u], __int_as_float(e[u].y), two_k));
        }
    }
}

// Stage, margins and scatter (the first three phases of the file header) for rows [0, nrows) described by `meta`,
// accumulating into acc (LDS, fixed point, see FixedAcc).
// The rows are taken in groups that fit the staging buffer:
//   stage  : the group's (column, value) pairs are copied to LDS as one flat run, kStageFlight entries per thread in
//            flight, the row number packed above the column; vec_val(vec_req(c), c) returns the {first, second}
//            operands of column c gathered from memory -- vec_req only requests (no branch, no use of what it
//            loads), so a thread's gathers wait for memory once -- and value * operand is staged with the entry;
//   margins: one wavefront per row (kFlight rows in flight) adds up its row's products; lane u hands the sums of its
//            u-th row to coef_of(row, first_sum, second_sum), which returns the row's coefficient;
//   scatter: every thread adds coefficient*value of its share of the staged entries to acc[column - c0].
// A row longer than `cap` is handled alone, straight from memory.
// Only the columns of the window [c0, c1) are accumulated: a vector too long for LDS is built one window at a
// time (the caller repeats the call per window; margins are recomputed).
template <bool SECOND, typename VecReq, typename VecVal, typename CoefFn>
__device__ __forceinline__ void csr_process_rows(const CsrView &A, RowMeta &meta, int nrows, int *acc, int c0, int c1,
                                                 const CsrStage &sg, FixedAcc &fx, uint32_t *su, int *poison,
                                                 VecReq vec_req, VecVal vec_val, CoefFn coef_of)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int cap = sg.cap;
    int2 *stage = sg.entry;
    int g0 = 0;
    while (g0 < nrows) {
        // group of consecutive rows that fits the staging buffer: rows g0..g1-1 with
        // pre[g1] - pre[g0] <= cap; a first row longer than cap is taken alone, unstaged
        const int base = meta.pre[g0];
        int g1 = nrows;
        bool direct = false;
        if (meta.pre[nrows] - base > cap) {            // (the same for every thread) not all remaining rows fit
            // the first row whose end lies past the buffer, by halving (every thread finds the same one)
            int lo = g0, hi = nrows - 1;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (meta.pre[mid + 1] - base > cap) hi = mid;
                else lo = mid + 1;
            }
            g1 = max(lo, g0 + 1);
            direct = meta.len[g0] > cap;
        }
        if (!direct) {
            // ---- stage: flat copy of the group's entries with their products
            const int total = meta.pre[g1] - base;
            uint32_t vmax = 0;
            // (the loop bound is the same for a whole wavefront: its lanes find their rows together)
            for (int p0 = threadIdx.x; p0 - lane < total; p0 += kStageFlight * kCsrThreads) {
                int64_t src[kStageFlight];
                int tag[kStageFlight], col[kStageFlight];
                float val[kStageFlight];
#pragma unroll
                for (int u = 0; u < kStageFlight; ++u)     // (a position past the end repeats an entry and is not stored)
                    src[u] = csr_stage_source(meta, g0, g1, base, total, p0 - lane + u * kCsrThreads, lane, u ? src[0] : 0, tag[u]);
#pragma unroll
                for (int u = 0; u < kStageFlight; ++u) {
                    col[u] = A.indices[src[u]];
                    val[u] = A.values[src[u]];
                }
                decltype(vec_req(0)) raw[kStageFlight];
#pragma unroll
                for (int u = 0; u < kStageFlight; ++u) raw[u] = vec_req(col[u]);
#pragma unroll
                for (int u = 0; u < kStageFlight; ++u) {
                    const int p = p0 + u * kCsrThreads;
                    const float2 f = vec_val(raw[u], col[u]);
                    vmax = max(vmax, abs_bits(val[u]));
                    if (p < total) {
                        stage[p] = make_int2(col[u] | tag[u], __float_as_int(val[u]));
                        sg.prod_a[p] = val[u] * f.x;
                        if (SECOND) sg.prod_b[p] = val[u] * f.y;
                    }
                }
            }
            csr_reduce_group<SECOND>(meta, g0, g1, base, total, vmax, acc, c0, c1, sg, fx, su, poison, coef_of);
        } else {
            // ---- one very long row, straight from memory (every wavefront computes the same sums)
            const int64_t s = meta.start[g0];
            float a1 = 0.0f, b1 = 0.0f;
            uint32_t vmax = 0;
            for (int k = lane; k < meta.len[g0]; k += kWave) {
                const int ck = A.indices[s + k];
                const float2 f = vec_val(vec_req(ck), ck);
                const float v = A.values[s + k];
                vmax = max(vmax, abs_bits(v));
                a1 += v * f.x;
                if (SECOND) b1 += v * f.y;
            }
            a1 = wave_sum_f32(a1);
            if (SECOND) b1 = wave_sum_f32(b1);
            vmax = wave_max_u32(vmax);                 // (the same in every wavefront)
            __syncthreads();
            if (threadIdx.x == 0) meta.coef[g0] = coef_of(g0, a1, b1);
            __syncthreads();
            const float cf = meta.coef[g0];
            fixed_admit(fx, fabsf(cf) * __uint_as_float(vmax), acc, c1 - c0, poison);
            const float two_k = ldexpf(1.0f, fx.k);
            for (int k = threadIdx.x; k < meta.len[g0]; k += kCsrThreads) {
                const int c = A.indices[s + k];
                if (c >= c0 && c < c1) atomicAdd(&acc[c - c0], fixed_term(cf, A.values[s + k], two_k));
            }
        }
        __syncthreads();
        g0 = g1;
    }
}

// ---- a mini-batch prepared ahead of its round
// What a worker step does before it first needs the model -- drawing its rows (Alg. 1, worker step 2: the sample stream),
// reading their extents, labels and cached margins, the prefix sums, and the copy of the rows' entries into one flat run
// -- does not depend on the model.  Between two rounds of one dq_run_rounds call an extra block per worker of the
// worker launch does all of that for the NEXT round, on compute units the launch leaves idle, and leaves it in
// memory as PrepRoom::stride 32-bit words per worker:
//   [0] 1 when the flat run is there (the batch has at most PrepRoom::cap entries), else 0   [1] number of entries
//   [2] the largest |value| among them, as bits, if they are more than kPrepNoMax   [3] 1 when the snapshot values are there
//   pre[kCsrMaxRows + 3], a word of the master's (WorkerArgs::dev_max; in the first worker's block), row[B] len[B] y[B]
//   z[B], each from a multiple of four words on      (RowMeta's fields)
//   pairs (column | row << kColBits, value bits), [1] of them; room for PrepRoom::snap_cap pairs further on the snapshot
//   at their columns, if there are no more of them than that
// The next round's blocks then start from one round trip to memory instead of a chain of five.

// Stage, margins and scatter for a prepared mini-batch without cached margins: `entry` is its flat run of `total` <= cap entries, `first`
// what the caller has already loaded of it (positions threadIdx.x + u * kCsrThreads, clamped to the buffer), meta
// holds the rows.  The rest as csr_process_rows.
template <typename VecReq, typename VecVal, typename CoefFn>
__device__ __forceinline__ void csr_process_prepared(const int2 *entry, const int2 (&first)[kStageFlight], int total,
                                                     RowMeta &meta, int nrows, int *acc, int c0, int c1, const CsrStage &sg,
                                                     FixedAcc &fx, uint32_t *su, int *poison, VecReq vec_req,
                                                     VecVal vec_val, CoefFn coef_of)
{
    uint32_t vmax = 0;
    const auto stage_batch = [&](int p0, const int2 (&e)[kStageFlight]) {
        int col[kStageFlight];
        decltype(vec_req(0)) raw[kStageFlight];
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u) {
            // (past the end `first` holds whatever the buffer held: column 0 is gathered instead)
            col[u] = p0 + u * kCsrThreads < total ? e[u].x & kColMask : 0;
            raw[u] = vec_req(col[u]);
        }
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u) {
            const int p = p0 + u * kCsrThreads;
            const float2 f = vec_val(raw[u], col[u]);
            const float val = __int_as_float(e[u].y);
            if (p < total) {
                vmax = max(vmax, abs_bits(val));
                sg.entry[p] = e[u];
                sg.prod_a[p] = val * f.x;
                sg.prod_b[p] = val * f.y;
            }
        }
    };
    stage_batch(threadIdx.x, first);
    for (int p0 = threadIdx.x + kStageFlight * kCsrThreads; p0 < total; p0 += kStageFlight * kCsrThreads) {
        int2 e[kStageFlight];
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u) e[u] = entry[min(p0 + u * kCsrThreads, total - 1)];
        stage_batch(p0, e);
    }
    csr_reduce_group<true>(meta, 0, nrows, 0, total, vmax, acc, c0, c1, sg, fx, su, poison, coef_of);
    __syncthreads();
}

// Up to here the preparing block, not the one that reads what it left, is what a launch waits for: then the reader forms
// the largest |value| (4753 columns, 8 workers of 13 rows: 14.9 us a round where the preparing block did, now 14.1).
constexpr int kPrepNoMax = kCsrThreads;

// The same with cached margins; the first kCsrInFlight entries, nearly always all of them, stay in the registers they were
// loaded into: `e` is the flat run's beginning, `entry` the run, `vmax` its largest |value|, and lane l of wavefront w holds row w + 16 l of the batch (its length, its
// first entry's position, and whatever coef_of(zdiff) needs besides its margin); the first operands are left in `operand`.  What a block waits for here is latency,
// one phase after another, so there are as few phases as the sums allow: products to LDS, barrier, margins and
// coefficients, barrier, scatter.  The sums are those of csr_reduce_group, bit for bit.
// Eight workers of 32 rows, 20,958 columns, from the block's start: products complete after 2.2 us, margins 2.8, scattered
// 3.6, where the general form took 2.7 (with the maximum), 3.7 and 4.5.
constexpr int kCsrInFlight = kStageFlight * kCsrThreads;

// GATED: a wavefront that has no entry among its 64 positions requests nothing for them, and up to 48 rows are added up two at
// a time to a wavefront; the whole block issues less (1349 columns, four workers of 36 rows of 9 entries: 12.5 -> 12.2 us a round;
// 3118 columns, eight workers of 39 rows of 10: 14.3 -> 13.9).  Not where the model is quantized here: 5000 columns, eight workers of
// 64 rows of 52 entries 11.8 us without and 12.1 with it.
template <bool GATED, typename VecReq, typename VecVal, typename CoefFn>
__device__ __forceinline__ void csr_process_in_flight(const int2 (&e)[kStageFlight], const int2 *entry, int total, float vmax, int nrows, int my_len,
                                                      int my_pre, float *coef, int *acc, int c0, int c1, float *prod,
                                                      FixedAcc &fx, uint32_t *su, int *poison, VecReq vec_req, VecVal vec_val, CoefFn coef_of,
                                                      float (&operand)[kStageFlight])
{
    int col[kStageFlight];
    decltype(vec_req(0, 0, 0)) raw[kStageFlight] = {};
    const int wave_first = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) & ~(kWave - 1));
#pragma unroll
    for (int u = 0; u < kStageFlight; ++u) {
        // (past the end `e` holds whatever the buffer held: column 0 is gathered instead)
        col[u] = static_cast<int>(threadIdx.x) + u * kCsrThreads < total ? e[u].x & kColMask : 0;
        if (!GATED || wave_first + u * kCsrThreads < total) raw[u] = vec_req(col[u], u, u);
    }
#pragma unroll
    for (int u = 0; u < kStageFlight; ++u) {
        const int p = threadIdx.x + u * kCsrThreads;
        if (p < total) {
            operand[u] = vec_val(raw[u], col[u]).x;
            prod[p] = __int_as_float(e[u].y) * operand[u];
        }
    }
    // What more there is, no more than as many again, requested together as well: one entry after the other, two trips to memory
    // each, cost 2236 columns, nine workers of 81 rows of 94 entries, 19.1 us a round, where it is 18.6 (4200 columns, Alg. 2, sixteen
    // workers of 128 rows of 52: 18.3 and 18.0).  Where the model is quantized here batches are light, and what is left of them
    // mostly less than one entry a thread: 4200 columns, eight workers of 64 rows of 75 entries 13.0 us, together 13.1.
    static_assert(kMaxStage <= 2 * kCsrInFlight, "a prepared mini-batch is taken in two batches");
    const int last = total - 1, rest = static_cast<int>(threadIdx.x) + kCsrInFlight, rest_first = wave_first + kCsrInFlight;
    const auto request_rest = [&](int2 (&more)[kStageFlight]) {
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u)
            if (rest_first + u * kCsrThreads < total) more[u] = entry[min(rest + u * kCsrThreads, last)];
    };
    if constexpr (!GATED) {
        for (int p = rest; p < total; p += kCsrThreads) {
            const int2 more = entry[p];
            const int c = more.x & kColMask;
            prod[p] = __int_as_float(more.y) * vec_val(vec_req(c, -1, p), c).x;
        }
    } else if (rest_first < total) {
        int2 more[kStageFlight] = {};
        request_rest(more);
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u)
            if (rest_first + u * kCsrThreads < total) raw[u] = vec_req(more[u].x & kColMask, -1, min(rest + u * kCsrThreads, last));
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u)
            if (rest + u * kCsrThreads < total)
                prod[rest + u * kCsrThreads] = __int_as_float(more[u].y) * vec_val(raw[u], more[u].x & kColMask).x;
    }
    const int lane = threadIdx.x & (kWave - 1);
    if (total <= kPrepNoMax) {
        const uint32_t top = wave_max_u32(static_cast<int>(threadIdx.x) < total ? abs_bits(__int_as_float(e[0].y)) : 0u);
        if (lane == 0) su[threadIdx.x / kWave] = top;
    }
    __syncthreads();
    if (total <= kPrepNoMax) vmax = __uint_as_float(wave_max_u32(lane < kCsrWaves ? su[lane] : 0u));
    // (a wavefront has one or two rows of the common batches of up to 32)
    if (nrows <= (GATED ? 3 : 2) * kCsrWaves) csr_lane_margins<2>(prod, total, nrows, my_len, my_pre, coef_of, coef);
    else csr_lane_margins<kFlight>(prod, total, nrows, my_len, my_pre, coef_of, coef);
    __syncthreads();                                     // (also behind the clearing of acc)
    fixed_admit(fx, coef_abs_sum(coef, 0, nrows) * vmax, acc, c1 - c0, poison);
    const float two_k = ldexpf(1.0f, fx.k);
    float cf[kStageFlight];
#pragma unroll
    for (int u = 0; u < kStageFlight; ++u) cf[u] = coef[(e[u].x >> kColBits) & (kCsrMaxRows - 1)];
#pragma unroll
    for (int u = 0; u < kStageFlight; ++u)
        if (static_cast<int>(threadIdx.x) + u * kCsrThreads < total && col[u] >= c0 && col[u] < c1)
            atomicAdd(&acc[col[u] - c0], fixed_term(cf[u], __int_as_float(e[u].y), two_k));
    if constexpr (!GATED) {
        for (int p = rest; p < total; p += kCsrThreads) {
            const int2 more = entry[p];
            const int c = more.x & kColMask;
            if (c >= c0 && c < c1)
                atomicAdd(&acc[c - c0], fixed_term(coef[(more.x >> kColBits) & (kCsrMaxRows - 1)], __int_as_float(more.y), two_k));
        }
    } else if (rest_first < total) {
        int2 more[kStageFlight] = {};
        request_rest(more);
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u) {
            const int c = more[u].x & kColMask;
            if (rest + u * kCsrThreads < total && c >= c0 && c < c1)
                atomicAdd(&acc[c - c0], fixed_term(coef[(more[u].x >> kColBits) & (kCsrMaxRows - 1)], __int_as_float(more[u].y), two_k));
        }
    }
    __syncthreads();
}

// ------------------------------------------------------------------ worker step
// how the model comes: as its message and the snapshot, as their difference, or as the model itself, not yet quantized
enum { kModelMessage, kModelDiff, kModelPending };

struct CsrWorkerArgs {
    CsrView A;
    const int32_t *idx;
    int B;
    const uint32_t *xq; const float *delta_x; int b_x;
    int64_t model_last_word;       // index of the last word of the model message
    const float *x_snap, *z_snap;
    float l2;
    float *alpha_out; int64_t ld;
    float *absmax_out, *l1norm_out;
    int sparsify, b;
    StreamKey key; uint32_t worker0;
    uint32_t *packed; int64_t ld_words, row_words;
    float *delta_out; int32_t *nnz_out; uint32_t *status;
    int cap;                       // staging capacity in entries
    int prep_cap;                  // most entries of a mini-batch prepared ahead (PrepRoom::cap; never more than cap)
    uint32_t *zero_word;           // nullable: set to 0 by one thread of the grid
    int win;                       // columns of the gradient held in LDS at a time (multiple of 4; >= d: all of it)
    int snap_cap;                  // PrepRoom::snap_cap
    int dev_max_at;               // word of prep_in where WorkerArgs::dev_max lies, 0: not given
    float *alpha_ws; int64_t ld_ws; // with several windows: M rows of workspace for the whole gradient, else null
    // sparsifier split over the identical blocks of a worker (beta_ws != null): each block sparsifies its slice into
    // row m of beta_ws and leaves the slice's largest magnitude and kept count; the quantization is a second launch
    // SLICED: a block leaves its columns of the gradient in row m of beta_ws and their largest magnitude in part_max, one
    // value per slice; with a sparsifier to come, part_max is the message rows, at whose heads the values wait
    // (no fields of their own: arguments that reach into one more 64-byte line cost every launch 0.2 us)
    float *beta_ws; float *part_max; int32_t *part_kept;
    const float *model_diff;       // nullable: (decoded model) - snapshot for every column, see WorkerArgs::model_diff
    // a mini-batch prepared ahead (see PrepLayout): prep_in (nullable) holds this round's, one block of prep_stride words
    // per worker; with prep_out the grid has one more block per worker (the last blockIdx.y), which prepares the round
    // whose streams carry next_iter into prep_out.  Both need B <= kCsrMaxRows, drawn rows (idx == null) and one window of columns per block (the whole vector, or
    // a slice).
    const int32_t *prep_in;
    int32_t *prep_out;
    int64_t prep_stride;
    uint32_t next_iter;
};

// MODEL == kModelDiff: the model comes as a.model_diff (one float per column) instead of the message and the snapshot.
// MODEL == kModelPending: it comes as x itself, and every block quantizes what it needs of it: the columns of its entries,
// and its slice's for the dense part (the blocks of worker 0 store those as the message).  That saves the launch of the
// message, 2.9 us, and costs two gathers per entry for one and a Philox block for each entry and quad: 20,958 columns, eight
// workers of 32 rows 13.1 -> 11.7 us a round (11.5 with the snapshot beside the prepared entries).  At 47,236 columns (two
// quads of a slice per thread, 75 entries a row) it costs more than the launch, 29.0 -> 30.6 us: see csr_run_layout.
// (Measured and dropped: x and its random word as a pair per column, left by the master, so that an entry takes an
// 8-byte gather and no Philox block: 13.0 us; the slice's own quads during the gathers instead of before them: 12.2 us.)
// COMMON: the gradient fits in LDS as one window (SLICED: always), the mini-batch in one pass of rows (B <= kCsrMaxRows),
// and the margins at the snapshot are cached (z_snap given) -- the kernel is then straight-line code with one set of the
// row-processing routines, which leaves the compiler far fewer values to keep alive across its phases.
// PREP: mini-batches may be prepared ahead (prep_in, prep_out); a single step has no use for that code, whose many values
// it would pay for in scalar registers kept elsewhere.
// SLICED: the blocks of a worker share its columns.  Every block stages the whole mini-batch and forms all margins, but
// scatters into, finishes and stores only the columns of its own slice, `win` of them: an eighth of the passes over
// the vector, which are what a block of the other form spends half of its time on (clearing, float window, maximum,
// quantization), and no limit on the width from LDS.  What needs the whole gradient -- scale, sparsifier,
// quantization -- is a later launch's, which finds the gradient in memory and its slices' maxima beside it.
// Measured: see csr_worker.
template <int MODEL, bool COMMON, bool SLICED, bool PREP>
__global__ __launch_bounds__(kCsrThreads) void csr_worker_kernel(const CsrWorkerArgs a)
{
    constexpr bool DIFF = MODEL == kModelDiff, PENDING = MODEL == kModelPending;
    touch_kernel_arguments<sizeof(CsrWorkerArgs)>();
    extern __shared__ __align__(16) float lds[];
    __shared__ RowMeta meta;
    __shared__ float sh_y[kCsrMaxRows];
    __shared__ uint32_t su[kCsrWaves];
    __shared__ int si[kCsrWaves];
    __shared__ double sd[kCsrWaves];
    __shared__ int sh_poison;
    __shared__ uint32_t sh_max;
    const int64_t d = a.A.d;
    const int win = a.win;                                     // columns per window, a multiple of 4
    float *alpha = lds;                                        // the window of the gradient being built: fixed-point sums
    int *acc = reinterpret_cast<int *>(lds);                   // while the rows are added, float32 afterwards
    if (threadIdx.x == 0) {                                    // (published by the barriers of the first row pass)
        sh_poison = 0;
        sh_max = 0u;
    }
    const CsrStage sg = csr_stage_in(lds + win, a.cap, !COMMON && a.z_snap == nullptr);

    const int m = blockIdx.x;
    const ModelMsg msg{a.xq, PENDING || a.b_x == 32 ? 1.0f : a.delta_x[0], a.b_x};
    // (PENDING: the fields of dq_vr_grad's outputs and of the difference carry the model and its largest magnitude)
    const Scale model_scale = PENDING ? make_scale(a.absmax_out[0], a.b_x) : Scale{};
    StreamKey model_key = a.key;
    model_key.worker = DQ_MASTER_ID;
    model_key.tag = DQ_TAG_MODEL;
    // identical copies of the worker that share the tail, or slices (a last one more prepares the next round instead)
    const int slice = blockIdx.y, nslices = static_cast<int>(gridDim.y) - (PREP && a.prep_out ? 1 : 0);
    // (at once without cached margins, behind the preparing block's part with them: 1400 columns, eight workers of 32 rows,
    // 13.1 us a round against 13.4 the other way; 3118 columns, eight workers of 39 rows, 13.9 against 14.1)
    const auto clear_zero_word = [&] {
        if (a.zero_word && m == 0 && slice == 0 && threadIdx.x == 0) *a.zero_word = 0u;
    };
    if (!COMMON) clear_zero_word();
    float *alpha_row = (!SLICED && !COMMON && a.alpha_ws) ? a.alpha_ws + static_cast<int64_t>(m) * a.ld_ws : nullptr;   // only with several windows

    const float inv_B = 1.0f / static_cast<float>(a.B);      // the mean over the mini-batch, as one multiplication per row
    const bool have_z = COMMON || a.z_snap != nullptr;
    uint32_t seen_max = 0;                                     // largest magnitude among the coordinates this thread finishes
    // the model value and the snapshot at column c: the field of column c starts at bit c*b_x of the message and
    // may continue in the next word; both words and the snapshot value are requested without any condition
    struct Gather { uint32_t w0, w1; float xs, diff; };
    const bool straddles = (32 % a.b_x) != 0;                 // (the same for every thread) else a field lies in one word
    auto vec_req = [&](int c) {
        if constexpr (DIFF || PENDING) {
            return Gather{0u, 0u, a.x_snap[c], a.model_diff[c]};     // (DIFF: the snapshot value is only used without cached margins)
        } else {
            const int w = (c * a.b_x) >> 5, last = static_cast<int>(a.model_last_word);   // (fewer than 2^20 words)
            return Gather{a.xq[w], straddles ? a.xq[w + 1 < last ? w + 1 : last] : 0u, a.x_snap[c], 0.0f};
        }
    };
    auto vec_val = [&](const Gather &g, int c) {
        if constexpr (DIFF) return make_float2(g.diff, g.xs);
        if constexpr (PENDING) {                               // (the random bits need no more than the column)
            const uint32_t word = stream_word(model_key, static_cast<uint64_t>(c));
            const int k = model_scale.inv_delta != 0.0f ? quantize_one(g.diff, model_scale, word) : 0;
            return make_float2(model_scale.delta * static_cast<float>(k) - g.xs, g.xs);
        }
        const uint32_t bits = __funnelshift_r(g.w0, g.w1, static_cast<unsigned>(c * a.b_x) & 31u);
        const float q = a.b_x == 32 ? __uint_as_float(bits)
                                    : msg.delta_x * static_cast<float>(sext_field(bits, 0, static_cast<unsigned>(a.b_x)));
        return make_float2(q - g.xs, g.xs);
    };
    auto coef_of = [&](int r, float dz, float zs) {
        if (meta.row[r] < 0) return 0.0f;
        if (have_z) zs = meta.z[r];
        return vr_slope_diff(sh_y[r], zs, dz) * inv_B;
    };
    // the rows of one pass: which sample, where its entries start, how many, its label and cached margin
    struct RowInfo { int row; int64_t start; int len; float y, z; };
    auto row_info = [&](int r0, const StreamKey &round_key) {
        RowInfo ri{-1, 0, 0, 1.0f, 0.0f};
        const int nrows = min(kCsrMaxRows, a.B - r0);
        if (static_cast<int>(threadIdx.x) < nrows) {
            const int r = r0 + threadIdx.x;
            int64_t i;
            if (a.idx) {
                i = a.idx[static_cast<int64_t>(m) * a.B + r];
            } else {
                StreamKey sk = round_key;
                sk.worker = a.worker0 + static_cast<uint32_t>(m);
                sk.tag = DQ_TAG_SAMPLE;
                i = __umulhi(stream_word(sk, static_cast<uint64_t>(r)), static_cast<uint32_t>(a.A.n));
            }
            if (static_cast<uint64_t>(i) < static_cast<uint64_t>(a.A.n)) {
                ri.row = static_cast<int>(i);
                ri.start = a.A.indptr[i];
                ri.len = static_cast<int>(a.A.indptr[i + 1] - ri.start);
                ri.y = a.A.y[i];
                ri.z = have_z ? a.z_snap[i] : 0.0f;
            }
        }
        return ri;
    };
    if (PREP && a.prep_out && slice == nslices) {
        // ---- the extra block: worker m's mini-batch of the next round, left in memory (see PrepLayout)
        StreamKey next_key = a.key;
        next_key.iter = a.next_iter;
        const int nrows = a.B;
        const RowInfo ri = row_info(0, next_key);
        if (static_cast<int>(threadIdx.x) < nrows) {
            meta.row[threadIdx.x] = ri.row;
            meta.start[threadIdx.x] = ri.start;
            meta.len[threadIdx.x] = ri.len;
        }
        csr_prefix_lengths(meta, nrows);
        const PrepLayout at(COMMON ? nrows : kCsrMaxRows);
        int32_t *out = a.prep_out + static_cast<int64_t>(m) * a.prep_stride;
        const int total = meta.pre[nrows];
        const bool fits = total <= a.prep_cap;
        if (static_cast<int>(threadIdx.x) < nrows) {
            out[at.row + threadIdx.x] = ri.row;
            out[at.len + threadIdx.x] = ri.len;
            out[at.pre + threadIdx.x] = meta.pre[threadIdx.x];
            out[at.y + threadIdx.x] = __float_as_int(ri.y);
            out[at.z + threadIdx.x] = __float_as_int(ri.z);
        }
        if (threadIdx.x == 0) {
            out[0] = fits ? 1 : 0;
            out[1] = total;
            out[at.pre + nrows] = total;
        }
        if (m == 0 && threadIdx.x == 0) out[at.dev_max] = 0;
        if (!fits) return;
        int2 *entry = reinterpret_cast<int2 *>(out + at.entries);
        const int lane = threadIdx.x & (kWave - 1);
        uint32_t vmax = 0;
        const bool snaps = COMMON && total <= a.snap_cap;      // (the same for every thread)
        float *entry_snap = reinterpret_cast<float *>(entry + a.snap_cap);
        for (int p0 = threadIdx.x; p0 - lane < total; p0 += kStageFlight * kCsrThreads) {
            int64_t src[kStageFlight];
            int tag[kStageFlight], col[kStageFlight];
            float val[kStageFlight];
#pragma unroll
            for (int u = 0; u < kStageFlight; ++u)
                src[u] = csr_stage_source(meta, 0, nrows, 0, total, p0 - lane + u * kCsrThreads, lane, u ? src[0] : 0, tag[u]);
#pragma unroll
            for (int u = 0; u < kStageFlight; ++u) {
                col[u] = a.A.indices[src[u]];
                val[u] = a.A.values[src[u]];
            }
#pragma unroll
            for (int u = 0; u < kStageFlight; ++u)
                if (p0 + u * kCsrThreads < total) entry[p0 + u * kCsrThreads] = make_int2(col[u] | tag[u], __float_as_int(val[u]));
            if (snaps) {
                float xs[kStageFlight];
#pragma unroll
                for (int u = 0; u < kStageFlight; ++u) xs[u] = a.x_snap[col[u]];
#pragma unroll
                for (int u = 0; u < kStageFlight; ++u)
                    if (p0 + u * kCsrThreads < total) entry_snap[p0 + u * kCsrThreads] = xs[u];
            }
            // (a position past the end repeats an entry of the batch)
#pragma unroll
            for (int u = 0; COMMON && u < kStageFlight; ++u) vmax = max(vmax, abs_bits(val[u]));
        }
        if constexpr (COMMON) {
            if (threadIdx.x == 0) out[3] = snaps ? 1 : 0;
            if (total <= kPrepNoMax) return;                   // (the same for every thread)
            vmax = wave_max_u32(vmax);
            if (lane == 0) atomicMax(&sh_max, vmax);           // (zero since before the barriers of the prefix sums)
            __syncthreads();
            if (threadIdx.x == 0) out[2] = static_cast<int>(sh_max);
        }
        return;
    }
    // PENDING: quad q of the model becomes its difference to the snapshot; the blocks of worker 0 also store the message,
    // each its own slice of it (all lanes of a wavefront make the call; x, xs: the quad's values, r its random words)
    const auto quantize_model_quad = [&](int64_t q, float4 x, float4 xs, const uint4 &r) {
        const int64_t quads = (d + 3) / 4;
        if (4 * q + 3 >= d && q < quads) {                     // the vector ends inside the quad
            const int64_t i = 4 * q;
            x.x = a.model_diff[i];
            x.y = i + 1 < d ? a.model_diff[i + 1] : 0.0f;
            x.z = i + 2 < d ? a.model_diff[i + 2] : 0.0f;
            x.w = 0.0f;
            xs.x = a.x_snap[i];
            xs.y = i + 1 < d ? a.x_snap[i + 1] : 0.0f;
            xs.z = i + 2 < d ? a.x_snap[i + 2] : 0.0f;
            xs.w = 0.0f;
        }
        int k0 = 0, k1 = 0, k2 = 0, k3 = 0;
        if (model_scale.inv_delta != 0.0f) {                   // (a degenerate scale: every code is zero)
            k0 = quantize_one(x.x, model_scale, r.x);
            k1 = quantize_one(x.y, model_scale, r.y);
            k2 = quantize_one(x.z, model_scale, r.z);
            k3 = quantize_one(x.w, model_scale, r.w);
        }
        if (m == 0) {                                          // (the same for the whole block)
            uint32_t *message = const_cast<uint32_t *>(a.xq);
            const int64_t at = q < quads ? q : quads;
            if (a.b_x == 8) store_quad_bits<8>(pack4<8, true, false>(k0, k1, k2, k3), at, quads, message);
            else if (a.b_x == 4) store_quad_bits<4>(q < quads ? pack4<4, true, false>(k0, k1, k2, k3) : 0u, at, quads, message);
            else store_quad_bits<2>(q < quads ? pack4<2, true, false>(k0, k1, k2, k3) : 0u, at, quads, message);
        }
        const float delta = model_scale.delta;
        return make_float4(delta * static_cast<float>(k0) - xs.x, delta * static_cast<float>(k1) - xs.y,
                           delta * static_cast<float>(k2) - xs.z, delta * static_cast<float>(k3) - xs.w);
    };
    if (COMMON) clear_zero_word();
    if (PENDING && m == 0 && slice == 0 && threadIdx.x == 0) {
        const_cast<float *>(a.delta_x)[0] = model_scale.delta;
        if (model_scale.bad && a.status) atomicOr(a.status, 1u);
    }
    // Alg. 2 once the rows are added (not SLICED: this block holds the sums of all columns), without the pass over the
    // whole vector.  A column that no row touches holds l2 * model_diff, which is bounded (WorkerArgs::dev_max); where the
    // largest of the touched ones, which every thread forms from the entries in its registers, is no less than the
    // bound, it is ||alpha||_inf, and all that is left is the block's own slice.  The values are those of the pass,
    // bit for bit.  Returns false (for every thread) where it is not.  72,000 x 20,958, 16 workers of 64 rows: the pass over
    // 5240 quads and the tail behind it took half of the kernel, 12.3 us; now 10.3.
    const int64_t tail_per = (((d + 3) / 4 + nslices - 1) / nslices + kWave - 1) / kWave * kWave, tail_first = tail_per * slice;
    const auto sparsify_touched = [&](const int2 (&e)[kStageFlight], const float (&operand)[kStageFlight], const int2 *entry, int total,
                                      const FixedAcc &fx, float dev_max, float4 own_diff, uint4 own_words) {
        const float unit = ldexpf(1.0f, -fx.k);
        uint32_t seen = 0;
#pragma unroll
        for (int u = 0; u < kStageFlight; ++u)
            if (static_cast<int>(threadIdx.x) + u * kCsrThreads < total) {
                float v = a.l2 * operand[u];
                v += static_cast<float>(acc[e[u].x & kColMask]) * unit;
                seen = max(seen, abs_bits(v));
            }
        for (int p = threadIdx.x + kCsrInFlight; p < total; p += kCsrThreads) {
            const int c = entry[p].x & kColMask;
            float v = a.l2 * a.model_diff[c];
            v += static_cast<float>(acc[c]) * unit;
            seen = max(seen, abs_bits(v));
        }
        seen = block_max_u32(seen, su);
        // (|Q(x) - x| is at most the scale and a rounding of x; a degenerate scale is none, and from one near the end of the range
        // the largest codes come back as infinity)
        const float rest = a.l2 * ((dev_max + msg.delta_x) * 1.001f);
        if (sh_poison || !(rest <= FLT_MAX) || msg.delta_x == 0.0f || msg.delta_x > FLT_MAX / 256.0f || !(seen >= abs_bits(rest))) return false;
        const SparsifyRule rule{__uint_as_float(seen), 0.0f, false};
        StreamKey key = a.key;
        key.worker = a.worker0 + static_cast<uint32_t>(m);
        key.tag = DQ_TAG_SPARSIFY;
        const int64_t quads = (d + 3) / 4, q_hi = min(quads, tail_first + tail_per);
        uint32_t bmax = 0;
        int kept = 0;
        for (int64_t q = tail_first + threadIdx.x; q < q_hi; q += kCsrThreads) {
            if (q != tail_first + threadIdx.x) {
                own_diff = reinterpret_cast<const float4 *>(a.model_diff)[q];
                own_words = stream_block(key, static_cast<uint32_t>(q));
            }
            const int4 sum = reinterpret_cast<const int4 *>(acc)[q];
            float4 v = make_float4(a.l2 * own_diff.x, a.l2 * own_diff.y, a.l2 * own_diff.z, a.l2 * own_diff.w);
            v.y = 4 * q + 1 < d ? v.y : 0.0f;                  // (past the end of the vector nothing was added)
            v.z = 4 * q + 2 < d ? v.z : 0.0f;
            v.w = 4 * q + 3 < d ? v.w : 0.0f;
            v.x = sparsify_one(v.x + static_cast<float>(sum.x) * unit, rule, own_words.x);
            v.y = sparsify_one(v.y + static_cast<float>(sum.y) * unit, rule, own_words.y);
            v.z = sparsify_one(v.z + static_cast<float>(sum.z) * unit, rule, own_words.z);
            v.w = sparsify_one(v.w + static_cast<float>(sum.w) * unit, rule, own_words.w);
            bmax = max(max(bmax, abs_bits(v.x)), max(max(abs_bits(v.y), abs_bits(v.z)), abs_bits(v.w)));
            kept += (v.x != 0.0f) + (v.y != 0.0f) + (v.z != 0.0f) + (v.w != 0.0f);
            store_quad(a.beta_ws + static_cast<int64_t>(m) * a.ld_ws, q, d, v);
        }
        block_max_u32_sum_i32(bmax, kept, su, si);
        if (threadIdx.x == 0) {
            a.part_max[static_cast<int64_t>(m) * nslices + slice] = __uint_as_float(bmax);
            a.part_kept[static_cast<int64_t>(m) * nslices + slice] = kept;
        }
        return true;
    };
    for (int64_t c0 = SLICED ? static_cast<int64_t>(slice) * win : 0; c0 < d; c0 += win) {
        const int64_t c1 = min(d, c0 + win);
        const int64_t c1p = min((d + 3) / 4 * 4, c0 + win);     // the window, up to a whole quad past the end of the vector
        FixedAcc fx{0.0f, 0};
        bool rows_done = false;
        // SLICED: the differences that the finished columns need, requested ahead of the rows (after the scatter they would be
        // one more trip to memory, 0.8 us; in a block that finishes all columns the registers they take cost as much)
        constexpr int kAhead = PENDING ? 1 : 2;
        float4 ahead[kAhead];
        bool have_ahead = false;
        if (PREP && a.prep_in) {
            // ---- this round's mini-batch was prepared: descriptors and the first entries are requested together
            // (a.B <= kCsrMaxRows, one window or slice)
            const PrepLayout at(COMMON ? a.B : kCsrMaxRows);   // (of the launch that left it: constant where registers are short)
            const int32_t *in = a.prep_in + static_cast<int64_t>(m) * a.prep_stride;
            const int2 *entry = reinterpret_cast<const int2 *>(in + at.entries);
            const int nrows = a.B;
            const int ready = in[0], total = in[1];
            int2 first[kStageFlight];
            float first_snap[kStageFlight];
            const float *entry_snap = reinterpret_cast<const float *>(entry + a.snap_cap);
            const auto request_first = [&] {
#pragma unroll
                for (int u = 0; u < kStageFlight; ++u)
                    first[u] = entry[min(static_cast<int>(threadIdx.x) + u * kCsrThreads, a.prep_cap - 1)];
            };
            const auto clear_window = [&] {
                for (int64_t j = 4ll * threadIdx.x; j < c1p - c0; j += 4ll * kCsrThreads)
                    *reinterpret_cast<int4 *>(acc + j) = make_int4(0, 0, 0, 0);
            };
            // (COMMON: lane l of wavefront w holds row w + 16 l, else thread r row r)
            const int lr = !COMMON ? static_cast<int>(threadIdx.x)
                                   : static_cast<int>(threadIdx.x) / kWave + (static_cast<int>(threadIdx.x) & (kWave - 1)) * kCsrWaves;
            const int tr = min(lr, nrows - 1);
            const int p_row = in[at.row + tr], p_len = in[at.len + tr], p_pre = in[at.pre + tr];
            const float p_y = __int_as_float(in[at.y + tr]), p_z = __int_as_float(in[at.z + tr]);
            request_first();
            if constexpr (COMMON) {
                const float vmax = __int_as_float(in[2]);
                const int have_snaps = PENDING ? in[3] : 0;
                const float dev_max = DIFF && !SLICED ? __int_as_float(a.prep_in[a.dev_max_at]) : 0.0f;
                if constexpr (PENDING)
#pragma unroll
                    for (int u = 0; u < kStageFlight; ++u)
                        first_snap[u] = entry_snap[min(static_cast<int>(threadIdx.x) + u * kCsrThreads, a.snap_cap - 1)];
                // (threads past the window read its last whole quad, all of them the same 16 bytes)
                const int first_col = static_cast<int>(c0) + 4 * static_cast<int>(threadIdx.x);
                const int last_quad = max(0, static_cast<int>(min<int64_t>(c1p, d / 4 * 4)) - 4);
                if constexpr (PENDING) {
                    float4 xv[kAhead], sv[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int at = min(first_col + 4 * kCsrThreads * u, last_quad);
                        xv[u] = *reinterpret_cast<const float4 *>(a.model_diff + at);
                        sv[u] = *reinterpret_cast<const float4 *>(a.x_snap + at);
                    }
                    clear_window();
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int64_t j = c0 + 4ll * threadIdx.x + 4ll * kCsrThreads * u;
                        if (j - 4 * (static_cast<int>(threadIdx.x) & (kWave - 1)) >= c1p) continue;      // (a whole wavefront)
                        const uint4 r = stream_block(model_key, static_cast<uint32_t>(j >> 2));
                        ahead[u] = quantize_model_quad(j >> 2, xv[u], sv[u], r);
                    }
                    have_ahead = true;
                }
                if constexpr (DIFF && SLICED) {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u)
                        ahead[u] = *reinterpret_cast<const float4 *>(a.model_diff + min(first_col + 4 * kCsrThreads * u, last_quad));
                    have_ahead = true;
                }
                if constexpr (!PENDING) clear_window();
                float operand[kStageFlight];
                // Alg. 2 with ||x - x_snap||_inf given: the slice's first quad and its random bits, ahead of the rows
                float4 own_diff = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                uint4 own_words = make_uint4(0u, 0u, 0u, 0u);
                const bool short_tail = DIFF && !SLICED && a.dev_max_at != 0 && a.beta_ws && !a.alpha_out;
                if (short_tail) {
                    const int64_t q = min(tail_first + threadIdx.x, (d + 3) / 4 - 1);      // (rows of model_diff are whole quads)
                    own_diff = reinterpret_cast<const float4 *>(a.model_diff)[q];
                    StreamKey key = a.key;
                    key.worker = a.worker0 + static_cast<uint32_t>(m);
                    key.tag = DQ_TAG_SPARSIFY;
                    own_words = stream_block(key, static_cast<uint32_t>(q));
                }
                if (ready) {                                      // (the same for every thread)
                    if (PENDING && !have_snaps)
#pragma unroll
                        for (int u = 0; u < kStageFlight; ++u)
                            first_snap[u] = a.x_snap[static_cast<int>(threadIdx.x) + u * kCsrThreads < total ? first[u].x & kColMask : 0];
                    csr_process_in_flight<!PENDING>(first, entry, total, vmax, nrows, lr < nrows ? p_len : 0, p_pre, meta.coef, acc,
                                          static_cast<int>(c0), static_cast<int>(c1), sg.prod_a, fx, su, &sh_poison,
                                          [&](int c, int u, int p) {           // (entry p at column c; u >= 0: one of the first)
                                              if constexpr (!PENDING) return vec_req(c);
                                              else return Gather{0u, 0u, u >= 0 ? first_snap[u] : have_snaps ? entry_snap[p] : a.x_snap[c], a.model_diff[c]};
                                          }, vec_val,
                                          [&](float dz) { return p_row < 0 ? 0.0f : vr_slope_diff(p_y, p_z, dz) * inv_B; }, operand);
                    rows_done = true;
                    if constexpr (DIFF && !SLICED) {
                        if (short_tail && sparsify_touched(first, operand, entry, total, fx, dev_max, own_diff, own_words)) return;
                    }
                }
            } else {
                clear_window();
            }
            if (!COMMON && ready) {
                if (lr < nrows) {
                    meta.row[lr] = p_row;
                    meta.len[lr] = p_len;
                    meta.pre[lr] = p_pre;
                    sh_y[lr] = p_y;
                    meta.z[lr] = p_z;
                }
                if (threadIdx.x == 0) meta.pre[nrows] = total;
                __syncthreads();
                // (one pass of rows in one window or slice, and not COMMON: no cached margins)
                csr_process_prepared(entry, first, total, meta, nrows, acc, static_cast<int>(c0), static_cast<int>(c1), sg, fx, su,
                                     &sh_poison, vec_req, vec_val, coef_of);
                rows_done = true;
            }
        }
        for (int r0 = 0; r0 < a.B && !rows_done; r0 += kCsrMaxRows) {     // passes of at most kCsrMaxRows rows
            const int nrows = min(kCsrMaxRows, a.B - r0);
            const RowInfo ri = row_info(r0, a.key);
            if (r0 == 0)                                       // (the window is cleared while the row loads are on their way)
                for (int64_t j = 4ll * threadIdx.x; j < c1p - c0; j += 4ll * kCsrThreads)
                    *reinterpret_cast<int4 *>(acc + j) = make_int4(0, 0, 0, 0);
            if (static_cast<int>(threadIdx.x) < nrows) {
                meta.row[threadIdx.x] = ri.row;
                meta.start[threadIdx.x] = ri.start;
                meta.len[threadIdx.x] = ri.len;
                sh_y[threadIdx.x] = ri.y;
                meta.z[threadIdx.x] = ri.z;
            }
            csr_prefix_lengths(meta, nrows);
            if (have_z)
                csr_process_rows<false>(a.A, meta, nrows, acc, static_cast<int>(c0), static_cast<int>(c1), sg, fx, su,
                                        &sh_poison, vec_req, vec_val, coef_of);
            else
                csr_process_rows<true>(a.A, meta, nrows, acc, static_cast<int>(c0), static_cast<int>(c1), sg, fx, su,
                                       &sh_poison, vec_req, vec_val, coef_of);
            if constexpr (COMMON) break;                       // (one pass)
        }
        // the window becomes float32: the dense part  l2*(q - snapshot)  plus the accumulated sums, zero past the end
        // of the vector; four coordinates per thread and step
        {
            const float unit = sh_poison ? __uint_as_float(0x7FC00000u) : ldexpf(1.0f, -fx.k);
            // (nothing was added past the end of the vector: the sums there are zero)
            const auto finish_quad = [&](int64_t j, float4 v) {
                const int4 sum = *reinterpret_cast<const int4 *>(acc + (j - c0));
                v.x += static_cast<float>(sum.x) * unit; v.y += static_cast<float>(sum.y) * unit;
                v.z += static_cast<float>(sum.z) * unit; v.w += static_cast<float>(sum.w) * unit;
                if constexpr (SLICED) *reinterpret_cast<float4 *>(a.beta_ws + static_cast<int64_t>(m) * a.ld_ws + j) = v;
                else *reinterpret_cast<float4 *>(alpha + (j - c0)) = v;
                if (SLICED && a.alpha_out) store_quad(a.alpha_out + static_cast<int64_t>(m) * a.ld, j >> 2, d, v);
                seen_max = max(max(seen_max, abs_bits(v.x)), max(max(abs_bits(v.y), abs_bits(v.z)), abs_bits(v.w)));
            };
            const auto slow_quad = [&](int64_t j) {
                float t[4];
                for (int e = 0; e < 4; ++e) {
                    if constexpr (DIFF) t[e] = j + e < d ? a.l2 * a.model_diff[j + e] : 0.0f;
                    else t[e] = j + e < d ? a.l2 * (model_value(msg, j + e) - a.x_snap[j + e]) : 0.0f;
                }
                finish_quad(j, make_float4(t[0], t[1], t[2], t[3]));
            };
            const int64_t whole = min(c1p, d / 4 * 4);            // whole quads of the vector end here
            if constexpr (PENDING) {
                // (a slice is whole wavefronts of quads, so the lanes of one go through this together)
                const auto finish_model_quad = [&](int64_t j, float4 df) {
                    const int64_t past = d - j;                  // coordinates left; those past the end stay zero
                    if (past > 0)
                        finish_quad(j, make_float4(a.l2 * df.x, past > 1 ? a.l2 * df.y : 0.0f, past > 2 ? a.l2 * df.z : 0.0f,
                                                   past > 3 ? a.l2 * df.w : 0.0f));
                };
                if (have_ahead) {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int64_t j = c0 + 4ll * threadIdx.x + 4ll * kCsrThreads * u;
                        if (j < c1p) finish_model_quad(j, ahead[u]);
                    }
                }
                const int64_t lane4 = 4 * (static_cast<int>(threadIdx.x) & (kWave - 1));
                for (int64_t j = c0 + 4ll * threadIdx.x + (have_ahead ? 4ll * kCsrThreads * kAhead : 0); j - lane4 < c1p;
                     j += 4ll * kCsrThreads) {
                    const int64_t at = min<int64_t>(j, d / 4 * 4 - 4);
                    const float4 x = *reinterpret_cast<const float4 *>(a.model_diff + at);
                    const float4 xs = *reinterpret_cast<const float4 *>(a.x_snap + at);
                    const float4 df = quantize_model_quad(j >> 2, x, xs, stream_block(model_key, static_cast<uint32_t>(j >> 2)));
                    if (j < c1p) finish_model_quad(j, df);
                }
            } else if constexpr (DIFF) {
                constexpr int kInitFlight = 6;                   // (as below: requested together, at clamped positions)
                if (have_ahead) {                                // (the same for every thread)
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int64_t j = c0 + 4ll * threadIdx.x + 4ll * kCsrThreads * u;
                        if (j < whole)
                            finish_quad(j, make_float4(a.l2 * ahead[u].x, a.l2 * ahead[u].y, a.l2 * ahead[u].z, a.l2 * ahead[u].w));
                    }
                }
                for (int64_t j0 = c0 + 4ll * threadIdx.x + (have_ahead ? 4ll * kCsrThreads * kAhead : 0); j0 < whole; j0 += 4ll * kCsrThreads * kInitFlight) {
                    float4 df[kInitFlight];
#pragma unroll
                    for (int u = 0; u < kInitFlight; ++u)
                        df[u] = *reinterpret_cast<const float4 *>(
                            a.model_diff + min<int64_t>(j0 + 4ll * kCsrThreads * u, whole - 4));
#pragma unroll
                    for (int u = 0; u < kInitFlight; ++u) {
                        const int64_t j = j0 + 4ll * kCsrThreads * u;
                        if (j < whole) finish_quad(j, make_float4(a.l2 * df[u].x, a.l2 * df[u].y, a.l2 * df[u].z, a.l2 * df[u].w));
                    }
                }
                if (threadIdx.x == 0 && whole >= c0 && whole < c1p) slow_quad(whole);      // the vector ends inside a quad
            } else if (a.b_x == 8) {
                // the loads of kInitFlight steps are requested together (at clamped positions: a load behind a
                // per-lane test would be waited for before the next one is issued)
                constexpr int kInitFlight = 6;
                for (int64_t j0 = c0 + 4ll * threadIdx.x; j0 < whole; j0 += 4ll * kCsrThreads * kInitFlight) {
                    float4 xs[kInitFlight];
                    uint32_t w[kInitFlight];
#pragma unroll
                    for (int u = 0; u < kInitFlight; ++u) {
                        const int64_t jc = min(j0 + 4ll * kCsrThreads * u, whole - 4);
                        xs[u] = *reinterpret_cast<const float4 *>(a.x_snap + jc);
                        w[u] = a.xq[jc >> 2];
                    }
#pragma unroll
                    for (int u = 0; u < kInitFlight; ++u) {
                        const int64_t j = j0 + 4ll * kCsrThreads * u;
                        if (j < whole)
                            finish_quad(j, make_float4(a.l2 * (msg.delta_x * static_cast<float>(sext_field(w[u], 0, 8)) - xs[u].x),
                                                       a.l2 * (msg.delta_x * static_cast<float>(sext_field(w[u], 8, 8)) - xs[u].y),
                                                       a.l2 * (msg.delta_x * static_cast<float>(sext_field(w[u], 16, 8)) - xs[u].z),
                                                       a.l2 * (msg.delta_x * static_cast<float>(sext_field(w[u], 24, 8)) - xs[u].w)));
                    }
                }
                if (threadIdx.x == 0 && whole >= c0 && whole < c1p) slow_quad(whole);      // the vector ends inside a quad
            } else {
                for (int64_t j = c0 + 4ll * threadIdx.x; j < c1p; j += 4ll * kCsrThreads) slow_quad(j);
            }
            if constexpr (!SLICED) __syncthreads();
        }
        if (alpha_row) {                                       // several windows: the finished one goes to memory
            for (int64_t j = c0 + threadIdx.x; j < c1p; j += kCsrThreads) alpha_row[j] = alpha[j - c0];
            __syncthreads();
        }
        if constexpr (COMMON || SLICED) break;                 // (one window)
    }
    if constexpr (SLICED) {
        const int64_t stride = a.sparsify ? a.ld_words : nslices;
        seen_max = wave_max_u32(seen_max);
        if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(&sh_max, seen_max);
        __syncthreads();
        if (threadIdx.x == 0) a.part_max[m * stride + slice] = __uint_as_float(sh_max);
        return;
    }
    // the whole gradient, padded with zeros to a whole quad: in LDS when it fits in one window, else in this worker's
    // workspace row (the block's own writes, visible to all its threads after the barrier above)
    float *av = alpha_row ? alpha_row : alpha;

    // 4. outputs
    if (a.alpha_out && slice == 0)
        for (int64_t j = threadIdx.x; j < d; j += kCsrThreads) a.alpha_out[static_cast<int64_t>(m) * a.ld + j] = av[j];
    if (!a.packed) {
        uint32_t vmax = 0;
        double s1 = 0.0;
        for (int64_t j = threadIdx.x; j < d; j += kCsrThreads) {
            vmax = max(vmax, abs_bits(av[j]));
            s1 += static_cast<double>(fabsf(av[j]));
        }
        vmax = block_max_u32(vmax, su);
        if (threadIdx.x == 0) a.absmax_out[m] = __uint_as_float(vmax);
        if (a.l1norm_out) {
            s1 = block_sum_f64(s1, sd);
            if (threadIdx.x == 0) a.l1norm_out[m] = static_cast<float>(s1);
        }
        return;
    }
    StreamKey key = a.key;
    key.worker = a.worker0 + static_cast<uint32_t>(m);
    if (a.beta_ws) {
        sparsify_slice_from_lds<true>(av, d, key, slice, nslices, a.beta_ws + static_cast<int64_t>(m) * a.ld_ws,
                                      a.part_max + static_cast<int64_t>(m) * nslices + slice,
                                      a.part_kept + static_cast<int64_t>(m) * nslices + slice, su, si, &seen_max);
        return;
    }
    const WorkerOut out{a.packed + static_cast<int64_t>(m) * a.ld_words, a.row_words, a.delta_out + m,
                        a.nnz_out ? a.nnz_out + m : nullptr, a.status};
    switch (a.b) {
    case 2: worker_tail_from_lds<2, true>(av, d, a.sparsify != 0, a.b, key, out, su, si, slice, nslices, &seen_max); break;
    case 4: worker_tail_from_lds<4, true>(av, d, a.sparsify != 0, a.b, key, out, su, si, slice, nslices, &seen_max); break;
    case 32: worker_tail_from_lds<32, true>(av, d, a.sparsify != 0, a.b, key, out, su, si, slice, nslices, &seen_max); break;
    default: worker_tail_from_lds<8, true>(av, d, a.sparsify != 0, a.b, key, out, su, si, slice, nslices, &seen_max); break;
    }
}

// Alg. 2, worker (ii) on gradients that a SLICED launch left in memory: grid (M, slices).  Each block takes ||alpha||_inf
// from the maxima that launch left per slice (alpha_parts of them, at alpha_max + m * alpha_max_stride), sparsifies a slice
// of the quads of row m in place and leaves the slice's largest magnitude and kept count.  Rows are padded with
// zeros to whole quads.  Everything is requested, and the first quad's random bits drawn, before anything is waited for.
// wire (nullable): wire_words words of each of its rows are set to zero, for sparse_message_parts_kernel.
__global__ __launch_bounds__(kCsrThreads) void sparsify_parts_kernel(
    float *__restrict__ rows, int64_t ld, int64_t d, const float *__restrict__ alpha_max, int64_t alpha_max_stride,
    int alpha_parts, StreamKey key, uint32_t worker0, float *__restrict__ part_max, int32_t *__restrict__ part_kept, int per,
    uint32_t *__restrict__ wire, int64_t ld_wire, int wire_words)
{
    touch_kernel_arguments<120>();
    __shared__ uint32_t su[kCsrWaves];
    __shared__ int si[kCsrWaves];
    const int m = blockIdx.x, slice = blockIdx.y, nslices = gridDim.y;
    const int64_t quads = (d + 3) / 4;
    const int64_t q_lo = min<int64_t>(quads, static_cast<int64_t>(per) * slice), q_hi = min<int64_t>(quads, q_lo + per), q_first = q_lo + threadIdx.x;
    float4 *row = reinterpret_cast<float4 *>(rows + static_cast<int64_t>(m) * ld);
    const PartsRaw maxima = parts_request(alpha_max + static_cast<int64_t>(m) * alpha_max_stride, alpha_parts);
    float4 v = row[min(q_first, quads - 1)];
    __builtin_amdgcn_sched_barrier(0);
    key.worker = worker0 + static_cast<uint32_t>(m);
    key.tag = DQ_TAG_SPARSIFY;
    uint4 w = stream_block(key, static_cast<uint32_t>(q_first));
    asm volatile("" ::"v"(w.x), "v"(w.y), "v"(w.z), "v"(w.w));
    __builtin_amdgcn_sched_barrier(0);
    if (wire) {
        uint32_t *words = wire + static_cast<int64_t>(m) * ld_wire;
        for (int w = slice * kCsrThreads + threadIdx.x; w < wire_words; w += nslices * kCsrThreads) words[w] = 0u;
    }
    const SparsifyRule rule{parts_absmax_of(maxima), 0.0f, false};
    uint32_t bmax = 0;
    int kept = 0;
    for (int64_t q = q_first; q < q_hi; q += kCsrThreads) {
        if (q != q_first) {
            v = row[q];
            w = stream_block(key, static_cast<uint32_t>(q));
        }
        v.x = sparsify_one(v.x, rule, w.x);
        v.y = sparsify_one(v.y, rule, w.y);
        v.z = sparsify_one(v.z, rule, w.z);
        v.w = sparsify_one(v.w, rule, w.w);
        bmax = max(max(bmax, abs_bits(v.x)), max(max(abs_bits(v.y), abs_bits(v.z)), abs_bits(v.w)));
        kept += (v.x != 0.0f) + (v.y != 0.0f) + (v.z != 0.0f) + (v.w != 0.0f);
        row[q] = v;
    }
    block_max_u32_sum_i32(bmax, kept, su, si);
    if (threadIdx.x == 0) {
        part_max[static_cast<int64_t>(m) * nslices + slice] = __uint_as_float(bmax);
        part_kept[static_cast<int64_t>(m) * nslices + slice] = kept;
    }
}

// ------------------------------------------------------------------ epoch prologue
// Grid (P): block p owns rows [p*per, (p+1)*per), in chunks of kFlushRows.  What bounds it is latency and the instructions
// of sixteen wavefronts on one compute unit: a block has one to itself (the sums of up to 35 k columns in LDS) and
// some fifteen thousand entries to fetch, each with a gather behind it.  So there is no staging and no barrier between
// the rows: L lanes of a wavefront take a row, ROWS such rows at a time straight from memory -- CHUNKS pieces of L
// entries of each requested together, then their gathers --, add up its margin and keep its coefficient in LDS.  Once all
// rows of the chunk have theirs, one barrier gives the bound that fixes the unit of the fixed-point sums (FixedAcc),
// and the same lanes add the rows' entries (from L2 now) to the columns.  A batch's first entries are requested before those
// of the one before are used: a trip to memory less for each.  72,000 rows of 52 entries, 20,958
// columns: 50.4 us with rows staged in LDS in groups of a hundred, five barrier-separated phases each; now 27.5 us by
// itself and 29 inside epochs; 80,000 rows of 100 entries, 60,000 columns 236 -> 64 us; 40,000 rows of 20, 2000 columns 14.7 -> 13.4 us.
constexpr int64_t kFullLds = 136 * 1024;                  // for the columns; 12.5 KB of static arrays beside them
constexpr int kTogether = 256;                            // positions of a row up to here are its own lanes' work

// The rows of a chunk in LDS, and where their entries lie: a scalar base and 32-bit byte offsets (1024 rows of fewer than
// 2^20 entries each), so that a load takes two instructions of address arithmetic.
struct FullChunk {
    const char *indices, *values;
    int rows;                                             // of the chunk
    const uint32_t *start;                                // of a row's entries, in bytes of either array
    const int *len;
    float *coef;                                          // the row's label until its coefficient is known
    __device__ __forceinline__ uint32_t index_at(uint32_t at) const { return *reinterpret_cast<const uint32_t *>(indices + at); }
    __device__ __forceinline__ float value_at(uint32_t at) const { return *reinterpret_cast<const float *>(values + at); }
};

// L lanes a row, ROWS * (64 / L) rows a batch, CHUNKS pieces of L entries at a time.
template <int L, int ROWS, int CHUNKS>
struct FullShapeOf {};

// ROWS * (64 / L) of the wavefront's rows, all per lane but `longest` (of the whole wavefront).  A row past the chunk's end has
// length 0, and a row of length 0 the start 0 of an entry that exists wherever any row has one.
template <int ROWS>
struct FullBatch {
    int row[ROWS], len[ROWS], longest;
    uint32_t st[ROWS];
};

template <int L, int ROWS>
__device__ __forceinline__ FullBatch<ROWS> full_batch(const FullChunk &ch, int r)
{
    constexpr int G = kWave / L;
    const int lane = threadIdx.x & (kWave - 1);
    FullBatch<ROWS> b;
    b.longest = 0;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        b.row[u] = r + u * G * kCsrWaves + (L == kWave ? 0 : lane / L);
        const int rc = min(b.row[u], ch.rows - 1), len = ch.len[rc];
        const uint32_t st = ch.start[rc];
        b.len[u] = b.row[u] < ch.rows ? len : 0;
        b.st[u] = b.len[u] > 0 ? st : 0u;
        if constexpr (L == kWave) {                       // (the same for all lanes: scalars)
            b.len[u] = __builtin_amdgcn_readfirstlane(b.len[u]);
            b.st[u] = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b.st[u])));
        }
        b.longest = max(b.longest, b.len[u]);
    }
    if constexpr (L != kWave) b.longest = static_cast<int>(wave_max_u32(static_cast<uint32_t>(b.longest)));
    return b;
}

template <int L, int ROWS, int CHUNKS>
__device__ __forceinline__ void full_fetch(const FullChunk &ch, const uint32_t (&st)[ROWS], const int (&len)[ROWS], int k,
                                           uint32_t (&col)[ROWS][CHUNKS], float (&val)[ROWS][CHUNKS])
{
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {                // (a lane past a row's end repeats its last entry)
            const uint32_t at = st[u] + min(4u * static_cast<uint32_t>(k + c * L), 4u * (max(len[u], 1) - 1u));
            col[u][c] = ch.index_at(at);
            val[u][c] = ch.value_at(at);
        }
}

// The wavefront's rows, a batch at a time: each_piece(batch, k, col, val, between) with the entries k, k + L, ... of its rows'
// lanes, then each_batch(batch).  A batch's first entries are requested while those before are worked on: each_piece calls
// `between` once it has requested what it needs itself.
template <int L, int ROWS, int CHUNKS, typename Start, typename Piece, typename Finish>
__device__ __forceinline__ void full_sweep(const FullChunk &ch, Start start, Piece each_piece, Finish each_batch)
{
    constexpr int G = kWave / L, kStep = ROWS * G * kCsrWaves;
    const int lane = threadIdx.x & (kWave - 1), in_row = lane % L, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int r = wave * G;
    if (r >= ch.rows) return;
    uint32_t col[ROWS][CHUNKS], next_col[ROWS][CHUNKS];
    float val[ROWS][CHUNKS], next_val[ROWS][CHUNKS];
    FullBatch<ROWS> b = full_batch<L, ROWS>(ch, r), next = b;
    if (b.longest > 0) full_fetch<L, ROWS, CHUNKS>(ch, b.st, b.len, in_row, col, val);
    for (;;) {
        const bool more = !(L == 16 && ROWS == 5) && r + kStep < ch.rows;      // (five rows are for all of a wavefront's at once)
        const auto between = [&] {
            if (!more) return;
            next = full_batch<L, ROWS>(ch, r + kStep);
            if (next.longest > 0) full_fetch<L, ROWS, CHUNKS>(ch, next.st, next.len, in_row, next_col, next_val);
        };
        start(b);
        if (b.longest > 0) each_piece(b, in_row, col, val, between);
        else between();
        for (int k = in_row + CHUNKS * L; k - in_row < min(b.longest, kTogether); k += CHUNKS * L) {
            full_fetch<L, ROWS, CHUNKS>(ch, b.st, b.len, k, col, val);
            each_piece(b, k, col, val, [] {});
        }
        each_batch(b);
        if (!more) break;
        r += kStep;
        b = next;
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
            for (int c = 0; c < CHUNKS; ++c) {
                col[u][c] = next_col[u][c];
                val[u][c] = next_val[u][c];
            }
    }
}

// Margins, losses and coefficients of the chunk's rows; the lanes' share of sum |coefficient| and the largest |value|.
template <int L, int ROWS, int CHUNKS>
__device__ __forceinline__ void full_margins(FullShapeOf<L, ROWS, CHUNKS>, const FullChunk &ch, const float *__restrict__ x, float *__restrict__ z_out,
                                             float inv_n, double &loss, float &csum, uint32_t &vmax)
{
    const int lane = threadIdx.x & (kWave - 1), in_row = lane % L;
    const auto x_at = [&](uint32_t col) { return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(x) + 4u * col); };
    float sum[ROWS];
    full_sweep<L, ROWS, CHUNKS>(ch, [&](const FullBatch<ROWS> &) {
#pragma unroll
        for (int u = 0; u < ROWS; ++u) sum[u] = 0.0f;
    }, [&](const FullBatch<ROWS> &b, int k, const uint32_t (&col)[ROWS][CHUNKS], const float (&val)[ROWS][CHUNKS], auto between) {
        float xv[ROWS][CHUNKS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
            for (int c = 0; c < CHUNKS; ++c) xv[u][c] = x_at(col[u][c]);
        between();
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
            for (int c = 0; c < CHUNKS; ++c) {
                vmax = max(vmax, abs_bits(val[u][c]));
                const int p = k + c * L;                  // (positions past kTogether: below)
                sum[u] += p < min(b.len[u], kTogether) ? val[u][c] * xv[u][c] : 0.0f;
            }
    }, [&](const FullBatch<ROWS> &b) {
        const auto &row = b.row;
        const auto &len = b.len;
        const auto &st = b.st;
        const int longest = b.longest;
        // what rows of more than kTogether entries have left: the whole wavefront's, eight pieces of 64 at a time
        if (longest > kTogether) {
#pragma unroll
            for (int u = 0; u < ROWS; ++u)
                for (int g = 0; g < kWave / L; ++g) {
                    const int n = __builtin_amdgcn_readlane(len[u], g * L);
                    const uint32_t s = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(st[u]), g * L));
                    if (n <= kTogether) continue;
                    constexpr int kFlight = 8;
                    float t = 0.0f;
                    for (int k = kTogether + lane; k - lane < n; k += kFlight * kWave) {
                        uint32_t col[kFlight];
                        float val[kFlight], xv[kFlight];
#pragma unroll
                        for (int v = 0; v < kFlight; ++v) {
                            const uint32_t at = s + 4u * min(k + v * kWave, n - 1);
                            col[v] = ch.index_at(at);
                            val[v] = ch.value_at(at);
                        }
#pragma unroll
                        for (int v = 0; v < kFlight; ++v) xv[v] = x_at(col[v]);
#pragma unroll
                        for (int v = 0; v < kFlight; ++v) {
                            vmax = max(vmax, abs_bits(val[v]));
                            t += k + v * kWave < n ? val[v] * xv[v] : 0.0f;
                        }
                    }
                    t = wave_sum_f32(t);
                    sum[u] += lane == g * L ? t : 0.0f;
                }
        }
        // the row's sum reaches its last lane (L = 16: two quad permutes and two row shifts); for L = 64 lane u takes row u
        float z = 0.0f, y = 0.0f;
        int at = -1;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            float t = sum[u];
            if constexpr (L == kWave) {
                t = wave_sum_f32(t);
                z = lane == u ? t : z;
                at = lane == u ? row[u] : at;
            } else {
                static_assert(L == 16, "lanes per row");
                t += __int_as_float(dpp_move_or_zero<0xb1, 0xf>(__float_as_int(t)));
                t += __int_as_float(dpp_move_or_zero<0x4e, 0xf>(__float_as_int(t)));
                t += __int_as_float(dpp_move_or_zero<0x114, 0xf>(__float_as_int(t)));
                t += __int_as_float(dpp_move_or_zero<0x118, 0xf>(__float_as_int(t)));
                // lane 15 of the row's lanes holds the sum; lane 15 - u is the one that evaluates row u
                t = __shfl(t, lane | (L - 1), kWave);
                z = in_row == L - 1 - u ? t : z;
                at = in_row == L - 1 - u ? row[u] : at;
            }
        }
        if (at >= 0 && at < ch.rows) {
            y = ch.coef[at];
            // (hardware exp, log and reciprocal, as in the dense kernel)
            const float coef = logistic_slope_fast(y, z) * inv_n;
            if (z_out) z_out[at] = z;
            loss += static_cast<double>(logistic_loss_fast(y * z));
            ch.coef[at] = coef;
            csum += fabsf(coef);
        }
    });
}

// The entries of the chunk's rows in columns lo .. lo + wide - 1 are added to acc.
template <int L, int ROWS, int CHUNKS>
__device__ __forceinline__ void full_scatter(FullShapeOf<L, ROWS, CHUNKS>, const FullChunk &ch, int *acc, uint32_t lo, uint32_t wide, float two_k)
{
    const int lane = threadIdx.x & (kWave - 1);
    float coef[ROWS];
    full_sweep<L, ROWS, CHUNKS>(ch, [&](const FullBatch<ROWS> &b) {
#pragma unroll
        for (int u = 0; u < ROWS; ++u) coef[u] = ch.coef[min(b.row[u], ch.rows - 1)];
    }, [&](const FullBatch<ROWS> &b, int k, const uint32_t (&col)[ROWS][CHUNKS], const float (&val)[ROWS][CHUNKS], auto between) {
        between();
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
            for (int c = 0; c < CHUNKS; ++c)
                if (k + c * L < min(b.len[u], kTogether) && col[u][c] - lo < wide)
                    atomicAdd(&acc[col[u][c] - lo], fixed_term(coef[u], val[u][c], two_k));
    }, [&](const FullBatch<ROWS> &b) {
        const auto &len = b.len;
        const auto &st = b.st;
        const int longest = b.longest;
        if (longest > kTogether) {
#pragma unroll
            for (int u = 0; u < ROWS; ++u)
                for (int g = 0; g < kWave / L; ++g) {
                    const int n = __builtin_amdgcn_readlane(len[u], g * L);
                    const uint32_t s = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(st[u]), g * L));
                    const float cf = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(coef[u]), g * L));
                    for (int k = kTogether + lane; k < n; k += kWave) {
                        const uint32_t c = ch.index_at(s + 4u * k);
                        if (c - lo < wide) atomicAdd(&acc[c - lo], fixed_term(cf, ch.value_at(s + 4u * k), two_k));
                    }
                }
        }
    });
}

__global__ __launch_bounds__(kCsrThreads) void csr_full_partial_kernel(
    const CsrView A, const float *__restrict__ x, float *__restrict__ z_out, float *__restrict__ partial, int64_t ldp,
    double *__restrict__ loss_partial, int win)
{
    extern __shared__ __align__(16) float lds[];
    __shared__ uint32_t sh_start[kFlushRows];
    __shared__ int sh_len[kFlushRows];
    __shared__ float sh_coef[kFlushRows];
    __shared__ double sh_loss[kCsrWaves];
    __shared__ uint32_t su[kCsrWaves];
    __shared__ float sf[kCsrWaves];
    int *acc = reinterpret_cast<int *>(lds);             // the window [c0, c1) of this block's partial sum, fixed point
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t per = (A.n + gridDim.x - 1) / gridDim.x;
    const int64_t i0 = blockIdx.x * per, i1 = min(A.n, i0 + per);
    const float inv_n = 1.0f / static_cast<float>(A.n);
    double loss = 0.0;                                   // the lanes that evaluate row scalars add to theirs
    float *mine = partial + static_cast<int64_t>(blockIdx.x) * ldp;
    for (int64_t j = 4ll * threadIdx.x; j < min<int64_t>(win, ldp); j += 4ll * kCsrThreads)
        *reinterpret_cast<int4 *>(acc + j) = make_int4(0, 0, 0, 0);
    if (i0 >= i1)                                        // a block without rows
        for (int64_t j = 4ll * threadIdx.x; j < ldp; j += 4ll * kCsrThreads)
            *reinterpret_cast<float4 *>(mine + j) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int64_t ib = i0; ib < i1; ib += kFlushRows) {
        const int cn = static_cast<int>(min<int64_t>(kFlushRows, i1 - ib));
        const auto scalar64 = [](int64_t v) {
            return (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32)))) << 32) |
                   static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
        };
        // (requested side by side, for rows that exist: one trip to memory; kFlushRows = kCsrThreads)
        const int64_t i = ib + min(static_cast<int>(threadIdx.x), cn - 1);
        const int64_t first = A.indptr[ib], last = A.indptr[ib + cn], row_first = A.indptr[i], row_last = A.indptr[i + 1];
        const float label = A.y[i];
        const uint64_t e0 = scalar64(first), e1 = scalar64(last);
        if (static_cast<int>(threadIdx.x) < cn) {
            sh_start[threadIdx.x] = static_cast<uint32_t>(static_cast<uint64_t>(row_first) - e0) * 4u;
            sh_len[threadIdx.x] = static_cast<int>(row_last - row_first);
            sh_coef[threadIdx.x] = label;
        }
        __syncthreads();
        const FullChunk ch{reinterpret_cast<const char *>(A.indices + e0), reinterpret_cast<const char *>(A.values + e0), cn,
                           sh_start, sh_len, sh_coef};
        // A row on a whole wavefront, or four rows side by side, which is worth the more the more rows there are and the shorter
        // they are (5000 columns): 80,000 rows of 28 entries, 312 a block, 21.0 us on quarters and 25.6 on whole wavefronts;
        // 30,000 of 20, 117 a block, 17.1 and 19.0, of 28 entries 19.0 and 19.3; up to 96 rows a block whole wavefronts are at
        // least as good: 8000 of 24 entries 15.8 and 13.7.
        const bool short_rows = cn > 96 && e1 - e0 <= static_cast<uint64_t>(cn > 192 ? 32 : 24) * static_cast<uint64_t>(cn);
        // Rows of a batch: a place without a row costs what one with a row does, so of two sizes the one that leaves fewer.  Whole
        // wavefronts, threes and fours: 72,000 rows of 52 entries, 18 a wavefront, 33.0 and 34.2 us; 20,242 of 75, five a
        // wavefront, 36.8 and 38.6; 8000 of 24, four a wavefront, 14.1 and 12.7.  (Sixes with nothing requested ahead: 33.9, 37.6,
        // 14.1.)  Quarters: 30,000 rows of 20, two turns, in pairs 14.6, in threes 15.8, all of five 17.6; 80,000 of 28, five turns, in
        // threes 20.8, all at once 20.4.
        const int turns = (cn + kCsrWaves - 1) / kCsrWaves, quarter_turns = (cn + 4 * kCsrWaves - 1) / (4 * kCsrWaves);
        const bool threes = (turns + 2) / 3 * 3 < (turns + 3) / 4 * 4, pairs = quarter_turns <= 2, fives = quarter_turns == 4 || quarter_turns == 5;
        const auto with_batches = [&](auto f) {
            if (!short_rows) {
                if (threes) f(FullShapeOf<kWave, 3, 2>{});
                else f(FullShapeOf<kWave, 4, 2>{});
            } else if (fives) {
                f(FullShapeOf<16, 5, 3>{});
            } else if (pairs) {
                f(FullShapeOf<16, 2, 3>{});
            } else {
                f(FullShapeOf<16, 3, 3>{});
            }
        };
        uint32_t vmax = 0;
        float csum = 0.0f;
        float *z_chunk = z_out ? z_out + ib : nullptr;
        with_batches([&](auto shape) { full_margins(shape, ch, x, z_chunk, inv_n, loss, csum, vmax); });
        csum = wave_sum_f32(csum);
        if (lane == 0) sf[wave] = csum;
        vmax = block_max_u32(vmax, su);                  // (its barriers also publish sf, the coefficients, the cleared sums)
        const float bound = wave_sum_f32(lane < kCsrWaves ? sf[lane] : 0.0f) * __uint_as_float(vmax);
        // The fixed-point sums go to this block's float32 partial vector after every chunk: a term is rounded relative to
        // the bound of everything in the accumulator, which grows with the number of rows, so that number is kept small.
        const bool finite = bound <= FLT_MAX;            // else Inf or NaN among the values or coefficients: all is NaN
        const int k_unit = fixed_exponent(finite ? bound : 0.0f);
        const float two_k = ldexpf(1.0f, k_unit), unit = finite ? ldexpf(1.0f, -k_unit) : __uint_as_float(0x7FC00000u);
        for (int64_t c0 = 0; c0 < ldp; c0 += win) {      // a window of columns at a time (one when the vector fits in LDS)
            const int64_t c1 = min(ldp, c0 + win);
            const uint32_t lo = static_cast<uint32_t>(c0), wide = static_cast<uint32_t>(c1 - c0);
            if (finite) with_batches([&](auto shape) { full_scatter(shape, ch, acc, lo, wide, two_k); });
            __syncthreads();
            for (int64_t j = c0 + 4ll * threadIdx.x; j < c1; j += 4ll * kCsrThreads) {
                const int4 sum = *reinterpret_cast<const int4 *>(acc + (j - c0));
                float4 v = make_float4(static_cast<float>(sum.x) * unit, static_cast<float>(sum.y) * unit,
                                       static_cast<float>(sum.z) * unit, static_cast<float>(sum.w) * unit);
                if (ib > i0) {
                    const float4 before = *reinterpret_cast<const float4 *>(mine + j);
                    v = make_float4(before.x + v.x, before.y + v.y, before.z + v.z, before.w + v.w);
                }
                *reinterpret_cast<float4 *>(mine + j) = v;
                *reinterpret_cast<int4 *>(acc + (j - c0)) = make_int4(0, 0, 0, 0);
            }
            __syncthreads();
        }
    }
    loss = wave_sum_f64(loss);
    if (lane == 0) sh_loss[wave] = loss;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = sh_loss[0];
        for (int w = 1; w < kCsrWaves; ++w) t += sh_loss[w];
        loss_partial[blockIdx.x] = t;
    }
}

// defined in grad_dense.hip
int launch_full_finish(const float *partial, int P, int64_t ldp, int64_t n, int64_t d, const float *x, float l2, float l1,
                       const double *loss_partial, float *g_out, double *obj_out, hipStream_t st);
int launch_worker_zero(const WorkerArgs &a, int64_t d, int64_t row_words, hipStream_t st);
int launch_quantize_pack_parts(const float *v, int64_t d, int64_t M, int64_t ld, int b, int field, const float *absmax,
                               int parts, const int32_t *count_parts, int32_t *count_out, const StreamKey &key,
                               uint32_t worker0, uint32_t *packed, int64_t ld_words, float *delta_out, uint32_t *status,
                               hipStream_t st);

// ------------------------------------------------------------------ host side
static int64_t csr_full_splits(int64_t n)
{
    int64_t P = ceil_div(n, 64);
    if (P > 256) P = 256;
    if (P < 1) P = 1;
    return P;
}

static_assert(kMaxSlices == kMaxParts, "a row's blocks leave a value each");

int64_t csr_workspace_bytes(int32_t op, const dq_problem *prob, int64_t M, int64_t)
{
    CsrPlan plan;
    if (!csr_plan(prob->d, true, plan)) return DQ_ERR_UNSUPPORTED;
    if (op == DQ_OP_FULL_GRAD) {
        const int64_t P = csr_full_splits(prob->n);
        return P * pad4(prob->d) * 4 + P * 8;
    }
    // a row per worker: the whole gradient when it does not fit in LDS, else the sparsified gradient when the
    // sparsifier is split over several blocks per worker (see csr_worker); then 8 values + 8 counts per worker: all
    // that a single step uses
    if (op == DQ_OP_WORKER_STEP) return csr_run_offset(prob->d, M);
    // then one more row, in which dq_run_rounds keeps (decoded model) - snapshot between two rounds of a call; then two
    // sets of prepared mini-batches (see PrepLayout), the one a round reads and the one it leaves for the next
    return csr_run_bytes(prob->d, M);
}

// Kernels that use more than 64 KB of dynamic LDS must be told so once (the limit is raised to the budget).
template <typename K>
static int allow_big_lds(K kernel, std::once_flag &once, hipError_t &once_rc)
{
    std::call_once(once, [&] {
        once_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      static_cast<int>(kLdsBudget - kCsrFixedLds));
    });
    DQ_HIP_TRY(once_rc);
    return DQ_OK;
}

int csr_full_grad(const dq_problem *prob, const float *x, float *g_out, float *z_out, double *obj_out, void *ws,
                  int64_t ws_bytes, hipStream_t st)
{
    const int64_t d = prob->d, n = prob->n;
    CsrPlan plan;
    if (!csr_plan(d, false, plan)) return DQ_ERR_UNSUPPORTED;
    if (ws_bytes < csr_workspace_bytes(DQ_OP_FULL_GRAD, prob, 0, 0) || !ws) return DQ_ERR_WORKSPACE;
    const int64_t ldp = pad4(d);
    const int P = static_cast<int>(csr_full_splits(n));
    float *partial = static_cast<float *>(ws);
    double *loss_partial = reinterpret_cast<double *>(partial + static_cast<int64_t>(P) * ldp);
    // equal windows of columns, one when the vector fits
    const int64_t win = pad4(ceil_div(ldp, ceil_div(ldp * 4, kFullLds)));
    static std::once_flag attr_once;
    static hipError_t attr_rc = hipSuccess;
    int rc = allow_big_lds(csr_full_partial_kernel, attr_once, attr_rc);
    if (rc != DQ_OK) return rc;
    const CsrView A{prob->indptr, prob->indices, prob->values, prob->y, n, d};
    csr_full_partial_kernel<<<dim3(P), dim3(kCsrThreads), static_cast<size_t>(win) * 4, st>>>(A, x, z_out, partial, ldp, loss_partial,
                                                                                              static_cast<int>(win));
    DQ_LAUNCH_CHECK();
    return launch_full_finish(partial, P, ldp, n, d, x, prob->l2, prob->l1, loss_partial, g_out, obj_out, st);
}

// Slices of a step split over the columns (0: the step is not split): eight per worker, fewer where that would be more
// blocks than compute units (one block more per worker prepares the next round); a slice holds whole groups of 64
// quads, so no word of a message belongs to two slices, and must fit in LDS beside `cap` staged entries.
struct CsrSlices {
    int count, win;
};

static CsrSlices csr_slices(int64_t d, int64_t M, const CsrPlan &plan, bool second)
{
    constexpr int64_t kUnits = 256;
    int64_t S = std::min<int64_t>(kMaxSlices, kUnits / M - 1);
    if (plan.nwin == 1) {
        // At least three slices (or the passes over the vector are not shared out enough), 4096 columns (rounds of 32 rows,
        // eight workers: 4096 columns 12.9 us split or not, 8192 13.2 against 15.0).  Above 8192 columns, where the unsplit step
        // has a master spread over the chip too, that master takes up to 32 messages at once and the one over parts sixteen
        // gradients after another, 1.9 us for every further sixteen: 14,000 columns, M = 32 10.4 + 3.6 us unsplit, 7.9 +
        // 5.8 split (a round 2-4 % longer, and from 49 workers on 2-9 %; M = 24 3 % shorter, M = 40 and 48 even to 3 %).
        // Unless so much of LDS is the vector's that fewer than 2048 entries can be staged beside it: 34,000 columns, M = 32 23.2
        // against 21.5 us, M = 64 29.4 against 26.5.
        if (d < 4096 || S < 3) return CsrSlices{0, 0};
        if (d > 2 * 4096 && plan.cap >= 2048 && (M % 32 == 0 || M > 48)) return CsrSlices{0, 0};
    }
    S = std::max<int64_t>(S, 2);
    const int64_t budget = kLdsBudget - kCsrFixedLds, each = second ? 16 : 12;
    for (; S <= kMaxSlices; ++S) {
        const int64_t win = ceil_div(ceil_div(d, S), 256) * 256;
        if (win * 4 + plan.cap * each > budget) continue;
        // (several windows: a block of the unsplit step takes them one after the other, as the compute units would these
        // slices if there were that many of them: 36,000 columns, M = 128 41 us a round either way, M = 256 49 against 59)
        const int64_t count = ceil_div(d, win);
        if (plan.nwin > 1 && ceil_div(M * count, kUnits) >= plan.nwin) break;
        return CsrSlices{static_cast<int>(count), static_cast<int>(win)};
    }
    return CsrSlices{0, 0};
}

// Whether (and how) a step is split over the columns.  Vectors of several LDS windows always are, if their outputs allow
// it and the slices do not outnumber the compute units as often as there are windows (8 workers, 32 rows, 47,236 columns: one block per worker and two windows 48.4 us; split, with the sparsifier and the
// quantization as launches of their own, 8.9 + 4.4 + 4.0 us).  Of the others those that can leave their quantization to
// the master (see `deferred`): at 20,958 columns worker step and master 10.4 + 3.1 us -> 7.9 + 3.9 us.  Not those with a
// sparsifier, which would need a launch for it between the two: 12.0 us as one launch, 8.8 + 3.9 as two.
static CsrSlices csr_step_slices(const dq_problem *prob, const WorkerArgs &a, const CsrPlan &plan)
{
    const CsrSlices none{0, 0};
    const bool count_ok = !a.nnz_out || (a.sparsify && a.b >= 4);      // after the sparsifier: count = kept coordinates
    if (!a.packed || a.b == 32 || !count_ok || !a.ws) return none;
    if (a.ws_bytes < csr_workspace_bytes(DQ_OP_WORKER_STEP, prob, a.M, a.B)) return none;
    if (plan.nwin == 1 && (a.sparsify || !a.deferred)) return none;
    return csr_slices(prob->d, a.M, plan, a.z_snap == nullptr);
}

// How a step runs, for csr_worker, which launches it, and for csr_run_layout, which must know it beforehand.
struct CsrStep {
    CsrPlan plan;
    CsrSlices sl;
    bool sliced;               // split over the columns
    unsigned blocks;           // per worker: the slices, or identical blocks that share the tail
    bool split_sparsifier;     // not split over the columns, every block sparsifies its share into the workspace
    bool common;               // csr_worker_kernel's COMMON
    bool can_prepare;          // mini-batches may be prepared a round ahead: one more block per worker
};

static bool csr_step(const dq_problem *prob, const WorkerArgs &a, CsrStep &s)
{
    const int64_t d = prob->d;
    if (!csr_plan(d, a.z_snap == nullptr, s.plan)) return false;
    s.sl = csr_step_slices(prob, a, s.plan);
    s.sliced = s.sl.count > 0;
    const bool one_window = s.sliced || s.plan.nwin == 1, count_ok = !a.nnz_out || (a.sparsify && a.b >= 4);
    // Few workers leave most compute units idle while each block spends a third of its time on the Philox rounds of
    // the final quantization: then several identical blocks per worker share that part (not when the nonzero count is
    // wanted and would need a sum across blocks, nor when the gradient lives in the per-worker workspace row).
    s.blocks = 1;
    if (a.packed && count_ok && s.plan.nwin == 1 && a.b != 32 && d >= 4096 && a.M * 4 <= 128) s.blocks = a.M * 8 <= 128 ? 8 : 4;
    if (s.sliced) s.blocks = static_cast<unsigned>(s.sl.count);
    // After the sparsifier the scale is ||beta||_inf, which needs every coordinate's random decision: sharing only the
    // quantization would leave each identical block a whole Philox-and-two-divisions pass over the vector (9 of the
    // 33 us of the step at d = 20958).  With workspace for a row per worker each block sparsifies its own slice into
    // memory instead and the quantization becomes a second launch that takes the scale from the slices' maxima.
    s.split_sparsifier = !s.sliced && s.blocks > 1 && a.sparsify && a.ws &&
                         a.ws_bytes >= csr_workspace_bytes(DQ_OP_WORKER_STEP, prob, a.M, a.B);
    s.common = one_window && a.B <= kCsrMaxRows && a.z_snap != nullptr;
    s.can_prepare = one_window && !a.idx && a.B <= kCsrMaxRows && a.M * (s.blocks + 1) <= 256;
    return true;
}

// The worker kernel quantizes the model where the step is split over the columns, its mini-batches are prepared ahead, its
// margins cached, the model's message whole words per 64 quads, no slice more than one quad per thread and the mini-batches
// light, as far as it is the faster (see csr_worker_kernel, csr_light_batches).
CsrRunLayout csr_run_layout(const dq_problem *prob, const WorkerArgs &a)
{
    CsrRunLayout out{};
    CsrStep s;
    if (!a.ws || !csr_step(prob, a, s) || a.ws_bytes < csr_workspace_bytes(DQ_OP_VR_GRAD, prob, a.M, a.B)) return out;
    char *base = static_cast<char *>(a.ws) + csr_run_offset(prob->d, a.M);
    const bool light = csr_light_batches(a.B, prob->n, prob->lda, kCsrInFlight, s.plan.cap);
    out.pending = s.sliced && s.common && s.can_prepare && (a.b_x == 2 || a.b_x == 4 || a.b_x == 8) && s.sl.win <= 4 * kCsrThreads && light;
    out.prep = csr_prep_room(prob->d, a.M, a.B, s.plan, out.pending);
    if (!out.pending) out.model_diff = reinterpret_cast<float *>(base);
    out.prep_sets[0] = reinterpret_cast<int32_t *>(base + (out.pending ? 0 : pad4(prob->d) * 4));
    out.prep_sets[1] = out.prep_sets[0] + a.M * out.prep.stride;
    // (the kernel's short_tail; anywhere else the master would read x_snap and the chip meet on one word for nothing.  With heavy
    // mini-batches looking at their entries once more takes longer than the pass over the columns, or they are not prepared: 4200
    // columns, sixteen workers, 6627 entries 17.9 us a round without and 18.3 with it, 4757 entries 16.2 and 15.8.)
    if (s.split_sparsifier && s.common && s.can_prepare && light) out.dev_max = PrepLayout(static_cast<int>(a.B)).dev_max;
    return out;
}

template <int MODEL, bool COMMON, bool SLICED, bool PREP>
static int csr_launch(const CsrWorkerArgs &k, dim3 grid, size_t lds, const WorkerArgs &a, hipStream_t st)
{
    const auto kernel = csr_worker_kernel<MODEL, COMMON, SLICED, PREP>;
    static std::once_flag attr_once;
    static hipError_t attr_rc = hipSuccess;
    const int rc = allow_big_lds(kernel, attr_once, attr_rc);
    if (rc != DQ_OK) return rc;
    if (a.ev_start && a.ev_stop)      // the kernel's own start and end times go to the two events
        hipExtLaunchKernelGGL(kernel, grid, dim3(kCsrThreads), static_cast<uint32_t>(lds), st, a.ev_start, a.ev_stop, 0u, k);
    else
        kernel<<<grid, dim3(kCsrThreads), lds, st>>>(k);
    DQ_LAUNCH_CHECK();
    return DQ_OK;
}

int csr_worker(const dq_problem *prob, const WorkerArgs &a, hipStream_t st)
{
    const int64_t d = prob->d;
    CsrStep step;
    if (!csr_step(prob, a, step)) return DQ_ERR_UNSUPPORTED;
    const CsrPlan &plan = step.plan;
    const int64_t row_words = a.packed ? (a.b == 32 ? d : packed_words(d, a.b)) : 0;
    if (a.deferred) *a.deferred = GradientParts{nullptr, 0, nullptr, nullptr, 0};
    if (a.prepared_next) *a.prepared_next = false;
    if (a.model_is_snapshot) return launch_worker_zero(a, d, row_words, st);
    if (plan.nwin > 1 && (!a.ws || a.ws_bytes < a.M * pad4(d) * 4)) return DQ_ERR_WORKSPACE;
    CsrWorkerArgs k{};
    k.A = CsrView{prob->indptr, prob->indices, prob->values, prob->y, prob->n, d};
    k.idx = a.idx; k.B = static_cast<int>(a.B);
    k.xq = a.xq; k.delta_x = a.delta_x; k.b_x = a.b_x; k.x_snap = a.x_snap; k.z_snap = a.z_snap; k.l2 = prob->l2;
    k.model_last_word = (a.b_x == 32 ? prob->d : packed_words(prob->d, a.b_x)) - 1;
    k.alpha_out = a.alpha_out; k.ld = a.ld; k.absmax_out = a.absmax_out; k.l1norm_out = a.l1norm_out;
    k.sparsify = a.sparsify; k.b = a.b;
    k.key = StreamKey{static_cast<uint32_t>(a.seed), static_cast<uint32_t>(a.seed >> 32), a.iter, 0u, DQ_TAG_GRAD};
    k.worker0 = a.worker0;
    k.packed = a.packed; k.ld_words = a.ld_words; k.row_words = row_words;
    k.delta_out = a.delta_out; k.nnz_out = a.nnz_out; k.status = a.status; k.zero_word = a.zero_word;
    k.cap = plan.cap; k.win = plan.win;
    k.alpha_ws = plan.nwin > 1 ? static_cast<float *>(a.ws) : nullptr; k.ld_ws = pad4(d);
    k.model_diff = a.b_x == 32 ? nullptr : a.model_diff;
    if (a.x_model) {
        k.model_diff = a.x_model;
        k.absmax_out = const_cast<float *>(a.absmax_model);
    }
    const CsrSlices sl = step.sl;
    const bool sliced = step.sliced, common = step.common;
    const unsigned slices = step.blocks;
    size_t lds = plan.lds;
    GradientParts parts{nullptr, 0, nullptr, nullptr, 0};
    float *alpha_max = nullptr;                          // the slices' maxima of the gradient itself
    int64_t alpha_max_stride = 0;
    if (sliced || step.split_sparsifier) {
        float *part_max = static_cast<float *>(a.ws) + a.M * k.ld_ws;
        int32_t *part_kept = reinterpret_cast<int32_t *>(part_max + a.M * kMaxSlices);
        parts = GradientParts{static_cast<float *>(a.ws), k.ld_ws, part_max, a.sparsify ? part_kept : nullptr, static_cast<int>(slices)};
        if (step.split_sparsifier) {
            k.beta_ws = static_cast<float *>(a.ws);
            k.part_max = part_max;
            k.part_kept = part_kept;
        }
    }
    if (sliced) {
        k.win = sl.win;
        lds = static_cast<size_t>(sl.win) * 4 + static_cast<size_t>(plan.cap) * (a.z_snap ? 12 : 16);
        k.beta_ws = static_cast<float *>(a.ws);
        // (before the sparsifier the maxima wait at the head of the message rows, which are written only after it)
        alpha_max = a.sparsify ? reinterpret_cast<float *>(a.packed) : const_cast<float *>(parts.part_max);
        alpha_max_stride = a.sparsify ? a.ld_words : static_cast<int64_t>(slices);
        k.part_max = alpha_max;
    }
    if (a.x_model && !(sliced && common)) return DQ_ERR_INVALID_ARG;       // (see csr_run_layout)
    // a round of dq_run_rounds that has a successor in its call prepares that round's mini-batches in one more block
    // per worker (on compute units the launch leaves idle), and reads its own if the round before left them
    if (step.can_prepare) {
        k.prep_in = a.prep_in;
        k.prep_out = a.prep_out;
        k.prep_stride = a.prep.stride; k.prep_cap = a.prep.cap; k.snap_cap = a.prep.snap_cap;
        k.dev_max_at = a.prep_in && a.dev_max ? PrepLayout(k.B).dev_max : 0;
        k.next_iter = a.iter + 1u;
    }
    if (a.prepared_next) *a.prepared_next = k.prep_out != nullptr;
    const dim3 grid(static_cast<unsigned>(a.M), slices + (k.prep_out ? 1u : 0u));
    const auto launch = [&](auto model, auto prep) {
        constexpr int MODEL = decltype(model)::value;
        constexpr bool PREP = decltype(prep)::value;
        if (sliced) return common ? csr_launch<MODEL, true, true, PREP>(k, grid, lds, a, st) : csr_launch<MODEL, false, true, PREP>(k, grid, lds, a, st);
        return common ? csr_launch<MODEL, true, false, PREP>(k, grid, lds, a, st) : csr_launch<MODEL, false, false, PREP>(k, grid, lds, a, st);
    };
    // (several windows one after the other: the kernel with the code of prepared mini-batches also where there are none)
    const bool prep = k.prep_in || k.prep_out || !(sliced || plan.nwin == 1);
    using Message = std::integral_constant<int, kModelMessage>;
    const int rc = a.x_model      ? csr_launch<kModelPending, true, true, true>(k, grid, lds, a, st)
                   : k.model_diff ? launch(std::integral_constant<int, kModelDiff>{}, std::true_type{})
                   : prep         ? launch(Message{}, std::true_type{})
                                  : launch(Message{}, std::false_type{});
    if (rc != DQ_OK) return rc;
    if (parts.parts == 0) return DQ_OK;
    if (sliced && a.sparsify) {
        const bool encode = a.encoded && a.wire && sparse_message_parts_ok(d, a.M, a.b, a.packed, a.ld_words, a.wire, a.ld_wire);
        sparsify_parts_kernel<<<dim3(static_cast<unsigned>(a.M), slices), dim3(kCsrThreads), 0, st>>>(
            k.beta_ws, k.ld_ws, d, alpha_max, alpha_max_stride, static_cast<int>(slices), k.key, a.worker0,
            const_cast<float *>(parts.part_max), const_cast<int32_t *>(parts.part_kept),
            static_cast<int>(sparse_parts_quads(d, static_cast<int>(slices))), encode ? a.wire : nullptr, a.ld_wire,
            encode ? static_cast<int>(dq_sparse_stream_words(d, a.b)) : 0);
        DQ_LAUNCH_CHECK();
        if (encode) {
            *a.encoded = true;
            return launch_sparse_message_parts(parts, d, a.M, a.b, k.key, a.worker0, a.packed, a.ld_words, a.wire, a.ld_wire, a.delta_out,
                                               a.nnz_out, a.wire_nnz, a.status, st);
        }
    }
    if (a.deferred) {                                    // the master quantizes while it aggregates
        *a.deferred = parts;
        return DQ_OK;
    }
    return launch_quantize_pack_parts(parts.rows, d, a.M, parts.ld, a.b, a.b, parts.part_max, parts.parts,
                                      a.nnz_out ? parts.part_kept : nullptr, a.nnz_out, k.key, a.worker0, a.packed,
                                      a.ld_words, a.delta_out, a.status, st);
}

}  // namespace dq
