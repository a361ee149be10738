// Pieces of the CSR worker step shared by the kernel of a step and that of whole rounds: the rows in flight, fixed-point
// accumulation of the scattered terms, margins.
#pragma once

#include "dq_common.h"
#include "elementwise.h"
#include "grad_common.h"

namespace dq {

constexpr int kCsrThreads = 1024;
constexpr int kCsrWaves = kCsrThreads / kWave;
constexpr int kColMask = (1 << kColBits) - 1;
constexpr int kFlight = 4;                       // rows a wavefront reduces at the same time
constexpr int kStageFlight = 4;                  // entries a thread stages at the same time (worker step)
constexpr int kFlushRows = 1024;                 // rows between two flushes of the fixed-point sums (full gradient)
constexpr int kChunkSlots = kMaxStage / kWave;   // see RowMeta::chunk_row

struct CsrView {
    const int64_t *indptr;
    const int32_t *indices;
    const float *values;
    const float *y;
    int64_t n, d;
};

// Per-block LDS metadata of the rows in flight.
struct RowMeta {
    int row[kCsrMaxRows];        // sample index, -1 = ignored
    int64_t start[kCsrMaxRows];  // first entry
    int len[kCsrMaxRows];
    int pre[kCsrMaxRows + 1];    // exclusive prefix sum of len
    float coef[kCsrMaxRows];
    float z[kCsrMaxRows];        // cached margin at the snapshot
    int chunk_row[kChunkSlots];  // the row that holds entry 64 c of the rows' concatenation, for the entries below 64 * kChunkSlots
};

// Fills meta.pre with the exclusive prefix sums of meta.len[0..nrows) (pre[nrows] = total).
// The first wavefront scans the lengths, kCsrMaxRows/64 consecutive rows per lane; all threads of
// the block must call it (barriers before and after).
__device__ __forceinline__ void csr_prefix_lengths(RowMeta &meta, int nrows)
{
    constexpr int kPer = kCsrMaxRows / kWave;
    __syncthreads();
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        int v[kPer], sum = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int r = lane * kPer + u;
            v[u] = r < nrows ? meta.len[r] : 0;
            sum += v[u];
        }
        int incl = sum;                                  // inclusive scan of the lane sums
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int up = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += up;
        }
        int run = incl - sum;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            meta.pre[lane * kPer + u] = run;
            run += v[u];
        }
        if (lane == kWave - 1) meta.pre[kCsrMaxRows] = run;
    }
    __syncthreads();
    // every row leaves its number at the multiples of 64 that it holds (an empty row holds none)
    if (static_cast<int>(threadIdx.x) < nrows) {
        const int lo = meta.pre[threadIdx.x], hi = meta.pre[threadIdx.x + 1];
        for (int c = (lo + kWave - 1) / kWave; c * kWave < hi && c < kChunkSlots; ++c) meta.chunk_row[c] = threadIdx.x;
    }
    __syncthreads();
}

// ---- fixed-point accumulation of the scattered terms
// LDS float atomic adds take about three cycles per lane on this part (measured: the 3328 adds of a 64-row
// mini-batch take 4.3-4.9 us however they are spread over wavefronts), integer ones a fifteenth of that, and an
// integer sum does not depend on the order of its terms.  So coefficient * value is accumulated in int32 as a multiple
// of the unit 2^-k, with k from a bound on the magnitude any column's sum can have reached: the sum over the groups
// of rows added so far of (sum of the group's |coefficient|) * (the group's largest |value|), times 2^k, stays
// <= 2^30, so a sum cannot overflow.  The coefficients of the variance-reduced gradient shrink with the distance
// between model and snapshot, and the unit shrinks with them.  A term is rounded to the nearest unit, i.e. within
// 2^-31 of that bound -- float32 addition loses up to 2^-25 of the partial sum per term, which is coarser for sums of
// the bound's order and finer for much smaller ones; either way far inside the tolerance of the gradient.  When a
// further group of rows raises the bound past a power of two, the window is first rescaled to the coarser unit.
// A value or coefficient that is not finite poisons the block: its result is NaN.
struct FixedAcc {
    float bound;            // see above; 0 while nothing but zeros has been added
    int k;                  // the unit is 2^-k
};

// k with bound * 2^k <= 2^30 (clamped so that 2^k and 2^-k are normal numbers)
__device__ __forceinline__ int fixed_exponent(float bound)
{
    int e = 0;
    (void)frexpf(bound, &e);                 // bound = m * 2^e with 0.5 <= m < 1; e = 0 for bound = 0
    return max(-100, min(100, 30 - e));
}

// A group of rows whose terms are bounded by group_bound (in sum, per column) is about to be added to acc[0..ncols):
// coarsen the unit if need be.  Every thread calls it with the same arguments, after a barrier that follows all
// earlier adds; a rescaled window is published by the barrier inside.
__device__ __forceinline__ void fixed_admit(FixedAcc &fx, float group_bound, int *acc, int ncols, int *poison)
{
    if (!(group_bound <= FLT_MAX)) {         // Inf or NaN among the values or coefficients
        if (threadIdx.x == 0) *poison = 1;
        return;
    }
    const float bound = fx.bound + group_bound;
    const int k_new = fixed_exponent(bound);
    if (fx.bound > 0.0f && k_new < fx.k) {
        const int sh = fx.k - k_new;
        for (int j = threadIdx.x; j < ncols; j += kCsrThreads)
            acc[j] = sh >= 31 ? 0 : (acc[j] + (1 << (sh - 1))) >> sh;       // nearest multiple of the new unit
        __syncthreads();
    }
    if (!(fx.bound > 0.0f) || k_new < fx.k) fx.k = k_new;
    fx.bound = bound;
}

// sum of |coef[r0..r1)| (at most kCsrMaxRows of them), the same value in every thread of the block
__device__ __forceinline__ float coef_abs_sum(const float *coef, int r0, int r1)
{
    const int lane = threadIdx.x & (kWave - 1);
    float t = 0.0f;
#pragma unroll
    for (int u = 0; u < kCsrMaxRows / kWave; ++u) {
        const int r = r0 + lane + kWave * u;
        const float c = coef[min(r, kCsrMaxRows - 1)];
        t += r < r1 ? fabsf(c) : 0.0f;
    }
    return wave_sum_f32(t);
}

__device__ __forceinline__ int fixed_term(float coef, float value, float two_k)
{
    return __float2int_rn(coef * value * two_k);          // (the scaling by a power of two is exact)
}

// The row of staged position p: the last r in [g0, g1) with pre[r] - base <= p, by halving steps of fixed number.
__device__ __forceinline__ int csr_row_of(const RowMeta &meta, int g0, int g1, int base, int p)
{
    int r = g0;
#pragma unroll
    for (int step = kCsrMaxRows / 2; step >= 1; step >>= 1) {
        const int cand = r + step;
        const int first = meta.pre[min(cand, g1)] - base;
        r = (cand < g1 && first <= p) ? cand : r;
    }
    return r;
}

// The same for the 64 consecutive positions P + lane of a wavefront when the group starts at row 0 (base = 0) and P is a
// multiple of 64, from the table of the rows at the multiples of 64 (RowMeta::chunk_row): the row of P is read there,
// and a lane's row lies as many rows further as start at or before its position among the next kNextRows (their
// starts are the same few LDS words for the whole wavefront).  More rows than that starting inside the chunk (short
// rows) is left to csr_row_of.  `p` = min(P + lane, total - 1).
constexpr int kNextRows = 4;
__device__ __forceinline__ int csr_row_in_chunk(const RowMeta &meta, int g1, int P, int p)
{
    const int r0 = meta.chunk_row[P >> 6];
    const int beyond = r0 + kNextRows + 1;
    if (beyond < g1 && meta.pre[min(beyond, kCsrMaxRows)] <= P + kWave - 1)       // (the same for all lanes)
        return csr_row_of(meta, 0, g1, 0, p);
    int r = r0;
#pragma unroll
    for (int j = 1; j <= kNextRows; ++j) {
        const int rj = r0 + j;
        const int first = meta.pre[min(rj, kCsrMaxRows)];
        r += (rj < g1 && first <= p) ? 1 : 0;
    }
    return r;
}

template <int FLIGHT, typename CoefFn>
__device__ __forceinline__ void csr_lane_margins(const float *prod, int total, int nrows, int my_len, int my_pre, CoefFn coef_of,
                                                 float *coef)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    float margin = 0.0f;
    for (int i = 0; wave + i * kCsrWaves < nrows; i += FLIGHT) {      // rows i .. i + FLIGHT - 1 of the wavefront
        int len[FLIGHT], off[FLIGHT], maxlen = 0;
        float sum[FLIGHT];
#pragma unroll
        for (int u = 0; u < FLIGHT; ++u) {                            // (lanes past the last row hold length 0)
            len[u] = __builtin_amdgcn_readlane(my_len, i + u);
            off[u] = __builtin_amdgcn_readlane(my_pre, i + u);
            maxlen = max(maxlen, len[u]);
            sum[u] = 0.0f;
        }
        for (int k = lane; k - lane < maxlen; k += kWave) {
            float v[FLIGHT];
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u) v[u] = prod[min(off[u] + k, total - 1)];
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u) sum[u] += k < len[u] ? v[u] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < FLIGHT; ++u) {
            const float t = wave_sum_f32(sum[u]);
            margin = lane == i + u ? t : margin;
        }
    }
    const int r = wave + lane * kCsrWaves;
    if (r < nrows) coef[r] = coef_of(margin);
}

}  // namespace dq
