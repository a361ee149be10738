// Sparse message format of Section 4.2 of the paper: a sparsified, quantized gradient is sent as
// its scale plus, per nonzero coordinate, ceil(log2 d) bits of position and b bits of value.
// Encoder: packed dense codes -> entry stream (order-preserving compaction); decoder: the inverse.
// Several blocks of 1024 threads share a row, each assembling its own words of the output in LDS with bitwise-OR
// atomics on disjoint bits (order-free, hence deterministic).
#include <algorithm>
#include <mutex>

#include "dq_common.h"
#include "elementwise.h"
#include "grad_launch.h"

namespace dq {

constexpr int kWireThreads = 1024;
constexpr int64_t kWireLdsWords = 36 * 1024;          // the longest stream or row: 144 KB
constexpr int64_t kEncodeSpan = 4096;                 // most stream words a block assembles

static inline int position_bits(int64_t d)
{
    int bits = 0;
    while ((int64_t{1} << bits) < d) ++bits;
    return bits;
}

// Exclusive prefix sum over the block's threads (two barriers); `scratch` holds one int per wavefront.  *total receives
// the block total.
__device__ __forceinline__ int block_scan_exclusive(int v, int *scratch, int *total)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int incl = wave_scan_i32(v);
    if (lane == kWave - 1) scratch[wave] = incl;
    __syncthreads();
    const int mine = lane < kWireThreads / kWave ? scratch[lane] : 0;      // (every wavefront scans the sixteen sums)
    *total = wave_sum_i32(mine);
    return wave_sum_i32(lane < wave ? mine : 0) + incl - v;
}

// One bit (the lowest) per nonzero field of a word.
template <int FIELD>
__device__ __forceinline__ uint32_t nonzero_fields(uint32_t w)
{
    if constexpr (FIELD == 8) w |= w >> 4;
    if constexpr (FIELD >= 4) w |= w >> 2;
    w |= w >> 1;
    return w & (FIELD == 8 ? 0x01010101u : FIELD == 4 ? 0x11111111u : 0x55555555u);
}

// What bounds it: latency, and the words one compute unit can write (the words past the used ones are zeroed, up to
// 144 KB a row).  So the capacity of a row is cut into spans of at most kEncodeSpan words, one block each.  Every block
// reads the whole row (at most 48 KB, from L2 after the first), thread t the words per*t .. per*t + per - 1 -- `per` is
// odd, so the reads from LDS meet no bank twice --, counts its nonzero fields and learns from one prefix sum the number
// of its first entry.  The entries of the block's span are then handed out one per thread, which finds its word by
// halving: the nonzeros of a text gradient crowd in the first columns, and left to the threads that counted them a few
// would emit most (by itself 8.1 -> 6.8 us in the first case below).  Measured at 47,236
// columns, 4 bits, 8 rows: one block per row with a prefix sum of twenty barriers per 16,384 coordinates 16.0 us, now
// 6.0 us; 20,958 columns, 16 rows: 10.6 us, now 5.3 us.
// Where the streams take the place of the rows one block does all spans of a row, which it has in LDS by then.
template <int FIELD>
__global__ __launch_bounds__(kWireThreads) void sparse_encode_kernel(
    const uint32_t *__restrict__ packed, int64_t ld_words, int row_words, int d, int pos_bits, uint32_t *__restrict__ stream,
    int64_t ld_stream, int cap_words, int span, int per, int32_t *__restrict__ nnz_out)
{
    extern __shared__ uint32_t sh[];
    __shared__ int sh_scan[kWireThreads / kWave];
    __shared__ int sh_first[kWireThreads];
    uint32_t *sh_stream = sh, *sh_row = sh + span;
    const int m = blockIdx.x;
    const uint32_t *row = packed + static_cast<int64_t>(m) * ld_words;
    // From five words a thread on eight are requested together, at clamped positions: one after the other they were `per` trips to
    // memory, 7 at 47,236 columns.  Up to three (20,958 columns of 4 bits) are done sooner one by one, most of all one alone: the
    // whole message of 1000 columns, 8 rows, 11.8 us, 12.5 with eight requests for it.
    const auto store_word = [&](int w, uint32_t v) {
        if (w >= row_words - 1) {                                 // fields past the last coordinate are not part of the row
            const int left = w >= row_words ? 0 : (d * FIELD - 1) % 32 + 1;
            v = left == 32 ? v : v & ((1u << left) - 1u);
        }
        sh_row[w] = v;
    };
    constexpr int kFlight = 8;
    if (per <= 3) {
        for (int w = threadIdx.x; w < per * kWireThreads; w += kWireThreads) store_word(w, row[min(w, row_words - 1)]);
    } else {
        for (int w0 = threadIdx.x; w0 < per * kWireThreads; w0 += kFlight * kWireThreads) {
            uint32_t v[kFlight];
#pragma unroll
            for (int u = 0; u < kFlight; ++u) v[u] = row[min(w0 + u * kWireThreads, row_words - 1)];
#pragma unroll
            for (int u = 0; u < kFlight; ++u)
                if (w0 + u * kWireThreads < per * kWireThreads) store_word(w0 + u * kWireThreads, v[u]);
        }
    }
    for (int w = threadIdx.x; w < span; w += kWireThreads) sh_stream[w] = 0u;
    __syncthreads();
    const int first = per * threadIdx.x;
    int count = 0, total;
    for (int j = 0; j < per; ++j) count += __popc(nonzero_fields<FIELD>(sh_row[first + j]));
    sh_first[threadIdx.x] = block_scan_exclusive(count, sh_scan, &total);        // (at most 2^17 entries of 25 bits)
    __syncthreads();
    const int E = pos_bits + FIELD;
    for (int w0 = blockIdx.y * span;;) {
        const int nw = min(span, cap_words - w0), lo = w0 * 32, hi = (w0 + nw) * 32;
        for (int e = lo / E + threadIdx.x; e < total && e * E < hi; e += kWireThreads) {
            int t = 0;                                            // the thread whose words hold entry e: the last with first <= e
#pragma unroll
            for (int step = kWireThreads / 2; step >= 1; step >>= 1) t += sh_first[t + step] <= e ? step : 0;
            int rank = e - sh_first[t], at = per * t - 1;
            uint32_t word = 0, mask = 0;
            for (int left = rank; left >= 0; left -= __popc(mask)) {      // ... then its word, and the field in it
                rank = left;
                word = sh_row[++at];
                mask = nonzero_fields<FIELD>(word);
            }
            for (; rank > 0; --rank) mask &= mask - 1;
            const int sh = __ffs(mask) - 1, bit = e * E, w = (bit >> 5) - w0;
            const uint64_t entry = static_cast<uint64_t>(at * (32 / FIELD) + sh / FIELD) |
                                   (static_cast<uint64_t>((word >> sh) & ((1u << FIELD) - 1u)) << pos_bits);
            const uint64_t shifted = entry << (bit & 31);         // E + 31 < 64 bits: at most two words
            if (w >= 0 && w < nw) atomicOr(sh_stream + w, static_cast<uint32_t>(shifted));
            if (w + 1 < nw && (shifted >> 32)) atomicOr(sh_stream + w + 1, static_cast<uint32_t>(shifted >> 32));
        }
        __syncthreads();
        uint32_t *out = stream + static_cast<int64_t>(m) * ld_stream + w0;
        for (int w = threadIdx.x; w < nw; w += kWireThreads) out[w] = sh_stream[w];
        w0 += gridDim.y * span;
        if (w0 >= cap_words) break;                               // (the same for every thread)
        for (int w = threadIdx.x; w < span; w += kWireThreads) sh_stream[w] = 0u;      // (each thread the words it has stored)
        __syncthreads();
    }
    if (threadIdx.x == 0 && blockIdx.y == 0) nnz_out[m] = total;
}

// The last step of a worker and the encoder in one launch, on sparsified gradients as sparsify_parts_kernel leaves them: rows
// of floats in slices of `per` quads (a multiple of 64), a largest magnitude and a kept count per slice.  Grid (M, slices).  What is
// kept has a nonzero code for b >= 4 (magnitudes of at least a third of the row's largest), or no code of the row has, so a
// slice's first entry in the stream is the sum of the counts before it.  Each block quantizes its slice, stores its words of the
// packed row and assembles its words of the stream, which that launch has zeroed: the first and the last may be its neighbours'
// too and are ORed to memory, those between are its own.  What bounds it is latency: launch, one trip to memory, a prefix
// sum per 1024 quads.  47,236 columns, 8 rows, 4 bits: quantizer and encoder 3.4 + 6.0 us, now 6.5 us.
template <int FIELD>
__global__ __launch_bounds__(kWireThreads) void sparse_message_parts_kernel(
    const float *__restrict__ rows, int64_t ld, int64_t d, int per, const float *__restrict__ part_max,
    const int32_t *__restrict__ part_kept, StreamKey key, uint32_t worker0, int pos_bits, uint32_t *__restrict__ packed,
    int64_t ld_words, uint32_t *__restrict__ stream, int64_t ld_stream, float *__restrict__ delta_out, int32_t *__restrict__ kept_out,
    int32_t *__restrict__ nnz_out, uint32_t *__restrict__ status)
{
    touch_kernel_arguments<120>();
    extern __shared__ uint32_t sh_stream[];
    __shared__ int sh_scan[2][kWireThreads / kWave];
    const int m = blockIdx.x, slice = blockIdx.y, nslices = gridDim.y;
    const int64_t quads = (d + 3) / 4, q_lo = min<int64_t>(quads, static_cast<int64_t>(per) * slice), q_hi = min<int64_t>(quads, q_lo + per);
    const float4 *row = reinterpret_cast<const float4 *>(rows + static_cast<int64_t>(m) * ld);
    const PartsRaw maxima = parts_request(part_max + static_cast<int64_t>(m) * nslices, nslices);
    int kept[kMaxParts];
#pragma unroll
    for (int s = 0; s < kMaxParts; ++s) kept[s] = part_kept[static_cast<int64_t>(m) * nslices + min(s, nslices - 1)];
    constexpr int kEach = 2;                             // quads side by side, a thread's at a time
    int64_t q = q_lo + kEach * threadIdx.x;
    float4 v[kEach];
    uint4 r[kEach];
#pragma unroll
    for (int u = 0; u < kEach; ++u) v[u] = row[min(q + u, quads - 1)];
    __builtin_amdgcn_sched_barrier(0);
    key.worker = worker0 + static_cast<uint32_t>(m);
    const bool busy = __any(q < q_hi);                   // (a wavefront behind the slice draws nothing)
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
        r[u] = make_uint4(0u, 0u, 0u, 0u);
        if (busy) {
            r[u] = stream_block(key, static_cast<uint32_t>(q + u));
            asm volatile("" ::"v"(r[u].x), "v"(r[u].y), "v"(r[u].z), "v"(r[u].w));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    const Scale scale = make_scale(parts_absmax_of(maxima), FIELD);
    int base = 0, mine = 0, sum = 0;
#pragma unroll
    for (int s = 0; s < kMaxParts; ++s) {
        if (s >= nslices) kept[s] = 0;
        base += s < slice ? kept[s] : 0;
        mine = s == slice ? kept[s] : mine;
        sum += kept[s];
    }
    const bool any = scale.inv_delta != 0.0f;
    if (slice == 0 && threadIdx.x == 0) {
        delta_out[m] = scale.delta;
        if (scale.bad && status) atomicOr(status, 1u);
        if (kept_out) kept_out[m] = sum;
        nnz_out[m] = any ? sum : 0;
    }
    const int E = pos_bits + FIELD, w0 = (base * E) >> 5, w1 = any && mine > 0 ? ((base + mine) * E + 31) >> 5 : w0;
    for (int w = threadIdx.x; w < w1 - w0; w += kWireThreads) sh_stream[w] = 0u;
    uint32_t *out = packed + static_cast<int64_t>(m) * ld_words;
    int turn = 0;
    for (int64_t q0 = q_lo; q0 < q_hi; q0 += kEach * kWireThreads, turn ^= 1) { // (the same number of turns for every thread)
        if (q0 != q_lo) {
            q = q0 + kEach * threadIdx.x;
#pragma unroll
            for (int u = 0; u < kEach; ++u) {
                v[u] = row[min(q + u, quads - 1)];
                r[u] = stream_block(key, static_cast<uint32_t>(q + u));
            }
        }
        int c[4 * kEach], count = 0;
        uint32_t bits[kEach];
#pragma unroll
        for (int u = 0; u < kEach; ++u) {
            const bool in = q + u < q_hi && any;
            c[4 * u] = in ? quantize_one(v[u].x, scale, r[u].x) : 0;
            c[4 * u + 1] = in ? quantize_one(v[u].y, scale, r[u].y) : 0;
            c[4 * u + 2] = in ? quantize_one(v[u].z, scale, r[u].z) : 0;
            c[4 * u + 3] = in ? quantize_one(v[u].w, scale, r[u].w) : 0;
            bits[u] = pack4<FIELD>(c[4 * u], c[4 * u + 1], c[4 * u + 2], c[4 * u + 3]);
            count += (c[4 * u] != 0) + (c[4 * u + 1] != 0) + (c[4 * u + 2] != 0) + (c[4 * u + 3] != 0);
        }
        if constexpr (FIELD == 4) {                      // (q is even: slices begin at multiples of 64 quads)
            if (q < q_hi) out[q / 2] = bits[0] | bits[1] << 16;
        } else {
#pragma unroll
            for (int u = 0; u < kEach; ++u)
                if (q + u < q_hi) out[q + u] = bits[u];
        }
        int total, at = block_scan_exclusive(count, sh_scan[turn], &total);
        if (count > 0)
#pragma unroll
            for (int e = 0; e < 4 * kEach; ++e)
                if (c[e] != 0) {
                    const int bit = (base + at) * E, w = (bit >> 5) - w0;
                    const uint64_t entry = static_cast<uint64_t>(4 * q + e) |
                                           (static_cast<uint64_t>(static_cast<uint32_t>(c[e]) & ((1u << FIELD) - 1u)) << pos_bits);
                    const uint64_t shifted = entry << (bit & 31);     // E + 31 < 64 bits: at most two words
                    if (w < w1 - w0) atomicOr(sh_stream + w, static_cast<uint32_t>(shifted));
                    if (w + 1 < w1 - w0 && (shifted >> 32)) atomicOr(sh_stream + w + 1, static_cast<uint32_t>(shifted >> 32));
                    ++at;
                }
        base += total;
    }
    __syncthreads();
    uint32_t *words = stream + static_cast<int64_t>(m) * ld_stream + w0;
    for (int w = threadIdx.x; w < w1 - w0; w += kWireThreads) {
        const uint32_t bits = sh_stream[w];
        if (w == 0 || w == w1 - w0 - 1) atomicOr(words + w, bits);
        else words[w] = bits;
    }
}

// A block owns `span` words of the dense row (all of them where the rows take the place of the streams) and takes from the
// stream, which it reads whole, the entries that fall there.
template <int FIELD>
__global__ __launch_bounds__(kWireThreads) void sparse_decode_kernel(
    const uint32_t *__restrict__ stream, int64_t ld_stream, const int32_t *__restrict__ nnz, int64_t d, int pos_bits,
    uint32_t *__restrict__ packed, int64_t ld_words, int row_words, int span)
{
    extern __shared__ uint32_t sh_row[];
    const int m = blockIdx.x, w0 = blockIdx.y * span, nw = min(span, row_words - w0);
    const uint32_t *in = stream + static_cast<int64_t>(m) * ld_stream;
    const int count = nnz[m];
    for (int w = threadIdx.x; w < nw; w += kWireThreads) sh_row[w] = 0u;
    __syncthreads();
    const int E = pos_bits + FIELD;
    for (int e = threadIdx.x; e < count; e += kWireThreads) {
        const int64_t bit = static_cast<int64_t>(e) * E;
        const int64_t w = bit >> 5;
        const int sh = static_cast<int>(bit & 31);
        uint64_t v = in[w];
        if (sh + E > 32) v |= static_cast<uint64_t>(in[w + 1]) << 32;
        const uint64_t entry = (v >> sh) & ((uint64_t{1} << E) - 1);
        const int64_t pos = static_cast<int64_t>(entry & ((uint64_t{1} << pos_bits) - 1));
        const uint32_t field = static_cast<uint32_t>(entry >> pos_bits);
        const int at = static_cast<int>((pos * FIELD) >> 5) - w0;
        if (pos < d && at >= 0 && at < nw) atomicOr(sh_row + at, field << ((pos * FIELD) & 31));
    }
    __syncthreads();
    uint32_t *out = packed + static_cast<int64_t>(m) * ld_words + w0;
    for (int w = threadIdx.x; w < nw; w += kWireThreads) out[w] = sh_row[w];
}

template <auto kernel>
static int allow_lds()
{
    // one flag and one result per kernel (every instantiation has its own): set once per process, safely from any thread
    static std::once_flag once;
    static hipError_t once_rc = hipSuccess;
    std::call_once(once, [&] {
        once_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      static_cast<int>(kWireLdsWords * 4));
    });
    DQ_HIP_TRY(once_rc);
    return DQ_OK;
}

int64_t sparse_parts_quads(int64_t d, int slices) { return ceil_div(ceil_div(ceil_div(d, 4), slices), kWave) * kWave; }

bool sparse_message_parts_ok(int64_t d, int64_t M, int b, const uint32_t *packed, int64_t ld_words, const uint32_t *wire,
                             int64_t ld_wire)
{
    if (b != 4 && b != 8) return false;
    const int64_t cap = ceil_div(d * (position_bits(d) + b), 32);
    return cap <= kWireLdsWords && ld_wire >= cap &&
           !ranges_overlap(packed, (M - 1) * ld_words + packed_words(d, b), wire, (M - 1) * ld_wire + cap);
}

int launch_sparse_message_parts(const GradientParts &parts, int64_t d, int64_t M, int b, const StreamKey &key, uint32_t worker0,
                                uint32_t *packed, int64_t ld_words, uint32_t *wire, int64_t ld_wire, float *delta_out,
                                int32_t *kept_out, int32_t *nnz_out, uint32_t *status, hipStream_t st)
{
    const int pb = position_bits(d), per = static_cast<int>(sparse_parts_quads(d, parts.parts));
    const size_t lds = static_cast<size_t>(std::min(ceil_div(4ll * per * (pb + b), 32) + 2, kWireLdsWords)) * 4;
    const dim3 grid(static_cast<unsigned>(M), static_cast<unsigned>(parts.parts)), block(kWireThreads);
    int rc;
#define DQ_MESSAGE(F)                                                                                                       \
    if ((rc = allow_lds<sparse_message_parts_kernel<F>>()) != DQ_OK) return rc;                                             \
    sparse_message_parts_kernel<F><<<grid, block, lds, st>>>(parts.rows, parts.ld, d, per, parts.part_max, parts.part_kept, key, worker0, pb, \
                                                             packed, ld_words, wire, ld_wire, delta_out, kept_out, nnz_out, status)
    if (b == 8) { DQ_MESSAGE(8); }
    else { DQ_MESSAGE(4); }
#undef DQ_MESSAGE
    DQ_LAUNCH_CHECK();
    return DQ_OK;
}

}  // namespace dq

using namespace dq;
static inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

extern "C" int64_t dq_sparse_stream_words(int64_t d, int32_t b)
{
    if (d <= 0 || b < 2 || b > 8) return DQ_ERR_INVALID_ARG;
    return (d * (position_bits(d) + b) + 31) / 32;
}

extern "C" int32_t dq_sparse_encode(const uint32_t *packed, int64_t ld_words, int64_t d, int64_t M, int32_t b,
                                    uint32_t *stream_out, int64_t ld_stream, int32_t *nnz_out, void *stream)
{
    if (d <= 0 || M <= 0 || !packed || !stream_out || !nnz_out) return DQ_ERR_INVALID_ARG;
    if (b != 2 && b != 4 && b != 8) return (b >= 2 && b <= 8) ? DQ_ERR_UNSUPPORTED : DQ_ERR_INVALID_ARG;
    const int64_t row_words = packed_words(d, b), cap = dq_sparse_stream_words(d, b);
    if (ld_words < row_words || ld_stream < cap || !aligned16(packed) || (M > 1 && ld_words % 4 != 0)) return DQ_ERR_INVALID_ARG;
    if (cap > kWireLdsWords) return DQ_ERR_UNSUPPORTED;
    const int pb = position_bits(d);
    // one block per compute unit over all rows, none with fewer than 512 words (each block reads its whole row again)
    const int64_t spans = std::max(ceil_div(cap, kEncodeSpan), std::min(ceil_div(256, M), ceil_div(cap, 512)));
    const int span = static_cast<int>(ceil_div(cap, spans));
    const int per = static_cast<int>(ceil_div(row_words, kWireThreads)) | 1;
    const size_t lds = (static_cast<size_t>(span) + static_cast<size_t>(per) * kWireThreads) * 4;
    const bool in_place = ranges_overlap(packed, (M - 1) * ld_words + row_words, stream_out, (M - 1) * ld_stream + cap);
    const dim3 grid(static_cast<unsigned>(M), in_place ? 1u : static_cast<unsigned>(ceil_div(cap, span))), block(kWireThreads);
    hipStream_t st = as_stream(stream);
    int rc;
#define DQ_ENCODE(F)                                                                                                     \
    if ((rc = allow_lds<sparse_encode_kernel<F>>()) != DQ_OK) return rc;                                                 \
    sparse_encode_kernel<F><<<grid, block, lds, st>>>(packed, ld_words, static_cast<int>(row_words), static_cast<int>(d), \
                                                      pb, stream_out, ld_stream, static_cast<int>(cap), span, per, nnz_out)
    if (b == 8) { DQ_ENCODE(8); }
    else if (b == 4) { DQ_ENCODE(4); }
    else { DQ_ENCODE(2); }
#undef DQ_ENCODE
    DQ_LAUNCH_CHECK();
    return DQ_OK;
}

extern "C" int32_t dq_sparse_decode(const uint32_t *stream_in, int64_t ld_stream, const int32_t *nnz, int64_t d, int64_t M,
                                    int32_t b, uint32_t *packed_out, int64_t ld_words, void *stream)
{
    if (d <= 0 || M <= 0 || !stream_in || !nnz || !packed_out) return DQ_ERR_INVALID_ARG;
    if (b != 2 && b != 4 && b != 8) return (b >= 2 && b <= 8) ? DQ_ERR_UNSUPPORTED : DQ_ERR_INVALID_ARG;
    const int64_t row_words = packed_words(d, b), cap = dq_sparse_stream_words(d, b);
    if (ld_words < row_words || ld_stream < cap) return DQ_ERR_INVALID_ARG;
    if (row_words > kWireLdsWords) return DQ_ERR_UNSUPPORTED;
    const int pb = position_bits(d);
    // (each block reads its row's whole stream: no more blocks than keep every thread busy with a word of its own)
    const bool in_place = ranges_overlap(packed_out, (M - 1) * ld_words + row_words, stream_in, (M - 1) * ld_stream + cap);
    const int span = static_cast<int>(ceil_div(row_words, in_place ? 1 : std::min(ceil_div(256, M), ceil_div(row_words, kWireThreads))));
    const size_t lds = static_cast<size_t>(span) * 4;
    const dim3 grid(static_cast<unsigned>(M), static_cast<unsigned>(ceil_div(row_words, span))), block(kWireThreads);
    hipStream_t st = as_stream(stream);
    int rc;
#define DQ_DECODE(F)                                                                                     \
    if ((rc = allow_lds<sparse_decode_kernel<F>>()) != DQ_OK) return rc;                                 \
    sparse_decode_kernel<F><<<grid, block, lds, st>>>(stream_in, ld_stream, nnz, d, pb, packed_out, ld_words, \
                                                      static_cast<int>(row_words), span)
    if (b == 8) { DQ_DECODE(8); }
    else if (b == 4) { DQ_DECODE(4); }
    else { DQ_DECODE(2); }
#undef DQ_DECODE
    DQ_LAUNCH_CHECK();
    return DQ_OK;
}
