// The rounds of a dq_run_rounds call on CSR features in one launch, on the compute units of one die (see die.h).
//
// A round on bag-of-words rows moves little: 72,000 x 20,958, eight workers of 32 rows of 52 entries, 13,000 entries, a model and
// eight gradients of 21,000 coordinates.  As launches (worker step, master) it is 11.4 us, of which the two launches and what each
// needs to get under way are half; like this 9.3 us (282 rounds a call: 3236 us, now 2680).  The blocks stay, and a round is:
//   members that are worker m's slice s (the first M * S of them, see csr_worker_kernel's SLICED): the model's message into
//     LDS, products, margins, coefficients, the slice's fixed-point sums, the slice of the gradient to memory (3.8 us)
//   -- exchange, with the slices' maxima (1.2 us) -- every member for its columns, `chunks` * 256 of them, and all workers: quantize,
//     aggregate, update the model (2.2 us)
//   -- exchange, with the models' maxima (1.2 us) -- quantize its columns of the model, which are its part of the message (0.5 us)
//   -- exchange (1.0 us) --
// What bounds it is the chain: 0.3 to 0.6 us for each of a dozen short phases between barriers.
// The model crosses as its message, 21 KB here, which every member reads whole and gathers from in LDS: gathers from the
// vector in L2 by 32 compute units at once are 53,000 requests, 1.4 us.
// One wavefront waits at an exchange; the others draw random words meanwhile, and lay out the mini-batches of the next
// round, which do not depend on the model: the rows two rounds ahead (one wavefront), their entries into registers.
// The arithmetic is that of the separate kernels in the same order: the results are theirs bit for bit.  Alg. 2 keeps its
// launches: with it, this kernel needs more registers than there are, and the waits for scratch memory are 50 us a round.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "csr_rows.h"
#include "die.h"
#include "grad_launch.h"

namespace dq {

constexpr int kNoRow = 0x7FFFFFFF;                        // where the rows past the last one begin
constexpr int kReadAhead = 4;                             // entries that a thread has under way where it reads them in the round

static_assert(kBusyWaves == kCsrWaves - 1 && kBusy == kBusyWaves * kWave, "one wavefront waits at exchanges");

// In the workspace; zero before the launch.
struct CsrRoundsControl {
    DieControl die;
    uint32_t slice[kDieUnits];                           // SHARED: the slices' largest magnitudes
};
static_assert(sizeof(CsrRoundsControl) <= kRoundsControl, "room in the workspace");

struct CsrRoundsArgs {
    CsrView A;
    const float *z_snap;
    int M, B, b, b_x;
    int S, win;                                          // slices of a worker, columns of one
    int chunks;                                          // of a member
    int cap;                                             // entries of a group of rows (CsrPlan::cap)
    int room;                                            // entries that LDS has room for
    float l2, scale, eta, theta, kappa;
    uint32_t k0, k1, iter0;                              // seed halves; iter of the first round of the call
    int t0, rounds, flag_first;                          // parity of the first round; its flag-bit case
    float *x, *yv, *xsum; const float *x_snap, *g_snap;
    uint32_t *xq; float *delta_x, *absmax_x;
    uint32_t *packed; int64_t ld_words;
    float *delta;
    uint32_t *status;
    float *rows; int64_t ld;                             // M gradients
    CsrRoundsControl *ctl;
    int want, join, shared;                              // parts; members wanted; SHARED whatever comes
    int patience;                                        // see die_join
};

struct CsrRoundsLds {
    RowMeta meta;
    float label[kCsrMaxRows];
    uint32_t slice[kDieUnits];                           // the slices' largest magnitudes
    float amax[kDieUnits], delta[kDieUnits];             // of the workers' gradients: largest magnitude, scale
    uint32_t top[2][kCsrWaves];
    __align__(16) uint32_t message[kMostChunks * kChunk * 16 / 32];    // this member's part of the model's
    int total, poison, dead, sh[3];
    uint32_t slice_max, value;
};
static_assert(sizeof(CsrRoundsLds) + 512 <= kRoundsFixedLds, "static LDS");

// The arguments, read again wherever they are used: more of them than there are scalar registers to keep them in.
typedef const CsrRoundsArgs __attribute__((address_space(4))) *CsrRoundsArgsPtr;

static __device__ uint32_t dies_taken[kDies];            // see die.h

// A round has `want` parts, a range of columns and at most one slice of a worker each.  A member has one of them and keeps the
// state of its columns in registers.  SHARED: where the members are too few, they have every `count`-th part each, one after the
// other, and keep the state in memory.
template <bool ACC, bool EACH, bool SHARED>
__device__ __forceinline__ void csr_rounds_of(int me, int count, CsrRoundsLds &l, float *lds, CsrRoundsArgsPtr a)
{
    const DieMember die{&a->ctl->die, me, count};
    int t = threadIdx.x, lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
    const bool messenger = wave == kCsrWaves - 1, planner = wave == kCsrWaves - 2;
    int d = static_cast<int>(a->A.d), M = a->M, B = a->B, b_x = a->b_x, chunks = a->chunks, C = chunks * kChunk;
    const int S = a->S, win = a->win;
    // What the compiler can work out beforehand for every round it keeps, where there are no registers for it in scratch memory,
    // and waits for that in every round: so the numbers that it would start from go through registers it cannot see across.
    const auto forget = [&]() {
        uint64_t args = reinterpret_cast<uint64_t>(a);
        uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(args)), hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(args >> 32));
        for (int *n : {&wave, &d, &M, &B, &b_x, &chunks}) *n = __builtin_amdgcn_readfirstlane(*n);
        asm volatile("" : "+s"(lo), "+s"(hi), "+s"(wave), "+s"(d), "+s"(M), "+s"(B), "+s"(b_x), "+s"(chunks));
        a = reinterpret_cast<CsrRoundsArgsPtr>(static_cast<uint64_t>(hi) << 32 | lo);
        asm volatile("" : "+v"(t));
        lane = t & (kWave - 1);
        C = chunks * kChunk;
    };
    const int tasks = M * S, parts = SHARED ? a->want : die.me + 1, stride = SHARED ? die.count : 1;
    const int message_words = (d * b_x + 31) / 32, message_room = (message_words + 1 + 3) / 4 * 4, room = a->room;
    int *acc = reinterpret_cast<int *>(lds);                              // the slice's sums
    uint32_t *model = reinterpret_cast<uint32_t *>(lds + win);            // the model's message
    float *prod = lds + win + message_room;                               // products; later the codes
    float *snap = prod + room;                                            // the snapshot
    uint32_t *codes = reinterpret_cast<uint32_t *>(prod);
    if (t == 0) l.dead = l.poison = 0;
    for (int j = 4 * t; j < win; j += 4 * kCsrThreads) *reinterpret_cast<int4 *>(acc + j) = make_int4(0, 0, 0, 0);
    for (int j = t; j < d; j += kCsrThreads) snap[j] = a->x_snap[j];

    // ---- mini-batches
    const int my_m = __builtin_amdgcn_readfirstlane(die.me / S);
    const bool has_task = die.me < tasks;
    // the planner's rows: lane + 64 u
    int64_t row_start[2] = {0, 0}, row_end[2] = {0, 0};
    float row_y[2] = {0.0f, 0.0f}, row_z[2] = {0.0f, 0.0f};
    const auto plan_rows = [&](int m, uint32_t iter) {   // draws them and requests their extents, labels, margins
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (u * kWave >= B) break;
            const int r = lane + kWave * u;
            row_start[u] = row_end[u] = 0;
            if (r < B) {
                const StreamKey key{a->k0, a->k1, iter, static_cast<uint32_t>(m), DQ_TAG_SAMPLE};
                const uint4 w = stream_block(key, static_cast<uint32_t>(r >> 2));
                const uint32_t word = r & 2 ? (r & 1 ? w.w : w.z) : (r & 1 ? w.y : w.x);
                const uint32_t i = __umulhi(word, static_cast<uint32_t>(a->A.n));
                row_start[u] = a->A.indptr[i];
                row_end[u] = a->A.indptr[i + 1];
                row_y[u] = a->A.y[i];
                row_z[u] = a->z_snap[i];
            }
        }
    };
    const auto leave_rows = [&]() {                      // ... and leaves them in LDS
        int base = 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (u * kWave >= B) break;
            const int len = static_cast<int>(row_end[u] - row_start[u]), r = lane + kWave * u, incl = wave_scan_i32(len);
            if (r < B) {
                const int pre = base + incl - len, end = base + incl;
                l.meta.start[r] = row_start[u];
                l.meta.len[r] = len;
                l.meta.pre[r] = pre;
                l.meta.pre[r + 1] = end;                 // (the next row's lane writes the same)
                l.label[r] = row_y[u];
                l.meta.z[r] = row_z[u];
                for (int c = (pre + kWave - 1) / kWave; c * kWave < end && c < kChunkSlots; ++c) l.meta.chunk_row[c] = r;
            }
            base += __builtin_amdgcn_readlane(incl, kWave - 1);
        }
        if (lane <= kNextRows) l.meta.pre[B + 1 + lane] = kNoRow;
        if (lane == 0) l.total = base;
    };
    // Entry p of the batch is thread p % kBusy's number p / kBusy.
    uint32_t at[kEntriesEach];                           // column, row above it
    float val[kEntriesEach];
    const auto fits = [&](int total) { return total <= room && total <= a->cap; };
    const auto request_entries = [&]() {
        const int total = __builtin_amdgcn_readfirstlane(l.total);
        if (messenger || !fits(total)) return;
        const int32_t *indices = a->A.indices;
        const float *values = a->A.values;
#pragma unroll
        for (int u0 = 0; u0 < kEntriesEach; u0 += 2) {
            if (wave * kWave + u0 * kBusy >= total) break;
            int r[2], p[2];
            int64_t src[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int first = min(wave * kWave + (u0 + u) * kBusy, (total - 1) & ~(kWave - 1));
                p[u] = min(first + lane, total - 1);
                r[u] = l.meta.chunk_row[first >> 6];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {                // the last row that starts at or before p: among the next few
                const int r0 = __builtin_amdgcn_readfirstlane(r[u]);
                int next[kNextRows + 1];                 // (past the last row: the end of the batch, then kNoRow)
#pragma unroll
                for (int n = 0; n <= kNextRows; ++n) next[n] = l.meta.pre[r0 + 1 + n];
                r[u] = r0;
#pragma unroll
                for (int n = 0; n < kNextRows; ++n) r[u] += next[n] <= p[u] ? 1 : 0;
                if (__any(next[kNextRows] <= p[u]))      // (more rows than that in 64 entries)
                    while (__any(l.meta.pre[r[u] + 1] <= p[u])) r[u] += l.meta.pre[r[u] + 1] <= p[u] ? 1 : 0;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) src[u] = l.meta.start[r[u]] + (p[u] - l.meta.pre[r[u]]);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                at[u0 + u] = static_cast<uint32_t>(indices[src[u]]) | static_cast<uint32_t>(r[u]) << kColBits;
                val[u0 + u] = values[src[u]];
            }
        }
    };
    uint32_t phase = 0;
    // An exchange; the others do `meanwhile` while the messenger waits.  What is to be read by other members has been waited
    // for by those who stored it, and a barrier passed since.  `arrived` gets, in the messenger's lane i, member i's value.  wait =
    // false: only the barrier.
    const auto exchange = [&](bool wait, uint32_t value, auto meanwhile, auto arrived) {
        forget();
        if (messenger) {
            if (wait) {
                __builtin_amdgcn_s_setprio(3);           // (the others are ahead of their time)
                const uint32_t v = die_wait(die, ++phase, value, &l.dead);
                arrived(v);
                __builtin_amdgcn_s_setprio(0);
            }
        } else {
            meanwhile();
        }
        __syncthreads();
        forget();
        return __builtin_amdgcn_readfirstlane(l.dead) == 0;
    };
    const bool has_units = wave < kUnitWaves;
    int tops = 0;
    const auto block_max = [&](uint32_t v) {
        uint32_t *top = l.top[tops];
        tops ^= 1;
        v = wave_max_u32(v);
        if (lane == 0) top[wave] = v;
        __syncthreads();
        return wave_max_u32(lane < kCsrWaves ? top[lane] : 0u);
    };
    const bool straddles = (32 % b_x) != 0;
    const auto model_code = [&](int c) {                 // from the message in LDS
        const int bit = c * b_x;
        const uint32_t lo = model[bit >> 5], hi = straddles ? model[(bit >> 5) + 1] : 0u;
        return sext_field(__funnelshift_r(lo, hi, static_cast<unsigned>(bit) & 31u), 0, static_cast<unsigned>(b_x));
    };

    // The member's columns: thread t has t + 960 n, and keeps their state.
    float xv[kColumns], yv[kColumns], sum[kColumns], gs[kColumns], xs_own[kColumns];
    const auto load_state = [&](int member) {
#pragma unroll
        for (int n = 0; n < kColumns; ++n) {
            const int j = t + n * kBusy, i = member * C + j;
            const bool in = !messenger && j < C && i < d;
            xv[n] = in ? load_fresh(a->x + i) : 0.0f;
            gs[n] = in ? a->g_snap[i] : 0.0f;
            if constexpr (ACC) {
                yv[n] = in ? load_fresh(a->yv + i) : 0.0f;
                sum[n] = in ? load_fresh(a->xsum + i) : 0.0f;
                xs_own[n] = in ? a->x_snap[i] : 0.0f;
            }
        }
    };
    if constexpr (!SHARED) load_state(die.me);

    // the random words of a new model
    uint32_t word[kColumns];
    const auto draw_model_words = [&](int member, uint32_t iter) {
#pragma unroll
        for (int n = 0; n < kColumns; ++n) {
            if (n * kBusy >= C) break;
            const uint32_t i = static_cast<uint32_t>(member * C + t + n * kBusy);
            const uint4 w = stream_block(StreamKey{a->k0, a->k1, iter, DQ_MASTER_ID, DQ_TAG_MODEL}, i >> 2);
            word[n] = i & 2 ? (i & 1 ? w.w : w.z) : (i & 1 ? w.y : w.x);
        }
    };
    if (a->flag_first || SHARED) draw_model_words(die.me, a->iter0 + 1u);
    float *const rows = a->rows;
    const int64_t ld = a->ld;
    float delta_x = a->flag_first ? 0.0f : a->delta_x[0];
    const int units = M * chunks;                        // wavefront w takes chunk (worker, member's chunk) number w + 14 p
    const uint32_t per_chunk = (65536u + static_cast<uint32_t>(chunks) - 1u) / static_cast<uint32_t>(chunks);
    const auto worker_of = [&](int unit) { return static_cast<int>(static_cast<uint32_t>(unit) * per_chunk >> 16); };    // unit / chunks
    const int first_round = !SHARED && !a->flag_first ? -1 : 0;           // (-1: only what round 0 needs beforehand)
    __syncthreads();
    for (int k = first_round; k < a->rounds; ++k) {
        const bool last = k == a->rounds - 1, flag = k == 0 && a->flag_first, active = k >= 0, gradients = active && !flag;
        forget();
        const uint32_t iter = a->iter0 + static_cast<uint32_t>(k);
        const bool ahead = !SHARED && has_task && !last;  // the next round's mini-batch is laid out in this one
        // ---- worker side: the slices of the gradients
        if (gradients && has_task) {                     // (the same for every thread)
            // the model's message, two pieces of a thread's together (past its end: zeros)
            const uint32_t size = static_cast<uint32_t>(message_words) * 4u;
            const uint32_t *xq = a->xq;
            const uint4 piece0 = load_fresh16(xq, size, 16u * static_cast<uint32_t>(t)),
                        piece1 = load_fresh16(xq, size, 16u * static_cast<uint32_t>(t + kCsrThreads));
            if (4 * t < message_words) *reinterpret_cast<uint4 *>(model + 4 * t) = piece0;
            if (4 * (t + kCsrThreads) < message_words) *reinterpret_cast<uint4 *>(model + 4 * (t + kCsrThreads)) = piece1;
#pragma unroll 1
            for (int w = 4 * (t + 2 * kCsrThreads); w < message_words; w += 4 * kCsrThreads)
                *reinterpret_cast<uint4 *>(model + w) = load_fresh16(xq, size, 4u * static_cast<uint32_t>(w));
        }
        if (gradients && has_task) {
            const float inv_B = 1.0f / static_cast<float>(B);
#pragma unroll 1
            for (int task = die.me; task < (SHARED ? tasks : die.me + 1); task += stride) {
                const int m = SHARED ? task / S : my_m, c0 = (task - m * S) * win, c1 = min(d, c0 + win);
                if constexpr (SHARED) {
                    __syncthreads();
                    if (planner) {
                        plan_rows(m, iter);
                        leave_rows();
                    }
                    __syncthreads();
                    request_entries();
                }
                const int total = __builtin_amdgcn_readfirstlane(l.total);
                const bool in_flight = fits(total);
                if (t == 0) l.slice_max = 0u;
                __syncthreads();                         // (the model's message)
                forget();
                FixedAcc fx{0.0f, 0};
                if (__builtin_expect(in_flight, 1)) {    // (the other code elsewhere: 9.3 us a round instead of 9.5)
                    uint32_t vmax = 0;
                    if (!messenger) {
#pragma unroll
                        for (int u0 = 0; u0 < kEntriesEach; u0 += 2) {
                            const int first = wave * kWave + u0 * kBusy;
                            if (first >= total) break;
#pragma unroll
                            for (int u = 0; u < 2; ++u) {        // (a position past the end repeats an entry)
                                const int c = static_cast<int>(at[u0 + u] & kColMask), e = first + u * kBusy + lane;
                                const float diff = delta_x * static_cast<float>(model_code(c)) - snap[c];
                                vmax = max(vmax, abs_bits(val[u0 + u]));
                                if (e < total) prod[e] = val[u0 + u] * diff;
                            }
                        }
                    }
                    vmax = wave_max_u32(vmax);
                    if (lane == 0) l.top[0][wave] = vmax;
                    __syncthreads();
                    forget();
                    const int lr = wave + lane * kCsrWaves, tr = min(lr, B - 1);
                    const int my_len = lr < B ? l.meta.len[tr] : 0, my_pre = l.meta.pre[tr];
                    const float my_y = l.label[tr], my_z = l.meta.z[tr];
                    const auto coef_of = [&](float dz) { return vr_slope_diff(my_y, my_z, dz) * inv_B; };
                    float margin = 0.0f;                 // lane l: of row wave + 16 l (sums as in csr_lane_margins)
#pragma unroll 1
                    for (int n = 0; wave + n * kCsrWaves < B; n += 2) {
                        int len[2], off[2];
                        float part[2] = {0.0f, 0.0f};
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            len[u] = __builtin_amdgcn_readlane(my_len, n + u);
                            off[u] = __builtin_amdgcn_readlane(my_pre, n + u);
                        }
                        const int longest = max(len[0], len[1]);
#pragma unroll 1
                        for (int e = lane; e - lane < longest; e += 3 * kWave) {
                            float q[2][3];
#pragma unroll
                            for (int u = 0; u < 2; ++u)
#pragma unroll
                                for (int w = 0; w < 3; ++w) q[u][w] = prod[min(off[u] + e + w * kWave, room - 1)];
#pragma unroll
                            for (int u = 0; u < 2; ++u)
#pragma unroll
                                for (int w = 0; w < 3; ++w) part[u] += e + w * kWave < len[u] ? q[u][w] : 0.0f;
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const float sum_r = wave_sum_f32(part[u]);
                            margin = lane == n + u ? sum_r : margin;
                        }
                    }
                    if (lr < B) l.meta.coef[lr] = coef_of(margin);
                    __syncthreads();
                    forget();
                    float csum = 0.0f;
                    {
                        const float c0v = fabsf(l.meta.coef[lane]), c1v = fabsf(l.meta.coef[lane + kWave]);
                        csum += lane < B ? c0v : 0.0f;   // (as coef_abs_sum; B <= 128)
                        csum += lane + kWave < B ? c1v : 0.0f;
                    }
                    vmax = wave_max_u32(lane < kCsrWaves ? l.top[0][lane] : 0u);
                    fixed_admit(fx, wave_sum_f32(csum) * __uint_as_float(vmax), acc, c1 - c0, &l.poison);
                    const float two_k = ldexpf(1.0f, fx.k);
                    if (!messenger) {
#pragma unroll
                        for (int u0 = 0; u0 < kEntriesEach; u0 += 2) {
                            const int first = wave * kWave + u0 * kBusy;
                            if (first >= total) break;
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                const int c = static_cast<int>(at[u0 + u] & kColMask) - c0;
                                const float cf = l.meta.coef[at[u0 + u] >> kColBits];
                                if (first + u * kBusy + lane < total && c >= 0 && c < c1 - c0) atomicAdd(&acc[c], fixed_term(cf, val[u0 + u], two_k));
                            }
                        }
                    }
                    __syncthreads();
                } else {
                    // ---- more entries than that: straight from memory, in the groups of rows that a step stages, by entries and not by
                    // rows, of which one can be most of the batch (a row a wavefront: 64 rows of lognormal length, sigma 2, 46.6 us a
                    // round, now 20.2; 32 of 1000 entries 84, now 51)
                    const int row_ends[2] = {lane < B ? l.meta.pre[lane + 1] : kNoRow, lane + kWave < B ? l.meta.pre[lane + kWave + 1] : kNoRow};
#pragma unroll 1
                    for (int g0 = 0, g1; g0 < B; g0 = g1) {
                        const int base = __builtin_amdgcn_readfirstlane(l.meta.pre[g0]), cap = a->cap;
                        g1 = B;
                        if (__builtin_amdgcn_readfirstlane(l.meta.pre[B]) - base > cap) {
                            int lo = g0, hi = B - 1;     // the first row whose end lies past the buffer
                            while (lo < hi) {
                                const int mid = (lo + hi) >> 1;
                                if (__builtin_amdgcn_readfirstlane(l.meta.pre[mid + 1]) - base > cap) hi = mid;
                                else lo = mid + 1;
                            }
                            g1 = max(lo, g0 + 1);
                        }
                        const int end = __builtin_amdgcn_readfirstlane(l.meta.pre[g1]);
                        // Entries from .. to of the batch, kReadAhead of a thread's requested together: take(entry, row, column, value).  A
                        // wavefront's 64 begin in the row that as many rows end before.
                        const auto each_entry = [&](int from, int to, auto take) {
#pragma unroll 1
                            for (int p0 = from + wave * kWave; p0 < to; p0 += kReadAhead * kCsrThreads) {
                                uint32_t where[kReadAhead];          // column, row above it
                                float v[kReadAhead];
#pragma unroll
                                for (int u0 = 0; u0 < kReadAhead; u0 += 2) {
                                    if (p0 + u0 * kCsrThreads >= to) break;
                                    int r[2], next[2][kNextRows + 1];
#pragma unroll
                                    for (int u = 0; u < 2; ++u) {
                                        const int first = min(p0 + (u0 + u) * kCsrThreads, to - 1);
                                        r[u] = __popcll(__ballot(row_ends[0] <= first)) + __popcll(__ballot(row_ends[1] <= first));
#pragma unroll
                                        for (int n = 0; n <= kNextRows; ++n) next[u][n] = l.meta.pre[r[u] + 1 + n];
                                    }
#pragma unroll
                                    for (int u = 0; u < 2; ++u) {
                                        const int p = min(p0 + (u0 + u) * kCsrThreads + lane, to - 1);
                                        int row = r[u];
#pragma unroll
                                        for (int n = 0; n < kNextRows; ++n) row += next[u][n] <= p ? 1 : 0;
                                        if (__any(next[u][kNextRows] <= p))
                                            while (__any(l.meta.pre[row + 1] <= p)) row += l.meta.pre[row + 1] <= p ? 1 : 0;
                                        const int64_t src = l.meta.start[row] + (p - l.meta.pre[row]);
                                        where[u0 + u] = static_cast<uint32_t>(a->A.indices[src]) | static_cast<uint32_t>(row) << kColBits;
                                        v[u0 + u] = a->A.values[src];
                                    }
                                }
#pragma unroll
                                for (int u = 0; u < kReadAhead; ++u) {
                                    const int p = p0 + u * kCsrThreads + lane;
                                    if (p < to) take(p, static_cast<int>(where[u] >> kColBits), static_cast<int>(where[u] & kColMask), v[u]);
                                }
                            }
                        };
                        const auto leave_coef = [&](int r, float dz) { l.meta.coef[r] = vr_slope_diff(l.label[r], l.meta.z[r], dz) * inv_B; };
                        if (g0 + t < g1 && l.meta.len[g0 + t] == 0) leave_coef(g0 + t, 0.0f);
                        // Products, as many as there is room for at a time, and the margins from them.  A row that goes on in the next
                        // piece is cut at a multiple of 64 entries, so each lane's sum goes on where it was.
                        uint32_t vmax = 0;
                        float part = 0.0f;               // of the one row of the wavefront that goes on
#pragma unroll 1
                        for (int p0 = base, p1; p0 < end; p0 = p1) {
                            p1 = end;
                            if (end - p0 > room) {
                                int lo = g0, hi = g1 - 1;        // the last row that starts within the room
                                while (lo < hi) {
                                    const int mid = (lo + hi + 1) >> 1;
                                    if (__builtin_amdgcn_readfirstlane(l.meta.pre[mid]) - p0 <= room) lo = mid;
                                    else hi = mid - 1;
                                }
                                const int first = __builtin_amdgcn_readfirstlane(l.meta.pre[lo]);
                                p1 = min(first + ((p0 + room - first) & ~(kWave - 1)), __builtin_amdgcn_readfirstlane(l.meta.pre[lo + 1]));
                            }
                            each_entry(p0, p1, [&](int p, int, int c, float v) {
                                vmax = max(vmax, abs_bits(v));
                                prod[p - p0] = v * (delta_x * static_cast<float>(model_code(c)) - snap[c]);
                            });
                            __syncthreads();
#pragma unroll 1
                            for (int r = g0 + wave; r < g1; r += kCsrWaves) {
                                const int first = __builtin_amdgcn_readfirstlane(l.meta.pre[r]), beyond = __builtin_amdgcn_readfirstlane(l.meta.pre[r + 1]);
                                if (beyond <= p0 || first >= p1 || first == beyond) continue;
                                float sum_r = first < p0 ? part : 0.0f;
                                const int to = min(beyond, p1) - p0;
#pragma unroll 2
                                for (int e = max(first - p0, 0) + lane; e < to; e += kWave) sum_r += prod[e];
                                if (beyond > p1) {
                                    part = sum_r;
                                } else {
                                    sum_r = wave_sum_f32(sum_r);
                                    if (lane == 0) leave_coef(r, sum_r);
                                }
                            }
                            __syncthreads();
                        }
                        vmax = block_max(vmax);
                        fixed_admit(fx, coef_abs_sum(l.meta.coef, g0, g1) * __uint_as_float(vmax), acc, c1 - c0, &l.poison);
                        const float two_k = ldexpf(1.0f, fx.k);
                        each_entry(base, end, [&](int, int r, int c, float v) {
                            if (c >= c0 && c < c1) atomicAdd(&acc[c - c0], fixed_term(l.meta.coef[r], v, two_k));
                        });
                        __syncthreads();
                    }
                    // (what the registers for entries held is of no use: no need to keep it meanwhile)
#pragma unroll
                    for (int u = 0; u < kEntriesEach; ++u) asm volatile("" : "=v"(at[u]), "=v"(val[u]));
                }
                forget();
                // the slice becomes float32: the dense part l2 * (q - snapshot) and the sums, zeros past the end of the vector
                const float unit = l.poison ? __uint_as_float(0x7FC00000u) : ldexpf(1.0f, -fx.k), l2 = a->l2;
                float *row = rows + m * ld;
                uint32_t seen = 0;
                const int last_quad = (c1 - c0 - 1) & ~3;
#pragma unroll 1
                for (int j0 = 4 * t; j0 <= last_quad; j0 += 8 * kCsrThreads) {
                    int4 terms[2];
                    float4 x0[2];
                    uint32_t bytes[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {        // (a quad past the end: the last one again, not used)
                        const int j = min(j0 + 4 * u * kCsrThreads, last_quad), c = c0 + j;
                        terms[u] = *reinterpret_cast<const int4 *>(acc + j);
                        x0[u] = *reinterpret_cast<const float4 *>(snap + c);
                        bytes[u] = model[c >> 2];        // (of use where a field is a byte)
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int j = j0 + 4 * u * kCsrThreads, c = c0 + j;
                        if (j > last_quad) continue;
                        *reinterpret_cast<int4 *>(acc + j) = make_int4(0, 0, 0, 0);
                        int code[4];
                        if (b_x == 8) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) code[e] = sext_field(bytes[u], 8u * e, 8u);
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e) code[e] = model_code(min(c + e, d - 1));
                        }
                        const float xs4[4] = {x0[u].x, x0[u].y, x0[u].z, x0[u].w};
                        const int sums[4] = {terms[u].x, terms[u].y, terms[u].z, terms[u].w};
                        float v[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            v[e] = l2 * (delta_x * static_cast<float>(code[e]) - xs4[e]);
                            v[e] += static_cast<float>(sums[e]) * unit;
                            if (c + e >= d) v[e] = 0.0f;
                            seen = max(seen, abs_bits(v[e]));
                        }
                        *reinterpret_cast<float4 *>(row + c) = make_float4(v[0], v[1], v[2], v[3]);
                    }
                }
                seen = wave_max_u32(seen);
                if (lane == 0) atomicMax(&l.slice_max, seen);
                wait_for_memory();
                __syncthreads();
                if (messenger && lane == 0) {
                    if constexpr (SHARED) a->ctl->slice[task] = l.slice_max;
                    else l.slice[task] = l.slice_max;    // (in the member's own place: its value at the exchange)
                    l.poison = 0;
                }
                if (SHARED && messenger) wait_for_memory();
            }
        }
        // ---- master side
        uint4 words[kPasses];
        const auto unit_of = [&](int p) { return min(wave + kUnitWaves * p, units - 1); };
        const auto draw_words = [&](int member) {
            if (!has_units) return;
#pragma unroll
            for (int p = 0; p < kPasses; ++p) {
                const int unit = unit_of(p), m = worker_of(unit), q = (member * chunks + unit - m * chunks) * (kChunk / 4) + lane;
                words[p] = stream_block(StreamKey{a->k0, a->k1, iter, static_cast<uint32_t>(m), DQ_TAG_GRAD}, static_cast<uint32_t>(q));
            }
        };
        if (!exchange(gradients, has_task ? l.slice_max : 0u, [&] {
                if (gradients && !SHARED) draw_words(die.me);
                if (ahead && planner) {
                    if (k == first_round) plan_rows(my_m, iter + 1u);
                    leave_rows();
                }
            }, [&](uint32_t v) {                         // the gradients' largest magnitudes
                if (lane < tasks) l.slice[lane] = SHARED ? load_fresh(a->ctl->slice + lane) : v;
                uint32_t amax = 0;
#pragma unroll
                for (int n0 = 0; n0 < 16; n0 += 4) {
                    if (n0 >= S) break;
#pragma unroll
                    for (int n = n0; n < n0 + 4; ++n) amax = max(amax, l.slice[min(lane * S + min(n, S - 1), kDieUnits - 1)]);
                }
                if (lane < M) l.amax[lane] = __uint_as_float(amax);
            })) break;
        uint32_t top = 0;
        if (active) {
            float4 v[kPasses];
            const auto load_rows = [&](int member) {
                if (!has_units) return;
#pragma unroll
                for (int p = 0; p < kPasses; ++p) {
                    const int unit = unit_of(p), m = worker_of(unit), q = (member * chunks + unit - m * chunks) * (kChunk / 4) + lane;
                    v[p] = load_fresh_f4(rows + m * ld, static_cast<uint32_t>(ld) * 4u, 16u * static_cast<uint32_t>(q));
                }
            };
            Scale scale[kPasses];                         // (while the rows are on their way)
            if (gradients) {
                if constexpr (!SHARED) load_rows(die.me);
                const int b = a->b;
                if (has_units) {
#pragma unroll
                    for (int p = 0; p < kPasses; ++p) scale[p] = make_scale(l.amax[worker_of(unit_of(p))], b);
                } else if (planner && lane < M) {
                    const Scale sc = make_scale(l.amax[lane], b);
                    l.delta[lane] = sc.delta;
                    if (die.me == 0 && sc.bad) atomicOr(a->status, 1u);
                    if (die.me == 0 && last) a->delta[lane] = sc.delta;
                }
            } else {
                if (last && die.me == 0 && t < M) a->delta[t] = 0.0f;
            }
#pragma unroll 1
            for (int member = die.me; member < parts; member += stride) {
                if constexpr (SHARED) {
                    __syncthreads();
                    load_state(member);
                    if (gradients) {
                        load_rows(member);
                        draw_words(member);
                    }
                }
                const int b = a->b;
                if (gradients) {
                    if (has_units) {
#pragma unroll
                        for (int p = 0; p < kPasses; ++p) {
                            int c[4] = {0, 0, 0, 0};
                            if (scale[p].inv_delta != 0.0f) {
                                c[0] = quantize_one(v[p].x, scale[p], words[p].x); c[1] = quantize_one(v[p].y, scale[p], words[p].y);
                                c[2] = quantize_one(v[p].z, scale[p], words[p].z); c[3] = quantize_one(v[p].w, scale[p], words[p].w);
                            }
                            codes[unit_of(p) * (kChunk / 4) + lane] = pack4<8>(c[0], c[1], c[2], c[3]);
                        }
                    }
                    __syncthreads();
                }
                if (last) {                              // the messages
                    const int quads = (d + 3) / 4;
                    uint32_t *packed = a->packed;
                    const int64_t ld_words = a->ld_words;
#pragma unroll 1
                    for (int unit = wave; unit < units; unit += kCsrWaves) {
                        const int m = worker_of(unit), q = (member * chunks + unit - m * chunks) * (kChunk / 4) + lane;
                        const uint32_t four = gradients && q < quads ? codes[unit * (kChunk / 4) + lane] : 0u;       // (past the end: zeros)
                        const int c0 = sext_field(four, 0, 8), c1 = sext_field(four, 8, 8), c2 = sext_field(four, 16, 8), c3 = sext_field(four, 24, 8);
                        uint32_t *out = packed + m * ld_words;
                        if (b == 8) store_quad_bits<8>(four, q, quads, out);
                        else if (b == 4) store_quad_bits<4>(q < quads ? pack4<4>(c0, c1, c2, c3) : 0u, q, quads, out);
                        else store_quad_bits<2>(q < quads ? pack4<2>(c0, c1, c2, c3) : 0u, q, quads, out);
                    }
                }
                const float eta = a->eta, kappa = a->kappa, theta = a->theta;
#pragma unroll
                for (int n = 0; n < kColumns; ++n) {
                    const int j = t + n * kBusy, i = member * C + j;
                    if (n * kBusy >= C) break;
                    if (messenger || j >= C || i >= d) continue;
                    float mean = 0.0f;
                    const auto apply = [&](float u) {    // one direction (Alg. 1 and 3, master (ii))
                        if constexpr (ACC) {
                            yv[n] = soft_threshold(yv[n] - eta * u, kappa);
                            xv[n] = xs_own[n] + theta * (yv[n] - xs_own[n]);
                            sum[n] = sum[n] + xv[n];
                        } else {
                            xv[n] = soft_threshold(xv[n] - eta * u, kappa);
                        }
                    };
                    if (flag) {
                        if constexpr (EACH)
                            for (int m = 0; m < M; ++m) apply(0.0f * 0.0f + gs[n]);
                    } else {
                        const uint32_t *word = codes + (j >> 2);
#pragma unroll 8
                        for (int m = 0; m < M; ++m) {
                            const float code = static_cast<float>(sext_field(word[m * (C / 4)], 8u * (j & 3), 8u)), delta = l.delta[m];
                            if constexpr (EACH) apply(delta * code + gs[n]);
                            else mean = fmaf(delta, code, mean);
                        }
                    }
                    if constexpr (!EACH) apply(a->scale * mean + gs[n]);
                    if (last || SHARED) {
                        a->x[i] = xv[n];
                        if constexpr (ACC) {
                            a->yv[i] = yv[n];
                            a->xsum[i] = sum[n];
                        }
                    }
                    top = max(top, abs_bits(xv[n]));
                }
                if constexpr (SHARED) wait_for_memory();
            }
            for (int w = t; w < kMostChunks * kChunk * 16 / 32; w += kCsrThreads) l.message[w] = 0u;
            top = block_max(top);
        }
        // ---- the model of the next round (Alg. 1, master (i))
        if (!exchange(active, top, [&] {
                if (ahead) request_entries();
            }, [&](uint32_t v) {
                v = wave_max_u32(v);
                if (lane == 0) l.value = v;
            })) break;
        if (active) {
            const Scale ms = make_scale(__uint_as_float(l.value), b_x);
            delta_x = ms.delta;
            if (die.me == 0 && t == 0) {
                a->absmax_x[(a->t0 + k) & 1] = __uint_as_float(l.value);
                if (last) a->delta_x[0] = ms.delta;
                if (ms.bad) atomicOr(a->status, 1u);
            }
#pragma unroll 1
            for (int member = die.me; member < parts; member += stride) {
                if (member != die.me) {
                    __syncthreads();
                    for (int w = t; w < kMostChunks * kChunk * 16 / 32; w += kCsrThreads) l.message[w] = 0u;
                    __syncthreads();
                    draw_model_words(member, iter + 1u);
                }
#pragma unroll
                for (int n = 0; n < kColumns; ++n) {
                    const int j = t + n * kBusy, i = member * C + j;
                    if (n * kBusy >= C) break;
                    if (messenger || j >= C || i >= d) continue;
                    const float x = SHARED ? load_fresh(a->x + i) : xv[n];
                    const int c = ms.inv_delta != 0.0f ? quantize_one(x, ms, word[n]) : 0;
                    if (b_x == 8) {
                        reinterpret_cast<uint8_t *>(l.message)[j] = static_cast<uint8_t>(c);
                        continue;
                    }
                    const int bit = j * b_x;             // (the field may continue in the next word)
                    const uint64_t bits = static_cast<uint64_t>(static_cast<uint32_t>(c) & ((1u << b_x) - 1u)) << (bit & 31);
                    if (static_cast<uint32_t>(bits)) atomicOr(l.message + (bit >> 5), static_cast<uint32_t>(bits));
                    if (bits >> 32) atomicOr(l.message + (bit >> 5) + 1, static_cast<uint32_t>(bits >> 32));
                }
                __syncthreads();
                const int per = C * b_x / 32, rest = message_words - member * per;
                if (messenger) {                         // (who has no other loads to wait for; a whole number of 32 bytes each)
                    uint32_t *out = a->xq + member * per;
                    for (int w = 4 * lane; w < min(per, rest); w += 4 * kWave) {
                        if (w + 3 < rest) {
                            *reinterpret_cast<uint4 *>(out + w) = *reinterpret_cast<const uint4 *>(l.message + w);
                        } else {
                            for (int n = w; n < rest; ++n) out[n] = l.message[n];
                        }
                    }
                }
            }
            if (messenger) wait_for_memory();
        }
        if (!exchange(active && !last, 0u, [&] {
                if (ahead && planner && k + 2 < a->rounds) plan_rows(my_m, iter + 2u);
                if (!planner || C > kBusy - kWave) draw_model_words(die.me, iter + 2u);
            }, [](uint32_t) {})) break;
    }
    if (t == 0) {
        if (l.dead) atomicOr(a->status, kGaveUp);
        die_leave(dies_taken, l.sh);
    }
}

template <bool ACC, bool EACH>
__global__ __launch_bounds__(kCsrThreads) void csr_rounds_kernel(const CsrRoundsArgs)
{
    extern __shared__ __align__(16) float lds[];
    __shared__ CsrRoundsLds l;
    const CsrRoundsArgsPtr a = (CsrRoundsArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    // (SHARED in the same kernel: as a second launch behind it, which mostly has nothing to do, it still had to wait for room on dies that
    // other launches held)
    const DieMember die = die_join(&a->ctl->die, dies_taken, static_cast<uint32_t>(a->join), a->patience, l.sh);
    if (die.me < 0) return;
    if (__builtin_expect(die.count == a->want && !a->shared, 1)) csr_rounds_of<ACC, EACH, false>(die.me, die.count, l, lds, a);
    else csr_rounds_of<ACC, EACH, true>(die.me, die.count, l, lds, a);
}

// ------------------------------------------------------------------ host side
int fill_u32(uint32_t *p, int64_t n, uint32_t value, hipStream_t st);

// (without a status word nobody would learn that the members gave up: die.h)
static bool csr_rounds_layout(const dq_problem *prob, const dq_run_config *cfg, const dq_run_state *st, int64_t rounds, CsrRoundsShape &s)
{
    return prob->layout == 1 && cfg->tau == 0 && st->z_snap && st->status && cfg->algo != DQ_ALGO_SPARSE && cfg->b != 32 &&
           csr_rounds_shape(prob->d, prob->n, prob->lda, cfg->M, cfg->B, cfg->b_x, rounds, s) &&
           st->ws_bytes >= csr_run_offset(prob->d, cfg->M) + kRoundsControl;
}

// A stream that may use a part of the compute units only (hipExtStreamCreateWithCUMask) need not have a whole die: with sixteen of each
// die's 32 a call waits 2 to 4 ms for one and then does its rounds with what there is, 27 us each over 282 rounds; as launches 11.5.
static bool whole_part(hipStream_t stream)
{
    // (default streams have no mask of their own; asked by this name for the legacy one's, the runtime crashes)
    if (stream == hipStreamLegacy || stream == hipStreamPerThread) return true;
    uint32_t mask[32] = {};
    int dev = 0, units = 0, in_mask = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipExtStreamGetCUMask(stream, sizeof(mask) / 4, mask) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    for (const uint32_t word : mask) in_mask += __builtin_popcount(word);
    return in_mask >= units;
}

bool csr_rounds_ok(const dq_problem *prob, const dq_run_config *cfg, const dq_run_state *st, int64_t rounds, hipStream_t stream)
{
    CsrRoundsShape s;
    return csr_rounds_layout(prob, cfg, st, rounds, s) && whole_part(stream);
}

// (for tests: no die is taken once all launches have ended)
int32_t csr_rounds_dies_taken(uint32_t *host)
{
    DQ_HIP_TRY(hipMemcpyFromSymbol(host, HIP_SYMBOL(dies_taken), sizeof(dies_taken)));
    return DQ_OK;
}

template <bool ACC, bool EACH>
static int csr_rounds_launch(const CsrRoundsArgs &a, size_t lds, hipStream_t stream)
{
    const auto kernel = csr_rounds_kernel<ACC, EACH>;
    static std::once_flag once;
    static hipError_t once_rc = hipSuccess;
    std::call_once(once, [&] {
        once_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      static_cast<int>(kRoundsLds));
    });
    DQ_HIP_TRY(once_rc);
    kernel<<<dim3(8u * static_cast<unsigned>(a.join)), dim3(kCsrThreads), lds, stream>>>(a);
    DQ_LAUNCH_CHECK();
    return DQ_OK;
}

int32_t csr_rounds(const dq_problem *prob, const dq_run_config *cfg, const dq_run_state *st, int64_t epoch, int64_t t0,
                   int64_t rounds, float eta, float theta, bool flag_first, int members, hipStream_t stream)
{
    const bool acc = cfg->algo == DQ_ALGO_ACC;
    const void *quads[] = {st->x, st->x_snap, st->g_snap, acc ? st->y : nullptr, acc ? st->xsum : nullptr, st->ws};
    for (const void *p : quads)
        if (p && !aligned16(p)) return DQ_ERR_INVALID_ARG;
    CsrRoundsShape s;
    if (!csr_rounds_layout(prob, cfg, st, rounds, s)) return DQ_ERR_UNSUPPORTED;
    CsrRoundsArgs a{};
    a.S = s.S; a.win = s.win; a.want = s.want; a.chunks = s.chunks; a.cap = s.cap; a.room = s.room;
    // the M rows of a step, its slices' results, then what dq_run_rounds has for itself
    a.ld = pad4(prob->d);
    a.rows = static_cast<float *>(st->ws);
    a.ctl = reinterpret_cast<CsrRoundsControl *>(static_cast<char *>(st->ws) + csr_run_offset(prob->d, cfg->M));
    a.join = members > 0 ? std::min(members, s.want) : s.want;
    a.shared = members > 0;
    const size_t lds = static_cast<size_t>(s.lds);
    a.A = CsrView{prob->indptr, prob->indices, prob->values, prob->y, prob->n, prob->d};
    a.z_snap = st->z_snap;
    a.M = static_cast<int>(cfg->M); a.B = static_cast<int>(cfg->B); a.b = cfg->b; a.b_x = cfg->b_x;
    a.l2 = prob->l2; a.scale = 1.0f / static_cast<float>(cfg->M); a.eta = eta; a.theta = theta; a.kappa = eta * prob->l1;
    a.k0 = static_cast<uint32_t>(cfg->seed); a.k1 = static_cast<uint32_t>(cfg->seed >> 32);
    a.x = st->x; a.yv = st->y; a.xsum = st->xsum; a.x_snap = st->x_snap; a.g_snap = st->g_snap;
    a.xq = st->xq; a.delta_x = st->delta_x; a.absmax_x = st->absmax_x;
    a.packed = st->packed; a.ld_words = st->ld_words; a.delta = st->delta; a.status = st->status;
    // A launch for every kMostRounds rounds, 5 ms or so: blocks of other streams' launches that are meant for the die wait that
    // long (the part deals a launch's blocks to the dies in turn).
    constexpr int64_t kMostRounds = 512;
    for (int64_t done = 0; done < rounds; done += kMostRounds) {
        a.iter0 = static_cast<uint32_t>(epoch * cfg->m + t0 + done);
        a.t0 = static_cast<int>((t0 + done) & 1); a.rounds = static_cast<int>(std::min(kMostRounds, rounds - done));
        a.flag_first = done == 0 && flag_first;
        // About as long as the rounds take, 10 us each, at most 2 to 4 ms: kernels of other streams end meanwhile, and with fewer members
        // the rounds take as much longer, 20 us each with 16 to 31 of 32, 35 with 8, 65 with 4, 244 with one.  (2 to 4 ms for calls of
        // eight rounds too: four processes 17.6 us for a round of each, like this 14.5, as launches 14.0.)
        a.patience = static_cast<int>(std::min<int64_t>(200000, 1000 * a.rounds));
        int rc = fill_u32(reinterpret_cast<uint32_t *>(a.ctl), sizeof(CsrRoundsControl) / 4, 0u, stream);
        if (rc != DQ_OK) return rc;
        const auto launch = [&](auto with_acc, auto each) {
            constexpr bool ACC = decltype(with_acc)::value, EACH = decltype(each)::value;
            return csr_rounds_launch<ACC, EACH>(a, lds, stream);
        };
        const std::true_type yes;
        const std::false_type no;
        if (acc) rc = cfg->each ? launch(yes, yes) : launch(yes, no);
        else rc = cfg->each ? launch(no, yes) : launch(no, no);
        if (rc != DQ_OK) return rc;
    }
    return DQ_OK;
}

}  // namespace dq
