// All rounds of a dq_run_rounds call on a small dense problem in one launch of one block (Alg. 1 and Alg. 3).
//
// At four workers, sixteen rows each and a thousand columns a round is two launches that the chip does nothing else
// beside: 7.4 + 3.2 us, of which the two launches themselves, the trips to memory at their starts and the passage of
// messages and model through memory are most.  One compute unit can do the round's arithmetic in less: 256 threads per
// worker hold the rows of its mini-batch in registers, one quad of columns each, exactly as a block of vr_dense_kernel
// does; the gradients' codes, the model and the snapshot stay in LDS from round to round; and since a round's rows do not
// depend on the model, the next round's are requested as soon as this round's are used up and arrive while the
// messages are quantized, aggregated and the model is updated and quantized.  Five barriers per round, no wait on any
// other block.  Only the last round's messages are stored: no one could have read the others.
// The arithmetic is that of the separate kernels in the same order: the results are theirs bit for bit.
// 2000 x 1000, 4 workers of 16 rows: 11.2 us a round as launches, now 6.6.
#include <algorithm>

#include "dq_common.h"
#include "elementwise.h"
#include "grad_common.h"
#include "grad_launch.h"

namespace dq {

// The limits: a block has 1024 threads, and a thread the registers for one quad of sixteen rows (64 of 128) beside what it
// works with.  A worker has 256 threads whatever the width, so that its sums across wavefronts are those of a block of
// vr_dense_kernel, bit for bit: narrower rows do not make room for more workers.
constexpr int kGroup = 256;                              // threads per worker, a quad of columns each
constexpr int kSmallWorkers = 4, kSmallRows = 16, kSmallD = 4 * kGroup;

static __device__ __align__(16) const float kNoSmallRow[kSmallD] = {};      // (see kNoRow in grad_dense.hip)

struct SmallArgs {
    const float *X; int64_t lda;
    const float *y, *z_snap;
    int n, d, M, B, b, b_x;
    float l2, scale, eta, theta, kappa;
    uint32_t k0, k1, iter0;                              // seed halves; iter of the first round of the call
    int t0, rounds, flag_first;                          // parity of the first round; its flag-bit case
    float *x, *yv, *xsum; const float *x_snap, *g_snap;
    uint32_t *xq; float *delta_x, *absmax_x;
    uint32_t *packed; int64_t ld_words;
    float *delta; uint32_t *status;
};

// x / y / sum / gradient / snapshot of the 256 quads: the state of the run while the kernel has it
struct SmallState {
    float4 x[kGroup], y[kGroup], sum[kGroup], g[kGroup], xs[kGroup], dx[kGroup];
};

template <bool ACC, bool EACH>
__global__ __launch_bounds__(kGroup *kSmallWorkers) void small_rounds_kernel(const SmallArgs a)
{
    constexpr int R = kSmallRows, kWaves = kGroup / kWave;
    __shared__ SmallState st;
    __shared__ float4 codes[kSmallWorkers][kGroup];
    __shared__ float deltas[kSmallWorkers];
    __shared__ float dots[kSmallWorkers][kWaves][R];
    __shared__ uint32_t wmax[kSmallWorkers][kWaves], xmax[kWaves];
    __shared__ int rows[kSmallWorkers][R];
    __shared__ float labels[kSmallWorkers][R], margins[kSmallWorkers][R];
    __shared__ uint32_t words[kGroup * 4 * 16 / 32 + 2];
    const int w = threadIdx.x / kGroup, t = threadIdx.x % kGroup;            // worker, quad of columns
    const int lane = threadIdx.x & (kWave - 1), gw = t / kWave;              // wavefront of the worker's four
    const int d = a.d, quads = (d + 3) / 4, col = 4 * t, last_col = (d + 3) / 4 * 4 - 4;
    const int nrows = a.B;
    const float inv_B = 1.0f / static_cast<float>(a.B);
    const bool first_group = w == 0;
    StreamKey grad{a.k0, a.k1, 0u, static_cast<uint32_t>(w), DQ_TAG_GRAD}, model{a.k0, a.k1, 0u, DQ_MASTER_ID, DQ_TAG_MODEL},
        sample{a.k0, a.k1, 0u, static_cast<uint32_t>(w), DQ_TAG_SAMPLE};

    // the rows of one round: drawn, with labels and margins, by the first wavefront of the worker ...
    const auto draw = [&](uint32_t iter) {
        if (gw == 0 && lane < nrows) {
            sample.iter = iter;
            const int i = static_cast<int>(__umulhi(stream_word(sample, static_cast<uint64_t>(lane)), static_cast<uint32_t>(a.n)));
            rows[w][lane] = i;
            labels[w][lane] = a.y[i];
            margins[w][lane] = a.z_snap[i];
        }
    };
    // ... and requested by all of it (a position past the last row loads zeros; a lane past the last column the row's last
    // quad, masked when it is used)
    float4 row[R];
    const uint32_t lane_offset = 4u * static_cast<uint32_t>(min(col, last_col));
    const auto request = [&]() {
        const int mine = rows[w][min(lane, nrows - 1)];
#pragma unroll
        for (int r = 0; r < R; ++r) {                    // (a scalar base per row and one 32-bit lane offset)
            const int64_t i = __builtin_amdgcn_readlane(mine, r);            // (lanes past the rows hold the last one)
            const char *base = reinterpret_cast<const char *>(r < nrows ? a.X + i * a.lda : kNoSmallRow);
            row[r] = *reinterpret_cast<const float4 *>(base + lane_offset);
        }
    };
    const bool ragged = __any(col + 3 >= d);              // (of this wavefront) some lane's quad is not whole
    const auto quad_of = [&](const float *v) { return load4_or_zero(v, col, d); };

    bool have_rows = false;
    if (!a.flag_first) {
        draw(a.iter0);
        have_rows = true;
    }
    if (first_group) {
        st.g[t] = quad_of(a.g_snap);
        st.xs[t] = quad_of(a.x_snap);
        st.x[t] = quad_of(a.x);
        if constexpr (ACC) {
            st.y[t] = quad_of(a.yv);
            st.sum[t] = quad_of(a.xsum);
        }
        if (!a.flag_first) {                             // the model of the first round comes as a message
            const ModelMsg msg{a.xq, a.delta_x[0], a.b_x};
            const int64_t last_word = (static_cast<int64_t>(d) * a.b_x + 31) / 32 - 1;
            const ModelQuad mq = model_quad_request<false>(msg, min(col, last_col), last_word);
            float q[4];
            model_quad_values<false>(msg, mq, col, d, q);
            const float4 xs = quad_of(a.x_snap);
            st.dx[t] = make_float4(q[0] - xs.x, q[1] - xs.y, q[2] - xs.z, q[3] - xs.w);
        }
    }
    __syncthreads();
    if (have_rows) request();
    for (int k = 0; k < a.rounds; ++k) {
        const bool last = k == a.rounds - 1, flag = k == 0 && a.flag_first;
        const uint32_t iter = a.iter0 + static_cast<uint32_t>(k);
        // (the seed's halves through registers the compiler cannot see across: else it keeps the ten round keys of every
        // stream, and spills for them)
        uint32_t k0 = a.k0, k1 = a.k1;
        asm volatile("" : "+s"(k0), "+s"(k1));
        grad.k0 = model.k0 = sample.k0 = k0;
        grad.k1 = model.k1 = sample.k1 = k1;
        // ---- worker side: the variance-reduced gradient, its scale and codes
        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (!flag) {                                     // (the same for every thread)
            const float4 dx = st.dx[t];
            if (ragged) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    row[r].x = col + 0 < d ? row[r].x : 0.0f;
                    row[r].y = col + 1 < d ? row[r].y : 0.0f;
                    row[r].z = col + 2 < d ? row[r].z : 0.0f;
                    row[r].w = col + 3 < d ? row[r].w : 0.0f;
                }
            }
            float prod[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                prod[r] = fmaf(row[r].x, dx.x, 0.0f);
                prod[r] = fmaf(row[r].y, dx.y, prod[r]);
                prod[r] = fmaf(row[r].z, dx.z, prod[r]);
                prod[r] = fmaf(row[r].w, dx.w, prod[r]);
            }
            const float mine = wave_sums16(prod);        // lane r: the wavefront's share of row r's product
            if (lane < R) dots[w][gw][lane] = mine;
            __syncthreads();
            const int lr = min(lane, R - 1);
            float dz = dots[w][0][lr];
#pragma unroll
            for (int i = 1; i < kWaves; ++i) dz += dots[w][i][lr];
            const int row_of = min(lr, nrows - 1);
            const float coef_l = lane < nrows ? vr_slope_diff(labels[w][row_of], margins[w][row_of], dz) * inv_B : 0.0f;
            float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float coef = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(coef_l), r));
                acc.x = fmaf(coef, row[r].x, acc.x);
                acc.y = fmaf(coef, row[r].y, acc.y);
                acc.z = fmaf(coef, row[r].z, acc.z);
                acc.w = fmaf(coef, row[r].w, acc.w);
            }
            v = make_float4(acc.x + a.l2 * dx.x, acc.y + a.l2 * dx.y, acc.z + a.l2 * dx.z, acc.w + a.l2 * dx.w);
            const uint32_t m = wave_max_u32(max(max(abs_bits(v.x), abs_bits(v.y)), max(abs_bits(v.z), abs_bits(v.w))));
            if (lane == 0) wmax[w][gw] = m;
        }
        __syncthreads();                                 // (all have read their labels and margins: the next round's may be drawn)
        if (!last) draw(iter + 1u);
        Scale s = make_scale(0.0f, a.b);
        int c[4] = {0, 0, 0, 0};
        if (!flag) {
            s = make_scale(__uint_as_float(max(max(wmax[w][0], wmax[w][1]), max(wmax[w][2], wmax[w][3]))), a.b);
            if (s.inv_delta != 0.0f) {
                grad.iter = iter;
                const uint4 r = stream_block(grad, static_cast<uint32_t>(t));
                c[0] = quantize_one(v.x, s, r.x); c[1] = quantize_one(v.y, s, r.y);
                c[2] = quantize_one(v.z, s, r.z); c[3] = quantize_one(v.w, s, r.w);
            }
            if (t == 0 && s.bad && a.status) atomicOr(a.status, 1u);
        }
        if (t == 0) deltas[w] = s.delta;
        codes[w][t] = make_float4(static_cast<float>(c[0]), static_cast<float>(c[1]), static_cast<float>(c[2]), static_cast<float>(c[3]));
        if (last) {                                      // the messages (every lane makes the call)
            uint32_t *out = a.packed + static_cast<int64_t>(w) * a.ld_words;
            const bool in = t < quads;
            if (a.b == 8) store_quad_bits<8>(in ? pack4<8>(c[0], c[1], c[2], c[3]) : 0u, t, quads, out);
            else if (a.b == 4) store_quad_bits<4>(in ? pack4<4>(c[0], c[1], c[2], c[3]) : 0u, t, quads, out);
            else store_quad_bits<2>(in ? pack4<2>(c[0], c[1], c[2], c[3]) : 0u, t, quads, out);
            if (t == 0) a.delta[w] = s.delta;
        }
        __syncthreads();
        if (!last) request();                            // the next round's rows: in flight until the next round's products
        // ---- master side, by the first worker's threads: aggregate, update, ||x||_inf
        float xn[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (first_group) {
            const float4 g4 = st.g[t], s4 = st.xs[t], x4 = st.x[t];
            const float gs[4] = {g4.x, g4.y, g4.z, g4.w}, xs[4] = {s4.x, s4.y, s4.z, s4.w};
            float yn[4] = {0.0f, 0.0f, 0.0f, 0.0f}, sm[4] = {0.0f, 0.0f, 0.0f, 0.0f}, sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            xn[0] = x4.x; xn[1] = x4.y; xn[2] = x4.z; xn[3] = x4.w;
            if constexpr (ACC) {
                const float4 y4 = st.y[t], t4 = st.sum[t];
                yn[0] = y4.x; yn[1] = y4.y; yn[2] = y4.z; yn[3] = y4.w;
                sm[0] = t4.x; sm[1] = t4.y; sm[2] = t4.z; sm[3] = t4.w;
            }
            for (int m = 0; m < a.M; ++m) {
                const float4 cv = codes[m][t];
                const float dm = deltas[m], vv[4] = {cv.x, cv.y, cv.z, cv.w};
                if constexpr (EACH) {
                    const float dir[4] = {dm * vv[0] + gs[0], dm * vv[1] + gs[1], dm * vv[2] + gs[2], dm * vv[3] + gs[3]};
                    master_apply_quad<ACC>(dir, xn, yn, xs, sm, true, a.eta, a.theta, a.kappa);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] = fmaf(dm, vv[e], sum[e]);
                }
            }
            if constexpr (!EACH) {
                const float dir[4] = {a.scale * sum[0] + gs[0], a.scale * sum[1] + gs[1], a.scale * sum[2] + gs[2],
                                      a.scale * sum[3] + gs[3]};
                master_apply_quad<ACC>(dir, xn, yn, xs, sm, true, a.eta, a.theta, a.kappa);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e >= d) xn[e] = 0.0f;
            st.x[t] = make_float4(xn[0], xn[1], xn[2], xn[3]);
            if constexpr (ACC) {
                st.y[t] = make_float4(yn[0], yn[1], yn[2], yn[3]);
                st.sum[t] = make_float4(sm[0], sm[1], sm[2], sm[3]);
            }
            const uint32_t m = wave_max_u32(max(max(abs_bits(xn[0]), abs_bits(xn[1])), max(abs_bits(xn[2]), abs_bits(xn[3]))));
            if (lane == 0) xmax[gw] = m;
            if (last)
                for (int i = t; i < kGroup * 4 * 16 / 32 + 2; i += kGroup) words[i] = 0u;
        }
        __syncthreads();
        // ---- the model of the next round
        if (first_group) {
            const float amax = __uint_as_float(max(max(xmax[0], xmax[1]), max(xmax[2], xmax[3])));
            const Scale ms = make_scale(amax, a.b_x);
            if (t == 0) {
                a.absmax_x[(a.t0 + k) & 1] = amax;
                if (ms.bad && a.status) atomicOr(a.status, 1u);
            }
            int q[4] = {0, 0, 0, 0};
            if (ms.inv_delta != 0.0f) {
                model.iter = iter + 1u;
                const uint4 r = stream_block(model, static_cast<uint32_t>(t));
                q[0] = quantize_one(xn[0], ms, r.x); q[1] = quantize_one(xn[1], ms, r.y);
                q[2] = quantize_one(xn[2], ms, r.z); q[3] = quantize_one(xn[3], ms, r.w);
            }
            const float4 xs = st.xs[t];
            st.dx[t] = make_float4(ms.delta * static_cast<float>(q[0]) - xs.x, ms.delta * static_cast<float>(q[1]) - xs.y,
                                   ms.delta * static_cast<float>(q[2]) - xs.z, ms.delta * static_cast<float>(q[3]) - xs.w);
            if (last) {
                if (t == 0) a.delta_x[0] = ms.delta;
                if (t < quads) or_quad_bits(words, t, a.b_x, q);
            }
        }
        __syncthreads();
    }
    if (first_group) {
        store_quad(a.x, t, d, st.x[t]);
        if constexpr (ACC) {
            store_quad(a.yv, t, d, st.y[t]);
            store_quad(a.xsum, t, d, st.sum[t]);
        }
        const int row_words = (d * a.b_x + 31) / 32;
        for (int i = t; i < row_words; i += kGroup) a.xq[i] = words[i];
    }
}

bool small_rounds_ok(const dq_problem *prob, const dq_run_config *cfg, const dq_run_state *st)
{
    return prob->layout == 0 && prob->d <= kSmallD && cfg->M <= kSmallWorkers && cfg->B <= kSmallRows && cfg->tau == 0 &&
           cfg->algo != DQ_ALGO_SPARSE && (cfg->b == 2 || cfg->b == 4 || cfg->b == 8) && cfg->b_x >= 2 && cfg->b_x <= 16 &&
           st->z_snap && !st->wire;
}

int32_t small_rounds(const dq_problem *prob, const dq_run_config *cfg, const dq_run_state *st, int64_t epoch, int64_t t0,
                     int64_t rounds, float eta, float theta, bool flag_first, hipStream_t stream)
{
    const bool acc = cfg->algo == DQ_ALGO_ACC;
    const void *quads[] = {st->x, st->x_snap, st->g_snap, acc ? st->y : nullptr, acc ? st->xsum : nullptr};
    for (const void *p : quads)
        if (p && !aligned16(p)) return DQ_ERR_INVALID_ARG;
    SmallArgs a{};
    a.X = prob->dense; a.lda = prob->lda; a.y = prob->y; a.z_snap = st->z_snap;
    a.n = static_cast<int>(prob->n); a.d = static_cast<int>(prob->d); a.M = static_cast<int>(cfg->M); a.B = static_cast<int>(cfg->B);
    a.b = cfg->b; a.b_x = cfg->b_x;
    a.l2 = prob->l2; a.scale = 1.0f / static_cast<float>(cfg->M); a.eta = eta; a.theta = theta; a.kappa = eta * prob->l1;
    a.k0 = static_cast<uint32_t>(cfg->seed); a.k1 = static_cast<uint32_t>(cfg->seed >> 32);
    a.x = st->x; a.yv = st->y; a.xsum = st->xsum; a.x_snap = st->x_snap; a.g_snap = st->g_snap;
    a.xq = st->xq; a.delta_x = st->delta_x; a.absmax_x = st->absmax_x;
    a.packed = st->packed; a.ld_words = st->ld_words; a.delta = st->delta; a.status = st->status;
    const dim3 block(static_cast<unsigned>(kGroup * cfg->M));
    // (a launch for every kMostRounds rounds: about 27 ms of one compute unit each)
    constexpr int64_t kMostRounds = 4096;
    for (int64_t done = 0; done < rounds; done += kMostRounds) {
        a.iter0 = static_cast<uint32_t>(epoch * cfg->m + t0 + done);
        a.t0 = static_cast<int>((t0 + done) & 1); a.rounds = static_cast<int>(std::min(kMostRounds, rounds - done));
        a.flag_first = done == 0 && flag_first;
        if (acc && cfg->each) small_rounds_kernel<true, true><<<dim3(1), block, 0, stream>>>(a);
        else if (acc) small_rounds_kernel<true, false><<<dim3(1), block, 0, stream>>>(a);
        else if (cfg->each) small_rounds_kernel<false, true><<<dim3(1), block, 0, stream>>>(a);
        else small_rounds_kernel<false, false><<<dim3(1), block, 0, stream>>>(a);
        DQ_LAUNCH_CHECK();
    }
    return DQ_OK;
}

}  // namespace dq
