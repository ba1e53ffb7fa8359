// Greedy shallow fusion (Section 2.3), one step over a batch of hypotheses, and
// the states' final weights.
//
// One workgroup of W wavefronts per hypothesis, its ASR scores and dense row in
// registers (group.h).  CTC and transducer modes first take the plain ASR
// argmax over the V + 1 classes, while the state's chain record is in flight;
// when that keeps blank (or, for CTC, the previous label) the LM is not
// consulted at all and the state stays.  Otherwise the group walks its state's
// backoff chain, forms fmaf(lambda, lm[v], asr[v]) per token and takes the
// argmax with lowest-index ties.  No MFMA: one fma and one compare per token.
//
// AED mode (Section 2.3): class V is <eos>, whose LM score is the state's
// final weight (the </s> score, precomputed per state); <eos> keeps the state.
#include <hip/hip_runtime.h>

#include <cmath>

#include "group.h"

namespace ngpu {

// A step is a chain of three dependent memory accesses (state, chain record,
// then dense row and arcs) and two exchanges, so its time is latency.
template <int MODE, int W, int NT, bool FULL>
__global__ __launch_bounds__(W * kWave) void step_kernel(DevTrie t, const float *__restrict__ asr, int64_t ld,
                                                         float lambda, int32_t *__restrict__ states,
                                                         int32_t *__restrict__ prev, int32_t *__restrict__ tokens) {
    extern __shared__ i32x4 lds4[];
    load_trie_args(t);
    load_args(asr, ld, lambda, states, prev, tokens);
    constexpr bool kRaw = MODE == kCtc || MODE == kTransducer;
    const int64_t b = blockIdx.x;
    const int V = t.vocab_size;
    Meet *meet = reinterpret_cast<Meet *>(lds4);
    const Group<W, NT, FULL> g(V, reinterpret_cast<i32x2 *>(meet + 1));
    const int wave = g.wave, lane = g.lane, zero = lane_zero();

    // the state, the previous label and blank's score go out first, then the
    // row, so that the wait for the state leaves the row in flight
    const float *src = asr + b * ld;
    const int s_l = states[b + zero];
    const int pv_l = MODE == kCtc ? prev[b + zero] : -1;
    const float rowV_l = MODE == kPlain ? 0.0f : src[V + zero];
    Words<NT> row, dw, dt;
    g.load_row(src, row);
    const RecordIndex ri = record_index(t, lane);
    g.clear_slots();
    int s = __builtin_amdgcn_readfirstlane(s_l);
    if (s < 0 || s >= t.num_states) {
        if (wave == 0 && lane == 0) {
            atomicAdd(&t.status[0], 1);
            tokens[b] = -1;
        }
        return;
    }
    const int4 rec = load_record(ri, s, lane);
    const float fin = MODE == kAed ? t.final_w[s + zero] : 0.0f;   // <eos> takes the state's final weight
    const int pv = __builtin_amdgcn_readfirstlane(pv_l);
    const float rowV = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(rowV_l)));
    g.mask_row(row);
    int label = -1;
    bool lm = true;
    if (kRaw) {
        unsigned key;
        g.raw_best(row, key, label);   // every token at -inf: the lowest, 0
        if (W > 1) {
            if (lane == 0) {
                meet->a[0][wave].w = label;
                meet->b[0][wave] = int(key);
            }
            lds_barrier();
            const int k = meet->b[0][lane & (W - 1)], tk = meet->a[0][lane & (W - 1)].w;
            const int e = winner_entry<W>(unsigned(k), tk);
            key = unsigned(__builtin_amdgcn_readlane(k, e));
            label = __builtin_amdgcn_readlane(tk, e);
        }
        if (float_key(or_lowest(rowV)) > key) label = V;      // blank only when strictly larger (highest index)
        lm = !(label == V || (MODE == kCtc && label == pv));  // blank or repeat: no LM, no move
    }
    if (lm) {
        const ChainHead h = head_of(rec);
        g.load_dense(t, unsigned(h.dense_row), dw, dt);
        const bool any = g.put_levels(t, rec, h);
        if (MODE == kCtc) {   // the previous label is no candidate
            const int p = pv - g.t0 - lane;
#pragma unroll
            for (int i = 0; i < NT; ++i) row.v[i] = p == kWave * i ? __float_as_int(-__builtin_inff()) : row.v[i];
        }
        float x[NT], bx;
        int nx[NT], bi;
        g.lm_values(h, dw, dt, any, x, nx);
#pragma unroll
        for (int i = 0; i < NT; ++i) x[i] = __builtin_fmaf(lambda, x[i], row.f(i));
        g.lane_best(x, bx, bi);
        int to = nx[0];
#pragma unroll
        for (int i = 1; i < NT; ++i) to = bi == kWave * i ? nx[i] : to;
        to &= kStateMask;
        unsigned key = float_key(bx);
        label = g.t0 + bi + lane;
        const int who = winner_lane(key, label);
        if (W > 1) {
            if (lane == who) {
                const i32x4 e = {int(key), label, to, 0};
                meet->a[1][wave] = e;
            }
            lds_barrier();
            const i32x4 e = meet->a[1][lane & (W - 1)];
            const int w = winner_entry<W>(unsigned(e.x), e.y);
            key = unsigned(__builtin_amdgcn_readlane(e.x, w));
            label = __builtin_amdgcn_readlane(e.y, w);
            to = __builtin_amdgcn_readlane(e.z, w);
        } else {
            key = unsigned(__builtin_amdgcn_readlane(int(key), who));
            label = __builtin_amdgcn_readlane(label, who);
            to = __builtin_amdgcn_readlane(to, who);
        }
        bool eos = false;
        if (MODE == kAed) {   // <eos> strictly above every token: the sentence ends, the state stays
            const float fw = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(fin)));
            eos = float_key(or_lowest(__builtin_fmaf(lambda, fw, rowV))) > key;
        }
        if (eos) {
            label = V;
        } else {
            if (MODE == kCtc && key == kInfKey && pv == 0) {
                // every candidate at -inf: the first one, and token 0 is none: token 1 (wavefront 0 writes)
                label = 1;
                const int put = __builtin_amdgcn_readfirstlane(g.slots[1].y);
                to = (put != 0 ? put : __builtin_amdgcn_readlane(dt.v[0], 1)) & kStateMask;
            }
            s = to;
        }
    }
    // every wavefront has read states[b] and prev[b] before the last barrier above
    if (wave == 0 && lane == 0) {
        tokens[b] = label;
        states[b] = s;
        if (MODE == kCtc) prev[b] = label;
    }
}

// A grid holds at most 2^32 - 1 work-items: larger batches go in several launches.
template <int MODE, int W, int NT>
static hipError_t launch_group(const DevTrie &t, const float *asr, int64_t B, int64_t ld, float lambda,
                               int32_t *states, int32_t *prev, int32_t *tokens, hipStream_t stream) {
    constexpr int64_t kMost = int64_t(UINT32_MAX) / (W * kWave);
    const size_t lds = sizeof(Meet) + size_t(W) * kWave * NT * sizeof(i32x2);
    const dim3 block(W * kWave);
    for (int64_t b0 = 0; b0 < B; b0 += kMost) {
        const dim3 grid{unsigned(B - b0 < kMost ? B - b0 : kMost)};
        int32_t *pv = prev ? prev + b0 : nullptr;
        if (t.vocab_size == W * kWave * NT)
            hipLaunchKernelGGL((step_kernel<MODE, W, NT, true>), grid, block, lds, stream, t, asr + b0 * ld, ld, lambda,
                               states + b0, pv, tokens + b0);
        else
            hipLaunchKernelGGL((step_kernel<MODE, W, NT, false>), grid, block, lds, stream, t, asr + b0 * ld, ld,
                               lambda, states + b0, pv, tokens + b0);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Wavefronts and tokens per lane, from sweeps over vocabularies and 8 to 12000
// hypotheses (CTC, us a step, without and from V = 513 on with the copies that
// reset the state; "before": row and walk in LDS, four wavefronts up to 1024
// hypotheses and one above, whatever the vocabulary).  Wavefronts pay off while
// the chip has room; beyond, each one repeats the walk and the exchanges.
//  - V <= 256: one of 4 a lane: 3.6 / 5.3 at V = 128, 8 / 4000 hypotheses [two of
//    2: 3.9 / 6.9; before: 4.5 / 5.8].
//  - V <= 512: one of 8: 3.7 / 5.9 at V = 400 [two of 4: 3.8 / 7.3; before: 4.4 / 6.8].
//  - V <= 1024: four of 4 up to 768 hypotheses: 4.6 at 300 [two of 8: 5.0; before:
//    5.4]; two of 8 above: 5.9 / 9.6 at 1500 / 4000 [6.1 / 10.8; before: 7.4 / 12.1], up
//    to V = 768 one of 12: 8.6 / 10.0 at V = 700, 2048 / 4096 [two of 8: 9.3 / 11.8;
//    before: 8.7 / 10.5].
//  - V <= 1536: eight of 4 up to 512 hypotheses (up to V = 1280 only 256: 8.1 at 400
//    with two of 10 [8.8; before: 8.6]), two of 10 or 12 above: 9.7 / 13.5 at V = 1100,
//    2048 / 4096 [four of 8: 11.5 / 17.1; before: 9.7 / 15.4].
//  - V <= 2048: eight of 4 up to 512 hypotheses: 4.0 / 5.1 at 8 / 300 [four of 8:
//    4.3 / 5.2; before: 5.0 / 5.8], four of 8 above: 15.5 at 4000 [17.9; before: 19.9].
//  - V <= 3072: eight of 8 up to 512 hypotheses, four of 10 or 12 above: 10.1 / 21.3 at
//    V = 2500, 900 / 4096 [eight of 8: 12.1 / 28.2; before: 11.0 / 29.0].
//  - V <= 4096: eight of 8: 4.6 / 6.1 / 27.9 at V = 4000, 8 / 300 / 4000 [four of 16:
//    5.2 / 6.7 / 28.0; before: 5.8 / 7.1 / 50].
//  - above: sixteen of 8 for few hypotheses, 5.4 at V = 8000, 8 [eight of 16: 5.7;
//    before: 7.6]; above 128 eight of 12 up to V = 6144, 10.8 / 15.9 / 38.5 at V = 5000,
//    400 / 900 / 4096 [sixteen of 8: 12.8 / 18.3 / 54.9; before: 11.1 / 17.5 / 75], and
//    eight of 16, 13.1 / 55.6 at V = 6200, 400 / 4096 [14.4 / 59.9; before: 13.8 / 92].
template <int MODE>
static hipError_t launch_mode(const DevTrie &t, const float *asr, int64_t B, int64_t ld, float lambda, int32_t *states,
                              int32_t *prev, int32_t *tokens, hipStream_t stream) {
    const int V = t.vocab_size;
#define NGPU_STEP(W, NT) return launch_group<MODE, W, NT>(t, asr, B, ld, lambda, states, prev, tokens, stream)
    if (V <= 256) NGPU_STEP(1, 4);
    if (V <= 512) NGPU_STEP(1, 8);
    if (V <= 1024) {
        if (B <= 768) NGPU_STEP(4, 4);
        if (V <= 768) NGPU_STEP(1, 12);
        NGPU_STEP(2, 8);
    }
    if (V <= 2048) {
        if (B <= (V <= 1280 ? 256 : 512)) NGPU_STEP(8, 4);
        if (V <= 1280) NGPU_STEP(2, 10);
        if (V <= 1536) NGPU_STEP(2, 12);
        NGPU_STEP(4, 8);
    }
    if (V <= 3072 && B > 512) {
        if (V <= 2560) NGPU_STEP(4, 10);
        NGPU_STEP(4, 12);
    }
    if (V <= 4096) NGPU_STEP(8, 8);
    if (B <= 128) NGPU_STEP(16, 8);
    if (V <= 6144) NGPU_STEP(8, 12);
    NGPU_STEP(8, 16);
#undef NGPU_STEP
}

hipError_t launch_fused_step(const DevTrie &t, const float *asr, int64_t B, int64_t ld, int mode, float lambda,
                             int32_t *states, int32_t *prev, int32_t *tokens, hipStream_t stream) {
    switch (mode) {
        case kPlain: return launch_mode<kPlain>(t, asr, B, ld, lambda, states, prev, tokens, stream);
        case kCtc: return launch_mode<kCtc>(t, asr, B, ld, lambda, states, prev, tokens, stream);
        case kAed: return launch_mode<kAed>(t, asr, B, ld, lambda, states, prev, tokens, stream);
        default: return launch_mode<kTransducer>(t, asr, B, ld, lambda, states, prev, tokens, stream);
    }
}

__global__ __launch_bounds__(256) void final_weights_kernel(DevTrie t, const int32_t *__restrict__ states, int64_t B,
                                                          float *__restrict__ out) {
    const int64_t b = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (b >= B) return;
    const int s = states[b];
    if (s < 0 || s >= t.num_states) {
        atomicAdd(&t.status[0], 1);
        out[b] = NAN;
        return;
    }
    out[b] = t.final_w[s];
}

hipError_t launch_final_weights(const DevTrie &t, const int32_t *states, int64_t B, float *out, hipStream_t stream) {
    hipLaunchKernelGGL(final_weights_kernel, dim3(unsigned((B + 255) / 256)), dim3(256), 0, stream, t, states, B,
                       out);
    return hipGetLastError();
}

}  // namespace ngpu
