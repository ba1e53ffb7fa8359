// The k best fused tokens of each hypothesis (beam-search expansion, Section
// 2.3: full-vocabulary scoring before selection), one workgroup of W
// wavefronts per hypothesis, its fused scores and next states in registers
// (group.h).
//
// Selection over the order-preserving keys of the fused scores, in a number of
// steps that hardly grows with k:
//   1. a lower bound of the k-th largest key: the smallest of at least k
//      disjoint parts' maxima.  The parts are wavefronts, rows of 16 lanes,
//      groups of 4 lanes or single lanes, the coarsest that number at least k:
//      at V = 1024, k = 16 (16 rows of 64 tokens) about 45 keys reach it;
//   2. while more keys reach the bound than a short list should hold, the
//      interval between it and the largest key is halved (one count over the
//      group, one barrier each; none for small k);
//   3. the keys that reach it go into a list in LDS, in token order, and each
//      finds its rank by counting the list's keys above its own (key, ~token:
//      all distinct, ties to the lower token); ranks below k are written out.
//      Where a value is shared by more tokens than the list holds, the keys
//      above it and the lowest tokens holding it are listed.
// The selection before it held a hypothesis in one wavefront (a bit-wise search
// over the keys up to V = 1024, one reduction and rescan per selected token
// above): 9.9 us for 1024 hypotheses of the 20M 6-gram at k = 16 and 84 us for 320
// at V = 5000, k = 32, against 7.5 and 10.1 here.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "group.h"

namespace ngpu {

template <int W>
constexpr int list_size() { return W * kWave > NGPU_LM_MAX_TOPK ? W * kWave : NGPU_LM_MAX_TOPK; }

template <int W, int NT, bool FULL>
__global__ __launch_bounds__(W * kWave) void topk_kernel(DevTrie t, const float *__restrict__ asr, int64_t ld,
                                                         float lambda, int k, const int32_t *__restrict__ states,
                                                         int32_t *__restrict__ tokens, float *__restrict__ scores,
                                                         int32_t *__restrict__ next) {
    extern __shared__ i32x4 lds4[];
    load_trie_args(t);
    load_args(asr, ld, lambda, k, states, tokens, scores, next);
    constexpr int kList = list_size<W>();
    const int64_t b = blockIdx.x;
    const int V = t.vocab_size;
    Meet *meet = reinterpret_cast<Meet *>(lds4);
    const Group<W, NT, FULL> g(V, reinterpret_cast<i32x2 *>(meet + 1));
    // the list takes the slots' place: every wavefront has read its slots before the barrier of the first exchange
    unsigned long long *lkey = reinterpret_cast<unsigned long long *>(meet + 1);   // kList: key, ~token
    i32x2 *lval = reinterpret_cast<i32x2 *>(lkey + kList);                         // kList: score, next state
    const int wave = g.wave, lane = g.lane, tid = threadIdx.x;
    int32_t *otok = tokens + b * k;
    float *osc = scores + b * k;
    int32_t *onx = next + b * k;

    const int s_l = states[b];   // issued before the row, so its wait leaves the row in flight
    Words<NT> row, dw, dt;
    g.load_row(asr + b * ld, row);
    const RecordIndex ri = record_index(t, lane);
    g.clear_slots();
    const int s = __builtin_amdgcn_readfirstlane(s_l);
    if (s < 0 || s >= t.num_states) {
        if (tid == 0) atomicAdd(&t.status[0], 1);
        for (int j = tid; j < k; j += W * kWave) {
            otok[j] = -1;
            osc[j] = NAN;
            onx[j] = -1;
        }
        return;
    }
    const int4 rec = load_record(ri, s, lane);
    const ChainHead h = head_of(rec);
    g.load_dense(t, unsigned(h.dense_row), dw, dt);
    const bool any = g.template put_levels<true>(t, rec, h);
    float x[NT];
    int nx[NT];
    unsigned key[NT];
    g.lm_values(h, dw, dt, any, x, nx);
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        x[i] = __builtin_fmaf(lambda, x[i], row.f(i));
        // a token's key lies from -inf's (also a NaN's) to +inf's, below ~0; past V: below every token's
        key[i] = FULL || kWave * i + lane < g.own ? float_key(or_lowest(x[i])) : 0u;
        m = max(m, key[i]);
    }

    int xi = 0;
    // value of every wavefront, entry l mod W in lane l
    auto gather = [&](unsigned a) -> unsigned {
        if (W == 1) return a;
        const int buf = xi & 1;
        ++xi;
        if (lane == 0) meet->b[buf][wave] = int(a);
        lds_barrier();
        return unsigned(meet->b[buf][lane & (W - 1)]);
    };
    // 1. the bound, and the largest key
    const int full = ((V >> 6) * kWave + g.range - 1) / g.range;   // wavefronts whose lanes all hold tokens
    unsigned part = m;
    if (k <= 16 * full) {
        part = max_over_waves<4>(part);
        if (k <= 4 * full) part = max_over_waves<16>(part);
    }
    const unsigned wtop = wave_max_u32(m);
    if (k <= full) part = wtop;
    const unsigned wlow = wave < full ? wave_max_u32(~part) : 0u;   // complement of the smallest part
    const unsigned top = __builtin_amdgcn_readfirstlane(max_over_waves<W>(gather(wtop)));
    unsigned lo = k <= kWave * full ? ~unsigned(__builtin_amdgcn_readfirstlane(max_over_waves<W>(gather(wlow)))) : 0u;
    if (lo == 0) lo = 1;   // every token's key is above 0

    // keys >= x in this wavefront, and in the group: total, and of the wavefronts before this one
    int total = 0, before = 0;
    auto count = [&](unsigned at) {
        int c = 0;
#pragma unroll
        for (int i = 0; i < NT; ++i) c += __builtin_popcountll(__ballot(key[i] >= at));
        const int e = int(gather(unsigned(c)));
        total = 0;
        before = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int n = W == 1 ? c : __builtin_amdgcn_readlane(e, w);
            before += w < wave ? n : 0;
            total += n;
        }
    };
    // 2. at least k keys reach lo, fewer than k reach hi (hi - lo modulo 2^32)
    const int want = min(kList, max(kWave, k + k / 4));
    unsigned hi = top + 1;
    count(lo);
    for (int halvings = 0; total > want && hi - lo > 1 && (halvings < 6 || total > kList); ++halvings) {
        const unsigned mid = lo + (hi - lo) / 2;
        const int t0 = total, b0 = before;
        count(mid);
        if (total >= k) {
            lo = mid;
        } else {
            hi = mid;
            total = t0;
            before = b0;
        }
    }
    // 3. the list
    int n = total;
    auto put = [&](bool take, int at, int i) {
        if (take) {
            lkey[at] = (static_cast<unsigned long long>(key[i]) << 32) | ~unsigned(g.token(i));
            lval[at] = i32x2{__float_as_int(x[i]), nx[i] & kStateMask};
        }
    };
    auto below = [&](unsigned long long mask) {
        return int(__builtin_amdgcn_mbcnt_hi(unsigned(mask >> 32), __builtin_amdgcn_mbcnt_lo(unsigned(mask), 0u)));
    };
    if (n <= kList) {
        int at = before;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const bool take = key[i] >= lo;
            const unsigned long long mask = __ballot(take);
            put(take, at + below(mask), i);
            at += __builtin_popcountll(mask);
        }
    } else {   // hi = lo + 1: the k-th key is lo, shared by more tokens than the list holds
        const int all_before = before;
        count(hi);
        const int above = total;
        int at = before, tie = above + all_before - before;
        n = k;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const bool over = key[i] >= hi, same = key[i] == lo;
            const unsigned long long mo = __ballot(over), ms = __ballot(same);
            put(over, at + below(mo), i);
            put(same && tie + below(ms) < k, tie + below(ms), i);
            at += __builtin_popcountll(mo);
            tie += __builtin_popcountll(ms);
        }
    }
    if (W > 1) lds_barrier();
    auto ranks = [&](auto per) {   // entries tid, tid + 64 W, ... of the list: ranked in one pass over it
        constexpr int R = decltype(per)::value;
        unsigned long long mine[R];
        int rank[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = tid + r * W * kWave;
            mine[r] = e < n ? lkey[e] : ~0ull;
            rank[r] = 0;
        }
#pragma unroll 8
        for (int q = 0; q < n; ++q) {
            const unsigned long long o = lkey[q];
#pragma unroll
            for (int r = 0; r < R; ++r) rank[r] += o > mine[r] ? 1 : 0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = tid + r * W * kWave;
            if (e < n && rank[r] < k) {
                const i32x2 val = lval[e];
                otok[rank[r]] = int(~unsigned(mine[r]));
                osc[rank[r]] = __int_as_float(val.x);
                onx[rank[r]] = val.y;
            }
        }
    };
    if (kList <= W * kWave || n <= W * kWave)
        ranks(std::integral_constant<int, 1>{});
    else if (kList <= 2 * W * kWave || n <= 2 * W * kWave)
        ranks(std::integral_constant<int, 2>{});
    else
        ranks(std::integral_constant<int, (kList + W * kWave - 1) / (W * kWave)>{});
}

// A grid holds at most 2^32 - 1 work-items: larger batches go in several launches.
template <int W, int NT>
static hipError_t launch(const DevTrie &t, const float *asr, int64_t B, int64_t ld, float lambda, int k,
                         const int32_t *states, int32_t *tokens, float *scores, int32_t *next, hipStream_t stream) {
    constexpr int64_t kMost = int64_t(UINT32_MAX) / (W * kWave);
    const size_t lds = sizeof(Meet) + std::max(size_t(list_size<W>()) * 16, size_t(W) * kWave * NT * sizeof(i32x2));
    const dim3 block(W * kWave);
    for (int64_t b0 = 0; b0 < B; b0 += kMost) {
        const dim3 grid{unsigned(B - b0 < kMost ? B - b0 : kMost)};
        if (t.vocab_size == W * kWave * NT)
            hipLaunchKernelGGL((topk_kernel<W, NT, true>), grid, block, lds, stream, t, asr + b0 * ld, ld, lambda, k,
                               states + b0, tokens + b0 * k, scores + b0 * k, next + b0 * k);
        else
            hipLaunchKernelGGL((topk_kernel<W, NT, false>), grid, block, lds, stream, t, asr + b0 * ld, ld, lambda, k,
                               states + b0, tokens + b0 * k, scores + b0 * k, next + b0 * k);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Wavefronts and tokens per lane, from sweeps over vocabularies, batches (8 to
// 12000) and k (1 to 200); us a call, in brackets the choice next to it.  Few
// hypotheses get more wavefronts each, which rank a long list sooner; many get
// fewer, since every wavefront repeats the walk, the exchanges and the counts.
//  - V <= 256: one wavefront, 6.1 at V = 128, 4000 hypotheses, k = 16 [two: 9.2];
//    two for large k and few hypotheses, 6.5 at 300, k = 100 [8.0].
//  - V <= 512 (V = 400): one up to k = 32, 6.9 at 4000, k = 16 [two: 9.4]; up to
//    1024 hypotheses two up to k = 96, 6.3 at 300, k = 64 [one: 7.4], four above,
//    10.3 at 300, k = 200 [two: 11.1]; beyond (1280 for large k) one, 10.0 / 24.6 at
//    4096, k = 64 / 200 [two: 12.0 / 26.2, four: 32.6 for 200], up to the 8192 where
//    two win.
//  - V <= 768: four of 4 a lane up to 1024 hypotheses (1536 for large k: 14.5 at 1025,
//    k = 200, one of 12 15.6); beyond one of 12, 8.4 / 10.5 / 13.2 / 26 at V = 700, 4096,
//    k = 1 / 16 / 64 / 200 [four: 12.6 / 16.4 / 20.4 / 34].
//  - V <= 1024: four of 4, 7.4 at 300, k = 64 [two of 8: 8.0], also for large k;
//    beyond 1024 hypotheses two of 8 up to k = 96, 9.5 / 17.1 at 2048 / 4096, k = 64
//    [four: 12.4 / 20.5].
//  - V <= 1536: four of 8 up to 768 hypotheses, also for large k; beyond two of 10
//    or 12 up to k = 96, 5.9 / 12.5 at V = 1100, 1024 / 4096, k = 1 [four: 7.3 / 16.8]
//    and 8.9 / 19.4 at k = 64, 1024 / 4096 [10.3 / 25].
//  - V <= 2048: four of 8, 6.9 / 19.1 at 300, k = 32 / 4000, k = 16 [eight of 4:
//    7.8 / 30.5].
//  - V <= 4096 (V = 4000): eight of 8 for few hypotheses, 6.0 at 8 [four of 16: 6.7],
//    four of 16 above, 8.8 / 32 at 300, k = 32 / 4000, k = 16 [9.3 / 41].
//  - above: eight of 12 up to V = 6144, 9.6 / 57 at V = 5000 [of 16: 10.4 / 63;
//    sixteen of 8: 18.2 / 110], of 16 above.
hipError_t launch_fused_topk(const DevTrie &t, const float *asr, int64_t B, int64_t ld, float lambda, int k,
                             const int32_t *states, int32_t *tokens, float *scores, int32_t *next,
                             hipStream_t stream) {
#define NGPU_TOPK(W, NT) return launch<W, NT>(t, asr, B, ld, lambda, k, states, tokens, scores, next, stream)
    const int V = t.vocab_size;
    if (V <= 256) {
        if (k > 64 && B <= 1024) NGPU_TOPK(2, 2);
        NGPU_TOPK(1, 4);
    }
    if (V <= 512) {
        if (k > 96 && B <= 1280) NGPU_TOPK(4, 2);
        if (k > 32 && (B <= 1024 || (k > 96 && B > 8192))) NGPU_TOPK(2, 4);
        NGPU_TOPK(1, 8);
    }
    if (V <= 768 && B > (k > 96 ? 1536 : 1024)) NGPU_TOPK(1, 12);
    if (V <= 1024) {
        if (k <= 96 && B > 1024) NGPU_TOPK(2, 8);
        NGPU_TOPK(4, 4);
    }
    if (V <= 1536 && k <= 96 && B > 768) {
        if (V <= 1280) NGPU_TOPK(2, 10);
        NGPU_TOPK(2, 12);
    }
    if (V <= 2048) NGPU_TOPK(4, 8);
    if (V <= 4096) {
        if (B <= 128) NGPU_TOPK(8, 8);
        NGPU_TOPK(4, 16);
    }
    if (V <= 6144) NGPU_TOPK(8, 12);
    NGPU_TOPK(8, 16);
#undef NGPU_TOPK
}

}  // namespace ngpu
