// Greedy shallow fusion (Section 2.3), one step over a batch of hypotheses, and
// the top-k beam expansion.
//
// One workgroup of W wavefronts per hypothesis (W = 4 for batches up to 1024,
// else 1), each wavefront owning every W-th stripe of 256 tokens.  CTC and
// transducer modes first take the plain ASR argmax over the V + 1 classes;
// when that keeps blank (or, for CTC, the previous label) the LM is not
// consulted at all and the state stays.  Otherwise the workgroup walks its
// state's backoff chain into an LDS row (the same walk as the advance kernel,
// with no HBM write of the row), merges the dense row of the order-1 ancestor,
// forms fmaf(lambda, lm[v], asr[v]) per token and takes the argmax with
// lowest-index ties: each lane keeps a running maximum over its tokens (read
// four at a time from LDS), the lanes' (value, index) pairs are reduced
// across the wavefront with DPP moves (the largest value, then the smallest
// index holding it), and the W wavefronts' winners meet as 64-bit keys
// (value, ~index) in one LDS exchange.  The winner's next state rides along with its key.  No
// MFMA: one fma and one compare per token.
//
// AED mode (Section 2.3): class V is <eos>, whose LM score is the state's
// final weight (the </s> score, precomputed per state); <eos> keeps the state.
#include <hip/hip_runtime.h>

#include "group.h"

namespace ngpu {

// Words of an ASR row buffer in LDS: the V tokens rounded up to whole
// stripes, so that the 16-byte reads of the scans stay inside it.  (Blank or
// <eos>, class V, travels in a register.)
__host__ __device__ inline int asr_row_words(int V) { return lds_row(V); }

// Per-lane argmax of row[v] over the owned tokens v < V.  Lane l reads tokens
// 4l .. 4l + 3 of each owned stripe with one 16-byte LDS read, so every lane
// meets its tokens in ascending order.
template <int W>
__device__ __forceinline__ void scan_row(const float *row, int V, int wave, int lane, float &bx, int &bi) {
    const int full = V & ~(kStripe - 1);
#pragma unroll 4
    for (int c = kStripe * wave; c < full; c += kStripe * W) {
        const int v0 = c + 4 * lane;
        const f32x4 a = *reinterpret_cast<const f32x4 *>(row + v0);
#pragma unroll
        for (int j = 0; j < 4; ++j) take_max(a[j], v0 + j, bx, bi);
    }
    if (full < V && owns_token<W>(full, wave)) {
        const int v0 = full + 4 * lane;
        const f32x4 a = *reinterpret_cast<const f32x4 *>(row + v0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (v0 + j < V) take_max(a[j], v0 + j, bx, bi);
    }
}

// Per-lane argmax of fmaf(lambda, lm[v], row[v]) over the owned tokens v < V,
// lm[v] from the walked LDS row; same reads as scan_row.
template <int W>
__device__ __forceinline__ void scan_fused(const ChainHead &h, const float *ls, const int *ln, const float *row,
                                           float lambda, int V, int wave, int lane, float &bx, int &bi) {
    auto four = [&](int v0, bool tail) {
        const f32x4 x = *reinterpret_cast<const f32x4 *>(ls + v0);
        const i32x4 n = *reinterpret_cast<const i32x4 *>(ln + v0);
        const f32x4 a = *reinterpret_cast<const f32x4 *>(row + v0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float lm;
            int nx;
            slot_value(h, x[j], n[j], lm, nx);
            const float f = __builtin_fmaf(lambda, lm, a[j]);
            const int v = v0 + j;
            if (!tail || v < V) take_max(f, v, bx, bi);
        }
    };
    const int full = V & ~(kStripe - 1);
#pragma unroll 4
    for (int c = kStripe * wave; c < full; c += kStripe * W) four(c + 4 * lane, false);
    if (full < V && owns_token<W>(full, wave)) four(full + 4 * lane, true);
}

// ASR row held in LDS (asr_row_words(V) words; the owned stripes are read).
template <int W>
struct LdsAsr {
    const float *row;
    __device__ __forceinline__ void argmax(int V, int wave, int lane, float &bx, int &bi) const {
        scan_row<W>(row, V, wave, lane, bx, bi);
    }
    __device__ __forceinline__ void fused(const ChainHead &h, const float *ls, const int *ln, float lambda, int V,
                                          int wave, int lane, float &bx, int &bi) const {
        scan_fused<W>(h, ls, ln, row, lambda, V, wave, lane, bx, bi);
    }
};

// Exchange area of W wavefronts: two alternating buffers of W (key, payload)
// pairs, so one barrier per exchange suffices (a buffer is written again only
// after every wavefront has passed the next exchange's barrier).
struct Exchange {
    unsigned long long key[2][4];
    int payload[2][4];
};

// Argmax over the W wavefronts' lanes of (bx, bi): lowest index among the
// largest values.  Returns the index (kNone when every value was -inf), its
// value and the payload the winning lane passed in; all uniform.
template <int W>
__device__ __forceinline__ int group_argmax(float bx, int bi, int payload, float &best, int &win_payload,
                                            Exchange *xc, int &xi, int wave, int lane) {
    static_assert(W == 1 || W == 2 || W == 4, "the exchange area holds at most four wavefronts");
    const unsigned long long mine = argmax_key(bx, bi);
    unsigned long long k = wave_argmax_key(bx, bi);
    // the lane whose key won hands over its payload (the lowest such lane: keys are unique but for kNone)
    const unsigned long long won = __builtin_amdgcn_read_exec() & __ballot(mine == k);
    const int src = won ? int(__builtin_ctzll(won)) : 0;
    int pl = __builtin_amdgcn_readlane(payload, src);
    if (W > 1) {
        const int buf = xi & 1;
        ++xi;
        if (lane == 0) {
            xc->key[buf][wave] = k;
            xc->payload[buf][wave] = pl;
        }
        lds_barrier();
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const unsigned long long o = xc->key[buf][i];
            const int op = xc->payload[buf][i];
            if (o > k) {
                k = o;
                pl = op;
            }
        }
        k = (static_cast<unsigned long long>(unsigned(__builtin_amdgcn_readfirstlane(int(unsigned(k >> 32))))) << 32) |
            unsigned(__builtin_amdgcn_readfirstlane(int(unsigned(k & 0xffffffffu))));
        pl = __builtin_amdgcn_readfirstlane(pl);
    }
    best = key_value(k);
    win_payload = pl;
    return argmax_index(k);
}

// Next state of token w in {0, 1} (stripe 0, owned by wavefront 0), shared
// with the other wavefronts.
template <int W>
__device__ __forceinline__ int first_token_state(const ChainHead &h, const float *ls, const int *ln, int w,
                                                 Exchange *xc, int &xi, int wave, int lane) {
    int ns = 0;
    if (wave == 0) {
        float lm;
        slot_value(h, ls[w], ln[w], lm, ns);
    }
    if (W > 1) {
        const int buf = xi & 1;
        ++xi;
        if (wave == 0 && lane == 0) xc->payload[buf][0] = ns;
        lds_barrier();
        ns = __builtin_amdgcn_readfirstlane(xc->payload[buf][0]);
    }
    return ns;
}

// One fused greedy step of a hypothesis held by W wavefronts.  asr: its V
// token ASR log-probabilities, whose copy into LDS was issued just before;
// rowV: class V (blank, or <eos> in AED mode).  s: valid state (uniform); pv:
// previous label (CTC).  Returns the label and updates s; all lanes of all W
// wavefronts return the same values.
template <int MODE, int W, bool SPLIT, class Index>
__device__ __forceinline__ int greedy_step(const DevTrie &t, const Index &ci, const LdsAsr<W> &asr, float rowV,
                                           float lambda, int &s, int pv, float *ls, int *ln, Exchange *xc, int &xi,
                                           int wave, int lane) {
    const int V = t.vocab_size;
    const float fin = MODE == kAed ? t.final_w[s] : 0.0f;   // <eos> takes the state's final weight
    // The chain record is fetched first: in CTC and transducer modes its load
    // overlaps the plain ASR argmax, which may still find that the LM is not needed.
    int nlev;
    memory_order_point();   // the ASR row's copies were issued before the record load
    const int4 rec = fetch_record(t, ci, s, lane, nlev);
    if (MODE == kCtc || MODE == kTransducer) {
        // the row, not the record: the record load (one instruction) stays in
        // flight through the argmax
        wait_lds_copies_but_last();
        float bx = -__builtin_inff(), av;
        int bi = kNone, unused;
        asr.argmax(V, wave, lane, bx, bi);
        int a = group_argmax<W>(bx, bi, 0, av, unused, xc, xi, wave, lane);
        if (a == kNone) a = 0;                    // every token at -inf: the first one, unless blank beats it
        if (rowV > av) a = V;                     // blank only when strictly larger (it has the highest index)
        if (a == V || (MODE == kCtc && a == pv)) return a;   // blank or repeat: no LM, no move
    }
    const ChainHead h = walk_record<W, SPLIT>(t, rec, nlev, ls, ln, lane, wave);
    // CTC: the previous label is no candidate; its slot reads NaN, which no
    // fused value built from it can pass under a strict '>'
    if (MODE == kCtc && pv >= 0 && pv < V && owns_token<W>(pv, wave) && lane == 0) {
        ls[pv] = __builtin_nanf("");
        ln[pv] = kFinal;
    }
    float bx = -__builtin_inff(), wv;
    int bi = kNone;
    asr.fused(h, ls, ln, lambda, V, wave, lane, bx, bi);
    // each lane's candidate next state rides along with its key (read from its own stripe)
    int cand = 0;
    if (bi != kNone) {
        float lm;
        slot_value(h, ls[bi], ln[bi], lm, cand);
    }
    int ns;
    int w = group_argmax<W>(bx, bi, cand, wv, ns, xc, xi, wave, lane);
    if (MODE == kAed && __builtin_fmaf(lambda, fin, rowV) > wv)
        return V;   // <eos> strictly above every token: the sentence ends, the state stays
    if (w == kNone) {   // every candidate at -inf: the first one
        w = (MODE == kCtc && pv == 0) ? 1 : 0;
        ns = first_token_state<W>(h, ls, ln, w, xc, xi, wave, lane);
    }
    s = ns;
    return w;
}

// LDS of one hypothesis: the walked row (ls, ln), nrows ASR rows, the exchange area.
__host__ __device__ inline size_t hyp_lds_bytes(int V, int nrows) {
    return (2 * size_t(lds_row(V)) + size_t(nrows) * size_t(asr_row_words(V))) * sizeof(float) + sizeof(Exchange);
}

// One fused step; one hypothesis per workgroup of W wavefronts.
template <int MODE, int W, bool SPLIT = false>
__global__ __launch_bounds__(W * kWave) void fused_step_kernel(DevTrie t, const float *__restrict__ asr, int64_t B,
                                                                int64_t ld, float lambda,
                                                                int32_t *__restrict__ states,
                                                                int32_t *__restrict__ prev,
                                                                int32_t *__restrict__ tokens) {
    extern __shared__ float lds[];
    load_trie_args(t);
    load_args(asr, B, ld, lambda, states, prev, tokens);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t b = blockIdx.x;
    if (b >= B) return;
    const int V = t.vocab_size;
    float *ls = lds;
    int *ln = reinterpret_cast<int *>(ls + lds_row(V));
    float *arow = reinterpret_cast<float *>(ln + lds_row(V));
    Exchange *xc = reinterpret_cast<Exchange *>(arow + asr_row_words(V));

    // the state, the previous label and blank's score go out first, then the
    // ASR row's copy into LDS, so their wait leaves the copy in flight
    const float *src = asr + b * ld;
    const int s_l = states[b];
    const int pv_l = MODE == kCtc ? prev[b] : -1;
    const float rowV_l = MODE == kPlain ? 0.0f : src[V];
    copy_stripes_dword<W>(src, arow, V, wave, lane);
    const ChainIndex ci = chain_index(t, lane);
    int s = __builtin_amdgcn_readfirstlane(s_l);
    const int pv = __builtin_amdgcn_readfirstlane(pv_l);
    const float rowV = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, rowV_l)));
    if (s < 0 || s >= t.num_states) {
        if (wave == 0 && lane == 0) {
            atomicAdd(&t.status[0], 1);
            tokens[b] = -1;
        }
        wait_lds_copies();   // no copy into LDS outlives the wavefront
        return;
    }
    int xi = 0;
    // every wavefront has read states[b] and prev[b] before the first exchange
    // barrier inside the step, and wavefront 0 writes them back after it
    const int label = greedy_step<MODE, W, SPLIT>(
        t, ci, LdsAsr<W>{arow}, rowV, lambda, s, pv, ls, ln, xc, xi, wave, lane);
    if (wave == 0 && lane == 0) {
        tokens[b] = label;
        states[b] = s;
        if (MODE == kCtc) prev[b] = label;
    }
}

// The k best fused scores of one hypothesis per wavefront (beam-search
// expansion), in descending order with lowest-index ties.  After the walk,
// each lane turns its slots into (fused value, next state) in place and keeps
// its own best; a round reduces the lanes' bests to the winner (one DPP
// reduction), and only the lane that held it marks the slot taken (bit 31 of
// its next state), writes the outputs and rescans its own tokens.  Cost:
// V / 64 per lane once, then k rounds of one reduction and one lane's rescan.
__global__ __launch_bounds__(kWave) void fused_topk_kernel(DevTrie t, const float *__restrict__ asr, int64_t B,
                                                           int64_t ld, float lambda, int k,
                                                           const int32_t *__restrict__ states,
                                                           int32_t *__restrict__ tokens, float *__restrict__ scores,
                                                           int32_t *__restrict__ next) {
    extern __shared__ float lds[];
    load_trie_args(t);
    load_args(asr, B, ld, lambda, k, states, tokens, scores, next);
    const int lane = threadIdx.x;
    const int64_t b = blockIdx.x;
    if (b >= B) return;
    const int V = t.vocab_size;
    float *ls = lds;
    int *ln = reinterpret_cast<int *>(ls + lds_row(V));
    float *arow = reinterpret_cast<float *>(ln + lds_row(V));
    int32_t *otok = tokens + b * k;
    float *osc = scores + b * k;
    int32_t *onx = next + b * k;
    const int s_l = states[b];   // issued before the row copy, so its wait leaves the copy in flight
    copy_to_lds_dword(asr + b * ld, arow, V, lane);
    const ChainIndex ci = chain_index(t, lane);
    const int s = __builtin_amdgcn_readfirstlane(s_l);
    if (s < 0 || s >= t.num_states) {
        if (lane == 0) atomicAdd(&t.status[0], 1);
        for (int j = lane; j < k; j += kWave) {
            otok[j] = -1;
            osc[j] = NAN;
            onx[j] = -1;
        }
        wait_lds_copies();   // no copy into LDS outlives the wavefront
        return;
    }
    const ChainHead h = walk_into_lds(t, ci, s, ls, ln, lane);   // its final wait covers the ASR row too
    constexpr int kTaken = int32_t(0x80000000u);
    float bx = -__builtin_inff();
    int bi = kNone;
    for (int c = 0; c < V; c += kStripe) {   // lane l: tokens c + 4l .. c + 4l + 3, rewritten in place
        const int v0 = c + 4 * lane;
        f32x4 x = *reinterpret_cast<const f32x4 *>(ls + v0);
        i32x4 n = *reinterpret_cast<const i32x4 *>(ln + v0);
        const f32x4 a = *reinterpret_cast<const f32x4 *>(arow + v0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float lm;
            int nx;
            slot_value(h, x[j], n[j], lm, nx);
            x[j] = __builtin_fmaf(lambda, lm, a[j]);
            n[j] = v0 + j < V ? nx : kTaken;   // padding past V counts as taken
            if (v0 + j < V) take_max(x[j], v0 + j, bx, bi);
        }
        *reinterpret_cast<f32x4 *>(ls + v0) = x;
        *reinterpret_cast<i32x4 *>(ln + v0) = n;
    }
    for (int j = 0; j < k; ++j) {
        float wv;
        int w = wave_argmax(bx, bi, wv);
        if (w == kNone) {   // everything left is -inf: the lowest index not yet taken
            int lo = kNone;
            for (int c = 0; c < V && lo == kNone; c += kStripe) {
                const int v0 = c + 4 * lane;
                const i32x4 n = *reinterpret_cast<const i32x4 *>(ln + v0);
#pragma unroll
                for (int q = 3; q >= 0; --q)
                    if (n[q] >= 0) lo = v0 + q;
            }
            w = int(~wave_max_u32(~(unsigned)lo));
        }
        if (lane == ((w & (kStripe - 1)) >> 2)) {   // the lane that owns token w
            otok[j] = w;
            osc[j] = ls[w];
            onx[j] = ln[w];
            ln[w] = ln[w] | kTaken;
            bx = -__builtin_inff();
            bi = kNone;
            for (int c = 0; c < V; c += kStripe) {
                const int v0 = c + 4 * lane;
                const f32x4 x = *reinterpret_cast<const f32x4 *>(ls + v0);
                const i32x4 n = *reinterpret_cast<const i32x4 *>(ln + v0);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (n[q] >= 0) take_max(x[q], v0 + q, bx, bi);
            }
        }
    }
}

// Inclusive prefix sum over the lanes of a wave (the DPP pattern of
// wave_max_u32 with additions).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned add_step(unsigned x) {
    return x + unsigned(__builtin_amdgcn_update_dpp(0, int(x), CTRL, ROW_MASK, 0xf, true));
}

__device__ __forceinline__ unsigned wave_incl_sum(unsigned x) {
    x = add_step<0x111, 0xf>(x);
    x = add_step<0x112, 0xf>(x);
    x = add_step<0x114, 0xf>(x);
    x = add_step<0x118, 0xf>(x);
    x = add_step<0x142, 0xa>(x);
    x = add_step<0x143, 0xc>(x);
    return x;
}

__device__ __forceinline__ unsigned wave_sum(unsigned x) {
    return unsigned(__builtin_amdgcn_readlane(int(wave_incl_sum(x)), kWave - 1));
}

// The k (distinct) sort keys in sk[0, k), with their scores and next states,
// written out in descending key order: lane l ranks entries l + 64 r (r < NR,
// k <= 64 NR) by counting the keys above them.
template <int NR>
__device__ __forceinline__ void rank_and_store(const unsigned long long *sk, const float *ssc, const int *snx, int k,
                                               int lane, int32_t *otok, float *osc, int32_t *onx) {
    unsigned long long mine[NR];
    int rank[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        mine[r] = lane + r * kWave < k ? sk[lane + r * kWave] : ~0ull;
        rank[r] = 0;
    }
#pragma unroll 8
    for (int q = 0; q < k; ++q) {
        const unsigned long long o = sk[q];
#pragma unroll
        for (int r = 0; r < NR; ++r) rank[r] += o > mine[r] ? 1 : 0;
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int e = lane + r * kWave;
        if (e < k) {
            otok[rank[r]] = int(~unsigned(mine[r] & 0xffffffffu));
            osc[rank[r]] = ssc[e];
            onx[rank[r]] = snx[e];
        }
    }
}

// The same selection in a number of steps that does not grow with k (V <=
// 256 * SPL): keys are the order-preserving images of the fused values
// (value_key; tokens past V get 0, below every token's key).
//   1. the threshold T, the largest key with at least k keys >= T (the k-th
//      largest key), by a binary search over its bits: a count of the keys
//      >= a candidate is a compare and add per register slot and one wave sum
//      (DPP).  The bits that a lower bound of T and the largest key share are
//      T's from the start, and the search stops as soon as a candidate has
//      exactly k keys >= it: then those are the k taken and no tie is cut;
//   2. every key above T is taken, and of the keys equal to T the lowest
//      token indices until k are taken (a token's rank among them from
//      ballots and lane-prefix counts: token 256 c + 4 l + j sits in slot
//      4 c + j of lane l, so index order is (c, lane, j));
//   3. the k taken entries are compacted into LDS as 64-bit sort keys
//      (value key, ~index) with their score and next state, and each lands
//      at its rank, the number of taken keys above it (keys are distinct).
template <int SPL>
__global__ __launch_bounds__(kWave) void fused_topk_select_kernel(DevTrie t, const float *__restrict__ asr,
                                                                  int64_t B, int64_t ld, float lambda, int k,
                                                                  const int32_t *__restrict__ states,
                                                                  int32_t *__restrict__ tokens,
                                                                  float *__restrict__ scores,
                                                                  int32_t *__restrict__ next) {
    constexpr int kN = 4 * SPL;
    extern __shared__ float lds[];
    load_trie_args(t);
    load_args(asr, B, ld, lambda, k, states, tokens, scores, next);
    const int lane = threadIdx.x;
    const int64_t b = blockIdx.x;
    if (b >= B) return;
    const int V = t.vocab_size;
    float *ls = lds;
    int *ln = reinterpret_cast<int *>(ls + lds_row(V));
    float *arow = reinterpret_cast<float *>(ln + lds_row(V));
    int32_t *otok = tokens + b * k;
    float *osc = scores + b * k;
    int32_t *onx = next + b * k;
    const int s_l = states[b];   // issued before the row copy, so its wait leaves the copy in flight
    copy_to_lds_dword(asr + b * ld, arow, V, lane);
    const ChainIndex ci = chain_index(t, lane);
    const int s = __builtin_amdgcn_readfirstlane(s_l);
    if (s < 0 || s >= t.num_states) {
        if (lane == 0) atomicAdd(&t.status[0], 1);
        for (int j = lane; j < k; j += kWave) {
            otok[j] = -1;
            osc[j] = NAN;
            onx[j] = -1;
        }
        wait_lds_copies();   // no copy into LDS outlives the wavefront
        return;
    }
    const ChainHead h = walk_into_lds(t, ci, s, ls, ln, lane);   // its final wait covers the ASR row too
    // slot i = 4 c + j of this lane is token 256 c + 4 lane + j
    float f[kN];
    int n[kN];
    unsigned key[kN];
#pragma unroll
    for (int c = 0; c < SPL; ++c) {
        const int v0 = c * kStripe + 4 * lane;
        const f32x4 x = *reinterpret_cast<const f32x4 *>(ls + v0);
        const i32x4 m = *reinterpret_cast<const i32x4 *>(ln + v0);
        const f32x4 a = *reinterpret_cast<const f32x4 *>(arow + v0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float lm;
            slot_value(h, x[j], m[j], lm, n[4 * c + j]);
            f[4 * c + j] = __builtin_fmaf(lambda, lm, a[j]);
            key[4 * c + j] = v0 + j < V ? value_key(f[4 * c + j]) : 0u;
        }
    }
    // 1. the threshold T.  It lies between a lower bound lo (for k <= 64 j,
    // the smallest over the lanes of a lane's j-th largest key: at least
    // 64 j >= k keys are >= it; 0 for k > 128) and the largest key, so the
    // bits above the highest one in which those two differ are T's already.
    unsigned lo = 0, mx = 0;
    if (k <= 2 * kWave) {
        unsigned m1 = 0, m2 = 0;   // the lane's largest and second largest key
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            m2 = max(m2, min(m1, key[i]));
            m1 = max(m1, key[i]);
        }
        mx = wave_max_u32(m1);
        lo = ~wave_max_u32(~(k <= kWave ? m1 : m2));
    } else {
        unsigned m1 = 0;
#pragma unroll
        for (int i = 0; i < kN; ++i) m1 = max(m1, key[i]);
        mx = wave_max_u32(m1);
    }
    const unsigned diff = lo ^ mx;
    const int top = diff ? 31 - __builtin_clz(diff) : -1;
    unsigned T = top < 0 ? mx : mx & ~((2u << top) - 1u);   // top = 31: no bit known (2u << 31 is 0)
    bool exact = false;   // the keys >= T number exactly k
    for (int bit = top; bit >= 0 && !exact; --bit) {
        const unsigned cand = T | (1u << bit);
        unsigned c = 0;
#pragma unroll
        for (int i = 0; i < kN; ++i) c += key[i] >= cand ? 1u : 0u;
        const int cnt = int(wave_sum(c));
        if (cnt >= k) T = cand;
        exact = cnt == k;
    }
    int above = k;
    if (!exact) {   // T is the k-th key itself: count the keys above it
        unsigned c = 0;
#pragma unroll
        for (int i = 0; i < kN; ++i) c += key[i] > T ? 1u : 0u;
        above = int(wave_sum(c));
    }
    // 2. taken entries: every key >= T when exact; otherwise T is the k-th
    // key itself, `above` keys exceed it, and of the keys equal to it the
    // lowest token indices are taken (bit i of tie_taken: slot i is such a tie)
    unsigned tie_taken = 0;
    if (!exact) {
        const int ties_needed = k - above;
        int ties_before = 0;   // ties at T in earlier stripes (uniform)
#pragma unroll
        for (int c = 0; c < SPL; ++c) {
            unsigned long long m[4];
            int below = 0;      // ties of this stripe in lower lanes
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                m[j] = __ballot(key[4 * c + j] == T);
                below += int(__builtin_amdgcn_mbcnt_hi(unsigned(m[j] >> 32),
                                                       __builtin_amdgcn_mbcnt_lo(unsigned(m[j]), 0u)));
            }
            int own = 0;        // ties of this lane in earlier slots of the stripe
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = 4 * c + j;
                const bool tie = key[i] == T;
                if (tie && ties_before + below + own < ties_needed) tie_taken |= 1u << i;
                own += tie ? 1 : 0;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) ties_before += __builtin_popcountll(m[j]);
        }
    }
    // 3. compaction into LDS (the walked row is in registers now), then ranks;
    // the exact case tests its keys directly, with no per-slot flags to build
    unsigned long long *sk = reinterpret_cast<unsigned long long *>(lds);
    float *ssc = reinterpret_cast<float *>(sk + k);
    int *snx = reinterpret_cast<int *>(ssc + k);
    auto compact = [&](auto taken) {
        int base = 0;
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            const bool tk = taken(i);
            const unsigned long long m = __ballot(tk);
            if (tk) {
                const int p = base + int(__builtin_amdgcn_mbcnt_hi(unsigned(m >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo(unsigned(m), 0u)));
                const int tok = (i >> 2) * kStripe + 4 * lane + (i & 3);
                sk[p] = (static_cast<unsigned long long>(key[i]) << 32) | unsigned(~unsigned(tok));
                ssc[p] = f[i];
                snx[p] = n[i];
            }
            base += __builtin_popcountll(m);
        }
    };
    if (exact)
        compact([&](int i) { return key[i] >= T; });
    else
        compact([&](int i) { return key[i] > T || ((tie_taken >> i) & 1u) != 0; });
    if (k <= kWave)
        rank_and_store<1>(sk, ssc, snx, k, lane, otok, osc, onx);
    else if (k <= 2 * kWave)
        rank_and_store<2>(sk, ssc, snx, k, lane, otok, osc, onx);
    else
        rank_and_store<4>(sk, ssc, snx, k, lane, otok, osc, onx);
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

hipError_t launch_fused_topk(const DevTrie &t, const float *asr, int64_t B, int64_t ld, float lambda, int k,
                             const int32_t *states, int32_t *tokens, float *scores, int32_t *next,
                             hipStream_t stream) {
    const size_t lds = (2 * size_t(lds_row(t.vocab_size)) + size_t(asr_row_words(t.vocab_size))) * sizeof(float);
    const dim3 grid(static_cast<unsigned>(B)), block(kWave);
    const int spl = (t.vocab_size + kStripe - 1) / kStripe;   // stripes per lane
    // V <= 1024: the selection with the row in registers, for every k (from
    // k = 6 on it beats one reduction per selected token; below that the two
    // are level: 10.1-10.5 us either way at k = 1 to 5 for 1024 hypotheses of
    // the 20M 6-gram).  Larger V: one reduction per selected token.  The k
    // taken entries (16 bytes each) may need more LDS than the row.
    const size_t lds_sel = lds > 16 * size_t(k) ? lds : 16 * size_t(k);
    switch (spl) {
        case 1:
            hipLaunchKernelGGL(fused_topk_select_kernel<1>, grid, block, lds_sel, stream, t, asr, B, ld, lambda, k,
                               states, tokens, scores, next);
            break;
        case 2:
            hipLaunchKernelGGL(fused_topk_select_kernel<2>, grid, block, lds_sel, stream, t, asr, B, ld, lambda, k,
                               states, tokens, scores, next);
            break;
        case 3:
            hipLaunchKernelGGL(fused_topk_select_kernel<3>, grid, block, lds_sel, stream, t, asr, B, ld, lambda, k,
                               states, tokens, scores, next);
            break;
        case 4:
            hipLaunchKernelGGL(fused_topk_select_kernel<4>, grid, block, lds_sel, stream, t, asr, B, ld, lambda, k,
                               states, tokens, scores, next);
            break;
        default:
            hipLaunchKernelGGL(fused_topk_kernel, grid, block, lds, stream, t, asr, B, ld, lambda, k, states, tokens,
                               scores, next);
    }
    return hipGetLastError();
}

// The same choice for one step per launch, where every launch pays the whole
// dependent chain once: four wavefronts stay ahead up to 1024 hypotheses
// (20M 6-gram, CTC: 8.54 against 8.70 us per step at 768, 8.95 against 9.12
// at 1024; 11.2 against 10.6 at 2048).
inline int step_waves_per_hyp(int64_t B) { return B <= 1024 ? 4 : 1; }

// Wavefronts that own one 256-token stripe each load only their stripe's part
// of every sparse level.
template <int W>
inline bool stripe_split(const DevTrie &t) {
    return W > 1 && (t.vocab_size + kStripe - 1) / kStripe == W;
}

template <int MODE, int W>
static hipError_t launch_step_w(const DevTrie &t, const float *asr, int64_t B, int64_t ld, float lambda,
                                int32_t *states, int32_t *prev, int32_t *tokens, hipStream_t stream) {
    if constexpr (W > 1) {
        if (stripe_split<W>(t)) {
            hipLaunchKernelGGL((fused_step_kernel<MODE, W, true>), dim3(unsigned(B)), dim3(W * kWave),
                               hyp_lds_bytes(t.vocab_size, 1), stream, t, asr, B, ld, lambda, states, prev, tokens);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((fused_step_kernel<MODE, W, false>), dim3(unsigned(B)), dim3(W * kWave),
                       hyp_lds_bytes(t.vocab_size, 1), stream, t, asr, B, ld, lambda, states, prev, tokens);
    return hipGetLastError();
}

template <int MODE>
static hipError_t launch_step_mode(const DevTrie &t, const float *asr, int64_t B, int64_t ld, float lambda,
                                   int32_t *states, int32_t *prev, int32_t *tokens, hipStream_t stream) {
    switch (step_waves_per_hyp(B)) {
        case 4: return launch_step_w<MODE, 4>(t, asr, B, ld, lambda, states, prev, tokens, stream);
        default: return launch_step_w<MODE, 1>(t, asr, B, ld, lambda, states, prev, tokens, stream);
    }
}

hipError_t launch_fused_step(const DevTrie &t, const float *asr, int64_t B, int64_t ld, int mode, float lambda,
                             int32_t *states, int32_t *prev, int32_t *tokens, hipStream_t stream) {
    switch (mode) {
        case kPlain: return launch_step_mode<kPlain>(t, asr, B, ld, lambda, states, prev, tokens, stream);
        case kCtc: return launch_step_mode<kCtc>(t, asr, B, ld, lambda, states, prev, tokens, stream);
        case kAed: return launch_step_mode<kAed>(t, asr, B, ld, lambda, states, prev, tokens, stream);
        default: return launch_step_mode<kTransducer>(t, asr, B, ld, lambda, states, prev, tokens, stream);
    }
}

}  // namespace ngpu
