// Whole greedy decode in one launch (Section 2.3): utterance b runs frames 0 ..
// len_b - 1 of asr[b * stride_b + t * stride_t + class], one workgroup per
// utterance.  Frame t + 1 depends on frame t through the state and the previous
// label only, so a frame is a chain of dependent steps: the state's chain
// record, its arcs, the fused scan, the argmax over the group, the next state.
// What is off that chain:
//  - the dense row: the state reached by emitting w has the dense row of w's
//    unigram, so the row is fetched together with the record instead of after
//    it (a state of order 1, a quarter of the frames on the 20M 6-gram and
//    three quarters on small models, then costs one memory round trip, not two);
//  - the ASR rows, loaded one or two frames ahead into registers;
//  - with several wavefronts, the plain argmax of frame t + 1 (CTC, transducer):
//    it is computed while frame t's record is in flight and shares frame t's
//    exchange, so a frame has one barrier.
#include <hip/hip_runtime.h>

#include "group.h"

namespace ngpu {

// How the ASR rows are loaded: as usual, or non-temporally, so that a stream
// larger than the 256 MB Infinity Cache leaves the dense rows, records and arcs
// in the caches.
constexpr int kKeep = 0, kStream = 2;   // aux bits of a buffer load: nt = 2

// W wavefronts per utterance, or one whose tokens are few (NT <= 8).
template <int MODE, int W, int NT, bool FULL, int CACHE>
__global__ __launch_bounds__(W * kWave) void decode_kernel(DevTrie t, int uni_base, const float *__restrict__ asr,
                                                           int64_t T, int64_t stride_t, int64_t stride_b,
                                                           const int32_t *__restrict__ lengths, float lambda,
                                                           int32_t *__restrict__ states, int32_t *__restrict__ prev,
                                                           int32_t *__restrict__ labels,
                                                           int32_t *__restrict__ label_states) {
    extern __shared__ i32x4 lds4[];
    constexpr bool kRaw = MODE == kCtc || MODE == kTransducer;
    const int64_t b = blockIdx.x;
    const int V = t.vocab_size;
    Meet *meet = reinterpret_cast<Meet *>(lds4);
    const Group<W, NT, FULL> g(V, reinterpret_cast<i32x2 *>(meet + 1));
    const int wave = g.wave, lane = g.lane;
    int32_t *lab = labels + b * T;
    int32_t *lst = label_states ? label_states + b * T : nullptr;
    const int zero = lane_zero();

    int64_t len = T;
    if (lengths) {
        len = __builtin_amdgcn_readfirstlane(lengths[b]);
        len = len < 0 ? 0 : (len > T ? T : len);
    }
    int s = __builtin_amdgcn_readfirstlane(states[b]);
    if (s < 0 || s >= t.num_states) {
        if (wave == 0) {
            if (lane == 0) atomicAdd(&t.status[0], 1);
            for (int64_t f = lane; f < T; f += kWave) {
                lab[f] = -1;
                if (lst) lst[f] = -1;
            }
        }
        return;
    }
    int pv = MODE == kCtc ? __builtin_amdgcn_readfirstlane(prev[b]) : -1;
    const RecordIndex ri = record_index(t, lane);

    Words<NT> cur, nxt, nn, dw, dt;
    float cur_v = 0.0f, nxt_v = 0.0f, nn_v = 0.0f, fin = 0.0f;
    auto load_row = [&](const float *row, Words<NT> &x, float &v) {
        g.template load_row<CACHE>(row, x);
        if (MODE != kPlain) v = row[V + zero];   // blank or <eos>
    };
    int4 rec;
    bool dirty = false;   // slots to clear
    auto fetch_rec = [&](int st) {
        rec = load_record(ri, st, lane);
        if (MODE == kAed) fin = t.final_w[st + zero];   // <eos> takes the state's final weight
    };

    const float *row = asr + b * stride_b;
    unsigned raw_key = 0;   // the frame's best class by its ASR scores alone: key and token
    int raw_tok = 0, xi = 0;
    // key of blank's score, NaN as -inf, taken off the chain while the frame before it runs
    auto blank_key_of = [](float v) {
        return unsigned(__builtin_amdgcn_readfirstlane(int(float_key(or_lowest(v)))));
    };
    unsigned blank_key = 0;
    if (len > 0) {
        load_row(row, cur, cur_v);
        fetch_rec(s);
        if (len > 1) row += stride_t;
        load_row(row, nxt, nxt_v);
        g.clear_slots();
        g.mask_row(cur);
        if (kRaw) {
            g.raw_best(cur, raw_key, raw_tok);
            blank_key = blank_key_of(cur_v);
            if (W > 1) {
                if (lane == 0) {
                    meet->a[0][wave].w = raw_tok;
                    meet->b[0][wave] = int(raw_key);
                }
                lds_barrier();
                const int k = meet->b[0][lane & (W - 1)], tk = meet->a[0][lane & (W - 1)].w;
                const int e = winner_entry<W>(unsigned(k), tk);
                raw_key = unsigned(__builtin_amdgcn_readlane(k, e));
                raw_tok = __builtin_amdgcn_readlane(tk, e);
                xi = 1;
            }
        }
        g.load_dense(t, unsigned(__builtin_amdgcn_readlane(rec.x, 0)), dw, dt);
    }
    for (int64_t f0 = 0; f0 < len; f0 += kWave) {
        const int64_t rest = len - f0;
        const int left = rest > (int64_t(1) << 30) ? 1 << 30 : int(rest);   // frames from f0 on
        const int n = left < kWave ? left : kWave;
        int keep_lab = -1, keep_st = -1;   // lane f: label and state of frame f0 + f
        for (int f = 0; f < n; ++f) {
            row += f + 2 < left ? stride_t : 0;   // row f + 2 (at the end the last row again, not used)
            load_row(row, nn, nn_v);
            g.mask_row(nxt);
            unsigned nr_key = 0, nr_blank = 0;
            int nr_tok = 0;
            if (kRaw) {
                g.raw_best(nxt, nr_key, nr_tok);
                nr_blank = blank_key_of(nxt_v);
            }
            int label = -1;
            bool lm = true;
            if (kRaw) {
                label = raw_tok;                                      // every token at -inf: the lowest, 0
                if (blank_key > raw_key) label = V;                   // blank only when strictly larger (highest index)
                lm = !(label == V || (MODE == kCtc && label == pv));  // blank or repeat: no LM, no move
            }
            unsigned fkey = 0;
            int ftok = 0, fto = 0, who = 0;
            if (lm) {
                const ChainHead h = head_of(rec);
                dirty |= g.put_levels(t, rec, h);
                if (MODE == kCtc) {   // the previous label is no candidate
                    const int p = pv - g.t0 - lane;
#pragma unroll
                    for (int i = 0; i < NT; ++i)
                        cur.v[i] = p == kWave * i ? __float_as_int(-__builtin_inff()) : cur.v[i];
                }
                float x[NT], bx;
                int nx[NT], bi;
                g.lm_values(h, dw, dt, dirty, x, nx);
#pragma unroll
                for (int i = 0; i < NT; ++i) x[i] = __builtin_fmaf(lambda, x[i], cur.f(i));
                g.lane_best(x, bx, bi);
                fto = nx[0];
#pragma unroll
                for (int i = 1; i < NT; ++i) fto = bi == kWave * i ? nx[i] : fto;
                fto &= kStateMask;
                fkey = float_key(bx);
                ftok = g.t0 + bi + lane;
                who = winner_lane(fkey, ftok);
            }
            if (W > 1) {
                const int buf = xi & 1;
                ++xi;
                if (lane == who) {   // the winning lane leaves its own values (no LM: lane 0, the plain argmax only)
                    const i32x4 e = {int(fkey), ftok, fto, nr_tok};
                    meet->a[buf][wave] = e;
                    if (kRaw) meet->b[buf][wave] = int(nr_key);
                }
                lds_barrier();
                const i32x4 e = meet->a[buf][lane & (W - 1)];
                if (lm) {
                    const int w = winner_entry<W>(unsigned(e.x), e.y);
                    fkey = unsigned(__builtin_amdgcn_readlane(e.x, w));
                    ftok = __builtin_amdgcn_readlane(e.y, w);
                    fto = __builtin_amdgcn_readlane(e.z, w);
                }
                if (kRaw) {
                    const int k = meet->b[buf][lane & (W - 1)];
                    const int w = winner_entry<W>(unsigned(k), e.w);
                    nr_key = unsigned(__builtin_amdgcn_readlane(k, w));
                    nr_tok = __builtin_amdgcn_readlane(e.w, w);
                }
            } else if (lm) {
                fkey = unsigned(__builtin_amdgcn_readlane(int(fkey), who));
                ftok = __builtin_amdgcn_readlane(ftok, who);
                fto = __builtin_amdgcn_readlane(fto, who);
            }
            bool moved = lm;
            if (MODE == kAed) {   // <eos> strictly above every token: the sentence ends, the state stays
                const float fw = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(fin)));
                const float rowV = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(cur_v)));
                if (float_key(or_lowest(__builtin_fmaf(lambda, fw, rowV))) > fkey) {
                    label = V;
                    moved = false;
                }
            }
            if (moved) {
                if (MODE == kCtc && fkey == kInfKey && pv == 0) {
                    // every candidate at -inf: the first one, and token 0 is none: token 1
                    ftok = 1;
                    if (wave == 0) {
                        const int put = __builtin_amdgcn_readfirstlane(g.slots[1].y);
                        fto = (put != 0 ? put : __builtin_amdgcn_readlane(dt.v[0], 1)) & kStateMask;
                    }
                    if (W > 1) {
                        const int buf = xi & 1;
                        ++xi;
                        if (wave == 0 && lane == 0) meet->b[buf][0] = fto;
                        lds_barrier();
                        fto = __builtin_amdgcn_readfirstlane(meet->b[buf][0]);
                    }
                }
                label = ftok;
                s = fto;
                // (after the last frame for nothing: no branch in the way of the common case)
                fetch_rec(s);
                g.load_dense(t, uni_base >= 0 ? unsigned(uni_base + label)
                                              : unsigned(__builtin_amdgcn_readfirstlane(t.dense_to[label]) & kStateMask),
                             dw, dt);
                if (dirty) g.clear_slots();
                dirty = false;
            }
            raw_key = nr_key;
            raw_tok = nr_tok;
            blank_key = nr_blank;
            cur = nxt;
            cur_v = nxt_v;
            nxt = nn;
            nxt_v = nn_v;
            if (MODE == kCtc) pv = label;
            keep_lab = lane == f ? label : keep_lab;
            keep_st = lane == f ? s : keep_st;
        }
        if (wave == 0 && lane < n) {   // one coalesced store per 64 frames
            lab[f0 + lane] = keep_lab;
            if (lst) lst[f0 + lane] = keep_st;
        }
    }
    if (wave == 0) {
        for (int64_t f = len + lane; f < T; f += kWave) {   // frames past the utterance's end
            lab[f] = -1;
            if (lst) lst[f] = s;
        }
        // every wavefront read states[b] and prev[b] before the first barrier;
        // with no frame at all the values written are the ones read
        if (lane == 0) {
            states[b] = s;
            if (MODE == kCtc) prev[b] = pv;
        }
    }
}

// (asm: the builtin maximum adds an instruction per loaded value to quiet NaNs)
__device__ __forceinline__ float max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// The lane's largest word, -inf where all are NaN.
template <int NT>
__device__ __forceinline__ float lane_max(const Words<NT> &x) {
    static_assert(NT % 2 == 0, "the last maximum takes -inf beside the last word");
    float r = max3(x.f(0), x.f(1), x.f(2));
#pragma unroll
    for (int i = 3; i < NT; i += 2) r = max3(r, x.f(i), i + 1 < NT ? x.f(i + 1) : -__builtin_inff());
    return r;
}
// Value of token 64 j + l (both uniform) of the words.
template <int LO, int HI, int NT>
__device__ __forceinline__ int pick(const Words<NT> &x, int j, int l) {
    if constexpr (HI - LO == 1) {
        return __builtin_amdgcn_readlane(x.v[LO], l);
    } else {
        constexpr int kMid = (LO + HI) / 2;
        return j < kMid ? pick<LO, kMid>(x, j, l) : pick<kMid, HI>(x, j, l);
    }
}

// One wavefront per utterance, 16 tokens a lane (20 and 32 for the batches in
// launch_mode): large batches, where the
// launch is bound by the ASR rows' stream and by instruction issue rather than
// by one utterance's chain.  COMPACT: the 4-byte dense rows, half the traffic;
// the winner's next state then follows from the row's rules (DevTrie).  The
// plain argmax needs the row's maximum only (three-input maxima): blank is
// above it or not, and a repeat is the previous label holding it; the winner's
// token is searched where the wave's maximum is found.  4096 utterances x 200
// frames, V = 1024: 813 us (822 in the kernel before, 8-byte slots and one frame's
// chain in line), 843 (847) on rows just written; without any LM work the stream
// of ASR rows (3.36 GB) alone takes 670.  V = 700, 100 frames: 326 us (654 before).
template <int MODE, int NT, bool FULL, bool COMPACT>
__global__ __launch_bounds__(kWave, (COMPACT ? 4 : 1)) void decode_wave_kernel(
    DevTrie t, int uni_base, const float *__restrict__ asr, int64_t T, int64_t stride_t, int64_t stride_b,
    const int32_t *__restrict__ lengths, float lambda, int32_t *__restrict__ states, int32_t *__restrict__ prev,
    int32_t *__restrict__ labels, int32_t *__restrict__ label_states) {
    extern __shared__ i32x4 lds4[];
    constexpr bool kRaw = MODE == kCtc || MODE == kTransducer;
    const int lane = threadIdx.x;
    const int64_t b = blockIdx.x;
    const int V = t.vocab_size;
    i32x2 *slots = reinterpret_cast<i32x2 *>(lds4);
    int32_t *lab = labels + b * T;
    int32_t *lst = label_states ? label_states + b * T : nullptr;
    const int zero = lane_zero();

    int64_t len = T;
    if (lengths) {
        len = __builtin_amdgcn_readfirstlane(lengths[b]);
        len = len < 0 ? 0 : (len > T ? T : len);
    }
    int s = __builtin_amdgcn_readfirstlane(states[b]);
    if (s < 0 || s >= t.num_states) {
        if (lane == 0) atomicAdd(&t.status[0], 1);
        for (int64_t f = lane; f < T; f += kWave) {
            lab[f] = -1;
            if (lst) lst[f] = -1;
        }
        return;
    }
    int pv = MODE == kCtc ? __builtin_amdgcn_readfirstlane(prev[b]) : -1;
    const RecordIndex ri = record_index(t, lane);
    Words<NT> bufa, bufb;
    float va = 0.0f, vb = 0.0f;
    auto load_row = [&](const float *row, Words<NT> &x, float &v) {
        x.load(row, V, lane);
        if (MODE != kPlain) v = row[V + zero];
    };
    int4 rec;
    Words<NT> dw, dt;
    float fin = 0.0f;
    int base_v = 0;
    auto fetch_rec = [&](int st) {
        rec = load_record(ri, st, lane);
        if (MODE == kAed) fin = t.final_w[st + zero];
    };
    auto fetch_dense = [&](unsigned row) {
        const uint64_t at = uint64_t(row * unsigned(V)) * 4;
        if (COMPACT) {
            dw.load(reinterpret_cast<const char *>(t.dense_c) + at, V, lane);
            base_v = t.dense_base[row + unsigned(zero)];
        } else {
            dw.load(reinterpret_cast<const char *>(t.dense_w) + at, V, lane);
            dt.load(reinterpret_cast<const char *>(t.dense_to) + at, V, lane);
        }
    };
    const float *row = asr + b * stride_b;
    if (len > 0) {
        load_row(row, bufa, va);
        fetch_rec(s);
        fetch_dense(unsigned(__builtin_amdgcn_readlane(rec.x, 0)));
    }
    int keep_lab = -1, keep_st = -1;
    auto frame = [&](int f, int left, Words<NT> &cur, float &cur_v, Words<NT> &nxt, float &nxt_v) {
        row += f + 1 < left ? stride_t : 0;
        if (!FULL) cur.pad(V, lane, -__builtin_inff());
        int label = -1;
        bool lm = true;
        if (kRaw) {
            const unsigned mk = wave_max_u32(float_key(lane_max(cur)));
            const float rowV = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(cur_v)));
            if (float_key(or_lowest(rowV)) > mk) {   // blank only when strictly larger
                label = V;
                lm = false;
            } else if (MODE == kCtc && mk == kInfKey) {   // no token above -inf: the first one, a repeat of label 0
                if (pv == 0) {
                    label = 0;
                    lm = false;
                }
            } else if (MODE == kCtc && pv >= 0 && pv < V) {
                const float at = __int_as_float(pick<0, NT>(cur, pv >> 6, pv & (kWave - 1)));
                if (float_key(at) == mk) {   // the previous label holds the maximum: a repeat unless a lower token does too
                    bool lower = false;
#pragma unroll
                    for (int i = 0; i < NT; ++i)
                        lower |= __ballot(kWave * i + lane < pv && float_key(cur.f(i)) == mk) != 0;
                    if (!lower) {
                        label = pv;
                        lm = false;
                    }
                }
            }
        }
        load_row(row, nxt, nxt_v);
        if (lm) {
            const ChainHead h = head_of(rec);
            const int nlev = h.nlev_group & 0xffff;
            const bool top = __builtin_amdgcn_readlane(rec.x, 1) >= t.top_begin;
            const i32x4 z = {0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < NT / 2; ++i) reinterpret_cast<i32x4 *>(slots)[kWave * i + lane] = z;
            for (int j = nlev; j >= 1; --j) {
                const int a0 = __builtin_amdgcn_readlane(rec.x, j), n = __builtin_amdgcn_readlane(rec.y, j) - a0;
                const float acc = __int_as_float(__builtin_amdgcn_readlane(rec.z, j));
                if (n == 0) continue;
                if (j == 1 && top)
                    put_arcs<true, false>(t, a0, n, acc, slots, 0, 0, lane);
                else
                    put_arcs<false, false>(t, a0, n, acc, slots, 0, 0, lane);
            }
            if (MODE == kCtc && pv >= 0 && pv < V && lane == 0) {   // no candidate: NaN never compares
                const i32x2 no = {0x7fc00000, kFinal};
                slots[pv] = no;
            }
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const i32x2 sl = slots[kWave * i + lane];
                const float acc = (COMPACT ? dw.v[i] : dt.v[i]) < 0 ? h.acc0 : h.acc1;
                const float dense = COMPACT ? acc - __builtin_fabsf(dw.f(i)) : acc + dw.f(i);
                cur.v[i] = __float_as_int(__builtin_fmaf(lambda, sl.y != 0 ? __int_as_float(sl.x) : dense, cur.f(i)));
            }
            const unsigned mk = wave_max_u32(float_key(lane_max(cur)));
            const float best = __int_as_float((mk & 0x80000000u) ? int(mk & 0x7fffffffu) : int(~mk));
            bool eos = false;
            if (MODE == kAed) {
                const float fw = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(fin)));
                const float rowV = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(cur_v)));
                eos = __builtin_fmaf(lambda, fw, rowV) > best;
            }
            if (eos) {
                label = V;
            } else {
                int w = 0, rank = 0, to = 0;
                bool own = false;
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    unsigned long long m = __ballot(cur.f(i) == best);
                    // no candidate above -inf (words past V are at -inf too): the
                    // first one.  Else the best is a token's: w < V.
                    if (i == 0 && mk == kInfKey) m = MODE == kCtc && pv == 0 ? 2 : 1;
                    const unsigned long long o = COMPACT ? __ballot(dw.v[i] >= 0) : 0;
                    if (m) {
                        const int l = int(__builtin_ctzll(m));
                        w = kWave * i + l;
                        if (COMPACT) {
                            rank += __builtin_popcountll(o & ((1ull << l) - 1ull));
                            own = (o >> l) & 1ull;
                        } else {
                            to = __builtin_amdgcn_readlane(dt.v[i], l);
                        }
                        break;
                    }
                    if (COMPACT) rank += __builtin_popcountll(o);
                }
                const int put = __builtin_amdgcn_readfirstlane(slots[w].y);
                if (COMPACT) to = own && t.compact_rank ? __builtin_amdgcn_readfirstlane(base_v) + rank : t.first[1] + w;
                label = w;
                s = (put != 0 ? put : to) & kStateMask;
                fetch_rec(s);
                fetch_dense(uni_base >= 0 ? unsigned(uni_base + w)
                                          : unsigned(__builtin_amdgcn_readfirstlane(t.dense_to[w]) & kStateMask));
            }
        }
        if (MODE == kCtc) pv = label;
        keep_lab = lane == f ? label : keep_lab;
        keep_st = lane == f ? s : keep_st;
    };
    for (int64_t f0 = 0; f0 < len; f0 += kWave) {
        const int64_t rest = len - f0;
        const int left = rest > (int64_t(1) << 30) ? 1 << 30 : int(rest);
        const int n = left < kWave ? left : kWave;
        for (int f = 0; f < n; f += 2) {   // the row buffers change places without copies (kWave is even)
            frame(f, left, bufa, va, bufb, vb);
            if (f + 1 < n) frame(f + 1, left, bufb, vb, bufa, va);
        }
        if (lane < n) {
            lab[f0 + lane] = keep_lab;
            if (lst) lst[f0 + lane] = keep_st;
        }
    }
    for (int64_t f = len + lane; f < T; f += kWave) {
        lab[f] = -1;
        if (lst) lst[f] = s;
    }
    if (lane == 0) {
        states[b] = s;
        if (MODE == kCtc) prev[b] = pv;
    }
}

// A launch's arguments.
struct Decode {
    DevTrie t;
    int uni_base;
    const float *asr;
    int64_t B, T, sb, st;
    const int32_t *lengths;
    float lambda;
    int32_t *states, *prev, *labels, *label_states;
    hipStream_t stream;
    // The ASR rows outgrow the Infinity Cache: stream them.  us a launch, kept
    // against streamed, repeated and (in brackets) first after the tensor was
    // written: 1.05 GB (256 x 1000, 20M 6-gram) 1824 / 1702 [1863 / 1810], 615 MB
    // (1000 x 150, V = 1024) 361 / 345 [403 / 383], 1.08 GB (3000 x 60, V = 1500) 460 /
    // 456 [494 / 472]; 246 MB (300 x 200) 327 / 327, 216 MB (600 x 60, V = 1500) 137 /
    // 144, 48 MB (40 x 200) 295 / 325: a smaller tensor may still be cached from its
    // writer.
    bool streams() const {
        const double row = 4.0 * (t.vocab_size + 1);
        return double(B) * double(T) * row > 256.0 * (1 << 20);
    }
};

// A grid holds at most 2^32 - 1 work-items: larger batches go in several launches.
template <int MODE, int W, int NT, bool FULL, int CACHE>
static hipError_t launch_group(const Decode &d) {
    constexpr int64_t kMost = int64_t(UINT32_MAX) / (W * kWave);
    const size_t lds = sizeof(Meet) + size_t(W) * kWave * NT * sizeof(i32x2);
    for (int64_t b0 = 0; b0 < d.B; b0 += kMost) {
        const dim3 grid{unsigned(d.B - b0 < kMost ? d.B - b0 : kMost)};
        hipLaunchKernelGGL((decode_kernel<MODE, W, NT, FULL, CACHE>), grid, dim3(W * kWave), lds, d.stream, d.t,
                           d.uni_base, d.asr + b0 * d.sb, d.T, d.st, d.sb, d.lengths ? d.lengths + b0 : nullptr, d.lambda,
                           d.states + b0, d.prev ? d.prev + b0 : nullptr, d.labels + b0 * d.T,
                           d.label_states ? d.label_states + b0 * d.T : nullptr);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Rows of up to 512 tokens are always kept: streamed, V = 128 took 143 against
// 136 us at 1500 utterances, 178 against 165 at 4000 (two rows share a line).  So
// are those of decode_wave_kernel: streamed, 4096 x 200 took 795 instead of 813 us
// repeated, but 888 instead of 843 on a tensor just written, which a decode
// after the acoustic model finds.
template <int MODE, int W, int NT>
static hipError_t launch_group(const Decode &d) {
    const bool full = d.t.vocab_size == W * kWave * NT;
    if constexpr (W > 1) {
        if (d.streams())
            return full ? launch_group<MODE, W, NT, true, kStream>(d) : launch_group<MODE, W, NT, false, kStream>(d);
    }
    return full ? launch_group<MODE, W, NT, true, kKeep>(d) : launch_group<MODE, W, NT, false, kKeep>(d);
}

template <int MODE, int NT, bool FULL, bool COMPACT>
static hipError_t launch_wave(const Decode &d) {
    hipLaunchKernelGGL((decode_wave_kernel<MODE, NT, FULL, COMPACT>), dim3(unsigned(d.B)), dim3(kWave),
                       size_t(kWave) * NT * sizeof(i32x2), d.stream, d.t, d.uni_base, d.asr, d.T, d.st, d.sb, d.lengths,
                       d.lambda, d.states, d.prev, d.labels, d.label_states);
    return hipGetLastError();
}

template <int MODE, int NT, bool FULL>
static hipError_t launch_wave(const Decode &d) {
    if constexpr (NT * kWave <= 1024)   // larger vocabularies have no compact rows
        if (d.t.dense_c) return launch_wave<MODE, NT, FULL, true>(d);
    return launch_wave<MODE, NT, FULL, false>(d);
}
template <int MODE, int NT>
static hipError_t launch_wave(const Decode &d) {
    return d.t.vocab_size == NT * kWave ? launch_wave<MODE, NT, true>(d) : launch_wave<MODE, NT, false>(d);
}

// Wavefronts and tokens per lane, from a sweep over vocabularies and batches
// (CTC, 100 frames; us a launch):
//  - V <= 512: one wavefront with 4 or 8 tokens a lane: no exchange at all.  128
//    tokens at 64 / 4000 utterances: 107 / 168 (two wavefronts: 133 / 335);
//    500 tokens: 116 / 231 with 8 a lane (two wavefronts with 4: 128 / 378).
//  - V <= 1024: four wavefronts up to 1024 utterances, one above (20M 6-gram):
//    204 against 277 at 512, 249 against 275 at 1024, 410 against 289 at 1500,
//    836 against 427 at 4096.  Two wavefronts (8 a lane) win only near 1500,
//    by 2 %.
//  - V <= 1280 (50 frames; "before": one wavefront per utterance above 512, rows
//    in LDS): eight wavefronts up to 768 utterances, two of 10 a lane up to 2048: 106
//    / 141 at V = 1100, 1024 / 1500 [four of 8: 129 / 211; before: 164 / 185]; one of 20
//    above: 176 / 189 at 2500 / 4096 [two of 10: 219 / 195; before: 336 / 248].
//  - V <= 1536: four of 6 above 768: 121 / 210 / 216 at V = 1300, 1024 / 2500 / 4096
//    [four of 8: 135 / 263 / 250; before: 194 / 332 / 249], but two of 12 at 1153 to
//    1536, which are all resident then (six a CU): 153 at 1500 [four of 6: 201; before:
//    210].
//  - V <= 2048: eight wavefronts while every utterance of the batch is resident
//    (156 against 181 for four at 64, 206 against 207 at 500, 100 frames), four above
//    (467 against 515 at 1200, 636 against 766 at 2500).  Four leave a nearly empty
//    second round at 1280 to 1536: one of 32 there, 204 / 152 at V = 2000, 1500
//    (CTC / transducer) [four: 218 / 153; before: 235 / 178].
//  - V <= 2560: eight of 8 up to 512 utterances, four of 10 above: 145 / 218 / 211 at
//    V = 2500, 700 / 1500 / 4096 (50 / 35 / 13 frames) [eight: 221 / 274 / 283; before:
//    264 / 384 / 282].
//  - V <= 4096: eight wavefronts of 8 a lane: 193 / 325 / 670 at 64 / 500 / 1200
//    (four of 16: 260 / 332 / 725; sixteen of 4: 189 / 402 / 831).
//  - above: sixteen of 8 a lane: 290 / 671 / 720 at 64 / 500 / 1200 (42 frames)
//    against 328 / 723 / 772 for eight of 16.
template <int MODE>
static hipError_t launch_mode(const Decode &d) {
    const int V = d.t.vocab_size;
    if (V <= 256) return launch_group<MODE, 1, 4>(d);
    if (V <= 512) return launch_group<MODE, 1, 8>(d);
    if (V <= 1024) {
        return d.B <= 1024 ? launch_group<MODE, 4, 4>(d) : launch_wave<MODE, 16>(d);
    }
    if (V <= 2048) {
        if (d.B <= 768) return launch_group<MODE, 8, 4>(d);
        if (V <= 1280) return d.B <= 2048 ? launch_group<MODE, 2, 10>(d) : launch_wave<MODE, 20>(d);
        if (V <= 1536) return d.B > 1152 && d.B <= 1536 ? launch_group<MODE, 2, 12>(d) : launch_group<MODE, 4, 6>(d);
        if (d.B > 1280 && d.B <= 1536) return launch_wave<MODE, 32>(d);
        return launch_group<MODE, 4, 8>(d);
    }
    if (V <= 2560 && d.B > 512) return launch_group<MODE, 4, 10>(d);
    if (V <= 4096) return launch_group<MODE, 8, 8>(d);
    return launch_group<MODE, 16, 8>(d);
}

hipError_t launch_fused_decode(const DevTrie &t, const float *asr, int64_t B, int64_t T, int64_t sb, int64_t st,
                               const int32_t *lengths, int mode, float lambda, int32_t *states, int32_t *prev,
                               int32_t *labels, int32_t *label_states, hipStream_t stream) {
    // Dense row of the state entered by emitting w: row 1 + w when every token
    // has a unigram (order-1 states are then numbered by token; <s>, if any,
    // comes last), else (-1) read from the empty context's row.
    const int n1 = (t.max_order > 2 ? t.first[2] : t.num_states) - 1;
    const int uni = t.max_order > 1 && n1 == t.vocab_size + (t.final_w ? 1 : 0) ? 1 : -1;
    const Decode d{t, uni, asr, B, T, sb, st, lengths, lambda, states, prev, labels, label_states, stream};
    switch (mode) {
        case kPlain: return launch_mode<kPlain>(d);
        case kCtc: return launch_mode<kCtc>(d);
        case kAed: return launch_mode<kAed>(d);
        default: return launch_mode<kTransducer>(d);
    }
}

}  // namespace ngpu
