// Device pieces shared by the fused kernels (step, whole decode, top-k).
//
// A hypothesis is held by a group of W wavefronts, one workgroup.  The tokens
// are dealt to the wavefronts in ranges of whole 64-token tiles, at most NT
// tiles each; lane l of a wavefront owns tokens 64 i + l of its range: their
// ASR scores and the dense row's entries sit in registers (one coalesced
// 256-byte load per tile).  Only the sparse levels go
// through LDS, one 8-byte slot {score, next state | kFinal} per token, all
// zero where no level holds the token; a wavefront writes and reads its own
// slots only, so the group needs no barrier for the walk.
//
// Loads go through buffer resources: lanes past the end of a row, a record or
// a level read 0 without a branch, so the compiler counts the loads in flight
// exactly and a wait for an early one leaves the later ones flying.  (Behind a
// per-lane branch, or after a load whose result some path never uses, it waits
// for every load of the wavefront: 256 utterances x 1000 frames took 2.25
// instead of 1.90 ms.)
#pragma once

#include "walk.h"

namespace ngpu {

enum { kPlain = 0, kCtc = 1, kTransducer = 2, kAed = 3 };

typedef int i32x2 __attribute__((ext_vector_type(2)));

// Largest vocabulary whose levels carry split counts at 256, 512 and 768.
constexpr int kSplitVocab = 1024;

// (readfirstlane: the compiler takes some of these pointers for lane-dependent
// and would put a loop over the lanes' values around every load)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t word_buffer(const void *p, int words) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint64_t u = (uint64_t(unsigned(__builtin_amdgcn_readfirstlane(int(a >> 32)))) << 32) |
                       unsigned(__builtin_amdgcn_readfirstlane(int(a)));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(u), short(0),
                                             __builtin_amdgcn_readfirstlane(words * 4), kBufferConfig);
}

// A zero that the compiler takes for a lane's own value: an address made with
// it is read by a vector load even where it is uniform (a scalar load would
// make later LDS waits wait for it too).
__device__ __forceinline__ int lane_zero() {
    int z = 0;
    asm volatile("" : "+v"(z));
    return z;
}

template <int NT>
struct Words {
    int v[NT];
    // words lane, lane + 64, ... of the n >= 0 words at p; 0 past them
    template <int CACHE = 0>
    __device__ __forceinline__ void load(const void *p, int n, int lane) {
        const __amdgpu_buffer_rsrc_t r = word_buffer(p, n);
        int at = lane * 4;
        asm volatile("" : "+v"(at));   // or the NT offsets are hoisted into registers of their own
#pragma unroll
        for (int i = 0; i < NT; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b32(r, at + kWave * i * 4, 0, CACHE);
    }
    __device__ __forceinline__ float f(int i) const { return __int_as_float(v[i]); }
    // words past the first n become x
    __device__ __forceinline__ void pad(int n, int lane, float x) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
            if (kWave * (i + 1) > n) v[i] = kWave * i + lane < n ? v[i] : __float_as_int(x);
    }
};

// Order-preserving key of x, -0 as +0 (value_key in four dependent steps).
__device__ __forceinline__ unsigned float_key(float x) {
    const int u = __float_as_int(x + 0.0f);
    return unsigned(u ^ ((u >> 31) | int(0x80000000u)));
}
constexpr unsigned kInfKey = 0x007fffffu;   // float_key(-inf)
// x, or -inf where x is NaN: a NaN score loses as under a strict '>' scan from
// -inf.  (Its key would lie above +inf's or, with the sign bit set, below
// -inf's, where a lane that holds no token would win against it.)
__device__ __forceinline__ float or_lowest(float x) { return __builtin_fmaxf(x, -__builtin_inff()); }

// The chain tables over the lanes: lane k holds the first state of order k
// (k >= 1, else a bound no state reaches), the address that record(s) = base +
// size * s starts from, and size = 16 max(k, 1), also the record's length.
struct RecordIndex {
    int first, size;
    uint64_t base;
};
__device__ __forceinline__ RecordIndex record_index(const DevTrie &t, int lane) {
    RecordIndex r{0x7fffffff, 16, 0};
#pragma unroll
    for (int j = 0; j < NGPU_LM_MAX_ORDER; ++j) {
        if (lane == j) {
            const int f = j == 0 ? 0 : t.first[j];
            r.first = j == 0 ? 0x7fffffff : f;
            r.size = 16 * (j > 0 ? j : 1);
            r.base = reinterpret_cast<uint64_t>(t.chain) + t.off_order[j] - uint64_t(r.size) * uint64_t(f);
        }
    }
    asm volatile("" ::"v"(r.first), "v"(r.size), "v"(r.base));
    return r;
}
// The chain record of the valid uniform state s: head in lane 0, level j - 1
// in lane j, zeros in the other lanes.
__device__ __forceinline__ int4 load_record(const RecordIndex &r, int s, int lane) {
    const int k = __builtin_popcountll(__ballot(s >= r.first));
    const unsigned size = unsigned(__builtin_amdgcn_readlane(r.size, k));
    const uint64_t base = (uint64_t(unsigned(__builtin_amdgcn_readlane(int(r.base >> 32), k))) << 32) |
                          unsigned(__builtin_amdgcn_readlane(int(unsigned(r.base)), k));
    const __amdgpu_buffer_rsrc_t b = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void *>(base + uint64_t(size) * unsigned(s)), short(0), int(size), kBufferConfig);
    return __builtin_bit_cast(int4, __builtin_amdgcn_raw_buffer_load_b128(b, lane * 16, 0, 0));
}

// Arcs [a0, a0 + n) of one order put into the slots of the tokens [t0, t0 +
// range) (FILTER: others may be among them), up to four 64-arc stripes per
// round trip.  The empty asm makes one wait for all the loads of a trip that
// the compiler sees; a load left pending on some path would make it wait for
// everything before the next load into those registers.
template <bool TOP, bool FILTER>
__device__ __forceinline__ void put_arcs(const DevTrie &t, int a0, int n, float acc, i32x2 *slots, int t0, int range,
                                         int lane) {
    auto put = [&](int place, int tok, int w, int next) {
        const int at = tok - t0;
        if (place < n && (!FILTER || unsigned(at) < unsigned(range))) {
            const i32x2 s = {__float_as_int(acc + __int_as_float(w)), next | kFinal};
            slots[at] = s;
        }
    };
    for (int c = 0; c < n; c += 4 * kWave) {
        int at8 = lane * 8, at12 = lane * 12;
        asm volatile("" : "+v"(at8), "+v"(at12));
        if (TOP) {
            const __amdgpu_buffer_rsrc_t r = word_buffer(t.top_arcs + (a0 - t.top_begin + c), 3 * (n - c));
            int x[4][3];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    x[u][q] = __builtin_amdgcn_raw_buffer_load_b32(r, at12 + kWave * 12 * u + 4 * q, 0, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u) asm volatile("" : "+v"(x[u][0]), "+v"(x[u][1]), "+v"(x[u][2]));
#pragma unroll
            for (int u = 0; u < 4; ++u) put(c + kWave * u + lane, x[u][0], x[u][1], x[u][2]);
        } else {
            const __amdgpu_buffer_rsrc_t r = word_buffer(t.arcs + (a0 + c), 2 * (n - c));
            if (n - c <= kWave) {
                i32x2 x = __builtin_bit_cast(i32x2, __builtin_amdgcn_raw_buffer_load_b64(r, at8, 0, 0));
                asm volatile("" : "+v"(x));
                put(c + lane, x.x, x.y, a0 + c + lane + t.to_delta);
            } else {
                i32x2 x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    x[u] = __builtin_bit_cast(i32x2,
                                              __builtin_amdgcn_raw_buffer_load_b64(r, at8 + kWave * 8 * u, 0, 0));
                asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    put(c + kWave * u + lane, x[u].x, x[u].y, a0 + c + kWave * u + lane + t.to_delta);
            }
        }
    }
}

// Meeting point of W <= 16 wavefronts: one entry each, two alternating
// buffers, so one barrier per exchange is enough (a buffer is written again
// only after every wavefront has passed the next exchange's barrier).
struct Meet {
    i32x4 a[2][16];
    int b[2][16];
};

// Waits until this wavefront's LDS writes are done, then for all wavefronts
// of the workgroup.  The memory clobber keeps the compiler from moving any
// memory access across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Maximum over W values that repeat every W lanes (W <= 16, a power of two).
template <int W>
__device__ __forceinline__ unsigned max_over_waves(unsigned x) {
    if (W >= 2) x = max(x, unsigned(__builtin_amdgcn_update_dpp(0, int(x), 0xB1, 0xf, 0xf, true)));    // lane ^ 1
    if (W >= 4) x = max(x, unsigned(__builtin_amdgcn_update_dpp(0, int(x), 0x4E, 0xf, 0xf, true)));    // lane ^ 2
    if (W >= 8) x = max(x, unsigned(__builtin_amdgcn_update_dpp(0, int(x), 0x141, 0xf, 0xf, true)));   // other half of 8
    if (W >= 16) x = max(x, unsigned(__builtin_amdgcn_update_dpp(0, int(x), 0x140, 0xf, 0xf, true)));  // other half of 16
    return x;
}

// The lane holding the wave's largest key, of several the one with the lowest
// token (tokens differ between lanes).
__device__ __forceinline__ int winner_lane(unsigned key, int tok) {
    const unsigned top = wave_max_u32(key);
    unsigned long long m = __ballot(key == top);
    if (m & (m - 1)) {
        const unsigned lo = wave_max_u32(key == top ? ~unsigned(tok) : 0u);
        m = __ballot(key == top && ~unsigned(tok) == lo);
    }
    return int(__builtin_ctzll(m));
}

// The same among W wavefronts' entries, entry l mod W in lane l.
template <int W>
__device__ __forceinline__ int winner_entry(unsigned key, int tok) {
    if (W == 1) return 0;
    const unsigned top = max_over_waves<W>(key);
    unsigned m = unsigned(__ballot(key == top)) & ((1u << W) - 1u);
    if (m & (m - 1)) {
        const unsigned lo = max_over_waves<W>(key == top ? ~unsigned(tok) : 0u);
        m = unsigned(__ballot(key == top && ~unsigned(tok) == lo)) & ((1u << W) - 1u);
    }
    return __builtin_ctz(m);
}

// A group's place and its tokens (dealt in tiles of TILE).
template <int W, int NT, bool FULL, int TILE = kWave>
struct Group {
    static constexpr int kRange = kWave * NT;
    static_assert(NT % 2 == 0, "slots are cleared two at a time");
    // each wavefront's range starts and ends at a multiple of 256: it loads only
    // its part of every level where the levels carry split counts
    static constexpr bool kSplit = W > 1 && W * kRange <= kSplitVocab && NT % 4 == 0;
    static constexpr bool kFilter = W > 1 && !kSplit;

    int wave, lane;
    int range;                 // tokens dealt to each wavefront but the last ones
    int t0, own;               // first token, tokens of this wavefront (none past V)
    i32x2 *slots;              // of this wavefront: slot of token t at t - t0
    int sh0, sh1;              // split counts below the range's two ends: shift
    unsigned mk0, mk1;         // and mask (0: none below the first, all below the last)

    __device__ __forceinline__ Group(int V, i32x2 *all_slots)
        : Group(V, W == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kWave)) {
        slots = all_slots + kRange * wave;
    }
    // wavefront `w` of a group (uniform); slots still to be set
    __device__ __forceinline__ Group(int V, int w) {
        wave = w;
        lane = threadIdx.x % kWave;
        // split counts fix the ranges' ends; otherwise every wavefront gets its share
        range = FULL || kSplit || W == 1 ? kRange : ((V + TILE - 1) / TILE + W - 1) / W * TILE;
        t0 = range * wave;
        own = min(max(V - t0, 0), range);
        const int q0 = wave * NT / 4, q1 = (wave + 1) * NT / 4;
        sh0 = q0 == 1 ? 0 : (q0 == 2 ? 9 : 19);
        sh1 = q1 == 1 ? 0 : (q1 == 2 ? 9 : 19);
        mk0 = q0 == 0 ? 0u : (q0 == 1 ? 0x1ffu : 0x3ffu);
        mk1 = q1 >= 4 ? 0u : (q1 == 1 ? 0x1ffu : 0x3ffu);
    }
    __device__ __forceinline__ int token(int i) const { return t0 + kWave * i + lane; }

    // this wavefront's ASR scores of a row; tokens past V lose against everything
    template <int CACHE = 0>
    __device__ __forceinline__ void load_row(const float *row, Words<NT> &x) const {
        x.template load<CACHE>(row + t0, own, lane);
    }
    __device__ __forceinline__ void mask_row(Words<NT> &x) const {
        if (!FULL) x.pad(own, lane, -__builtin_inff());
    }
    __device__ __forceinline__ void load_dense(const DevTrie &t, unsigned row, Words<NT> &dw, Words<NT> &dt) const {
        const uint64_t at = uint64_t(row * unsigned(t.vocab_size) + unsigned(t0)) * 4;   // rows x V < 2^27
        dw.load(reinterpret_cast<const char *>(t.dense_w) + at, own, lane);
        dt.load(reinterpret_cast<const char *>(t.dense_to) + at, own, lane);
    }
    __device__ __forceinline__ void clear_slots() const {
        const i32x4 z = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < NT / 2; ++i) reinterpret_cast<i32x4 *>(slots)[kWave * i + lane] = z;
    }
    // The record's sparse levels into the slots, order 2 first, so that the
    // highest order holding a token is the last to write it (LDS operations of
    // a wavefront complete in order; tokens within a level are distinct).
    // Returns whether any slot may have been written.
    // DEEP: first finds the levels that hold arcs of this wavefront, which pays
    // where chains are deep (uniform states of a 10-gram: 9.7 against 10.5 us for
    // 3001 queries) and costs where they are short (decode: 1.5 %).
    template <bool DEEP = false>
    __device__ __forceinline__ bool put_levels(const DevTrie &t, const int4 &rec, const ChainHead &h) const {
        const int nlev = h.nlev_group & 0xffff;
        const bool top = __builtin_amdgcn_readlane(rec.x, 1) >= t.top_begin;   // a level holds arcs of one order
        auto part = [&](unsigned splits, int n, int &lo) {   // of a level's n arcs
            lo = 0;
            if (kSplit) {
                lo = int((splits >> sh0) & mk0);
                n = (mk1 ? int((splits >> sh1) & mk1) : n) - lo;
            }
            return n;
        };
        auto put = [&](int j, int a0, int n) {
            const float acc = __int_as_float(__builtin_amdgcn_readlane(rec.z, j));
            if (j == 1 && top)
                put_arcs<true, kFilter>(t, a0, n, acc, slots, t0, own, lane);
            else
                put_arcs<false, kFilter>(t, a0, n, acc, slots, t0, own, lane);
        };
        bool any = false;
        if (DEEP) {
            int lo;   // lane j: level j - 1
            const int n = part(unsigned(rec.w), rec.y - rec.x, lo), a0 = rec.x + lo;
            unsigned todo = unsigned(__ballot(n > 0)) & ((2u << nlev) - 2u);   // lane 0 holds the head
            any = todo != 0;
            while (todo) {
                const int j = 31 - __builtin_clz(todo);
                todo &= ~(1u << j);
                put(j, __builtin_amdgcn_readlane(a0, j), __builtin_amdgcn_readlane(n, j));
            }
        } else {
            for (int j = nlev; j >= 1; --j) {
                int lo;
                const int a0 = __builtin_amdgcn_readlane(rec.x, j);
                const int n = part(unsigned(__builtin_amdgcn_readlane(rec.w, j)),
                                   __builtin_amdgcn_readlane(rec.y, j) - a0, lo);
                if (n == 0) continue;
                any = true;
                put(j, a0 + lo, n);
            }
        }
        return any;
    }
    // LM score and (flagged) next state of every token of the lane.
    __device__ __forceinline__ void lm_values(const ChainHead &h, const Words<NT> &dw, const Words<NT> &dt, bool any,
                                              float (&x)[NT], int (&nx)[NT]) const {
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            x[i] = (dt.v[i] < 0 ? h.acc0 : h.acc1) + dw.f(i);
            nx[i] = dt.v[i];
        }
        if (any) {   // uniform; else no sparse level holds a token of this wavefront
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const i32x2 s = slots[kWave * i + lane];
                x[i] = s.y != 0 ? __int_as_float(s.x) : x[i];
                nx[i] = s.y != 0 ? s.y : nx[i];
            }
        }
    }
    // The lane's largest value and its place 64 i; ties stay with the lowest token.
    // Never NaN, and above -inf only for a token below V.
    __device__ __forceinline__ void lane_best(const float (&x)[NT], float &bx, int &bi) const {
        bx = or_lowest(x[0]);
        bi = 0;
#pragma unroll
        for (int i = 1; i < NT; ++i) {
            const bool g = x[i] > bx;
            bx = g ? x[i] : bx;
            bi = g ? kWave * i : bi;
        }
    }
    // The wavefront's best class of an ASR row alone: key and token.
    __device__ __forceinline__ void raw_best(const Words<NT> &row, unsigned &key, int &tok) const {
        float x[NT], bx;
        int bi;
#pragma unroll
        for (int i = 0; i < NT; ++i) x[i] = row.f(i);
        lane_best(x, bx, bi);
        const unsigned k = float_key(bx);
        const int src = winner_lane(k, t0 + bi + lane);
        key = unsigned(__builtin_amdgcn_readlane(int(k), src));
        tok = __builtin_amdgcn_readlane(t0 + bi + lane, src);
    }
};

}  // namespace ngpu
