// Batched full-vocabulary backoff query (Algorithm 1, batched over hypotheses).
//
// One group of wavefronts per hypothesis (group.h), the dense row's entries in
// registers, the sparse levels through LDS slots; the finished rows leave with
// non-temporal stores (they are not read again here, so they should not
// displace the dense rows and arcs from the L2).  Where V and the outputs'
// alignment allow, a lane holds tokens 256 i + 4 l .. 4 l + 3, so that loads and
// stores are 16 bytes a lane and a wavefront's store instruction writes 1 KiB.
//
// Large batches at V = 1024 use an XCD-aware distribution (grouped kernel):
// workgroups are dispatched round-robin over the eight XCDs, so workgroup i
// serves dense-row group i % 8, and each XCD's L2 holds an eighth of the dense
// rows instead of all of them.  No MFMA: the work is gathers, scatters and one
// fp32 add per token.
#include <hip/hip_runtime.h>

#include <cmath>

#include "group.h"

namespace ngpu {

// Dense entries of a wavefront's range, four consecutive tokens a lane.
template <int NT>
struct Quads {
    f32x4 w[NT / 4];
    i32x4 to[NT / 4];
    template <class G>
    __device__ __forceinline__ void load(const DevTrie &t, const G &g, int row) {
        const uint64_t at = uint64_t(unsigned(row) * unsigned(t.vocab_size) + unsigned(g.t0)) * 4;   // rows x V < 2^27
        const __amdgpu_buffer_rsrc_t rw = word_buffer(reinterpret_cast<const char *>(t.dense_w) + at, g.own);
        const __amdgpu_buffer_rsrc_t rt = word_buffer(reinterpret_cast<const char *>(t.dense_to) + at, g.own);
        int off = g.lane * 16;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int i = 0; i < NT / 4; ++i) {
            w[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, off + 1024 * i, 0, 0));
            to[i] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rt, off + 1024 * i, 0, 0));
        }
    }
    // The finished rows of the range, where `any` slots were written taken from them.
    template <bool FULL, class G>
    __device__ __forceinline__ void store(const G &g, const ChainHead &h, bool any, float *orow, int32_t *nrow) const {
#pragma unroll
        for (int i = 0; i < NT / 4; ++i) {
            const int v = kStripe * i + 4 * g.lane;
            f32x4 x;
            i32x4 n = to[i];
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = (n[j] < 0 ? h.acc0 : h.acc1) + w[i][j];
            if (any) {
                const i32x4 a = *reinterpret_cast<const i32x4 *>(g.slots + v);
                const i32x4 c = *reinterpret_cast<const i32x4 *>(g.slots + v + 2);
                x[0] = a.y ? __int_as_float(a.x) : x[0];
                n[0] = a.y ? a.y : n[0];
                x[1] = a.w ? __int_as_float(a.z) : x[1];
                n[1] = a.w ? a.w : n[1];
                x[2] = c.y ? __int_as_float(c.x) : x[2];
                n[2] = c.y ? c.y : n[2];
                x[3] = c.w ? __int_as_float(c.z) : x[3];
                n[3] = c.w ? c.w : n[3];
            }
            n &= kStateMask;
            if (FULL || v < g.own) {   // own is a multiple of 4
                __builtin_nontemporal_store(x, reinterpret_cast<f32x4 *>(orow + v));
                __builtin_nontemporal_store(n, reinterpret_cast<i32x4 *>(nrow + v));
            }
        }
    }
};

// One group per hypothesis.  VEC: 16-byte loads and stores (V a multiple of 4,
// the outputs 16-byte aligned); else lane l holds tokens 64 i + l.
template <int W, int NT, bool FULL, bool VEC>
__global__ __launch_bounds__(W * kWave) void advance_kernel(DevTrie t, const int32_t *__restrict__ states,
                                                            float *__restrict__ scores, int32_t *__restrict__ next) {
    extern __shared__ i32x4 lds4[];
    load_trie_args(t);
    load_args(states, scores, next);
    const int V = t.vocab_size;
    const int64_t b = blockIdx.x;
    const Group<W, NT, FULL, VEC ? kStripe : kWave> g(V, reinterpret_cast<i32x2 *>(lds4));
    const int lane = g.lane;
    float *orow = scores + b * V + g.t0;
    int32_t *nrow = next + b * V + g.t0;
    const int s_l = states[b + lane_zero()];
    const RecordIndex ri = record_index(t, lane);
    g.clear_slots();
    const int s = __builtin_amdgcn_readfirstlane(s_l);
    if (s < 0 || s >= t.num_states) {
        if (g.wave == 0 && lane == 0) atomicAdd(&t.status[0], 1);
        for (int v = lane; v < g.own; v += kWave) {
            orow[v] = NAN;
            nrow[v] = -1;
        }
        return;
    }
    const int4 rec = load_record(ri, s, lane);
    const ChainHead h = head_of(rec);
    if constexpr (VEC) {
        Quads<NT> d;
        d.load(t, g, h.dense_row);
        const bool any = g.template put_levels<true>(t, rec, h);
        d.template store<FULL>(g, h, any, orow, nrow);
    } else {
        Words<NT> dw, dt;
        g.load_dense(t, unsigned(h.dense_row), dw, dt);
        const bool any = g.template put_levels<true>(t, rec, h);
        float x[NT];
        int n[NT];
        g.lm_values(h, dw, dt, any, x, n);
#pragma unroll
        for (int i = 0; i < NT; ++i)
            if (FULL || kWave * i + lane < g.own) {
                __builtin_nontemporal_store(x[i], orow + kWave * i + lane);
                __builtin_nontemporal_store(n[i] & kStateMask, nrow + kWave * i + lane);
            }
    }
}

// Chain head of state s (one per lane).
__device__ __forceinline__ ChainHead lane_head(const DevTrie &t, int s) {
    int k = 0, fk = 0;
    uint64_t off = t.off_order[0];
#pragma unroll
    for (int j = 1; j < NGPU_LM_MAX_ORDER; ++j) {
        if (s >= t.first[j]) {   // first[] ascends; entries past the last order equal S
            k = j;
            fk = t.first[j];
            off = t.off_order[j];
        }
    }
    return *reinterpret_cast<const ChainHead *>(t.chain + off + size_t(s - fk) * 16u * size_t(k > 0 ? k : 1));
}

// The XCD-grouped mapping, W independent wavefronts (one workgroup each) per
// hypothesis: each scans kGroups consecutive hypotheses (lane i loads the state
// and chain head of hypothesis i) and answers its range of the tokens of the ones
// whose dense row lies in its group; the W kGroups workgroups of a chunk together
// cover every hypothesis once.  The scan knows the dense row, so its loads go
// out before the record's.  One wavefront per workgroup: one that finds no
// hypothesis of its group frees its slot at once.
template <int W, int NT, bool FULL>
__global__ __launch_bounds__(kWave) void advance_grouped_kernel(DevTrie t, const int32_t *__restrict__ states,
                                                                int64_t B, float *__restrict__ scores,
                                                                int32_t *__restrict__ next) {
    extern __shared__ i32x4 lds4[];
    const int V = t.vocab_size;
    const int grp = int(blockIdx.x % kGroups);
    const int64_t base = int64_t(blockIdx.x / (W * kGroups)) * kGroups;
    Group<W, NT, FULL, kStripe> g(V, int((blockIdx.x / kGroups) % W));
    g.slots = reinterpret_cast<i32x2 *>(lds4);
    const int lane = g.lane;
    const RecordIndex ri = record_index(t, lane);
    int s_l = -1, dense_l = -1;
    bool mine = false;
    const int64_t bl = base + lane;
    if (lane < kGroups && bl < B) {
        s_l = states[bl];
        if (s_l < 0 || s_l >= t.num_states) {
            s_l = -1;
            mine = (bl % kGroups) == grp;   // an invalid state's row is written by one owner
        } else {
            const ChainHead hd = lane_head(t, s_l);
            mine = chain_group(hd) == grp;
            dense_l = hd.dense_row;
        }
    }
    // The scan's loads are complete here; otherwise the wait for them stays at
    // the head of the loop, where it would also drain the previous hypothesis's
    // stores before the next one's loads are issued.
    asm volatile("" : "+v"(s_l), "+v"(dense_l));
    uint64_t todo = __ballot(mine);
    while (todo) {
        const int i = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int64_t b = base + i;
        float *orow = scores + b * V + g.t0;
        int32_t *nrow = next + b * V + g.t0;
        const int s = __builtin_amdgcn_readlane(s_l, i);
        if (s < 0) {
            if (lane == 0 && g.wave == 0) atomicAdd(&t.status[0], 1);
            for (int v = lane; v < g.own; v += kWave) {
                orow[v] = NAN;
                nrow[v] = -1;
            }
            continue;
        }
        Quads<NT> d;
        d.load(t, g, __builtin_amdgcn_readlane(dense_l, i));
        const int4 rec = load_record(ri, s, lane);
        g.clear_slots();
        const ChainHead h = head_of(rec);
        const bool any = g.template put_levels<true>(t, rec, h);
        d.template store<FULL>(g, h, any, orow, nrow);
    }
}

// A grid holds at most 2^32 - 1 work-items: larger batches go in several launches.
template <int W, int NT>
static hipError_t launch(const DevTrie &t, const int32_t *states, int64_t B, float *scores, int32_t *next,
                         hipStream_t stream, bool vec) {
    constexpr int64_t kMost = int64_t(UINT32_MAX) / (W * kWave);
    const size_t lds = size_t(W) * kWave * NT * sizeof(i32x2);
    const dim3 block(W * kWave);
    const bool full = t.vocab_size == W * kWave * NT;
    for (int64_t b0 = 0; b0 < B; b0 += kMost) {
        const dim3 grid{unsigned(B - b0 < kMost ? B - b0 : kMost)};
        float *sc = scores + b0 * t.vocab_size;
        int32_t *nx = next + b0 * t.vocab_size;
        if (vec && full)
            hipLaunchKernelGGL((advance_kernel<W, NT, true, true>), grid, block, lds, stream, t, states + b0, sc, nx);
        else if (vec)
            hipLaunchKernelGGL((advance_kernel<W, NT, false, true>), grid, block, lds, stream, t, states + b0, sc, nx);
        else
            hipLaunchKernelGGL((advance_kernel<W, NT, false, false>), grid, block, lds, stream, t, states + b0, sc, nx);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

// W wavefronts per hypothesis in the grouped mapping, while its dispatch size in
// work-items fits: whether it was launched.
template <int W, int NT>
static bool launch_grouped(const DevTrie &t, const int32_t *states, int64_t B, float *scores, int32_t *next,
                           hipStream_t stream) {
    const int64_t groups = W * ((B + kGroups - 1) / kGroups) * kGroups;
    if (groups * kWave > int64_t(UINT32_MAX)) return false;
    const dim3 grid{unsigned(groups)}, block{kWave};
    const size_t lds = size_t(kWave) * NT * sizeof(i32x2);
    if (t.vocab_size == W * kWave * NT)
        hipLaunchKernelGGL((advance_grouped_kernel<W, NT, true>), grid, block, lds, stream, t, states, B, scores, next);
    else
        hipLaunchKernelGGL((advance_grouped_kernel<W, NT, false>), grid, block, lds, stream, t, states, B, scores,
                           next);
    return true;
}

// Launch shapes, us a call from sweeps over vocabularies and 1 to 65536 hypotheses
// (6-grams of 1M n-grams, V = 1024 the 20M 6-gram; from V = 513 on also 4-grams of
// 120 V n-grams; "before": one wavefront per hypothesis with its row in LDS above 1024
// hypotheses, four below, grouped from 20480 on).  Two things decide beside the
// number of wavefronts: whether each has whole 256-token stripes to do (three, five
// and six are as good as powers of two), and, for large batches, whether rows are
// whole 128-byte lines (V % 32 == 0): else stores of a line that two wavefronts share
// must come close together.
//  - V <= 256: one wavefront of 4 tokens a lane: 28.5 at V = 128, 60000 [two of 2:
//    56; before: 48].
//  - V <= 512: two of 4 up to 1024 hypotheses, 4.0 at V = 400, 600; one of 8 above,
//    6.0 / 33.6 at 5000 / 60000 [two of 4: 8.1 / 53; before: 6.9 / 54].
//  - V <= 768: three of 4 up to 768 hypotheses, one of 12 above: 5.0 / 5.8 at V = 600,
//    1500 / 3000 [two of 8: 5.1 / 6.1; before: 4.9 / 6.0].  Whole lines: one of 12 up to
//    8192, and always up to V = 640, 7.1 / 11.3 / 42 at V = 544, 6000 / 12000 / 60000 [two
//    of 8: 7.9 / 11.9 / 47; before: 7.1 / 11.1 / 53]; else two of 8, 14.0 / 59 at V = 768,
//    12000 / 60000 [one: 15.1 / 65].  Other rows: two of 8 from 4096, 8.8 at V = 600,
//    6000 [one: 9.0; three: 9.5], three of 4 from 8192, 15.3 / 62 at 12000 / 60000 [four
//    of 4: 18.3 / 77; before: 15.6 / 77].  Without 16-byte stores four of 4 from 4096
//    on above V = 640, 90 at V = 701, 65536 [three: 112].
//  - V <= 1024, whole lines: four of 4 up to 768 hypotheses, 4.3 at 512 [two of 8:
//    4.7; before: 4.5]; two of 8 above, 5.75 / 9.3 / 21.6 at 1500 / 4000 / 10000 [6.2 /
//    11.3 / 22.6; before: 7.3 / 10.8 / 23.1]; at V = 1024 grouped from 20480 on, 40.6 /
//    103 at 22000 / 65536 [two of 8: 43 / 123].  V = 800, 60000: two of 8 72 [four of
//    4: 97; before, grouped: 88].
//  - V <= 1024, other rows: four of 4: 8.5 / 57.5 at V = 999, 3000 / 30000 [two of 8:
//    9.0 / 76; before: 11.7 / 91]; 97.5 at V = 1000, 60000 [120; before: 116].  With
//    16-byte stores two of 8 win at a few thousand: 5.9 at V = 1000, 2000 [6.7].
//  - V <= 1536: five of 4 up to V = 1280 and 512 hypotheses, six of 4 above it up to 128,
//    3.45 / 3.6 at V = 1280 / 1504, 64 [four of 8: 3.7 / 3.8; before: 3.6 / 3.7]; three of 8
//    up to 2048, 4.6 / 5.8 at V = 1504, 700 / 1500 [four of 8: 4.7 / 6.4; before: 4.6 /
//    6.2], for whole lines up to V = 1280 always, 7.5 / 20.4 / 87 at V = 1056, 3000 / 12000
//    / 60000 [four of 8: 8.5 / 23.5 / 101; before: 7.9 / 22.1 / 95]; else four of 8, 39 /
//    110 at V = 1100, 20480 / 60000 [three: 48 / 130; before: 53 / 140].  Above V = 1280
//    from 20480 on: whole lines grouped, three of 8, 41 / 114 at V = 1408 [four of 8: 44 /
//    122; before: 48 / 127]; other rows four of 12 (fewer workgroups at once, whose
//    stores of shared lines come closer), 50 / 151 at V = 1300, 20480 / 65536 [four of
//    8: 54 / 181; before: 60 / 175].
//  - V <= 2048: four of 8: 11.5 at V = 2048, 3000 [eight of 4: 14.9; before: 14.6]; from
//    20480 on grouped: whole lines four of 8, 60 / 186 at V = 2048, 20480 / 65536 [plain:
//    70 / 217; before: 64 / 195], other rows four of 12, 66 / 204 at V = 1800 [plain: 73 /
//    235; of 8: 71 / 223; before: 74 / 222].
//  - V <= 3072: up to V = 2304 three of 12 up to 4096 hypotheses (1024 without 16-byte stores), 4.7 / 7.7 at V = 2304,
//    300 / 1500 [eight of 8: 5.5 / 9.1; before: 5.0 / 8.6]; above it four of 12 up to 1024,
//    5.3 at V = 2500, 512 [eight of 8: 5.7; before: 5.2]; from 20480 on grouped: whole
//    lines four of 12, 67 / 101 at V = 2304, 20480 / 32768 [plain: 79 / 123; before: 71 /
//    113], other rows eight of 8, 105 / 164 at V = 3000 [plain: 116 / 191; before: 119 /
//    186].
//  - V <= 4096: eight of 8: 18.4 at V = 3000, 3000 [sixteen of 4: 28; before: 22.3];
//    grouped from 20480 on, 128 / 202 at V = 4096, 20480 / 32768 [plain: 154 / 246;
//    before: 138 / 215].
//  - above: eight of 16: 4.7 / 7.6 / 45 at V = 8000, 8 / 300 / 3000 [sixteen of 8:
//    5.1 / 9.3 / 46; before: 6.2 / 8.1 / 73]; grouped from 20480 on, 202 at V = 6000,
//    20480 [plain: 251; before: 226].
constexpr int64_t kGroupedMinBatch = 20480;

hipError_t launch_advance(const DevTrie &t, const int32_t *states, int64_t B, float *scores, int32_t *next,
                          hipStream_t stream) {
    const int V = t.vocab_size;
    const bool vec = V % 4 == 0 && reinterpret_cast<uintptr_t>(scores) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(next) % 16 == 0;
    const bool lines = V % 32 == 0;   // rows of whole 128-byte lines
    const bool large = B >= kGroupedMinBatch;
#define NGPU_ADVANCE(W, NT) return launch<W, NT>(t, states, B, scores, next, stream, vec)
#define NGPU_GROUPED(W, NT)                                                                                 \
    do {                                                                                                    \
        if (vec && large && launch_grouped<W, NT>(t, states, B, scores, next, stream)) return hipGetLastError(); \
    } while (0)
    if (V <= 256) NGPU_ADVANCE(1, 4);
    if (V <= 512) {
        if (B <= 1024) NGPU_ADVANCE(2, 4);
        NGPU_ADVANCE(1, 8);
    }
    if (V <= 768) {
        if (B > 768 && (B <= 4096 || (lines && (V <= 640 || B <= 8192)))) NGPU_ADVANCE(1, 12);
        if (!vec && V > 640 && B > 4096) NGPU_ADVANCE(4, 4);
        if (B > 768 && (B <= 8192 || lines)) NGPU_ADVANCE(2, 8);
        NGPU_ADVANCE(3, 4);
    }
    if (V <= 1024) {
        if (V == 1024) NGPU_GROUPED(2, 8);
        if (B > 768 && (lines || (vec && B <= 6144))) NGPU_ADVANCE(2, 8);
        NGPU_ADVANCE(4, 4);
    }
    if (V <= 1280) {
        if (B <= 512) NGPU_ADVANCE(5, 4);
        if (B <= 2048 || lines) NGPU_ADVANCE(3, 8);
        NGPU_ADVANCE(4, 8);
    }
    if (V <= 1536) {
        if (B <= 128) NGPU_ADVANCE(6, 4);
        if (B <= 2048) NGPU_ADVANCE(3, 8);
        if (lines) NGPU_GROUPED(3, 8);
        if (!lines && large) NGPU_ADVANCE(4, 12);
        NGPU_ADVANCE(4, 8);
    }
    if (V <= 2048) {
        if (lines) NGPU_GROUPED(4, 8);
        NGPU_GROUPED(4, 12);
        NGPU_ADVANCE(4, 8);
    }
    if (V <= 3072) {
        if (V <= 2304 && B <= (vec ? 4096 : 1024)) NGPU_ADVANCE(3, 12);
        if (B <= 1024) NGPU_ADVANCE(4, 12);
        if (lines) NGPU_GROUPED(4, 12);
    }
    if (V <= 4096) {
        NGPU_GROUPED(8, 8);
        NGPU_ADVANCE(8, 8);
    }
    NGPU_GROUPED(8, 16);
    NGPU_ADVANCE(8, 16);
#undef NGPU_ADVANCE
#undef NGPU_GROUPED
}

}  // namespace ngpu
