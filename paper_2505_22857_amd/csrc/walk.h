// Device pieces shared by every kernel: the chain records of a state, kernel
// arguments, waits and the wave maximum.
//
// The backoff walk of state s (Algorithm 1):
//   1. its chain record (head + one entry per state of order >= 2 on its
//      backoff chain) arrives in one vector load: lane 0 reads the head, lane
//      j the entry of level j - 1.  The record's address and length follow from
//      s alone (its order), so nothing waits on the head to fetch the levels.
//   2. the dense row of the order-1 ancestor (which already folds in the empty
//      context) gives every token a weight and a next state.
//   3. the sparse levels go on top, order 2 first and the query state's order
//      last, so the highest order that holds a token wins.  Arcs below the
//      highest order are 8-byte records {token, weight} whose next state is
//      their index plus a constant; those of the highest order carry it, in 12
//      bytes.  A wavefront that owns whole 256-token stripes of the row loads
//      only its part of a level (arcs are sorted by token and the levels carry
//      their counts below each stripe).
//   4. a token that no level holds scores acc + its dense weight, acc = acc0
//      where the dense entry is flagged as backed off to the empty context,
//      else acc1.
#pragma once

#include <hip/hip_runtime.h>

#include "trie.h"

namespace ngpu {

constexpr int kWave = 64;
constexpr int kStripe = 256;                   // tokens per split count of a level
constexpr int32_t kFinal = 0x40000000;         // next-state bit: slot written by a sparse level
constexpr int32_t kStateMask = 0x3fffffff;
static_assert(int64_t(kStateMask) + 1 == NGPU_LM_MAX_STATES, "state ids fit the bits below the flags");

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Word 3 of a raw (unformatted, unswizzled) buffer resource on gfx9-family
// chips: 32-bit data format; reads past the resource's byte range return 0.
constexpr int kBufferConfig = 0x00020000;

// Kernel arguments are otherwise loaded (scalar loads) where first used, each
// waited for before the next is issued; in a latency-bound launch that puts
// several scalar memory round trips before the first state load.  Passing
// them to empty asm statements at the kernel's start issues all their loads at
// once, with one wait; later reads reuse the values (kernel arguments are
// constant) or hit the scalar cache.  The asm statements count as memory
// accesses, so uniform loads from global memory after them are vector loads.
// Used by the kernels that serve one hypothesis a group and end (query, step,
// top-k), at every batch size: kernels with a loop over hypotheses or frames
// would hold the values in scalar registers throughout and spill.
template <class T>
__device__ __forceinline__ void load_arg(const T &v) {
    asm volatile("" ::"s"(v));
}
template <class... T>
__device__ __forceinline__ void load_args(const T &...v) {
    (load_arg(v), ...);
}

__device__ __forceinline__ void load_trie_args(const DevTrie &t) {
    load_args(t.chain, t.dense_w, t.dense_to, t.arcs, t.top_arcs, t.status, t.num_states, t.vocab_size, t.top_begin,
              t.to_delta);
    load_args(t.first[1], t.first[2], t.first[3], t.first[4], t.first[5], t.first[6], t.first[7], t.first[8],
              t.first[9]);
    load_args(t.off_order[0], t.off_order[1], t.off_order[2], t.off_order[3], t.off_order[4], t.off_order[5],
              t.off_order[6], t.off_order[7], t.off_order[8], t.off_order[9]);
    static_assert(NGPU_LM_MAX_ORDER == 10, "the chain tables above have NGPU_LM_MAX_ORDER entries");
}

__device__ __forceinline__ int chain_group(const ChainHead &h) { return h.nlev_group >> 16; }

__device__ __forceinline__ ChainHead head_of(const int4 &r) {
    ChainHead h;
    h.dense_row = __builtin_amdgcn_readlane(r.x, 0);
    h.acc1 = __int_as_float(__builtin_amdgcn_readlane(r.y, 0));
    h.acc0 = __int_as_float(__builtin_amdgcn_readlane(r.z, 0));
    h.nlev_group = __builtin_amdgcn_readlane(r.w, 0);
    return h;
}

// One step of the wave maximum: each lane takes the larger of its value and
// the value DPP control CTRL moves into it (lanes with no source, or outside
// ROW_MASK, see 0, which never wins since the values are unsigned).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned max_step(unsigned k) {
    const unsigned o = unsigned(__builtin_amdgcn_update_dpp(0, int(k), CTRL, ROW_MASK, 0xf, true));
    return o > k ? o : k;
}

// Wave-wide maximum of an unsigned value, uniform in every lane.  An inclusive
// scan within each row of 16 lanes (row_shr 1, 2, 4, 8), then row 15
// broadcast into rows 1 and 3 and row 31 into rows 2 and 3, leaves the
// maximum in lane 63.
__device__ __forceinline__ unsigned wave_max_u32(unsigned k) {
    k = max_step<0x111, 0xf>(k);
    k = max_step<0x112, 0xf>(k);
    k = max_step<0x114, 0xf>(k);
    k = max_step<0x118, 0xf>(k);
    k = max_step<0x142, 0xa>(k);
    k = max_step<0x143, 0xc>(k);
    return unsigned(__builtin_amdgcn_readlane(int(k), kWave - 1));
}

}  // namespace ngpu
