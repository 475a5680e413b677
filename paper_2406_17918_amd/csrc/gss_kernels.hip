// HIP kernels of the cache-backed multi-hop neighbor sampler, written for gfx950 (CDNA4, wave64).
//
// Kernel map:
//   fill_full_kernel   StaticSample / Initialize (Alg. 1, Alg. 2) and FCR CacheRefresh (Alg. 3):
//                      one half-wavefront per cache row, all per-layer tables of a relation in one pass.
//   step_tick_kernel   one launch carries one phase of every step in flight that is ready for it
//                      (the slices own consecutive ranges of a one-dimensional grid).  The phases of a hop:
//     sample  per frontier node (one half-wavefront): read the cached row, partial refresh (Alg. 2
//             RefreshCache / OTF-Partial / shared rho-refresh), draw the fanout (SampleFromCache),
//             write the picks and insert them into the dedupe table;
//     mark    per pick: look up the table, flag first occurrences, ranks and totals per tile, offsets, counts;
//     emit    per pick: local ids, COO in (dst-major, slot-minor) order, new src_nodes;
//     settle  mark and emit in one launch, for steps that have the launches to themselves.
//
// Nothing here is a dense contraction, so no MFMA: the work is row reads, keyed integer hashing
// (Philox4x32-10), group-level ranking through LDS broadcasts and ballots, and atomics on the dedupe table.
#include <hip/hip_ext.h>

#include <cstring>
#include <type_traits>

#include "gss_device.h"

namespace gss {

// ------------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11).  One block = four 32-bit words.
//   draw   x64 = (w1 << 32) | w0
//   the two per-slot draws of a visited node share one block (purpose word 2):
//   EVICT reads words (0,1), PICK reads words (2,3).
//   priority(index) = x64 with its low 16 bits replaced by the index (no ties).
// ------------------------------------------------------------------------------------------
struct Block4 { uint32_t w0, w1, w2, w3; };

// a ^ b ^ c in one instruction (the three-input bitwise op of gfx950; 0x96 is the truth table of the three-way xor):
// written out, the compiler emits two xors per word and round, a quarter of a block's vector instructions
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ Block4 philox4x32_10(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1,
                                                uint32_t c2, uint32_t c3) {
  asm("" : "+s"(k0), "+s"(k1));
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;   // one 32x32->64 multiply gives hi and lo
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    c0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    c1 = (uint32_t)p1;
    c2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return Block4{c0, c1, c2, c3};
}

struct DrawKey {
  uint32_t k0, k1;     // rng_seed lo / hi
  uint32_t node;       // counter word 0
  uint32_t step;       // counter word 2
  uint32_t tag;        // layer << 8 | relation << 16 (the purpose is OR-ed in per draw)
};
__device__ __forceinline__ Block4 draw_block(const DrawKey& K, uint32_t purpose, uint32_t index, uint32_t attempt) {
  return philox4x32_10(K.k0, K.k1, K.node, index | (attempt << 16), K.step, K.tag | purpose);
}
__device__ __forceinline__ uint64_t lo64(const Block4& b) { return ((uint64_t)b.w1 << 32) | b.w0; }
__device__ __forceinline__ uint64_t hi64(const Block4& b) { return ((uint64_t)b.w3 << 32) | b.w2; }
__device__ __forceinline__ uint64_t priority(uint64_t x64, uint32_t index) { return (x64 & ~0xFFFFull) | index; }
// floor(x64 * m / 2^64) for m < 2^32
__device__ __forceinline__ uint32_t below(uint64_t x64, uint32_t m) {
  const uint64_t t = (uint64_t)(uint32_t)x64 * m;
  const uint64_t u = (x64 >> 32) * m + (t >> 32);
  return (uint32_t)(u >> 32);
}
constexpr int ITEMS_PER_THREAD = TILE / TILE_THREADS;   // consecutive pick slots a thread of a tile phase owns
constexpr uint64_t PRIO_NONE = ~0ull;   // larger than every real priority (their low 16 bits are < 64)

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }
struct Wg { int x, y; };   // position of the workgroup within its slice's grid

__device__ __forceinline__ int64_t load_indptr(const void* indptr, int is64, int64_t v) {
  return is64 ? ((const int64_t*)indptr)[v] : (int64_t)((const int32_t*)indptr)[v];
}

// ------------------------------------------------------------------------------------------
// Groups of W lanes.  A cache row of k <= 32 slots occupies half a wavefront (W = 32), and a
// wavefront works on two nodes at once (every Philox block and every compare is shared by both);
// rows of 33 .. 64 slots take the whole wavefront (W = 64).
// Lanes of a group talk through a small LDS scratch: a lane writes its item, every lane then reads
// item i at the same address (an LDS broadcast), which replaces per-iteration cross-lane moves.
// LDS operations of one wavefront execute in order, so no barrier is needed inside a group; the
// accesses are volatile to keep the compiler from reordering them.
// ------------------------------------------------------------------------------------------
template <int W>
struct GroupLdsT {
  uint64_t prio[2 * W];  // priorities by slot, or by adjacency position in the k < deg < 2k regime
  uint64_t ab[2 * W];    // lo: value fixed in the slot (or -1); hi: this round's candidate (or -2)
  int32_t out[2 * W];    // values compacted in position order
};
template <int W> using MaskT = typename std::conditional<W == 64, uint64_t, uint32_t>::type;   // one bit per lane of a group
__device__ __forceinline__ int mask_popc(uint32_t m) { return __popc(m); }
__device__ __forceinline__ int mask_popc(uint64_t m) { return __popcll((unsigned long long)m); }
__device__ __forceinline__ int mask_ffs(uint32_t m) { return __ffs((int)m); }
__device__ __forceinline__ int mask_ffs(uint64_t m) { return __ffsll((unsigned long long)m); }
template <int W>
struct GrpT {
  static constexpr int WIDTH = W;
  static constexpr int PER_WAVE = 64 / W;               // groups of a wavefront (W = 21: three, and lane 63 has no group)
  static constexpr int PER_WG = (TILE_THREADS / 64) * PER_WAVE;   // groups of a workgroup
  static constexpr bool POW2 = (W & (W - 1)) == 0;
  static constexpr int LOG2_WIDTH = W == 64 ? 6 : (W == 32 ? 5 : (W == 16 ? 4 : (W == 8 ? 3 : 0)));
  using Mask = MaskT<W>;
  // LDS address space made explicit: volatile accesses through a generic pointer would be emitted as
  // flat memory instructions instead of ds_read / ds_write.
  typedef __attribute__((address_space(3))) volatile GroupLdsT<W>* LdsPtr;
  int sub;                 // lane within the group
  int half;                // group within the wavefront
  bool idle;               // a lane beyond the wavefront's last group (only when W does not divide 64): it takes no part
  int ahead;               // see set_redraws: attempt << 8 | number of the pending slot that the lane draws for
  int redraws;
  LdsPtr L;
  // The visits of a phase redraw n slots each (a constant of the launch).  Lane (attempt a, pending slot q) = a * n + q.
  __device__ __forceinline__ void set_redraws(int n) {
    redraws = n > 0 ? n : 1;
    const int a = sub / redraws;
    ahead = (a << 8) | (sub - a * redraws);
  }
  __device__ __forceinline__ void init(GroupLdsT<W>* lds) {        // `lds`: one scratch per group of the workgroup
    if constexpr (W == 32 || W == 64) {
      sub = (int)(threadIdx.x & (unsigned)(W - 1));
      half = W == 32 ? (int)((threadIdx.x >> 5) & 1u) : 0;
      idle = false;
      L = (LdsPtr)&lds[threadIdx.x / (unsigned)W];
    } else {
      const int lane = (int)(threadIdx.x & 63u);
      half = lane / W;
      idle = half >= PER_WAVE;
      if (idle) half = PER_WAVE - 1;
      sub = lane - half * W;
      L = (LdsPtr)&lds[(int)(threadIdx.x >> 6) * PER_WAVE + half];
    }
  }
  __device__ __forceinline__ int index_in_workgroup() const { return (int)(threadIdx.x >> 6) * PER_WAVE + half; }
  __device__ __forceinline__ Mask below() const { return ((Mask)1 << sub) - (Mask)1; }          // the lanes before this one
  __device__ __forceinline__ bool in(Mask m) const { return ((m >> sub) & (Mask)1) != 0; }       // is this lane's bit set
  __device__ __forceinline__ static Mask all() { return (W == 64 || W == 32) ? ~(Mask)0 : (Mask)(((Mask)1 << (W & 31)) - (Mask)1); }
  // the lanes of the wavefront that come after lane i of their group
  __device__ __forceinline__ static uint64_t wave_lanes_after(int i) {
    const uint64_t one = (uint64_t)all() & ~(((uint64_t)2 << i) - 1ull);
    if constexpr (W == 64) return one;
    uint64_t m = 0ull;
#pragma unroll
    for (int q = 0; q < PER_WAVE; ++q) m |= one << (q * W);
    return m;
  }
  __device__ __forceinline__ static Mask first(int n) { return n >= W ? all() : (((Mask)1 << n) - (Mask)1); }
};
using GroupLds = GroupLdsT<32>;
using Grp = GrpT<32>;
using GroupLdsPtr = Grp::LdsPtr;
template <int W>
__device__ __forceinline__ MaskT<W> grp_ballot(const GrpT<W>& G, bool pred) {
  const uint64_t b = __ballot(pred);
  if constexpr (W == 64) return b;
  else if constexpr (W == 32) return G.half ? (uint32_t)(b >> 32) : (uint32_t)b;
  else return (uint32_t)(b >> (G.half * W)) & GrpT<W>::all();
}
__device__ __forceinline__ uint32_t below_mask(int sub) { return (1u << sub) - 1u; }

// number of the n priorities in LDS smaller than p (all priorities are distinct)
template <int W>
__device__ __forceinline__ int grp_rank(const GrpT<W>& G, int n, uint64_t p) {
  int r = 0;
#pragma unroll 4
  for (int i = 0; i < n; ++i) r += (G.L->prio[i] < p) ? 1 : 0;
  return r;
}
// The same over the first n entries with n the same in every lane of the wavefront (a slot count of the launch, not of
// the node): the loop counter stays in scalar registers and four entries are compared per round.  Entries from n up to the
// next multiple of four must hold PRIO_NONE (every lane of a group stores its slot's priority, PRIO_NONE beyond the row).
template <int W>
__device__ __forceinline__ int grp_rank_uniform(const GrpT<W>& G, int n, uint64_t p) {
  const int n4 = (__builtin_amdgcn_readfirstlane(n) + 3) & ~3;
  int r = 0;
  for (int i = 0; i < n4; i += 4) {
    const uint64_t q0 = G.L->prio[i], q1 = G.L->prio[i + 1], q2 = G.L->prio[i + 2], q3 = G.L->prio[i + 3];
    r += (q0 < p) ? 1 : 0;          // (one compare and one add-with-carry each)
    r += (q1 < p) ? 1 : 0;
    r += (q2 < p) ? 1 : 0;
    r += (q3 < p) ? 1 : 0;
  }
  return r;
}
template <int W>
__device__ __forceinline__ void grp_rank2(const GrpT<W>& G, int n, uint64_t p0, uint64_t p1, int& r0, int& r1) {
  r0 = 0; r1 = 0;
#pragma unroll 4
  for (int i = 0; i < n; ++i) {
    const uint64_t q = G.L->prio[i];
    r0 += (q < p0) ? 1 : 0;
    r1 += (q < p1) ? 1 : 0;
  }
}

// Takes the proposals of n pending slots in order, attempt by attempt and slot by slot: lane `i * stride + q` holds the
// proposal `cand` of attempt i < drawn for pending slot number q, which is slot `slot` of the row.  A slot is fixed to its first
// proposal that no fixed slot holds.
template <int W>
__device__ __forceinline__ void take_in_order(const GrpT<W>& G, int cand, int slot, int n, int stride, int drawn, MaskT<W>& fixed, int& val) {
  using Mask = MaskT<W>;
  G.L->ab[G.sub] = (uint64_t)(uint32_t)cand | ((uint64_t)(uint32_t)slot << 32);
  Mask open = GrpT<W>::first(n);                                          // pending, by number
  for (int i = 0; i < drawn && open != 0; ++i)
    for (Mask m = open; m != 0; m &= m - (Mask)1) {                       // (the same in all lanes of the group)
      const int q = mask_ffs(m) - 1;
      const uint64_t e = G.L->ab[i * stride + q];
      const int c = (int)(uint32_t)e, j = (int)(uint32_t)(e >> 32);
      if (grp_ballot(G, G.in(fixed) && val == c) == (Mask)0) {
        if (G.sub == j) val = c;
        fixed |= (Mask)1 << j;
        open &= ~((Mask)1 << q);
      }
    }
}

// Round-major rejection fill.  Slots of `pend` need an id, slots of `fixed` hold one in `val`.
// In round a every pending slot j draws pos = below(deg; index=j, attempt=a) and proposes
// adj[pos]; it is accepted unless the id is already in the row or proposed by a lower pending slot
// in the same round (which is what slot-ascending sequential processing of a round yields).
// FEW: few slots are pending (a partial refresh): instead of every lane scanning all k slots, the
// group walks over the pending slots, and every lane compares its own id with that slot's proposal.  The n_new pending
// slots of a visit leave lanes over, which draw the slots' next attempts in the same block (set_redraws): a second round
// is then a walk over LDS instead of another Philox block and another trip to the adjacency (with n_new = 4 and 32 lanes
// half of the wavefronts needed one or more).  Up to four attempts where a repeat is likely and the adjacency is a few
// cache lines (deg < 8 k), two up to deg < 32 k; the neighbors of a hub lie in a line each, and there one attempt nearly
// always does.
// The fill of a whole row (FEW = false: every slot pending) does the same from its second round on.
template <bool FEW, int W>
__device__ __forceinline__ int grp_rejection_fill(const GrpT<W>& G, MaskT<W> pend, MaskT<W> fixed, int val, int k,
                                                  const int32_t* __restrict__ adj, uint32_t deg,
                                                  const DrawKey& K, uint32_t purpose, int32_t* state) {
  constexpr int GRP = W;
  if constexpr (FEW) {
    const int most = deg < 8u * (uint32_t)k ? 4 : (deg < 32u * (uint32_t)k ? 2 : 1);
    const int drawn = min(most, GRP / G.redraws);                         // attempts at once: every pending slot has a lane for each
    for (uint32_t a = 0; pend != 0; a += (uint32_t)drawn) {
      if (a >= 65536u - 4u) {   // acceptance probability is > 1/2 per draw: unreachable for a simple graph
        if (G.sub == 0) atomicOr(&state[ST_ERROR], ERR_REJECT_OVERFLOW);
        break;
      }
      if (G.in(pend)) G.L->out[mask_popc(pend & G.below())] = G.sub;
      const int n = mask_popc(pend), my_a = G.ahead >> 8, my_q = G.ahead & 0xFF;
      const int slot = G.L->out[my_q];
      int cand = -3;
      if (my_a < drawn && my_q < n) cand = adj[below(lo64(draw_block(K, purpose, (uint32_t)slot, a + (uint32_t)my_a)), deg)];
      take_in_order(G, cand, slot, n, G.redraws, drawn, fixed, val);
      pend &= ~fixed;
    }
    return val;
  }
  // A whole row (nothing is fixed yet).  First round: a slot only has to differ from the lower slots' proposals, and the
  // comparisons are collected as wavefront masks (one vector instruction per slot).
  const bool in_row = G.sub < k;
  int cand = in_row ? adj[below(lo64(draw_block(K, purpose, (uint32_t)G.sub, 0)), deg)] : -3;
  G.L->out[G.sub] = cand;
  uint64_t taken = 0ull;
#pragma unroll 4
  for (int i = 0; i < k; ++i) taken |= __ballot(G.L->out[i] == cand) & GrpT<W>::wave_lanes_after(i);
  const bool acc = in_row && !((taken >> lane_id()) & 1ull);
  if (acc) val = cand;
  fixed = grp_ballot(G, acc);
  pend &= ~fixed;
  for (uint32_t a = 1; pend != 0;) {
    if (a >= 65536u - (uint32_t)GRP) {   // acceptance probability is > 1/2 per draw: unreachable for a simple graph
      if (G.sub == 0) atomicOr(&state[ST_ERROR], ERR_REJECT_OVERFLOW);
      break;
    }
    // The slots left are few: a round would run the whole Philox block and a trip to the adjacency for a handful of lanes.
    // Instead the lanes draw the slots' next GRP / n attempts at once (lane = attempt * n + number of the pending slot; a
    // proposal is a pure function of slot and attempt), which are then taken in order from LDS.
    const int n = mask_popc(pend);
    if (G.in(pend)) G.L->out[mask_popc(pend & G.below())] = G.sub;
    const float inv = __builtin_amdgcn_rcpf((float)n);                    // (sub + 1/2) / n is never near a whole number
    const int my_a = (int)(((float)G.sub + 0.5f) * inv), my_q = G.sub - my_a * n, drawn = (int)(((float)GRP + 0.5f) * inv);
    const int slot = G.L->out[my_q];
    cand = -3;
    if (my_a < drawn) cand = adj[below(lo64(draw_block(K, purpose, (uint32_t)slot, a + (uint32_t)my_a)), deg)];
    take_in_order(G, cand, slot, n, n, drawn, fixed, val);
    pend &= ~fixed;
    a += (uint32_t)drawn;
  }
  return val;
}

// k < deg < 2k <= 2 W: the group owns adjacency positions sub and sub + W.  The `want` eligible
// positions of smallest priority are written to L->out[0..want) in ascending position order.
template <int W>
__device__ __forceinline__ void grp_select_positions(const GrpT<W>& G, int d, int want, bool elig0, bool elig1,
                                                     int a0, int a1, const DrawKey& K, uint32_t purpose) {
  const int p0 = G.sub, p1 = G.sub + W;
  uint64_t q0 = PRIO_NONE, q1 = PRIO_NONE;
  if (elig0) q0 = priority(lo64(draw_block(K, purpose, (uint32_t)p0, 0)), (uint32_t)p0);
  if (elig1) q1 = priority(lo64(draw_block(K, purpose, (uint32_t)p1, 0)), (uint32_t)p1);
  G.L->prio[p0] = q0;
  G.L->prio[p1] = q1;
  int r0, r1;
  grp_rank2(G, d, q0, q1, r0, r1);
  const bool s0 = elig0 && r0 < want, s1 = elig1 && r1 < want;
  const MaskT<W> m0 = grp_ballot(G, s0), m1 = grp_ballot(G, s1);
  if (s0) G.L->out[mask_popc(m0 & G.below())] = a0;
  if (s1) G.L->out[mask_popc(m0) + mask_popc(m1 & G.below())] = a1;
}

// The same where the ids of some slots are excluded (retained: lanes of `kept`, id in `val`): of the d positions at most
// `want` more than k are eligible, so they usually fit the group's lanes when they are moved together: one Philox block and
// one rank among the eligible ones instead of two blocks and two ranks among d.
template <int W>
__device__ __forceinline__ void grp_redraw_positions(const GrpT<W>& G, int d, int want, int k, MaskT<W> kept, int val,
                                                     const int32_t* __restrict__ adj, const DrawKey& K, uint32_t purpose) {
  bool e0 = G.sub < d, e1 = G.sub + W < d;
  const int a0 = e0 ? adj[G.sub] : -1, a1 = e1 ? adj[G.sub + W] : -1;
  if (G.sub < k) G.L->out[G.sub] = G.in(kept) ? val : -1;
#pragma unroll 4
  for (int j = 0; j < k; ++j) {
    const int rv = G.L->out[j];
    e0 &= (rv != a0);
    e1 &= (rv != a1);
  }
  const MaskT<W> m0 = grp_ballot(G, e0), m1 = grp_ballot(G, e1);
  const int n0 = mask_popc(m0), n = n0 + mask_popc(m1);
  if (n > W) {
    grp_select_positions(G, d, want, e0, e1, a0, a1, K, purpose);
    return;
  }
  if (e0) G.L->ab[mask_popc(m0 & G.below())] = (uint64_t)(uint32_t)a0 | ((uint64_t)(uint32_t)G.sub << 32);
  if (e1) G.L->ab[n0 + mask_popc(m1 & G.below())] = (uint64_t)(uint32_t)a1 | ((uint64_t)(uint32_t)(G.sub + W) << 32);
  const uint64_t mine = G.L->ab[G.sub];
  const uint32_t pos = (uint32_t)(mine >> 32);
  uint64_t p = PRIO_NONE;
  if (G.sub < n) p = priority(lo64(draw_block(K, purpose, pos, 0)), pos);
  G.L->prio[G.sub] = p;
  const bool sel = G.sub < n && grp_rank(G, n, p) < want;
  const MaskT<W> m = grp_ballot(G, sel);
  if (sel) G.L->out[mask_popc(m & G.below())] = (int)(uint32_t)mine;
}

// FILL_FULL for one row: returns the value of slot `sub` (-1 beyond the row).
template <int W>
__device__ __forceinline__ int grp_fill_full_row(const GrpT<W>& G, const int32_t* __restrict__ adj, uint32_t deg, int k,
                                                 const DrawKey& K, uint32_t purpose, int32_t* state) {
  constexpr int GRP = W;
  if (deg <= (uint32_t)k) return ((uint32_t)G.sub < deg) ? adj[G.sub] : -1;
  if (deg < 2u * (uint32_t)k) {
    const int d = (int)deg;
    const bool e0 = G.sub < d, e1 = G.sub + GRP < d;
    const int a0 = e0 ? adj[G.sub] : -1, a1 = e1 ? adj[G.sub + GRP] : -1;
    grp_select_positions(G, d, k, e0, e1, a0, a1, K, purpose);
    return (G.sub < k) ? G.L->out[G.sub] : -1;
  }
  const int v = grp_rejection_fill<false>(G, GrpT<W>::first(k), (MaskT<W>)0, -1, k, adj, deg, K, purpose, state);
  return (G.sub < k) ? v : -1;
}

// REFRESH_PART for one full row of a node with deg > k (Alg. 2 RefreshCache): the n_new slots of smallest
// EVICT priority (`sb`: the slot's EVICT/PICK block) are redrawn from adj(v) \ retained.  `val` is the slot's
// current id; returns its new one and the mask of redrawn slots.
template <int W>
__device__ __forceinline__ int grp_refresh_part(const GrpT<W>& G, int val, int k, int n_new, const Block4& sb,
                                                const int32_t* __restrict__ adj, uint32_t deg, const DrawKey& K,
                                                int32_t* state, MaskT<W>& evict) {
  const int sub = G.sub;
  const MaskT<W> slots = GrpT<W>::first(k);
  const uint64_t e = (sub < k) ? priority(lo64(sb), (uint32_t)sub) : PRIO_NONE;
  G.L->prio[sub] = e;
  // The n_new slots of smallest priority.  Priorities are uniform 64-bit numbers, so the slots below the
  // (n_new + 5) / k quantile nearly always include them: then a slot only has to be compared with those few (a slot
  // above the mark has at least n_new slots below it and is not ranked at all).  The wavefront walks over the slots
  // that are below the mark in either of its groups - a scalar loop; a slot above the mark in one's own group adds
  // nothing to a rank below it.  If a group has fewer than n_new slots below the mark, every slot is ranked among all.
  uint64_t mark = PRIO_NONE;
  if (n_new + 5 < k) mark = (uint64_t)(uint32_t)(4294967040.0f * (float)(n_new + 5) / (float)k) << 32;
  const bool low = e < mark;
  const uint64_t wave_low = __ballot(low), wave_here = __ballot(sub == 0);
  uint64_t scan = wave_low;
  bool enough = __popcll((unsigned long long)wave_low) >= n_new;
  if constexpr (W == 32) {
    const uint32_t lo = (uint32_t)wave_low, hi = (uint32_t)(wave_low >> 32);
    enough = (__popc(lo) >= n_new || !(wave_here & 1ull)) && (__popc(hi) >= n_new || !((wave_here >> 32) & 1ull));
    scan = lo | hi;
  } else if constexpr (W < 32) {
    enough = true;
    scan = 0ull;
#pragma unroll
    for (int q = 0; q < GrpT<W>::PER_WAVE; ++q) {
      const uint32_t m = (uint32_t)(wave_low >> (q * W)) & GrpT<W>::all();
      enough = enough && (__popc(m) >= n_new || !((wave_here >> (q * W)) & 1ull));
      scan |= m;
    }
  }
  int er;
  if (enough) {
    er = low ? 0 : k;
    for (uint64_t m = scan; m != 0; m &= m - 1) er += (G.L->prio[__builtin_ctzll(m)] < e) ? 1 : 0;
  } else {
    er = grp_rank_uniform(G, k, e);
  }
  evict = grp_ballot(G, sub < k && er < n_new);
  const MaskT<W> retained = slots & ~evict;
  if (deg < 2u * (uint32_t)k) {
    // priority regime: a position is eligible unless its id sits in a retained slot
    grp_redraw_positions(G, (int)deg, n_new, k, retained, val, adj, K, P_FILL_PART);
    if (G.in(evict)) val = G.L->out[mask_popc(evict & G.below())];
  } else {
    val = grp_rejection_fill<true>(G, evict, retained, val, k, adj, deg, K, P_FILL_PART, state);
  }
  return val;
}

// ------------------------------------------------------------------------------------------
// fill_full_kernel: a workgroup takes chunks of FILL_CHUNK rows.
//   A  one thread per row reads indptr (base, degree) into LDS and flags rows with deg > k;
//   B  rows with deg <= k (83-89 % of all rows in the power-law workloads) are plain copies of the
//      adjacency: one thread per table cell, coalesced, every load independent of the others;
//   C  the flagged rows are compacted into a list, and (row, table) pairs are dealt to the eight
//      32-lane groups, so both halves of every wavefront run the Philox / rejection code together.
// ------------------------------------------------------------------------------------------
// A row of S slots: value `val` of slot `sub`, -1 in the slots beyond the group's lanes.
template <int W>
__device__ __forceinline__ void store_row(int32_t* row, int sub, int S, int val) {
  if (sub < S) row[sub] = val;
  if (W < 32 && sub + W < S) row[sub + W] = -1;
}
constexpr int FILL_CHUNK = 64;    // rows per chunk: small enough that a few thousand workgroups share the rejection work
template <int W>
__global__ __launch_bounds__(256) void fill_full_kernel(FillParams P) {
  __shared__ GroupLdsT<W> lds[GrpT<W>::PER_WG];
  __shared__ long long row_base[FILL_CHUNK];
  __shared__ int row_deg[FILL_CHUNK];
  __shared__ int row_at[FILL_CHUNK];          // table row of the node, -1: the node keeps no row (degree split)
  __shared__ int heavy_rows[FILL_CHUNK];
  __shared__ int wave_heavy[4];
  GrpT<W> G;
  G.init(lds);
  G.set_redraws(P.n_new);
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int sshift = (P.S == 64) ? 6 : (P.S == 32) ? 5 : 4;
  const int64_t nchunks = (P.n_dst + FILL_CHUNK - 1) / FILL_CHUNK;
  for (int64_t chunk = blockIdx.x; chunk < nchunks; chunk += gridDim.x) {
    const int64_t v0 = chunk * FILL_CHUNK;
    const int rows = (int)((P.n_dst - v0 < FILL_CHUNK) ? (P.n_dst - v0) : FILL_CHUNK);
    // ---- A: degrees ----
    bool heavy = false;
    if (tid < rows) {
      const int64_t b = load_indptr(P.indptr, P.is64, v0 + tid);
      const int64_t d = load_indptr(P.indptr, P.is64, v0 + tid + 1) - b;
      row_base[tid] = b;
      row_deg[tid] = (int)d;                       // degrees are < 2^31 (checked when the graph is validated)
      const int at = P.row_of ? P.row_of[v0 + tid] : (int)(v0 + tid);
      row_at[tid] = at;
      heavy = d > P.k && at >= 0;
    }
    const uint64_t hm = __ballot(heavy);
    if (lane == 0) wave_heavy[wave] = __popcll(hm);
    __syncthreads();
    int before = 0, nheavy = 0;
    for (int q = 0; q < 4; ++q) { const int c = wave_heavy[q]; if (q < wave) before += c; nheavy += c; }
    if (heavy) heavy_rows[before + __popcll(hm & ((1ull << lane) - 1ull))] = tid;
    // ---- B: light rows, one thread per four cells (16-byte stores; one table after the other) ----
    const int quads = rows << (sshift - 2);
    for (int c = tid; c < quads; c += 256) {
      const int row = c >> (sshift - 2), slot = (c << 2) & (P.S - 1);
      const int d = row_deg[row];
      if (d > P.k || row_at[row] < 0) continue;
      const int32_t* const from = P.indices + row_base[row] + slot;
      int4 val = make_int4(-1, -1, -1, -1);
      if (slot < d) val.x = from[0];
      if (slot + 1 < d) val.y = from[1];
      if (slot + 2 < d) val.z = from[2];
      if (slot + 3 < d) val.w = from[3];
      const int64_t at = ((int64_t)row_at[row] << sshift) + slot;
      for (int t = 0; t < P.ntab; ++t) *reinterpret_cast<int4*>(P.table[t] + at) = val;
    }
    __syncthreads();
    // ---- C: heavy rows, one W-lane group per (row, table) ----
    const int items = nheavy * P.ntab;
    for (int it = G.idle ? items : G.index_in_workgroup(); it < items; it += GrpT<W>::PER_WG) {
      const int row = heavy_rows[it / P.ntab], t = it % P.ntab;
      const int64_t v = v0 + row;
      DrawKey K{P.seed_lo, P.seed_hi, (uint32_t)v, P.stepword, (P.layer_word[t] << 8) | (P.relation << 16)};
      int val;
      if (P.src_table[t]) {
        // layer-wide partial refresh: the row of the previous epoch (possibly the same memory) with n_new slots redrawn
        val = (G.sub < P.k) ? P.src_table[t][((int64_t)row_at[row] << sshift) + G.sub] : -1;
        Block4 sb{0u, 0u, 0u, 0u};
        if (G.sub < P.k) sb = draw_block(K, P_EVICT, (uint32_t)G.sub, 0);
        MaskT<W> evict;
        val = grp_refresh_part(G, val, P.k, P.n_new, sb, P.indices + row_base[row], (uint32_t)row_deg[row], K, P.state, evict);
      } else {
        val = grp_fill_full_row(G, P.indices + row_base[row], (uint32_t)row_deg[row], P.k, K, P_FILL_FULL, P.state);
      }
      store_row<W>(P.table[t] + ((int64_t)row_at[row] << sshift), G.sub, P.S, val);
    }
    __syncthreads();
  }
}

// fill_heavy_kernel: the same rows for a table set that has been filled before.  Rows of nodes with at most k
// neighbors hold the whole adjacency and never change, so a later refresh only recomputes the rows of the nodes
// with more (a list made once at set-up): one 32-lane group per (row, table), no chunk staging, no barriers.
template <int W>
__global__ __launch_bounds__(256) void fill_heavy_kernel(FillParams P, const int32_t* __restrict__ heavy, int64_t nheavy) {
  __shared__ GroupLdsT<W> lds[GrpT<W>::PER_WG];
  GrpT<W> G;
  G.init(lds);
  if (G.idle) return;
  G.set_redraws(P.n_new);
  constexpr int GROUPS = GrpT<W>::PER_WG;
  const int sshift = (P.S == 64) ? 6 : (P.S == 32) ? 5 : 4;
  const int64_t items = nheavy * P.ntab;
  for (int64_t it = (int64_t)blockIdx.x * GROUPS + G.index_in_workgroup(); it < items; it += (int64_t)gridDim.x * GROUPS) {
    const int64_t v = heavy[it / P.ntab];
    const int t = (int)(it % P.ntab);
    const int64_t b = load_indptr(P.indptr, P.is64, v);
    const uint32_t deg = (uint32_t)(load_indptr(P.indptr, P.is64, v + 1) - b);
    const int64_t at = (P.row_of ? (int64_t)P.row_of[v] : v) << sshift;
    DrawKey K{P.seed_lo, P.seed_hi, (uint32_t)v, P.stepword, (P.layer_word[t] << 8) | (P.relation << 16)};
    int val;
    if (P.src_table[t]) {
      val = (G.sub < P.k) ? P.src_table[t][at + G.sub] : -1;
      Block4 sb{0u, 0u, 0u, 0u};
      if (G.sub < P.k) sb = draw_block(K, P_EVICT, (uint32_t)G.sub, 0);
      MaskT<W> evict;
      val = grp_refresh_part(G, val, P.k, P.n_new, sb, P.indices + b, deg, K, P.state, evict);
    } else {
      val = grp_fill_full_row(G, P.indices + b, deg, P.k, K, P_FILL_FULL, P.state);
    }
    store_row<W>(P.table[t] + at, G.sub, P.S, val);
  }
}

// ------------------------------------------------------------------------------------------
// Dedupe table: per key (node type offset + id) the smallest "order word" inserted in this hop.
//   direct layout  one 64-bit word per node: (~version << 32) | order, reduced with atomicMin.
//   hashed layout  open addressing, linear probing, 16-byte entries:
//                    keyver = (version << 32) | key     claimed with a 64-bit CAS
//                    val    = (~version << 32) | order  reduced with a 64-bit atomicMin
// Words of an older version count as empty (their high half is larger), so nothing is cleared
// between hops.  Device-scope atomics are the scarce resource here (about 26 per ns on the whole
// chip, against 50-200 random loads per ns), so every insert first LOADS the word and skips the
// atomic when the stored order is already smaller.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t hash_key(uint32_t key) {
  uint32_t h = key * 0x9E3779B1u;
  return h ^ (h >> 15);
}

__device__ __forceinline__ uint64_t load_relaxed(const uint64_t* p) {
  return __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Reduces word *w with (version, order).  Returns the previous order of this version, or 0xFFFFFFFF.
__device__ __forceinline__ uint32_t word_min(uint64_t* w, uint32_t ver, uint32_t order) {
  const uint64_t myval = ((uint64_t)(~ver) << 32) | order;
  uint64_t cur = load_relaxed(w);
  if (cur > myval) cur = atomicMin((unsigned long long*)w, (unsigned long long)myval);
  return ((uint32_t)(cur >> 32) == ~ver) ? (uint32_t)cur : 0xFFFFFFFFu;
}

// Inserts (key, order).  Returns the previous order for the key in this version, or 0xFFFFFFFF.
__device__ __forceinline__ uint32_t table_insert_min(const DedupeTable& H, uint32_t ver, uint32_t key,
                                                     uint32_t order, int32_t* state) {
  if (H.direct) return word_min(&H.direct[key], ver, order);
  const uint64_t mine = ((uint64_t)ver << 32) | key;
  uint64_t h = hash_key(key) & H.mask;
  for (uint64_t probes = 0; probes <= H.mask; ++probes) {
    unsigned long long* kv = (unsigned long long*)&H.entries[h].keyver;
    uint64_t cur = __hip_atomic_load(kv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint32_t)(cur >> 32) != ver) {           // empty or stale: try to claim it
      const uint64_t old = atomicCAS(kv, (unsigned long long)cur, (unsigned long long)mine);
      cur = (old == cur) ? mine : old;
    }
    if (cur == mine) return word_min(&H.entries[h].val, ver, order);
    h = (h + 1) & H.mask;
  }
  atomicOr(&state[ST_ERROR], ERR_TABLE_FULL);
  return 0xFFFFFFFFu;
}

__device__ __forceinline__ uint32_t table_lookup(const DedupeTable& H, uint32_t ver, uint32_t key, int32_t* state) {
  if (H.direct) return (uint32_t)H.direct[key];
  const uint64_t mine = ((uint64_t)ver << 32) | key;
  uint64_t h = hash_key(key) & H.mask;
  for (uint64_t probes = 0; probes <= H.mask; ++probes) {
    const HashEntry e = H.entries[h];
    if (e.keyver == mine) return (uint32_t)e.val;
    if ((uint32_t)(e.keyver >> 32) != ver) break;   // hit an empty slot: the key was never inserted
    h = (h + 1) & H.mask;
  }
  atomicOr(&state[ST_ERROR], ERR_TABLE_MISS);
  return 0u;
}

// Relation / node type r of a slice.  The compact launch builds a slice's arguments in registers, where nothing
// can be indexed at run time: its layout (one relation, one node type) has nothing to index anyway.
struct HopParamsMonoRegs : HopParamsMono { static constexpr bool IN_REGISTERS = true; };
template <class HP, class = void> struct in_registers { static constexpr bool value = false; };
template <class HP> struct in_registers<HP, decltype((void)HP::IN_REGISTERS)> { static constexpr bool value = true; };
template <class HP>
__device__ __forceinline__ const RelParam& rel_of(const HP& P, int r) {
  if constexpr (in_registers<HP>::value) return P.rel[0]; else return P.rel[r];
}
template <class HP>
__device__ __forceinline__ const TypeParam& type_of(const HP& P, int t) {
  if constexpr (in_registers<HP>::value) return P.type[0]; else return P.type[t];
}
template <class HP>
__device__ __forceinline__ int frontier_count(const HP& P, int t) {
  const int o = type_of(P, t).count_override;
  return o >= 0 ? o : P.state[ST_COUNTS + P.hop * P.T + t];
}

// Live tiles of a hop.  Pick slots are laid out by host-known upper bounds (relation r owns the tiles from
// slot_base[r] / TILE on), but only the first ceil(F * f / TILE) tiles of a relation hold picks, F being the
// frontier size of its dst type, known on the device.  The insert, mark and emit phases walk the concatenation
// of the live ranges: live index j -> (relation, tile).  first[r] = live index of relation r's first tile,
// first[R] = number of live tiles, nslots[r] = F * f.
struct LiveLds {
  int first[GSS_MAX_RELATIONS + 1];
  uint32_t nslots[GSS_MAX_RELATIONS];
  int base[GSS_MAX_RELATIONS + 1];       // first tile of a relation, dead tiles counted; base[R] = all tiles
  int src_type[GSS_MAX_RELATIONS];
};
template <class HP>
__device__ __forceinline__ void live_tiles_setup(const HP& P, LiveLds* L) {
  if constexpr (HP::MAX_R == 1) return;          // one relation: nothing to look up (live_count, live_tile)
  if ((int)threadIdx.x < P.R) {
    // (one vector load per lane; a loop over the relations with scalar loads costs a round trip to the scalar cache each)
    const RelParam& RP = P.rel[threadIdx.x];
    const int dst_type = RP.dst_type, src_type = RP.src_type, base = RP.slot_base / TILE;
    L->base[threadIdx.x] = base;
    L->src_type[threadIdx.x] = src_type;
    if (threadIdx.x == 0) L->base[P.R] = P.num_tiles_ub;
    int count = P.type[dst_type].count_override;
    if (count < 0) count = P.state[ST_COUNTS + P.hop * P.T + dst_type];
    L->nslots[threadIdx.x] = (uint32_t)count * (uint32_t)P.f;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int q = 0; q < P.R; ++q) { L->first[q] = run; run += (int)((L->nslots[q] + TILE - 1) / TILE); }
    L->first[P.R] = run;
  }
  __syncthreads();
}
// Number of live tiles of the hop.
template <class HP>
__device__ __forceinline__ int live_count(const HP& P, const LiveLds* L) {
  if constexpr (HP::MAX_R == 1) return (int)(((uint32_t)frontier_count(P, 0) * (uint32_t)P.f + TILE - 1) / TILE);
  return L->first[P.R];
}
// Live index of relation r's first tile.
template <class HP>
__device__ __forceinline__ int live_first(const LiveLds* L, int r) {
  if constexpr (HP::MAX_R == 1) return 0;
  return L->first[r];
}
struct LiveTile { int r; uint32_t local0, nslots; };
template <class HP>
__device__ __forceinline__ LiveTile live_tile(const HP& P, const LiveLds* L, int j) {
  if constexpr (HP::MAX_R == 1) return LiveTile{0, (uint32_t)j * TILE, (uint32_t)frontier_count(P, 0) * (uint32_t)P.f};
  int r = 0;
  while (r + 1 < P.R && j >= L->first[r + 1]) ++r;
  return LiveTile{r, (uint32_t)(j - L->first[r]) * TILE, L->nslots[r]};
}

// ------------------------------------------------------------------------------------------
// sample phase: rows wg.y < R of the slice's grid: relation y, one 32-lane group per frontier node.
//               rows wg.y >= R: node type y-R, one thread per frontier node (insert the dst
//               nodes into the dedupe table with order = frontier index, copy them to src_nodes).
// ------------------------------------------------------------------------------------------
// Node type t of a hop, one thread per frontier node: the dst nodes enter the dedupe table (order = frontier index)
// and head the hop's src_nodes.  Workgroup x of the P.gxd that share the work.
template <class HP>
__device__ __forceinline__ void dst_node_rows(const HP& P, int t, int x) {
  const TypeParam& TP = type_of(P, t);
  const int F = frontier_count(P, t);
  for (int i = x * (int)blockDim.x + (int)threadIdx.x; i < F; i += P.gxd * (int)blockDim.x) {
    const int v = TP.frontier[i];
    if ((uint32_t)v >= (uint32_t)TP.n_nodes) { atomicOr(&P.state[ST_ERROR], ERR_SEED_RANGE); continue; }
    TP.src_nodes[i] = v;
    if (P.hop > 0 && P.ht.direct) {
      // Beyond the seeds the dst nodes are distinct (the previous hop's dedupe made them so), and a frontier index is
      // smaller than every pick's order word: whatever the picks of the same launch do to the node's word with their
      // atomic minimum, before or after, a plain store of the frontier index leaves the minimum there.  (Random
      // device-scope atomics run at 27 per ns on the whole chip, whatever the table size; plain stores at 50-180.)
      __hip_atomic_store((unsigned long long*)&P.ht.direct[TP.key_off + (uint32_t)v], ((unsigned long long)(~P.ver) << 32) | (uint32_t)i,
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      continue;
    }
    const uint32_t old = table_insert_min(P.ht, P.ver, TP.key_off + (uint32_t)v, (uint32_t)i, P.state);
    if (old < EDGE_BIT && old != (uint32_t)i) atomicOr(&P.state[ST_ERROR], ERR_SEED_DUP);
  }
}

template <class HP, int W>
__device__ __forceinline__ void sample_phase(const HP& P, const Wg wg, GroupLdsT<W>* lds) {
  if (wg.y >= P.R) {
    dst_node_rows(P, wg.y - P.R, wg.x);
    return;
  }
  using Mask = MaskT<W>;
  GrpT<W> G;
  G.init(lds);
  if (G.idle) return;                 // (no barrier below: the phase is a per-group loop)
  G.set_redraws(P.n_new);
  const int r = wg.y;
  const RelParam& RP = rel_of(P, r);
  const RelConst& RC = P.rc(r);
  const int grp = wg.x * GrpT<W>::PER_WG + G.index_in_workgroup();
  // the first node id is loaded before the frontier size is known (both loads travel together);
  // `frontier_cap` is the allocated length of the frontier array
  const int v_first = (grp < type_of(P, RP.dst_type).frontier_cap) ? type_of(P, RP.dst_type).frontier[grp] : 0;
  const int F = frontier_count(P, RP.dst_type);
  const int ngrp = P.gx * GrpT<W>::PER_WG;
  const int k = P.k, f = P.f, sub = G.sub;
  const int32_t* __restrict__ frontier = type_of(P, RP.dst_type).frontier;
  const uint32_t src_key_off = type_of(P, RP.src_type).key_off;

  int v_ahead = v_first;
  for (int i = grp; i < F; i += ngrp) {
    const int v = v_ahead;
    if (i + ngrp < F) v_ahead = frontier[i + ngrp];   // the id of the group's next node travels while this one is worked on
    const uint32_t g0 = (uint32_t)RP.slot_base + (uint32_t)i * (uint32_t)f;
    if ((uint32_t)v >= (uint32_t)RC.n_dst) {        // reported by the node-type pass; emit nothing
      if (sub < f) P.picks[g0 + sub] = -1;
      continue;
    }
    DrawKey K{P.seed_lo, P.seed_hi, (uint32_t)v, P.step, (P.layer_word << 8) | ((uint32_t)r << 16)};
    int val;
    bool sel;
    // Degree split: the node's table row comes from the row map; nodes without a row are sampled
    // like Full Batch Load.  The adjacency bounds are requested together with the map entry.
    int at = v;
    bool uncached = P.mode == GSS_MODE_FBL;
    int64_t b = 0, d64 = 0;
    if (RC.row_of) {
      at = RC.row_of[v];
      b = load_indptr(RC.indptr, RC.is64, v);
      d64 = load_indptr(RC.indptr, RC.is64, (int64_t)v + 1) - b;
      uncached |= at < 0;
    } else if (uncached) {
      b = load_indptr(RC.indptr, RC.is64, v);
      d64 = load_indptr(RC.indptr, RC.is64, (int64_t)v + 1) - b;
    }
    if (uncached) {
      // Full Batch Load: no cache, a uniform min(deg,f)-subset straight from the adjacency,
      // keyed by the step and the hop's own layer (also when the cached nodes share one table)
      K.tag = ((uint32_t)P.layer << 8) | ((uint32_t)r << 16);
      val = grp_fill_full_row(G, RC.indices + b, (uint32_t)d64, f, K, P_FBL, P.state);
      sel = (int64_t)sub < (d64 < f ? d64 : (int64_t)f);
    } else {
    int32_t* row = RP.table + (int64_t)at * P.S;
    val = (sub < k) ? row[sub] : -1;
    // On a refresh step the adjacency bounds (and the shared-mode stamp) are loaded together with
    // the row rather than after it: one round trip less on the critical path of every visited node.
    long long stamp = -1;
    const bool fetch_mode = P.mode == GSS_MODE_OTF_FETCH && P.n_new > 0;
    if (P.refresh_now || fetch_mode) {
      if (!RC.row_of) {
        b = load_indptr(RC.indptr, RC.is64, v);
        d64 = load_indptr(RC.indptr, RC.is64, (int64_t)v + 1) - b;
      }
      if (P.mode == GSS_MODE_SHARED_OTF) stamp = RC.stamp[at];
    }
    const int len = mask_popc(grp_ballot(G, val >= 0));

    // ---- does this visit refresh the row? (only full rows can belong to a node with deg > k) ----
    bool refresh = false;
    const uint32_t deg = (uint32_t)d64;
    if (P.refresh_now && len == k) {
      bool due = true;
      if (P.mode == GSS_MODE_SHARED_OTF) {
        due = stamp != (long long)P.step;
        if (due && sub == 0) RC.stamp[at] = (long long)P.step;
      }
      refresh = due && d64 > k;
    }
    // OTF Fetch: a node with more than k neighbors takes n_new of its f neighbors fresh from the adjacency
    // and only f - n_new from the (full) row
    const bool fetch = fetch_mode && d64 > k;
    const int fdraw = fetch ? f - P.n_new : f;
    // one Philox block per slot serves both per-slot draws: EVICT (words 0,1) and PICK (words 2,3)
    Block4 sb{0u, 0u, 0u, 0u};
    if ((refresh || len > fdraw) && sub < k) sb = draw_block(K, P_EVICT, (uint32_t)sub, 0);

    if (refresh) {
      Mask evict;
      val = grp_refresh_part(G, val, k, P.n_new, sb, RC.indices + b, deg, K, P.state, evict);
      if (G.in(evict)) row[sub] = val;
    }

    // ---- draw the fanout from the row ----
    if (len <= fdraw) {
      sel = sub < len;
    } else {
      const uint64_t pp = (sub < len) ? priority(hi64(sb), (uint32_t)sub) : PRIO_NONE;
      G.L->prio[sub] = pp;
      const int rank = grp_rank_uniform(G, k, pp);       // (slots from len on hold PRIO_NONE)
      int start = 0;
      if (P.shared) start = min(P.band_offset, len - fdraw);
      sel = sub < len && rank >= start && rank < start + fdraw;
    }
    if (fetch) {
      // the cached picks move to lanes 0 .. fdraw-1 (ascending slot order); lanes fdraw .. f-1 draw fresh
      // neighbors from adj(v) \ {cached picks} by the redraw procedure of the partial refresh, on this
      // f-wide list instead of the row
      const Mask selm0 = grp_ballot(G, sel);
      if (sel) G.L->out[mask_popc(selm0 & G.below())] = val;
      int cv = (sub < fdraw) ? G.L->out[sub] : -1;
      const Mask kept = GrpT<W>::first(fdraw);                        // fdraw < f <= W
      const Mask redraw = GrpT<W>::first(f) & ~kept;
      const int32_t* adj = RC.indices + b;
      const uint32_t deg = (uint32_t)d64;
      if (deg < 2u * (uint32_t)f) {
        grp_redraw_positions(G, (int)deg, P.n_new, f, kept, cv, adj, K, P_FETCH);
        if (G.in(redraw)) cv = G.L->out[mask_popc(redraw & G.below())];
      } else {
        cv = grp_rejection_fill<true>(G, redraw, kept, cv, f, adj, deg, K, P_FETCH, P.state);
      }
      val = cv;
      sel = sub < f;
    }
    }
    const Mask selm = grp_ballot(G, sel);
    const int cnt = mask_popc(selm);
    if (sel) {
      const uint32_t g = g0 + (uint32_t)mask_popc(selm & G.below());
      P.picks[g] = val;
      bool inserts = !P.insert_split;                  // (bit 1, the LDS stage, is only ever set in the staged builds)
      if constexpr (std::is_base_of<HopParamsStaged, HP>::value) inserts = !(P.insert_split & 1);
      if (inserts) table_insert_min(P.ht, P.ver, src_key_off + (uint32_t)val, EDGE_BIT | g, P.state);
    }
    if (sub >= cnt && sub < f) P.picks[g0 + sub] = -1;
  }
}

// Optional first stage of the dedupe, per tile, in LDS ("LDS-staged unique, spilling to the global table"): the tile's
// picks enter an open-addressing table of 2 * TILE 64-bit words, (key << 32) | slot within the tile, reduced with
// a 64-bit LDS minimum; only the pick that holds the smallest slot of its id within the tile goes on to the global
// table - the others could not win there anyway.  Returns, per thread, which of its ITEMS_PER_THREAD picks go on.
// All threads of the workgroup call it (barriers inside); `key[q]` is only read where `valid` has bit q set.
constexpr int TILE_HASH = 2 * TILE;
struct DedupeLds { unsigned long long word[TILE_HASH]; };
__device__ __forceinline__ uint32_t tile_firsts(DedupeLds* D, const uint32_t* key, uint32_t valid, uint32_t slot0) {
  unsigned long long* tab = D->word;
  for (int i = (int)threadIdx.x; i < TILE_HASH; i += (int)blockDim.x) tab[i] = ~0ull;
  __syncthreads();
  uint32_t home[ITEMS_PER_THREAD];
#pragma unroll
  for (int q = 0; q < ITEMS_PER_THREAD; ++q) {
    home[q] = 0u;
    if (!((valid >> q) & 1u)) continue;
    const unsigned long long mine = ((unsigned long long)key[q] << 32) | (slot0 + (uint32_t)q);
    uint32_t h = (key[q] * 0x9E3779B1u) >> 21;                    // 11 bits: TILE_HASH entries
    for (;;) {                                                    // (at most TILE of the 2 TILE entries are ever taken)
      unsigned long long cur = __hip_atomic_load(&tab[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (cur == ~0ull &&                                         // empty: try to take it (on failure `cur` = who did)
          __hip_atomic_compare_exchange_strong(&tab[h], &cur, mine, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
        break;                                                    // taken: this pick is the smallest so far
      if ((uint32_t)(cur >> 32) == key[q]) {
        __hip_atomic_fetch_min(&tab[h], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        break;
      }
      h = (h + 1u) & (uint32_t)(TILE_HASH - 1);
    }
    home[q] = h;
  }
  __syncthreads();
  uint32_t first = 0u;
#pragma unroll
  for (int q = 0; q < ITEMS_PER_THREAD; ++q)
    if (((valid >> q) & 1u) && (uint32_t)__hip_atomic_load(&tab[home[q]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == slot0 + (uint32_t)q)
      first |= 1u << q;
  __syncthreads();                                                // (the table is cleared again for the next tile)
  return first;
}

// ------------------------------------------------------------------------------------------
// Visit-once steps (see ChainArgs): chain phase and place phase.
// ------------------------------------------------------------------------------------------
// Marks node v as visited in this step with holding index Q (`mine` = (~version << 32) | Q).  True for exactly one
// of the picks that name the same node in one step.
__device__ __forceinline__ bool claim_visit(uint64_t* visit, uint32_t v, uint64_t mine) {
  unsigned long long* w = (unsigned long long*)&visit[v];
  const uint64_t cur = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((uint32_t)(cur >> 32) == (uint32_t)(mine >> 32)) return false;      // visited already
  // (a word of another version can only turn into one of this step's version)
  return atomicCAS(w, (unsigned long long)cur, (unsigned long long)mine) == cur;
}
// The same for a seed (holding index Q < num_seeds).  A seed must be visited as a seed even if a pick of another seed
// names it and claims it before its own group gets to it: words of later versions and smaller indices are smaller, so an
// atomic minimum lets the seed take the entry over (the pick's entry in list 1 then points at an index the visit table
// no longer holds, and is skipped).
__device__ __forceinline__ void claim_seed(uint64_t* visit, uint32_t v, uint64_t mine) {
  __hip_atomic_fetch_min((unsigned long long*)&visit[v], (unsigned long long)mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The one visit of node v in this step, by the hop c that reaches it first: read the row, refresh it when the step
// refreshes (Alg. 2 RefreshCache on the shared table: once per node and step), rank the slots once by PICK priority,
// and take for every hop h = c .. L-1 the ranks [band[h], band[h] + f[h]) ("Shared Cache Design": per-layer bands of
// one per-(step, node) ranking) - what the per-hop sample phase computes when it meets the node again in hop h.
// Nodes without a cache row (degree split) draw every hop straight from the adjacency, keyed by the hop's layer.
// Returns hop c's pick number `sub` (-1 beyond the node's picks).
template <class HP>
__device__ __forceinline__ int visit_node(const HP& P, const ChainArgs& C, const Grp& G, int c, int v, uint32_t Q) {
  const RelParam& RP = rel_of(P, 0);
  const RelConst& RC = P.rc(0);
  const int k = P.k, sub = G.sub;
  DrawKey K{P.seed_lo, P.seed_hi, (uint32_t)v, P.step, P.layer_word << 8};
  int at = v;
  int64_t b = 0, d64 = 0;
  if (RC.row_of) at = RC.row_of[v];
  if (RC.row_of || P.refresh_now) {
    b = load_indptr(RC.indptr, RC.is64, v);
    d64 = load_indptr(RC.indptr, RC.is64, (int64_t)v + 1) - b;
  }
  int mine = -1;
  if (at < 0) {
    for (int h = c; h < C.L; ++h) {
      const int f = C.f(h);
      K.tag = C.layer(h) << 8;
      int val = grp_fill_full_row(G, RC.indices + b, (uint32_t)d64, f, K, P_FBL, P.state);
      const int cnt = (int)(d64 < f ? d64 : (int64_t)f);
      if (sub >= cnt) val = -1;
      if (sub < f) C.held[C.off[h] + Q * (uint32_t)f + (uint32_t)sub] = val;
      if (h == c) mine = val;
    }
    return mine;
  }
  int32_t* row = RP.table + (int64_t)at * P.S;
  int val = (sub < k) ? row[sub] : -1;
  const int len = __popc(grp_ballot(G, val >= 0));
  const bool refresh = P.refresh_now && len == k && d64 > k;
  bool ranked = false;
  for (int h = c; h < C.L; ++h) ranked |= len > C.f(h);
  Block4 sb{0u, 0u, 0u, 0u};
  if ((refresh || ranked) && sub < k) sb = draw_block(K, P_EVICT, (uint32_t)sub, 0);
  if (refresh) {
    uint32_t evict;
    val = grp_refresh_part(G, val, k, P.n_new, sb, RC.indices + b, (uint32_t)d64, K, P.state, evict);
    if ((evict >> sub) & 1u) row[sub] = val;
  }
  int rank = 0;
  if (ranked) {
    const uint64_t pp = (sub < len) ? priority(hi64(sb), (uint32_t)sub) : PRIO_NONE;
    G.L->prio[sub] = pp;
    rank = grp_rank_uniform(G, k, pp);                  // (slots from len on hold PRIO_NONE)
  }
  for (int h = c; h < C.L; ++h) {
    const int f = C.f(h);
    bool sel = sub < len;
    if (len > f) {
      const int start = min(C.band(h), len - f);
      sel = sub < len && rank >= start && rank < start + f;
    }
    const uint32_t selm = grp_ballot(G, sel);
    const int cnt = __popc(selm);
    if (sel) G.L->out[__popc(selm & below_mask(sub))] = val;       // picks in slot order, through LDS
    const int pick = (sub < cnt) ? G.L->out[sub] : -1;
    if (sub < f) C.held[C.off[h] + Q * (uint32_t)f + (uint32_t)sub] = pick;
    if (h == c) mine = pick;
  }
  return mine;
}

// chain phase of hop c: one 32-lane group per node of the frontier of hop c, eight groups per workgroup, striding.
// The nodes that hop c reaches first - the seeds for c = 0, else list c - are visited.  Unless c is the last hop, hop
// c's picks of every frontier node - of the ones just visited, and of the nodes of earlier hops, whose picks are held -
// then claim their nodes: a pick that comes first appends its node to list c + 1.
struct ChainLds { uint32_t start[CHAIN_MAX_HOPS * CHAIN_SEGS + 2]; };
template <bool AHEAD, class HP>
__device__ __forceinline__ void chain_phase(const HP& P, const ChainArgs& C, const Wg wg, GroupLds* lds, ChainLds* CL) {
  Grp G;
  G.init(lds);
  G.set_redraws(P.n_new);
  const int c = P.hop, sub = G.sub, L = C.L;
  const int grp = wg.x * (int)(blockDim.x >> 5) + (int)(threadIdx.x >> 5);
  const int ngrp = P.gx * (int)(blockDim.x >> 5);
  const RelConst& RC = P.rc(0);
  const uint64_t vtag = (uint64_t)(~P.visit_ver()) << 32;
  const uint32_t F0 = (uint32_t)C.V[0];
  const bool claims = c + 1 < L;
  // ---- the items: seeds (unless only list c has work to do), then the segments of lists 1 .. c ----
  const int first_list = claims ? 0 : c;                 // the last hop only visits
  const uint32_t nseeds = first_list == 0 ? F0 : 0u;
  const int h0 = first_list > 1 ? first_list : 1;        // first list kept in segments
  const int nsegs = c >= h0 ? (c - h0 + 1) * CHAIN_SEGS : 0;
  if (c == 0 && wg.x == 0 && threadIdx.x < CHAIN_MAX_HOPS * CHAIN_SEGS) C.counts_next[threadIdx.x * COUNT_STRIDE] = 0u;
  if (nsegs > 0) {
    if ((int)threadIdx.x < nsegs) {
      const uint32_t n = C.counts[(h0 * CHAIN_SEGS + (int)threadIdx.x) * COUNT_STRIDE];
      const uint32_t cap = C.lcap[h0 + (int)threadIdx.x / CHAIN_SEGS];
      if (n > cap) atomicOr(&P.state[ST_ERROR], ERR_TABLE_FULL);
      CL->start[threadIdx.x + 1] = n < cap ? n : cap;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
      // exclusive prefix of the segment sizes (size of segment q at start[q + 1] -> its first item at start[q]) by the
      // first wavefront, two segments per lane: a lane's stores depend, through the shuffles, on the loads of every
      // lane below it, which are the only other readers of the words it overwrites
      const int l = (int)threadIdx.x;
      static_assert(CHAIN_MAX_HOPS * CHAIN_SEGS <= 128, "two segments per lane");
      const uint32_t a = 2 * l < nsegs ? CL->start[2 * l + 1] : 0u, b = 2 * l + 1 < nsegs ? CL->start[2 * l + 2] : 0u;
      uint32_t inc = a + b;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = (uint32_t)__shfl_up((int)inc, o);
        if (l >= o) inc += t;
      }
      const uint32_t ex = nseeds + inc - (a + b);
      if (2 * l < nsegs) CL->start[2 * l] = ex;
      if (2 * l + 1 < nsegs) CL->start[2 * l + 1] = ex + a;
      if (l == 63) CL->start[nsegs] = nseeds + inc;
    }
    __syncthreads();
  }
  const uint32_t total = nsegs > 0 ? CL->start[nsegs] : nseeds;
  const int32_t* __restrict__ seeds = type_of(P, 0).frontier;
  const int fc = C.f(c);
  // item g -> the node: its id (seeds) or its list entry (Q << 32 | v), and the list it is in
  auto item = [&](uint32_t g, int& h) -> uint64_t {
    if (g < nseeds) { h = 0; return ((uint64_t)g << 32) | (uint32_t)seeds[g]; }
    int q = 0;                                           // the segment that holds item g (start[] is ascending)
    for (int step = 64; step > 0; step >>= 1)
      if (q + step < nsegs && CL->start[q + step] <= g) q += step;
    h = h0 + q / CHAIN_SEGS;
    return C.list[C.loff[h] + (uint32_t)(q % CHAIN_SEGS) * C.lcap[h] + (g - CL->start[q])];
  };
  int h_ahead = 0;
  uint64_t e_ahead = (AHEAD && (uint32_t)grp < total) ? item((uint32_t)grp, h_ahead) : 0ull;
  for (uint32_t g = (uint32_t)grp; g < total; g += (uint32_t)ngrp) {
    // ---- which node (the group's next item travels while this one is worked on - not in the build held to 64
    //      vector registers, where the item in flight meant two registers spilled to scratch memory, and a kernel that
    //      uses scratch memory is followed by 4.5 us of idle time before the next launch starts) ----
    uint64_t e;
    int h;
    if constexpr (AHEAD) {
      e = e_ahead;
      h = h_ahead;
      if (g + (uint32_t)ngrp < total) e_ahead = item(g + (uint32_t)ngrp, h_ahead);
    } else {
      e = item(g, h);
    }
    const int v = (int)(uint32_t)e;
    const uint32_t Q = (uint32_t)(e >> 32);
    const bool fresh = h == c;                           // first reached by this hop: to be visited
    // (list 1 may name a seed that a pick claimed before the seed's own visit took the entry over)
    if (h == 1 && C.visit[v] != (vtag | Q)) continue;
    // ---- hop c's picks of the node: drawn now, or held since its visit ----
    int id = -1;
    if (c == 0) {
      if ((uint32_t)v < (uint32_t)RC.n_dst) {
        // the seed's entry of the visit table: nobody waits for the result.  (A repeated seed is visited twice; the
        // place phase reports it, and the step's results are discarded.)
        if (sub == 0) claim_seed(C.visit, (uint32_t)v, vtag | Q);
        id = visit_node(P, C, G, 0, v, Q);
      } else {
        // an id out of range (the place phase reports it): it holds no picks
        for (int h = 0; h < L; ++h)
          if (sub < C.f(h)) C.held[C.off[h] + Q * (uint32_t)C.f(h) + (uint32_t)sub] = -1;
      }
    } else if (fresh) {
      id = visit_node(P, C, G, c, v, Q);
    } else if (sub < fc) {
      id = C.held[C.off[c] + Q * (uint32_t)fc + (uint32_t)sub];
    }
    if (!claims) continue;
    // ---- every pick claims its node; the winners join list c + 1 ----
    const uint32_t Qc = (uint32_t)C.V[c] + Q * (uint32_t)fc + (uint32_t)sub;
    bool won = false;
    if (id >= 0) won = claim_visit(C.visit, (uint32_t)id, vtag | Qc);
    const uint64_t wm = __ballot(won);                   // both nodes of the wavefront: they share a segment
    if (wm != 0ull) {
      const uint32_t seg = (g >> 1) % CHAIN_SEGS;
      const int leader = __ffsll((unsigned long long)wm) - 1;
      uint32_t base = 0u;
      if (lane_id() == leader) base = atomicAdd(&C.counts[((c + 1) * CHAIN_SEGS + seg) * COUNT_STRIDE], (uint32_t)__popcll(wm));
      base = (uint32_t)__shfl((int)base, leader);
      if (won) {
        const uint32_t at = base + (uint32_t)__popcll(wm & ((1ull << lane_id()) - 1ull));
        if (at < C.lcap[c + 1]) C.list[C.loff[c + 1] + seg * C.lcap[c + 1] + at] = ((uint64_t)Qc << 32) | (uint32_t)id;
        // (beyond the capacity: cannot happen; the next chain phase reports the counter)
      }
    }
  }
}

// place phase of hop h: tiles of pick slots in frontier order.  Slot i * f + j takes pick j of frontier node i from
// the holding area (through the node's holding index in the visit table) and enters it into the dedupe table; rows
// wg.y >= 1 of the slice handle the dst nodes.  From here on the hop looks like any other: mark, emit.
template <class HP>
__device__ __forceinline__ void place_phase(const HP& P, const Wg wg, LiveLds* live, DedupeLds* D) {
  if (wg.y >= 1) {
    dst_node_rows(P, 0, wg.x);
    return;
  }
  live_tiles_setup(P, live);
  const TypeParam& TP = type_of(P, 0);
  const uint32_t f = (uint32_t)P.f;
  const bool staged = (P.insert_split & 2) != 0;
  for (int j = wg.x; j < live_count(P, live); j += P.gx) {
    const LiveTile lt = live_tile(P, live, j);
    const uint32_t nslots = lt.nslots;
    const uint32_t g = lt.local0 + ITEMS_PER_THREAD * threadIdx.x;       // one relation: its slots start at 0
    uint32_t i = g / f, jj = g - i * f;
    int id[ITEMS_PER_THREAD];
    uint32_t Q = 0;
    bool have = false;
#pragma unroll
    for (int q = 0; q < ITEMS_PER_THREAD; ++q) {
      id[q] = -1;
      if (g + q < nslots) {
        if (!have || jj == 0u) {            // the first slot of the thread, or a new frontier node
          have = true;
          const int v = TP.frontier[i];
          Q = 0xFFFFFFFFu;
          if ((uint32_t)v < (uint32_t)TP.n_nodes) {
            const uint64_t w = P.visit[v];
            if ((uint32_t)(w >> 32) == ~P.visit_ver()) Q = (uint32_t)w;
            else atomicOr(&P.state[ST_ERROR], ERR_TABLE_MISS);   // (cannot happen: every frontier node was visited)
          }
        }
        if (Q != 0xFFFFFFFFu) id[q] = P.held[Q * f + jj];
      }
      if (++jj == f) { jj = 0u; ++i; }
    }
    if (g < nslots) *reinterpret_cast<int4*>(P.picks + g) = make_int4(id[0], id[1], id[2], id[3]);
    if (P.insert_split & 1) continue;     // (uniform: the hop has an insert phase, which enters the picks into the table)
    uint32_t key[ITEMS_PER_THREAD], go = 0u;
#pragma unroll
    for (int q = 0; q < ITEMS_PER_THREAD; ++q) {
      key[q] = TP.key_off + (uint32_t)id[q];
      if (id[q] >= 0) go |= 1u << q;
    }
    if (staged) go = tile_firsts(D, key, go, ITEMS_PER_THREAD * threadIdx.x);
#pragma unroll
    for (int q = 0; q < ITEMS_PER_THREAD; ++q)
      if ((go >> q) & 1u) table_insert_min(P.ht, P.ver, key[q], EDGE_BIT | (g + q), P.state);
  }
}

// ------------------------------------------------------------------------------------------
// insert phase (large hops only; smaller ones insert in the sample phase): per pick, reduce the dedupe
// table word of its id with the pick's slot.  Four consecutive slots per thread, four independent
// table accesses in flight - in the sample phase the insert is the tail of a long dependent chain.
// ------------------------------------------------------------------------------------------
template <bool STAGED, class HP>
__device__ __forceinline__ void insert_phase(const HP& P, const Wg wg, LiveLds* live, DedupeLds* D) {
  // The workgroup's first tile is requested before the live counts are known (if it lies in relation 0 its
  // address does not depend on them, and the buffer covers every tile of the grid): the picks travel while the
  // counts are fetched.
  int4 pv_first = make_int4(-1, -1, -1, -1);
  if (wg.x < P.num_tiles_ub)
    pv_first = *reinterpret_cast<const int4*>(P.picks + (uint32_t)rel_of(P, 0).slot_base + (uint32_t)wg.x * TILE + 4u * threadIdx.x);
  live_tiles_setup(P, live);
  if (!STAGED || (P.insert_split & 2) == 0) {
    for (int j = wg.x; j < live_count(P, live); j += P.gx) {
      const LiveTile lt = live_tile(P, live, j);
      const RelParam& RP = rel_of(P, lt.r);
      const uint32_t nslots = lt.nslots;
      const uint32_t loc = lt.local0 + 4u * threadIdx.x;
      const uint32_t g = (uint32_t)RP.slot_base + loc;
      if (loc >= nslots) continue;
      const int4 pv = (j == wg.x && lt.r == 0) ? pv_first : *reinterpret_cast<const int4*>(P.picks + g);
      const uint32_t key_off = type_of(P, RP.src_type).key_off;
      const int id[4] = {pv.x, pv.y, pv.z, pv.w};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (loc + q < nslots && id[q] >= 0) table_insert_min(P.ht, P.ver, key_off + (uint32_t)id[q], EDGE_BIT | (g + q), P.state);
    }
    return;
  }
  // with the LDS stage: every thread of the workgroup takes part in every tile (barriers)
  if constexpr (STAGED)
  for (int j = wg.x; j < live_count(P, live); j += P.gx) {
    const LiveTile lt = live_tile(P, live, j);
    const RelParam& RP = rel_of(P, lt.r);
    const uint32_t nslots = lt.nslots;
    const uint32_t loc = lt.local0 + 4u * threadIdx.x;
    const uint32_t g = (uint32_t)RP.slot_base + loc;
    int4 pv = make_int4(-1, -1, -1, -1);
    if (loc < nslots) pv = (j == wg.x && lt.r == 0) ? pv_first : *reinterpret_cast<const int4*>(P.picks + g);
    const uint32_t key_off = type_of(P, RP.src_type).key_off;
    const int id[4] = {pv.x, pv.y, pv.z, pv.w};
    uint32_t key[4], go = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      key[q] = key_off + (uint32_t)id[q];
      if (loc + q < nslots && id[q] >= 0) go |= 1u << q;
    }
    go = tile_firsts(D, key, go, 4u * threadIdx.x);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((go >> q) & 1u) table_insert_min(P.ht, P.ver, key[q], EDGE_BIT | (g + q), P.state);
  }
}

// exclusive scan of two small counters over a 256-thread workgroup; returns totals in tot0/tot1
__device__ __forceinline__ void block_scan2(int v0, int v1, int& ex0, int& ex1, int& tot0, int& tot1, int* lds) {
  const int lane = lane_id(), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int i0 = v0, i1 = v1;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int a = __shfl_up(i0, o), b = __shfl_up(i1, o);
    if (lane >= o) { i0 += a; i1 += b; }
  }
  __syncthreads();
  if (lane == 63) { lds[w] = i0; lds[16 + w] = i1; }
  __syncthreads();
  int b0 = 0, b1 = 0, t0 = 0, t1 = 0;
  for (int q = 0; q < nw; ++q) {
    const int a = lds[q], b = lds[16 + q];
    if (q < w) { b0 += a; b1 += b; }
    t0 += a; t1 += b;
  }
  ex0 = b0 + i0 - v0; ex1 = b1 + i1 - v1; tot0 = t0; tot1 = t1;
}

// ------------------------------------------------------------------------------------------
// mark and emit phases, or settle phase: from the picks of a hop and the dedupe table (complete: an earlier launch did the
// inserts) to the block, one workgroup per tile of TILE pick slots.  A pick is the first occurrence of its id if the table holds
// its own slot; the first occurrences are numbered in slot order (after the dst nodes), a repeat takes the number of its first.
//
// Lane l of wavefront w owns the slots 256 w + 64 q + l, q = 0 .. 3: a ballot is then a mask of 64 consecutive slots, and
// ranks are bit counts (no shuffles, no scan).  The numbers of the first occurrences are handed on 16 slots a word (a bit
// mask and the number of the first one): half a byte per slot or less, where a rank word per slot took four, and small enough
// for the repeats' random reads to hit the caches.
//
// mark, emit (steps that share launches with others): mark stores each pick's order word, the ranks and the tile's totals.
// Hops of up to EMIT_SCAN_TILES tiles: every workgroup of the emit phase turns the totals into offsets for itself, in LDS (a
// few KB from L2, next to the loads of its picks).  Larger hops: the workgroup of the mark phase that finishes last does it
// once.  It is found with counters, and its
// hand-off needs no fence: the totals are relaxed device-scope atomics, complete before the counter moves.  But the counters
// are three more round trips at the end of the mark phase: where a launch is short that costs more than the repeated scans
// (1,024-seed FCR steps on the 169k-node graph: launches of 11.9 us instead of 11.2).
// settle (blocking steps, which have a launch to themselves): one pass with hand-offs between workgroups, one launch less.  Every
// hand-off is ONE 64-bit word that carries its own validity (a version tag), stored and loaded with relaxed device-scope
// atomics: no fence, nothing to clear between hops.
//   agg[j]    tile j's totals: tag 32 | edges 16 | firsts 16; a tile sums the words of the tiles before it
//   pref      the running totals after every LOOKBACK_BLOCK tiles (per relation, per node type): a tile reads at most
//             LOOKBACK_BLOCK words, 16 per thread
//   recs[g / 16]  tag 17 | number of the first one 31 | mask 16
// A workgroup only waits for workgroups with smaller numbers of the same slice, which start earlier or at the same time
// (dispatch is in order on every XCD), so the waits end; they are bounded all the same.
// ------------------------------------------------------------------------------------------
constexpr int ITEMS = TILE / TILE_THREADS;   // pick slots per thread
static_assert(ITEMS == 4 && TILE_THREADS == 256, "four wavefronts of four ballots each");
constexpr uint32_t NO_PICK = 0xFFFFFFFFu;
constexpr int SPIN_LIMIT = 1 << 20;          // polls of a hand-off word (about a microsecond each) before giving up

__device__ __forceinline__ void store_relaxed(uint64_t* p, uint64_t v) {
  __hip_atomic_store((unsigned long long*)p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Waits until word *p, last seen as `w`, carries `tag` above bit SHIFT.
template <int SHIFT>
__device__ __forceinline__ uint64_t await_word(const uint64_t* p, uint64_t w, uint32_t tag, int32_t* state) {
  int polls = 0;
  while ((uint32_t)(w >> SHIFT) != tag) {
    if (++polls > SPIN_LIMIT) { atomicOr(&state[ST_ERROR], ERR_HANDOFF); return 0ull; }
    __builtin_amdgcn_s_sleep(1);
    w = load_relaxed(p);
  }
  return w;
}

struct SettleLds {
  uint32_t wave[4];                          // firsts | edges << 16 of the tile, per wavefront
  uint32_t sum_first[4], sum_edge[4];        // sums over the tiles before, per wavefront
  uint32_t tot_first[GSS_MAX_NODE_TYPES], tot_edge[GSS_MAX_RELATIONS];
  union {
    uint64_t recs[TILE / 16];                // settle: the tile's own words of recs[]
    struct {                                 // mark, emit: scratch of the offsets' scan
      int scan[32];
      uint32_t rel_first[GSS_MAX_RELATIONS], add_first[GSS_MAX_RELATIONS], add_edge[GSS_MAX_RELATIONS];
    };
    int is_last;
  };
  uint2 off[EMIT_SCAN_TILES];                // emit: new nodes and edges before a tile
};

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o);
  return v;
}

// Sums of the firsts / edges words of the tiles [from, to) over the workgroup; of the firsts only those of the relations
// in the set `same`, of the edges only those of tiles >= edge_from.  (One barrier inside; L->sum_* must be free.)
template <class HP>
__device__ __forceinline__ void sum_tiles(const HP& P, const LiveLds* live, SettleLds* L, int from, int to, uint32_t same, int edge_from,
                                          uint32_t& firsts, uint32_t& edges) {
  uint32_t sf = 0u, se = 0u;
  for (int i = from + (int)threadIdx.x; i < to; i += TILE_THREADS) {
    const uint32_t v = (uint32_t)await_word<32>(P.agg + i, load_relaxed(P.agg + i), P.ver, P.state);
    bool count_first = true;
    if constexpr (HP::MAX_R > 1) {
      int r = 0;
      while (r + 1 < P.R && i >= live->first[r + 1]) ++r;
      count_first = (same >> r) & 1u;
    }
    if (count_first) sf += v & 0xFFFFu;
    if (HP::MAX_R == 1 || i >= edge_from) se += v >> 16;
  }
  sf = wave_sum(sf);
  se = wave_sum(se);
  if (lane_id() == 0) { L->sum_first[threadIdx.x >> 6] = sf; L->sum_edge[threadIdx.x >> 6] = se; }
  __syncthreads();
  firsts = L->sum_first[0] + L->sum_first[1] + L->sum_first[2] + L->sum_first[3];
  edges = L->sum_edge[0] + L->sum_edge[1] + L->sum_edge[2] + L->sum_edge[3];
}

// Relations with source type s, as a bit set.
template <class HP>
__device__ __forceinline__ uint32_t relations_from(const HP& P, int s) {
  if constexpr (HP::MAX_R == 1) return 1u;
  uint32_t m = 0u;
  for (int q = 0; q < P.R; ++q) m |= (rel_of(P, q).src_type == s ? 1u : 0u) << q;
  return m;
}

// The hop's counts (num_src per node type = the next frontier, num_edges per relation) from the totals in tot_*, and,
// after the last hop, the device state (counts of every hop, error flag) to pinned host memory: the step needs no copy
// command after its kernels.
template <class HP>
__device__ __forceinline__ void write_counts(const HP& P, const uint32_t* tot_first, const uint32_t* tot_edge) {
  if (threadIdx.x == 0) {
    for (int r = 0; r < P.R; ++r) P.state[ST_COUNTS + P.edge_count_off + P.hop * P.R + r] = (int32_t)tot_edge[r];
    for (int s = 0; s < P.T; ++s) P.state[ST_COUNTS + (P.hop + 1) * P.T + s] = frontier_count(P, s) + (int32_t)tot_first[s];
  }
  if (P.state_host == nullptr) return;
  __syncthreads();   // this workgroup's own count stores are visible to all its threads
  for (int i = (int)threadIdx.x; i < P.state_words; i += (int)blockDim.x)
    P.state_host[i] = i == ST_ERROR ? __hip_atomic_load(&P.state[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : P.state[i];
}
template <class HP>
__device__ __forceinline__ void write_zero_counts(const HP& P, SettleLds* L) {
  for (int i = (int)threadIdx.x; i < GSS_MAX_RELATIONS; i += TILE_THREADS) L->tot_edge[i] = 0u;
  for (int i = (int)threadIdx.x; i < GSS_MAX_NODE_TYPES; i += TILE_THREADS) L->tot_first[i] = 0u;
  __syncthreads();
  write_counts(P, L->tot_first, L->tot_edge);
}

// Order word of every pick of the thread in tile `lt` (first slot g0 + own); NO_PICK where a slot holds none (order words are
// smaller).  The picks themselves are read again where they are needed: registers are what limits this kernel.
template <class HP>
__device__ __forceinline__ void load_order_words(const HP& P, const LiveTile& lt, uint32_t g0, uint32_t own, bool have, const int* ahead, uint32_t* w) {
  const uint32_t key_off = type_of(P, rel_of(P, lt.r).src_type).key_off;
  int id[ITEMS];
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    const uint32_t s = own + 64u * q;
    id[q] = -1;
    if (lt.local0 + s < lt.nslots) id[q] = have ? ahead[q] : P.picks[g0 + s];
  }
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {               // four independent table reads in flight
    w[q] = NO_PICK;
    if (id[q] >= 0) w[q] = table_lookup(P.ht, P.ver, key_off + (uint32_t)id[q], P.state);
  }
}
// First occurrences and picks among the wavefront's slots.
__device__ __forceinline__ void count_wave(const uint32_t* w, uint32_t mine, uint32_t& nf, uint32_t& ne) {
  nf = ne = 0u;
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    nf += (uint32_t)__popcll(__ballot(w[q] == mine + 64u * q));
    ne += (uint32_t)__popcll(__ballot(w[q] != NO_PICK));
  }
}
// Lane l < 16 of a wavefront: mask of the first occurrences among the slots 16 l .. 16 l + 15, and the number of the first
// of them, `num` being that of the wavefront's first.
__device__ __forceinline__ uint32_t firsts_of_16(const uint32_t* w, uint32_t mine, int lane, uint32_t& num) {
  uint64_t m = 0ull, below = 0ull;
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    const uint64_t b = __ballot(w[q] == mine + 64u * q);
    if (lane >= 4 * q) { num += (uint32_t)__popcll(below); m = b; }
    below = b;
  }
  const int sh = 16 * (lane & 3);
  num += (uint32_t)__popcll(m & ((1ull << sh) - 1ull));
  return (uint32_t)(m >> sh) & 0xFFFFu;
}

// Tile totals -> offsets (off[tile]: new nodes and edges before it) and totals (L->tot_*), by one workgroup.  First
// occurrences run over the relations of one source type in ascending order; edges restart per relation.  Four tiles per thread
// and turn.  (FRESH: the totals were written in this launch.)
template <bool FRESH, class HP>
__device__ __forceinline__ void scan_tiles(const HP& P, const LiveLds* live, SettleLds* L, uint2* off) {
  for (int s = 0; s < P.T; ++s) {
    int run_first = 0;
    for (int r = 0; r < P.R; ++r) {
      if (rel_of(P, r).src_type != s) continue;
      const int ntiles = HP::MAX_R == 1 ? live_count(P, live) : live->first[r + 1] - live->first[r];
      const uint32_t* const agg = P.tile_sums + rel_of(P, r).slot_base / TILE;
      uint2* const to = off + rel_of(P, r).slot_base / TILE;
      int run_edge = 0;
      for (int c = 0; c < ntiles; c += 4 * TILE_THREADS) {
        const int t0 = c + 4 * (int)threadIdx.x;
        int pf[4], pe[4], sf = 0, se = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t v = 0u;
          if (t0 + q < ntiles) v = FRESH ? __hip_atomic_load(agg + t0 + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : agg[t0 + q];
          pf[q] = (int)(v & 0xFFFFu); pe[q] = (int)(v >> 16);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) { sf += pf[q]; se += pe[q]; }
        int exf, exe, tf, te;
        block_scan2(sf, se, exf, exe, tf, te, L->scan);
        exf += run_first; exe += run_edge;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (t0 + q < ntiles) to[t0 + q] = make_uint2((uint32_t)exf, (uint32_t)exe);
          exf += pf[q]; exe += pe[q];
        }
        run_first += tf; run_edge += te;
        if (c + 4 * TILE_THREADS < ntiles) __syncthreads();
      }
      if (threadIdx.x == 0) L->tot_edge[r] = (uint32_t)run_edge;
      if constexpr (HP::MAX_R > 1) __syncthreads();
    }
    if (threadIdx.x == 0) L->tot_first[s] = (uint32_t)run_first;
  }
  __syncthreads();
}

// Do the workgroups of the emit phase scan the tile totals themselves?  (Several relations: only if all tiles, dead ones
// between the relations included, fit - they are scanned in one go.)
template <class HP>
__device__ __forceinline__ bool scans_in_emit(const HP& P, int ntiles) {
  return (HP::MAX_R == 1 ? ntiles : P.num_tiles_ub) <= EMIT_SCAN_TILES;
}

// scan_tiles for the emit phase of a graph with several relations: ONE scan over the tiles of all relations (a dead tile
// counts nothing), then the prefix at the start of a relation is taken off again and, for new nodes, the totals of the earlier
// relations from the same source type are put on.
template <class HP>
__device__ __forceinline__ void scan_tiles_of_all(const HP& P, const LiveLds* live, SettleLds* L) {
  const int t0 = 4 * (int)threadIdx.x;
  int rel[4], pf[4], pe[4], sf = 0, se = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) rel[q] = 0;
  for (int r = 1; r < P.R; ++r) {
    const int b = live->base[r];
#pragma unroll
    for (int q = 0; q < 4; ++q) rel[q] += t0 + q >= b ? 1 : 0;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = rel[q];
    uint32_t v = 0u;
    if (t0 + q - live->base[r] < live->first[r + 1] - live->first[r]) v = P.tile_sums[t0 + q];
    pf[q] = (int)(v & 0xFFFFu); pe[q] = (int)(v >> 16);
    sf += pf[q]; se += pe[q];
  }
  int exf, exe, tf, te;
  block_scan2(sf, se, exf, exe, tf, te, L->scan);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    L->off[t0 + q] = make_uint2((uint32_t)exf, (uint32_t)exe);
    exf += pf[q]; exe += pe[q];
  }
  __syncthreads();
  const int me = (int)threadIdx.x;
  if (me < 64) {                         // (one wavefront: its LDS operations are in order)
    volatile uint32_t* const per_rel = L->rel_first;
    uint2 at = make_uint2(0u, 0u), end = make_uint2((uint32_t)tf, (uint32_t)te);
    if (me < P.R) {
      const int b = live->base[me], nb = live->base[me + 1];
      at = b < EMIT_SCAN_TILES ? L->off[b] : end;
      if (nb < EMIT_SCAN_TILES && me + 1 < P.R) end = L->off[nb];
      per_rel[me] = end.x - at.x;
      L->tot_edge[me] = end.y - at.y;
      L->add_edge[me] = 0u - at.y;
    }
    const int my_type = me < P.R ? live->src_type[me] : -1;
    uint32_t earlier = 0u, of_type = 0u;
    for (int q = 0; q < P.R; ++q) {
      const uint32_t n = per_rel[q];
      const int s = live->src_type[q];
      if (q < me && s == my_type) earlier += n;
      if (s == me) of_type += n;
    }
    if (me < P.R) L->add_first[me] = earlier - at.x;
    if (me < P.T) L->tot_first[me] = of_type;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) { L->off[t0 + q].x += L->add_first[rel[q]]; L->off[t0 + q].y += L->add_edge[rel[q]]; }
  __syncthreads();
}

// Is this the last of the n workgroups of the slice that get here?  (Called by all its threads.)  Two levels of counters:
// additions to one address take 11 ns each.  The last one to see a counter clears it for the next hop.
template <class HP>
__device__ __forceinline__ bool last_workgroup(const HP& P, const Wg wg, int n, SettleLds* L) {
  if (threadIdx.x == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the tiles' totals have reached memory
    const int way = wg.x % DONE_WAYS, ways = min(n, DONE_WAYS), share = n / DONE_WAYS + (way < n % DONE_WAYS ? 1 : 0);
    uint32_t* c = P.done + (1 + way) * COUNT_STRIDE;
    bool last = atomicAdd(c, 1u) == (uint32_t)share - 1u;
    if (last) {
      *c = 0u;
      last = atomicAdd(P.done, 1u) == (uint32_t)ways - 1u;
      if (last) *P.done = 0u;
    }
    L->is_last = last ? 1 : 0;
  }
  __syncthreads();
  const bool last = L->is_last != 0;
  __syncthreads();
  return last;
}

template <class HP>
__device__ __forceinline__ void mark_phase(const HP& P, const Wg wg, SettleLds* L, LiveLds* live) {
  const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
  const uint32_t own = 256u * (uint32_t)wave + (uint32_t)lane;           // first of the thread's slots within a tile
  // The picks of the workgroup's first tile are requested before the live counts are known: in relation 0 their address
  // does not depend on them, and the buffer covers every tile of the grid.
  int ahead[ITEMS];
  if (wg.x < P.num_tiles_ub) {
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) ahead[q] = P.picks[(uint32_t)wg.x * TILE + own + 64u * q];
  }
  live_tiles_setup(P, live);
  const int ntiles = live_count(P, live);
  if (ntiles == 0) {
    if (wg.x == 0 && !scans_in_emit(P, 0)) write_zero_counts(P, L);
    return;
  }
  if (wg.x >= ntiles) return;
  for (int j = wg.x; j < ntiles; j += P.gx) {
    const LiveTile lt = live_tile(P, live, j);
    const uint32_t g0 = (uint32_t)rel_of(P, lt.r).slot_base + lt.local0;  // (relation slot bases are multiples of TILE)
    uint32_t w[ITEMS];
    load_order_words(P, lt, g0, own, j == wg.x && lt.r == 0, ahead, w);
    const uint32_t mine = EDGE_BIT | (g0 + own);
    uint32_t nf, ne;
    count_wave(w, mine, nf, ne);
    if (j != wg.x) __syncthreads();               // (the words of the tile before have been read)
    if (lane == 0) L->wave[wave] = nf | (ne << 16);
    __syncthreads();
    uint32_t before = 0u, total = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) { const uint32_t c = L->wave[q]; if (q < wave) before += c; total += c; }
    if (threadIdx.x == 0) __hip_atomic_store(P.tile_sums + g0 / TILE, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) P.order[g0 + own + 64u * q] = w[q];
    uint32_t num = before & 0xFFFFu;
    const uint32_t mask = firsts_of_16(w, mine, lane, num);
    if (lane < 16) P.ranks[(g0 >> 4) + 16u * (uint32_t)wave + (uint32_t)lane] = mask | (num << 16);
  }
  if (scans_in_emit(P, ntiles)) return;
  if (last_workgroup(P, wg, min(ntiles, P.gx), L)) {
    scan_tiles<true>(P, live, L, P.tile_off);
    write_counts(P, L->tot_first, L->tot_edge);
  }
}

// Number of the new node whose first occurrence is slot g, without the offset of the dst nodes.
template <class HP>
__device__ __forceinline__ uint32_t number_of(uint32_t rank, uint32_t tile_first, uint32_t g) {
  return tile_first + (rank >> 16) + (uint32_t)__popc(rank & ((1u << (g & 15u)) - 1u));
}

template <class HP>
__device__ __forceinline__ void emit_phase(const HP& P, const Wg wg, SettleLds* L, LiveLds* live) {
  const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
  const uint32_t own = 256u * (uint32_t)wave + (uint32_t)lane;
  live_tiles_setup(P, live);
  const int ntiles = live_count(P, live);
  // (the grid is sized by an estimate: a workgroup beyond the live tiles has nothing to emit; workgroup 0 stays for the
  // hop's counts)
  const bool scans = scans_in_emit(P, ntiles);
  if (wg.x >= ntiles && !(wg.x == 0 && scans)) return;
  uint32_t w[ITEMS];
  auto load_words = [&](int j) {
    const LiveTile lt = live_tile(P, live, j);
    const uint32_t g0 = (uint32_t)rel_of(P, lt.r).slot_base + lt.local0;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) w[q] = P.order[g0 + own + 64u * q];
  };
  if (wg.x < ntiles) load_words(wg.x);            // (they travel while the totals are scanned)
  if (scans) {
    if constexpr (HP::MAX_R == 1) scan_tiles<false>(P, live, L, L->off); else scan_tiles_of_all(P, live, L);
    if (wg.x == 0) write_counts(P, L->tot_first, L->tot_edge);
  }
  for (int j = wg.x; j < ntiles; j += P.gx) {
    const LiveTile lt = live_tile(P, live, j);
    const RelParam& RP = rel_of(P, lt.r);
    const uint32_t g0 = (uint32_t)RP.slot_base + lt.local0;
    if (j != wg.x) load_words(j);
    uint32_t e = scans ? L->off[g0 / TILE].y : P.tile_off[g0 / TILE].y;
    uint32_t rank[ITEMS], tile_first[ITEMS];      // of the pick's first occurrence, four in flight; and the id, if it is the first
    int id[ITEMS];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
      rank[q] = tile_first[q] = 0u;
      if (w[q] != NO_PICK && w[q] >= EDGE_BIT) {
        const uint32_t g1 = w[q] & ~EDGE_BIT;
        rank[q] = P.ranks[g1 >> 4];
        tile_first[q] = scans ? L->off[g1 / TILE].x : P.tile_off[g1 / TILE].x;
        if (g1 == g0 + own + 64u * q) id[q] = P.picks[g1];
      }
    }
    uint32_t ne = 0u;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) ne += (uint32_t)__popcll(__ballot(w[q] != NO_PICK));
    if (j != wg.x) __syncthreads();
    if (lane == 0) L->wave[wave] = ne;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) if (q < wave) e += L->wave[q];
    const uint32_t num_dst = (uint32_t)frontier_count(P, RP.src_type);
    const uint32_t f = (uint32_t)P.f, i0 = lt.local0 / f, rem0 = lt.local0 - i0 * f;
    int32_t* __restrict__ src_nodes = type_of(P, RP.src_type).src_nodes;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
      const uint64_t valid = __ballot(w[q] != NO_PICK);
      if (w[q] != NO_PICK) {
        uint32_t to = w[q];                       // a dst node: its frontier index
        if (w[q] >= EDGE_BIT) {
          const uint32_t g1 = w[q] & ~EDGE_BIT;
          to = num_dst + number_of<HP>(rank[q], tile_first[q], g1);
          if (g1 == g0 + own + 64u * q) src_nodes[to] = id[q];     // the first occurrence publishes the new source node
        }
        const uint32_t at = e + (uint32_t)__popcll(valid & ((1ull << lane) - 1ull));
        RP.src_local[at] = (int)to;
        // slot / f through a multiplication: exact for rem0 + slot < 1088 and f <= 64
        RP.dst_local[at] = (int)(i0 + (((rem0 + own + 64u * q) * P.f_mul) >> 20));
      }
      e += (uint32_t)__popcll(valid);
    }
  }
}

// Running totals up to and including tile j (the last of its block or of the hop) -> L->tot_*: own totals in firsts / edges
// where there is one relation, else summed up per relation and source type.
template <class HP>
__device__ __forceinline__ void totals(const HP& P, const LiveLds* live, SettleLds* L, int j, int b0, uint32_t firsts, uint32_t edges) {
  if constexpr (HP::MAX_R == 1) {
    if (threadIdx.x == 0) { L->tot_first[0] = firsts; L->tot_edge[0] = edges; }
  } else {
    const uint64_t* prev = P.pref + (size_t)(b0 / LOOKBACK_BLOCK - 1) * (size_t)(P.R + P.T);
    auto before = [&](int at) { return b0 ? (uint32_t)await_word<32>(prev + at, load_relaxed(prev + at), P.ver, P.state) : 0u; };
    __syncthreads();
    if ((int)threadIdx.x < P.T) L->tot_first[threadIdx.x] = before(P.R + (int)threadIdx.x);
    for (int r = 0; r < P.R; ++r) {
      uint32_t f_, e_;
      __syncthreads();
      sum_tiles(P, live, L, max(b0, live->first[r]), min(j + 1, live->first[r + 1]), ~0u, 0, f_, e_);
      if (threadIdx.x == 0) {
        L->tot_edge[r] = e_ + before(r);
        L->tot_first[rel_of(P, r).src_type] += f_;
      }
    }
  }
}

template <class HP>
__device__ __forceinline__ void settle_phase(const HP& P, const Wg wg, SettleLds* L, LiveLds* live) {
  const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
  const uint32_t own = 256u * (uint32_t)wave + (uint32_t)lane;           // first of the thread's slots within a tile
  // The picks of the workgroup's tile are requested before the live counts are known: in relation 0 their address does
  // not depend on them, and the buffer covers every tile of the grid.
  int ahead[ITEMS];
  if (wg.x < P.num_tiles_ub) {
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) ahead[q] = P.picks[(uint32_t)wg.x * TILE + own + 64u * q];
  }
  live_tiles_setup(P, live);
  const int ntiles = live_count(P, live);
  if (ntiles == 0) {
    if (wg.x == 0) write_zero_counts(P, L);
    return;
  }
  // One tile per workgroup, if the grid - sized by an estimate - has enough of them; else consecutive tiles, and what other
  // workgroups wait for goes out for all of them first: the totals of every tile, then the numbers of every tile, then the
  // edges (the tiles are then looked at three times; taken one after the other, every tile would wait for the one before).
  const int per = (ntiles + P.gx - 1) / P.gx;
  const int j0 = wg.x * per, n = min(per, ntiles - j0);
  const uint32_t ver = P.ver, tag17 = P.ver & 0x1FFFFu;
  for (int it = 0; it < (per > 1 ? 3 * n : n); ++it) {
    const int turn = it < n ? 0 : it < 2 * n ? 1 : 2, j = j0 + it - turn * n;
    const bool totals_turn = per == 1 || turn == 0, numbers_turn = per == 1 || turn == 1, edges_turn = per == 1 || turn == 2;
    const LiveTile lt = live_tile(P, live, j);
    const RelParam& RP = rel_of(P, lt.r);
    const uint32_t g0 = (uint32_t)RP.slot_base + lt.local0;              // (relation slot bases are multiples of TILE)
    uint32_t w[ITEMS];
    load_order_words(P, lt, g0, own, per == 1 && lt.r == 0, ahead, w);
    const uint32_t mine = EDGE_BIT | (g0 + own);  // the order word that makes the thread's first slot a first occurrence
    uint32_t nf, ne;
    count_wave(w, mine, nf, ne);
    __syncthreads();                              // (the words of the tile before have been read)
    if (lane == 0) L->wave[wave] = nf | (ne << 16);
    __syncthreads();
    uint32_t before = 0u, total = 0u;             // firsts | edges << 16: of the wavefronts before this one, of the tile
#pragma unroll
    for (int q = 0; q < 4; ++q) { const uint32_t c = L->wave[q]; if (q < wave) before += c; total += c; }
    if (totals_turn && threadIdx.x == 0) store_relaxed(P.agg + j, ((uint64_t)ver << 32) | total);
    if (!numbers_turn && !edges_turn) continue;
    // ---- the tiles before: offset of the new nodes of this source type, and of the relation's edges ----
    const int b0 = j / LOOKBACK_BLOCK * LOOKBACK_BLOCK;
    uint32_t off_first = 0u, off_edge = 0u;
    if (j > b0) sum_tiles(P, live, L, b0, j, relations_from(P, RP.src_type), live_first<HP>(live, lt.r), off_first, off_edge);
    if (b0) {
      const uint64_t* prev = P.pref + (size_t)(b0 / LOOKBACK_BLOCK - 1) * (size_t)(P.R + P.T);
      off_edge += (uint32_t)await_word<32>(prev + lt.r, load_relaxed(prev + lt.r), ver, P.state);
      off_first += (uint32_t)await_word<32>(prev + P.R + RP.src_type, load_relaxed(prev + P.R + RP.src_type), ver, P.state);
    }
    const bool last = j == ntiles - 1;
    const bool block_end = j + 1 == b0 + LOOKBACK_BLOCK;
    uint32_t e = off_edge + (before >> 16);       // of the wavefront's first edge
    // ---- numbers of the first occurrences, 16 slots a word ----
    {
      uint32_t num = (uint32_t)frontier_count(P, RP.src_type) + off_first + (before & 0xFFFFu);
      const uint32_t mask = firsts_of_16(w, mine, lane, num);
      const uint64_t rec = ((uint64_t)tag17 << 47) | ((uint64_t)num << 16) | mask;
      if (lane < 16 && numbers_turn) {
        store_relaxed(P.recs + (g0 >> 4) + 16u * (uint32_t)wave + (uint32_t)lane, rec);
      }
      if (lane < 16) L->recs[16 * wave + lane] = rec;
    }
    if (numbers_turn && (block_end || last)) totals(P, live, L, j, b0, off_first + (total & 0xFFFFu), off_edge + (total >> 16));
    __syncthreads();
    if (numbers_turn && block_end && !last && (int)threadIdx.x < P.R + P.T) {
      const int q = (int)threadIdx.x;
      store_relaxed(P.pref + (size_t)(b0 / LOOKBACK_BLOCK) * (size_t)(P.R + P.T) + q,
                    ((uint64_t)ver << 32) | (q < P.R ? L->tot_edge[q] : L->tot_first[q - P.R]));
    }
    if (numbers_turn && last) write_counts(P, L->tot_first, L->tot_edge);
    if (!edges_turn) continue;
    // ---- the repeats' numbers (first occurrences are never later), four words in flight ----
    uint64_t rec[ITEMS];
    int id[ITEMS];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
      const uint32_t g1 = w[q] & ~EDGE_BIT;
      rec[q] = 0ull;
      if (w[q] != NO_PICK && w[q] >= EDGE_BIT)
        rec[q] = (g1 ^ g0) < TILE ? L->recs[(g1 & (TILE - 1)) >> 4] : load_relaxed(P.recs + (g1 >> 4));
      if (w[q] == mine + 64u * q) id[q] = P.picks[g1];
    }
    const uint32_t f = (uint32_t)P.f, i0 = lt.local0 / f, rem0 = lt.local0 - i0 * f;
    int32_t* __restrict__ src_nodes = type_of(P, RP.src_type).src_nodes;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
      const uint64_t valid = __ballot(w[q] != NO_PICK);
      if (w[q] != NO_PICK) {
        uint32_t to = w[q];                       // a dst node: its frontier index
        if (w[q] >= EDGE_BIT) {
          const uint32_t g1 = w[q] & ~EDGE_BIT;
          const uint64_t v = await_word<47>(P.recs + (g1 >> 4), rec[q], tag17, P.state);
          to = (uint32_t)(v >> 16) & 0x7FFFFFFFu;
          to += (uint32_t)__popc((uint32_t)v & ((1u << (g1 & 15u)) - 1u));
          if (w[q] == mine + 64u * q) src_nodes[to] = id[q];     // the first occurrence publishes the new source node
        }
        const uint32_t at = e + (uint32_t)__popcll(valid & ((1ull << lane) - 1ull));
        RP.src_local[at] = (int)to;
        // slot / f through a multiplication: exact for rem0 + slot < 1088 and f <= 64
        RP.dst_local[at] = (int)(i0 + (((rem0 + own + 64u * q) * P.f_mul) >> 20));
      }
      e += (uint32_t)__popcll(valid);
    }
  }
}

// ------------------------------------------------------------------------------------------
// step_tick_kernel: a one-dimensional grid holds the workgroups of all slices back to back (slice i
// owns [end[i-1], end[i]), x-major within its gx * gy rectangle), so no workgroup is launched in vain.
// ------------------------------------------------------------------------------------------
template <int W, bool STAGED>
union TickLds {
  GroupLdsT<W> group[GrpT<W>::PER_WG];
  SettleLds settle;
  typename std::conditional<STAGED, DedupeLds, int>::type stage;    // only in the builds with the LDS stage of the dedupe
};
// Scalar registers, not vector registers or LDS, decide how many workgroups a CU holds: with the 106 the
// compiler takes by itself 6 were resident per CU (measured: 191 per XCD at the peak of a full tick), capped at
// 96 it is 7 (223 per XCD); the spills go to lanes of a vector register.  Capping further for 8 costs more in
// spill code than the slots bring.
// The workgroup `block` of the slice with arguments P.
template <int W, bool DENSE, class HP>
__device__ __forceinline__ void run_slice(const HP& P, int block, const ChainArgs* C = nullptr) {
  // rows 0 .. gy-1 of the slice are gx workgroups wide, the gyd rows after them gxd (sample phase: the
  // rows of the node types need one thread per frontier node, not one 32-lane group)
  Wg wg;
  wg.x = block;
  wg.y = 0;
  while (wg.y < P.gy && wg.x >= P.gx) { wg.x -= P.gx; ++wg.y; }
  if (wg.y == P.gy && P.gxd > 0)
    while (wg.x >= P.gxd) { wg.x -= P.gxd; ++wg.y; }
  constexpr bool STAGED = std::is_base_of<HopParamsStaged, HP>::value;
  __shared__ TickLds<W, STAGED> lds;
  __shared__ LiveLds live;
  __shared__ typename std::conditional<std::is_same<HP, HopParamsChain>::value && W == 32, ChainLds, int>::type chain_lds;
  (void)chain_lds;
  switch (P.phase) {
    case PH_SAMPLE: sample_phase(P, wg, lds.group); break;
    case PH_INSERT: insert_phase<STAGED>(P, wg, &live, reinterpret_cast<DedupeLds*>(&lds.stage)); break;
    case PH_MARK:   mark_phase(P, wg, &lds.settle, &live); break;
    case PH_EMIT:   emit_phase(P, wg, &lds.settle, &live); break;
    case PH_SETTLE: settle_phase(P, wg, &lds.settle, &live); break;
    default:
      if constexpr (std::is_same<HP, HopParamsChain>::value && W == 32) {     // (only this build holds the visit-once code)
        if (P.phase == PH_PLACE) place_phase(P, wg, &live, reinterpret_cast<DedupeLds*>(&lds.stage));
        else if (P.phase == PH_CHAIN) chain_phase<!DENSE>(P, *C, wg, lds.group, &chain_lds);
      }
      break;
  }
}
__device__ __forceinline__ void report_start(const LaunchMark& m) {
  if (m.started && blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(m.started, m.number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
template <class TP, int W, bool DENSE = false>
__device__ __forceinline__ void tick_body(const TP& M_by_value) {
  // The builds that carry a chain's arguments read their arguments where the launch put them, in the kernel argument
  // segment (constant memory: scalar loads with run-time offsets), not through the by-value parameter: indexing that with
  // the slice number made the compiler copy the whole structure to scratch memory there (from 8 slices on).  The other
  // builds keep the parameter: with the pointer the 1,024-seed FCR workload ran 4 % slower.
  typedef const __attribute__((address_space(4))) TP* KernargPtr;
  const TP& M = (TP::HAS_CHAIN || TP::Slice::MAX_R > 1) ? *(const TP*)(KernargPtr)__builtin_amdgcn_kernarg_segment_ptr() : M_by_value;
  int z = 0;
#pragma unroll
  for (int i = 0; i < TP::SLICES - 1; ++i) z += ((int)blockIdx.x >= M.end[i]) ? 1 : 0;
  report_start(M.mark);                  // (not first: its argument then travels with the bounds)
  const ChainArgs* chain = nullptr;
  if constexpr (TP::HAS_CHAIN) chain = &M.chain;
  run_slice<W, DENSE>(M.s[z], (int)blockIdx.x - (z ? M.end[z - 1] : 0), chain);
}
// Two builds of the same kernel.  With its scalar registers capped at 96 the kernel takes 67-72 vector registers:
// seven workgroups per CU.  The dense build is held to 64 (eight workgroups per CU) and pays for it with more scalar
// registers parked in vector lanes.  Launches of several times the chip's capacity gain from the eighth workgroup
// (65,536-seed steps -4 %, the seven-relation workload -1.5 %); ordinary ticks, whose time is set by the dependent
// chains of a few narrow slices, lose 3-6 % on the workloads with a refresh in the sample phase.
template <class TP, int W>
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_sgpr(96))) void step_tick_kernel(TP M) { tick_body<TP, W>(M); }
template <class TP, int W = 32>
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_sgpr(96), amdgpu_waves_per_eu(8, 8))) void step_tick_dense_kernel(TP M) {
  tick_body<TP, W, true>(M);
}
// The compact form for one-relation graphs: the slice's full arguments are put together from the launch's shared
// part, the slice's own part and the slot's entry of the device table (one more scalar load at the start).
template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_sgpr(96))) void step_tick_mono_kernel(TickMono<D> M) {
  int z = 0;
#pragma unroll
  for (int i = 0; i < D - 1; ++i) z += ((int)blockIdx.x >= M.end[i]) ? 1 : 0;
  const MonoSlice& c = M.s[z];
  report_start(M.mark);
  // (constant address space: scalar loads.  Entries only change between launches.)
  const __attribute__((address_space(4))) SlotConst& sc = ((const __attribute__((address_space(4))) SlotConst*)(uintptr_t)M.h.slots)[c.slot];
  HopParamsMonoRegs H;
  H.ht.direct = sc.ht.direct; H.ht.entries = sc.ht.entries; H.ht.mask = sc.ht.mask;
  H.state = sc.state;
  H.state_host = c.publish ? sc.state_host : nullptr;
  H.picks = sc.picks; H.order = sc.order; H.tile_off = sc.tile_off;
  if (c.phase == PH_SETTLE) { H.agg = sc.agg; H.recs = sc.recs; H.pref = sc.pref; }
  else { H.tile_sums = sc.tile_sums; H.ranks = sc.ranks; H.done = sc.done; }
  H.phase = c.phase;
  H.gx = c.gx; H.gy = c.gy; H.gxd = c.gxd; H.gyd = c.gyd;
  H.R = 1; H.T = 1;
  H.hop = c.hop; H.f = c.f; H.k = M.h.k; H.S = M.h.S;
  H.n_new = c.n_new; H.mode = M.h.mode; H.refresh_now = c.refresh_now; H.band_offset = c.band_offset;
  H.num_tiles_ub = c.num_tiles_ub; H.edge_count_off = M.h.edge_count_off;
  H.f_mul = (1u << 20) / (uint32_t)c.f + 1u; H.state_words = M.h.state_words;
  H.shared = M.h.shared; H.layer = c.layer;
  H.insert_split = c.insert_split; H.slot = c.slot;
  H.ver = c.ver; H.step = c.step; H.layer_word = c.layer_word; H.seed_lo = M.h.seed_lo; H.seed_hi = M.h.seed_hi;
  H.rel[0].table = c.table; H.rel[0].src_local = c.src_local; H.rel[0].dst_local = c.dst_local;
  H.rel[0].slot_base = 0; H.rel[0].src_type = 0; H.rel[0].dst_type = 0;
  H.type[0].frontier = c.frontier; H.type[0].src_nodes = c.src_nodes;
  H.type[0].key_off = M.h.key_off; H.type[0].n_nodes = M.h.n_nodes;
  H.type[0].count_override = c.count_override; H.type[0].frontier_cap = c.frontier_cap;
  H.relc[0] = M.h.relc;
  run_slice<32, false>(H, (int)blockIdx.x - (z ? M.end[z - 1] : 0));
}

// ------------------------------------------------------------------------------------------
// Graph validation, cache read-out, checksum
// ------------------------------------------------------------------------------------------
__global__ void validate_graph_kernel(const void* indptr, int is64, int64_t n_dst, const int32_t* indices,
                                      int64_t nnz, int64_t n_src, int32_t* state) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nth = (int64_t)gridDim.x * blockDim.x;
  bool bad = false;
  if (tid == 0) bad |= load_indptr(indptr, is64, 0) != 0 || load_indptr(indptr, is64, n_dst) != nnz;
  for (int64_t v = tid; v < n_dst; v += nth) {
    const int64_t d = load_indptr(indptr, is64, v + 1) - load_indptr(indptr, is64, v);
    bad |= d < 0 || d >= (int64_t(1) << 31);
  }
  for (int64_t e = tid; e < nnz; e += nth) bad |= (uint64_t)(int64_t)indices[e] >= (uint64_t)n_src;
  if (bad) atomicOr(&state[ST_ERROR], ERR_GRAPH);
}

__global__ void cache_read_kernel(const int32_t* table, const int32_t* row_of, int64_t n, int k, int S, int32_t* out) {
  const int64_t total = n * k;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < total; c += (int64_t)gridDim.x * blockDim.x) {
    const int64_t v = c / k;
    const int j = (int)(c - v * k);
    const int64_t at = row_of ? (int64_t)row_of[v] : v;
    out[c] = at >= 0 ? table[at * S + j] : -1;
  }
}

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__global__ void cache_checksum_kernel(const int32_t* table, const int32_t* row_of, int64_t n, int k, int S,
                                      unsigned long long* out) {
  const int64_t total = n * k;
  uint64_t sum = 0;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < total; c += (int64_t)gridDim.x * blockDim.x) {
    const int64_t v = c / k;
    const int j = (int)(c - v * k);
    const int64_t at = row_of ? (int64_t)row_of[v] : v;
    const int val = at >= 0 ? table[at * S + j] : -1;
    sum += mix64((uint64_t)c * 0x9E3779B97F4A7C15ull + (uint64_t)(uint32_t)val);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint32_t lo = __shfl_down((uint32_t)sum, o), hi = __shfl_down((uint32_t)(sum >> 32), o);
    sum += ((uint64_t)hi << 32) | lo;
  }
  if (lane_id() == 0) atomicAdd(out, (unsigned long long)sum);
}

// The same checksum without any allocation: every workgroup reduces one chunk of CK_CHUNK cells into its own word of a
// static scratch array (no atomics, nothing to clear), and a second one-workgroup kernel adds the words up into the
// caller's device word.  The array's name is only a host-side stand-in: kernels get the address that
// hipGetSymbolAddress returns for the current device (each GPU holds its own copy).
constexpr int CK_CHUNK = 16384;
constexpr int CK_MAX_PARTIALS = (int)(GSS_CHECKSUM_STATIC_MAX_CELLS / CK_CHUNK);
static __device__ __align__(256) unsigned long long scratch[CK_MAX_PARTIALS];   // 128 KB on every GPU the library runs on

__device__ __forceinline__ uint64_t block_sum_u64(uint64_t sum, unsigned long long* lds) {   // 256 threads; valid in thread 0
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint32_t lo = __shfl_down((uint32_t)sum, o), hi = __shfl_down((uint32_t)(sum >> 32), o);
    sum += ((uint64_t)hi << 32) | lo;
  }
  if (lane_id() == 0) lds[threadIdx.x >> 6] = sum;
  __syncthreads();
  return lds[0] + lds[1] + lds[2] + lds[3];
}

__global__ __launch_bounds__(256) void checksum_partials_kernel(const int32_t* table, const int32_t* row_of, int64_t n, int k,
                                                                int S, unsigned long long* partials) {
  __shared__ unsigned long long lds[4];
  const int64_t total = n * k, c0 = (int64_t)blockIdx.x * CK_CHUNK;
  uint64_t sum = 0;
  for (int i = (int)threadIdx.x; i < CK_CHUNK; i += 256) {
    const int64_t c = c0 + i;
    if (c >= total) break;
    const int64_t v = c / k;
    const int j = (int)(c - v * k);
    const int64_t at = row_of ? (int64_t)row_of[v] : v;
    const int val = at >= 0 ? table[at * S + j] : -1;
    sum += mix64((uint64_t)c * 0x9E3779B97F4A7C15ull + (uint64_t)(uint32_t)val);
  }
  const uint64_t t = block_sum_u64(sum, lds);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

__global__ __launch_bounds__(256) void checksum_finish_kernel(const unsigned long long* partials, int count, unsigned long long* out) {
  __shared__ unsigned long long lds[4];
  uint64_t sum = 0;
  for (int i = (int)threadIdx.x; i < count; i += 256) sum += partials[i];
  const uint64_t t = block_sum_u64(sum, lds);
  if (threadIdx.x == 0) *out = t;
}

// Row map of the degree split (built once, when the sampler is created).  Nodes are taken in chunks
// of 1024: count the nodes with deg > theta per chunk, scan the chunk counts (one workgroup), then
// number the nodes of every chunk.
constexpr int MAP_CHUNK = 1024;
__device__ __forceinline__ bool has_row(const void* indptr, int is64, int64_t v, int64_t n, int32_t theta) {
  return v < n && load_indptr(indptr, is64, v + 1) - load_indptr(indptr, is64, v) > (int64_t)theta;
}
__global__ __launch_bounds__(MAP_CHUNK) void row_map_count_kernel(const void* indptr, int is64, int64_t n, int32_t theta,
                                                                  int32_t* chunk_counts) {
  __shared__ int lds[32];
  const int64_t nchunks = (n + MAP_CHUNK - 1) / MAP_CHUNK;
  for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
    const int flag = has_row(indptr, is64, c * MAP_CHUNK + threadIdx.x, n, theta) ? 1 : 0;
    int e0, e1, t0, t1;
    block_scan2(flag, 0, e0, e1, t0, t1, lds);
    if (threadIdx.x == 0) chunk_counts[c] = t0;
    __syncthreads();
  }
}
__global__ __launch_bounds__(MAP_CHUNK) void row_map_scan_kernel(int64_t nchunks, int32_t* chunk_counts, int32_t* num_rows) {
  __shared__ int lds[32];
  int run = 0;
  for (int64_t c0 = 0; c0 < nchunks; c0 += MAP_CHUNK) {
    const int64_t c = c0 + threadIdx.x;
    const int cnt = c < nchunks ? chunk_counts[c] : 0;
    int e0, e1, t0, t1;
    block_scan2(cnt, 0, e0, e1, t0, t1, lds);
    if (c < nchunks) chunk_counts[c] = run + e0;
    run += t0;
    __syncthreads();
  }
  if (threadIdx.x == 0) *num_rows = run;
}
__global__ __launch_bounds__(MAP_CHUNK) void row_map_assign_kernel(const void* indptr, int is64, int64_t n, int32_t theta,
                                                                   const int32_t* chunk_counts, int32_t* row_of) {
  __shared__ int lds[32];
  const int64_t nchunks = (n + MAP_CHUNK - 1) / MAP_CHUNK;
  for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
    const int64_t v = c * MAP_CHUNK + threadIdx.x;
    const int flag = has_row(indptr, is64, v, n, theta) ? 1 : 0;
    int e0, e1, t0, t1;
    block_scan2(flag, 0, e0, e1, t0, t1, lds);
    if (v < n) row_of[v] = flag ? chunk_counts[c] + e0 : -1;
    __syncthreads();
  }
}

// list[row_of[v]] = v for the nodes that have a row in the map
__global__ void list_from_map_kernel(const int32_t* __restrict__ map, int64_t n, int32_t* __restrict__ list) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
    const int r = map[v];
    if (r >= 0) list[r] = (int32_t)v;
  }
}

// ------------------------------------------------------------------------------------------
// Feature gather (the value side of the K-V cache: out[i] = H[ids[i]]), the one HBM-bound kernel of the library.
// A row is ceil(row_bytes / sizeof(VEC)) chunks, the last one moved back so that it ends with the row (it may repeat bytes
// of the one before), so every row from sizeof(VEC) bytes on moves in VEC accesses, whatever its length and address: the
// hardware takes unaligned 16-byte accesses.  (Chosen by alignment instead, rows of an odd number of bf16 values moved byte by
// byte.)  The chunks of all rows are dealt out to the threads in order: no lane idles however many chunks a row has, and
// every thread has GATHER_UNROLL rows in flight (1, 2, 4, 8: two and four are within 1 %, eight 5 % slower).  The output is
// written around the caches (non-temporal stores: nothing of it is read here again, and the table's popular rows keep
// their place): 133k rows of 400 bytes 21.1 us instead of 24.7 with ordinary stores and 26.3 with 32 lanes per row - 5.05 TB/s,
// a plain copy reaches 4.8 on this card; 1,501 rows of 5,732 bytes 3.9 us instead of 9.6, 100k rows of 301 bf16 22.6 instead of 77.6.
// ------------------------------------------------------------------------------------------
constexpr int GATHER_UNROLL = 2, GATHER_CHUNKS = 256 * GATHER_UNROLL;      // chunks of a workgroup
template <class VEC> struct __attribute__((packed, aligned(1))) Unaligned { VEC v; };
template <class VEC>
__device__ __forceinline__ void store_streaming(char* at, const VEC& v) {
  if constexpr (sizeof(VEC) == 16) {
    typedef uint32_t Quad __attribute__((ext_vector_type(4), aligned(1)));
    __builtin_nontemporal_store(Quad{v.x, v.y, v.z, v.w}, reinterpret_cast<Quad*>(at));
  } else {
    reinterpret_cast<Unaligned<VEC>*>(at)->v = v;
  }
}
template <class VEC>
__global__ __launch_bounds__(256) void gather_rows_kernel(const char* __restrict__ table, int64_t num_rows, int64_t row_bytes, int chunks,
                                                          uint32_t inv_chunks, const int32_t* __restrict__ ids, int64_t num_ids,
                                                          char* __restrict__ out) {
  // chunk c0 + n of the workgroup, c0 = row0 * chunks + rest: row row0 + (rest + n) / chunks
  const int64_t c0 = (int64_t)blockIdx.x * GATHER_CHUNKS, row0 = c0 / chunks;
  const uint32_t rest = (uint32_t)(c0 - row0 * chunks), left = (uint32_t)min(num_ids - row0, (int64_t)0x7FFFFFFF);
  ids += row0;
  out += row0 * row_bytes;
  uint32_t q[GATHER_UNROLL];             // row of the chunk, from row0 on
  int32_t id[GATHER_UNROLL];
  VEC v[GATHER_UNROLL];
  auto within = [&](int u) {             // first byte of the chunk within its row
    const uint32_t n = rest + 256u * u + threadIdx.x;
    return min((int64_t)((n - q[u] * (uint32_t)chunks) * (uint32_t)sizeof(VEC)), row_bytes - (int64_t)sizeof(VEC));
  };
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u) {
    const uint32_t n = rest + 256u * u + threadIdx.x;
    q[u] = chunks == 1 ? n : __umulhi(n, inv_chunks);        // n / chunks: exact for n <= 1024 + chunks, chunks <= 2^16
    id[u] = ids[min(q[u], left - 1u)];
  }
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u) {
    const bool ok = (uint32_t)id[u] < (uint32_t)min(num_rows, (int64_t)0x80000000ll);
    v[u] = reinterpret_cast<const Unaligned<VEC>*>(table + (ok ? (int64_t)id[u] : 0ll) * row_bytes + within(u))->v;
    if (!ok) v[u] = VEC{};
  }
#pragma unroll
  for (int u = 0; u < GATHER_UNROLL; ++u)
    if (q[u] < left) store_streaming(out + (int64_t)q[u] * row_bytes + within(u), v[u]);
}

__global__ void store_slot_kernel(SlotConst* at, SlotConst value) {
  if (threadIdx.x == 0) *at = value;
}

__global__ void fill_i64_kernel(long long* p, int64_t n, long long value) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = value;
}

// ------------------------------------------------------------------------------------------
// Launch wrappers (host)
// ------------------------------------------------------------------------------------------
static inline unsigned clamp_grid(int64_t want, int64_t cap) {
  if (want < 1) want = 1;
  return (unsigned)(want < cap ? want : cap);
}

hipError_t launch_fill_full(const FillParams& P, hipStream_t st, LaunchTimer* timer) {
  const unsigned grid = clamp_grid((P.n_dst + FILL_CHUNK - 1) / FILL_CHUNK, 8192);
  hipEvent_t start = nullptr, stop = nullptr;
  void (*const kernel)(FillParams) = P.k > 32 ? fill_full_kernel<64> : P.k > 20 ? fill_full_kernel<32> : P.k > 16 ? fill_full_kernel<21>
                                                                     : fill_full_kernel<16>;   // lanes per heavy row
  if (timer && timer->bracket(KID_FILL_FULL, &start, &stop))      // the events get the dispatch's own start / end times
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, start, stop, 0, P);
  else
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, P);
  return hipGetLastError();
}

hipError_t launch_fill_heavy(const FillParams& P, const int32_t* heavy, int64_t nheavy, hipStream_t st, LaunchTimer* timer) {
  if (nheavy <= 0) return hipSuccess;
  const int groups = P.k > 32 ? 4 : P.k > 20 ? 8 : P.k > 16 ? 12 : 16;
  const unsigned grid = clamp_grid((nheavy * P.ntab + groups - 1) / groups, 16384);
  hipEvent_t start = nullptr, stop = nullptr;
  void (*const kernel)(FillParams, const int32_t*, int64_t) =
      P.k > 32 ? fill_heavy_kernel<64> : P.k > 20 ? fill_heavy_kernel<32> : P.k > 16 ? fill_heavy_kernel<21> : fill_heavy_kernel<16>;
  if (timer && timer->bracket(KID_FILL_FULL, &start, &stop))
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, start, stop, 0, P, heavy, nheavy);
  else
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, P, heavy, nheavy);
  return hipGetLastError();
}

hipError_t launch_list_from_map(const int32_t* map, int64_t n, int32_t* list, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(list_from_map_kernel, dim3(clamp_grid((n + 255) / 256, 8192)), dim3(256), 0, st, map, n, list);
  return hipGetLastError();
}

int tick_capacity(int R, int T) {
  if (R == 1 && T == 1) return TICK_MONO_SLICES;
  if (R <= HopParamsSmall::MAX_R && T <= HopParamsSmall::MAX_T) return 9;
  if (R <= HopParamsMid::MAX_R && T <= HopParamsMid::MAX_T) return 6;
  return 4;
}

template <class HP, int D>
static hipError_t launch_tick_t(const HopParams* P, int n, const RelConst* relc_host, const RelConst* relc_dev,
                                const ChainArgs* chain, const LaunchMark& mark, hipStream_t st, LaunchTimer* timer,
                                hipEvent_t done, bool dense, int width = 0) {
  using TP = TickT<HP, D>;
  static_assert(sizeof(TP) <= 4000, "kernel arguments are limited to 4 KB");
  TP M;
  M.mark = mark;
  if constexpr (TP::HAS_CHAIN) {
    if (chain) M.chain = *chain; else memset(static_cast<void*>(&M.chain), 0, sizeof M.chain);
  } else if (chain) {
    return hipErrorInvalidValue;
  }
  int total = 0;
  for (int i = 0; i < D; ++i) {
    const HopParams& src = P[i < n ? i : 0];        // unused slices repeat the first and own no workgroup
    static_cast<HopCommon&>(M.s[i]) = static_cast<const HopCommon&>(src);
    for (int r = 0; r < HP::MAX_R; ++r) M.s[i].rel[r] = src.rel[r];
    for (int t = 0; t < HP::MAX_T; ++t) M.s[i].type[t] = src.type[t];
    M.s[i].set_consts(relc_host, relc_dev);
    if (i < n) total += src.gx * src.gy + src.gxd * src.gyd;
    M.end[i] = total;
  }
  hipEvent_t start = nullptr, stop = nullptr;
  // rows of more than 32 slots: the build with one node per wavefront (it has no dense variant, and no chain code);
  // rows of up to 20 / 16 slots on one-relation graphs: the builds with three / four nodes per wavefront
  const bool wide = P[0].k > 32;
  void (*kernel)(TP) = dense ? step_tick_dense_kernel<TP> : step_tick_kernel<TP, 32>;
  if constexpr (TP::HAS_CHAIN) {
    if (wide || (width != 0 && width != 32)) return hipErrorInvalidValue;
  } else if (wide) {
    if (width != 0 && width != 64) return hipErrorInvalidValue;
    kernel = step_tick_kernel<TP, 64>;
  } else if (width == 21 || width == 16) {
    if constexpr (std::is_same<HP, HopParamsMono>::value) {
      if (width == 21) kernel = dense ? step_tick_dense_kernel<TP, 21> : step_tick_kernel<TP, 21>;
      else kernel = dense ? step_tick_dense_kernel<TP, 16> : step_tick_kernel<TP, 16>;
    } else {
      return hipErrorInvalidValue;
    }
  } else if (width != 0 && width != 32) {
    return hipErrorInvalidValue;
  }
  if (timer && timer->bracket(KID_STEP_TICK, &start, &stop))
    hipExtLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(256), 0, st, start, stop, 0, M);
  else if (done)   // the dispatch itself completes the event: no separate marker between this launch and the next
    hipExtLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(256), 0, st, nullptr, done, 0, M);
  else
    hipLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(256), 0, st, M);
  if (timer && done) {
    const hipError_t e = hipEventRecord(done, st);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

// The compact launch: slices of one-relation graphs, up to TICK_MONO_SLICES of them.
static hipError_t launch_tick_mono(const HopParams* P, int n, const RelConst* relc_host, const SlotConst* slots_dev,
                                   const LaunchMark& mark, hipStream_t st, LaunchTimer* timer, hipEvent_t done) {
  using TM = TickMono<TICK_MONO_SLICES>;
  static_assert(sizeof(TM) <= 4000, "kernel arguments are limited to 4 KB");
  TM M;
  memset(static_cast<void*>(&M), 0, sizeof M);
  M.mark = mark;
  const HopParams& A = P[0];
  M.h.relc = relc_host[0];
  M.h.slots = slots_dev;
  M.h.key_off = A.type[0].key_off; M.h.n_nodes = A.type[0].n_nodes;
  M.h.k = A.k; M.h.S = A.S; M.h.mode = A.mode; M.h.shared = A.shared;
  M.h.state_words = A.state_words; M.h.edge_count_off = A.edge_count_off;
  M.h.seed_lo = A.seed_lo; M.h.seed_hi = A.seed_hi;
  int total = 0;
  for (int i = 0; i < TICK_MONO_SLICES; ++i) {
    const HopParams& src = P[i < n ? i : 0];        // unused slices repeat the first and own no workgroup
    MonoSlice& c = M.s[i];
    c.table = src.rel[0].table; c.src_local = src.rel[0].src_local; c.dst_local = src.rel[0].dst_local;
    c.frontier = src.type[0].frontier; c.src_nodes = src.type[0].src_nodes;
    c.count_override = src.type[0].count_override; c.frontier_cap = src.type[0].frontier_cap;
    c.num_tiles_ub = src.num_tiles_ub; c.gx = src.gx; c.gxd = src.gxd; c.band_offset = src.band_offset;
    c.ver = src.ver; c.step = src.step; c.layer_word = src.layer_word;
    c.slot = (uint8_t)src.slot; c.phase = (uint8_t)src.phase; c.hop = (uint8_t)src.hop; c.layer = (uint8_t)src.layer;
    c.f = (uint8_t)src.f; c.n_new = (uint8_t)src.n_new; c.refresh_now = (uint8_t)src.refresh_now;
    c.insert_split = (uint8_t)src.insert_split;
    c.publish = src.state_host ? 1 : 0; c.gy = (uint8_t)src.gy; c.gyd = (uint8_t)src.gyd;
    if (src.rel[0].slot_base != 0 || src.f > 255 || src.n_new > 255 || src.gy > 255 || src.gyd > 255)
      return hipErrorInvalidValue;
    if (i < n) total += src.gx * src.gy + src.gxd * src.gyd;
    M.end[i] = total;
  }
  hipEvent_t start = nullptr, stop = nullptr;
  if (timer && timer->bracket(KID_STEP_TICK, &start, &stop))
    hipExtLaunchKernelGGL(step_tick_mono_kernel<TICK_MONO_SLICES>, dim3((unsigned)total), dim3(256), 0, st, start, stop, 0, M);
  else if (done)
    hipExtLaunchKernelGGL(step_tick_mono_kernel<TICK_MONO_SLICES>, dim3((unsigned)total), dim3(256), 0, st, nullptr, done, 0, M);
  else
    hipLaunchKernelGGL(step_tick_mono_kernel<TICK_MONO_SLICES>, dim3((unsigned)total), dim3(256), 0, st, M);
  if (timer && done) {
    const hipError_t e = hipEventRecord(done, st);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t launch_tick(const HopParams* P, int n, const RelConst* relc_host, const RelConst* relc_dev,
                       const SlotConst* slots_dev, bool chain_build, const ChainArgs* chain, const LaunchMark& mark, hipStream_t st,
                       LaunchTimer* timer, hipEvent_t done, bool dense, int width) {
  if (n < 1 || n > tick_capacity(P[0].R, P[0].T)) return hipErrorInvalidValue;
  const int R = P[0].R, T = P[0].T;
  if (chain_build) {
    if (R != 1 || T != 1 || n > CHAIN_TICK_SLICES) return hipErrorInvalidValue;
    if (n <= 4) return launch_tick_t<HopParamsChain, 4>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense);
    return launch_tick_t<HopParamsChain, CHAIN_TICK_SLICES>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense);
  }
  if (chain) return hipErrorInvalidValue;
  if (P[0].insert_split & 2) {      // the sampler uses the LDS stage of the dedupe: a build of its own (one relation, rows of up to 32 slots)
    if (R != 1 || T != 1 || n > 12 || P[0].k > 32) return hipErrorInvalidValue;
    return launch_tick_t<HopParamsStaged, 12>(P, n, relc_host, relc_dev, nullptr, mark, st, timer, done, dense);
  }
  const bool narrow = width == 21 || width == 16;
  if (narrow && (chain_build || (P[0].insert_split & 2) || R != 1 || T != 1 || n > 12)) return hipErrorInvalidValue;
  if (R == 1 && T == 1 && n > 12) {
    if (!slots_dev || P[0].k > 32) return hipErrorInvalidValue;   // (the compact form has no build for wide rows)
    return launch_tick_mono(P, n, relc_host, slots_dev, mark, st, timer, done);
  }
  if (R == 1 && T == 1) {
    if (n <= 4) return launch_tick_t<HopParamsMono, 4>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense, width);
    if (n <= 8) return launch_tick_t<HopParamsMono, 8>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense, width);
    return launch_tick_t<HopParamsMono, 12>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense, width);
  }
  if (R <= HopParamsSmall::MAX_R && T <= HopParamsSmall::MAX_T) {
    if (n <= 3) return launch_tick_t<HopParamsSmall, 3>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense);
    if (n <= 6) return launch_tick_t<HopParamsSmall, 6>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense);
    return launch_tick_t<HopParamsSmall, 9>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense);
  }
  if (R <= HopParamsMid::MAX_R && T <= HopParamsMid::MAX_T) {
    if (n <= 3) return launch_tick_t<HopParamsMid, 3>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense);
    return launch_tick_t<HopParamsMid, 6>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense);
  }
  if (n <= 2) return launch_tick_t<HopParams, 2>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense);
  return launch_tick_t<HopParams, 4>(P, n, relc_host, relc_dev, chain, mark, st, timer, done, dense);
}

hipError_t launch_validate_graph(const void* indptr, int is64, int64_t n_dst, const int32_t* indices, int64_t nnz,
                                 int64_t n_src, int32_t* state, hipStream_t st) {
  const int64_t work = nnz > n_dst ? nnz : n_dst;
  const unsigned grid = clamp_grid((work + 255) / 256, 8192);
  hipLaunchKernelGGL(validate_graph_kernel, dim3(grid), dim3(256), 0, st, indptr, is64, n_dst, indices, nnz, n_src, state);
  return hipGetLastError();
}

hipError_t launch_cache_read(const int32_t* table, const int32_t* row_of, int64_t n, int k, int S, int32_t* out,
                             hipStream_t st) {
  const unsigned grid = clamp_grid((n * k + 255) / 256, 8192);
  hipLaunchKernelGGL(cache_read_kernel, dim3(grid), dim3(256), 0, st, table, row_of, n, k, S, out);
  return hipGetLastError();
}

hipError_t launch_cache_checksum(const int32_t* table, const int32_t* row_of, int64_t n, int k, int S,
                                 unsigned long long* out, hipStream_t st) {
  const unsigned grid = clamp_grid((n * k + 255) / 256, 4096);
  hipLaunchKernelGGL(cache_checksum_kernel, dim3(grid), dim3(256), 0, st, table, row_of, n, k, S, out);
  return hipGetLastError();
}

hipError_t launch_cache_checksum_static(const int32_t* table, const int32_t* row_of, int64_t n, int k, int S,
                                        unsigned long long* out, hipStream_t st) {
  constexpr int MAX_DEVICES = 64;
  static unsigned long long* scratch_of[MAX_DEVICES];     // device address of `scratch`, per device (set once; racing
  int dev = -1;                                            // first calls store the same value)
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  if (!scratch_of[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    scratch_of[dev] = (unsigned long long*)p;
  }
  const int64_t total = n * k;
  if (total > (int64_t)GSS_CHECKSUM_STATIC_MAX_CELLS) return hipErrorInvalidValue;
  const int chunks = (int)((total + CK_CHUNK - 1) / CK_CHUNK);
  unsigned long long* partials = scratch_of[dev];
  if (chunks > 0)
    hipLaunchKernelGGL(checksum_partials_kernel, dim3((unsigned)chunks), dim3(256), 0, st, table, row_of, n, k, S, partials);
  hipLaunchKernelGGL(checksum_finish_kernel, dim3(1), dim3(256), 0, st, (const unsigned long long*)partials, chunks, out);
  return hipGetLastError();
}

hipError_t launch_build_row_map(const void* indptr, int is64, int64_t n, int32_t theta, int32_t* chunk_counts,
                                int32_t* row_of, int32_t* num_rows, hipStream_t st) {
  const int64_t nchunks = (n + MAP_CHUNK - 1) / MAP_CHUNK;
  const unsigned grid = clamp_grid(nchunks, 4096);
  if (nchunks > 0) hipLaunchKernelGGL(row_map_count_kernel, dim3(grid), dim3(MAP_CHUNK), 0, st, indptr, is64, n, theta, chunk_counts);
  hipLaunchKernelGGL(row_map_scan_kernel, dim3(1), dim3(MAP_CHUNK), 0, st, nchunks, chunk_counts, num_rows);
  if (nchunks > 0) hipLaunchKernelGGL(row_map_assign_kernel, dim3(grid), dim3(MAP_CHUNK), 0, st, indptr, is64, n, theta, chunk_counts, row_of);
  return hipGetLastError();
}

template <class VEC>
static hipError_t launch_gather_t(const void* table, int64_t num_rows, int64_t row_bytes, const int32_t* ids, int64_t num_ids,
                                  void* out, hipStream_t st) {
  const int chunks = (int)((row_bytes + (int64_t)sizeof(VEC) - 1) / (int64_t)sizeof(VEC));
  const uint32_t inv = (uint32_t)(((1ull << 32) + (uint64_t)chunks - 1) / (uint64_t)chunks);   // (chunks == 1: not used)
  const int64_t most = (int64_t)1 << 30;                 // workgroups of a launch
  const int64_t rows = most * GATHER_CHUNKS / chunks;    // ... and the rows they take
  for (int64_t i = 0; i < num_ids; i += rows) {
    const int64_t n = num_ids - i < rows ? num_ids - i : rows, wgs = (n * chunks + GATHER_CHUNKS - 1) / GATHER_CHUNKS;
    hipLaunchKernelGGL(gather_rows_kernel<VEC>, dim3((unsigned)wgs), dim3(256), 0, st, (const char*)table, num_rows, row_bytes, chunks,
                       inv, ids + i, n, (char*)out + i * row_bytes);
  }
  return hipGetLastError();
}

hipError_t launch_gather_rows(const void* table, int64_t num_rows, int64_t row_bytes, const int32_t* ids, int64_t num_ids,
                              void* out, hipStream_t st) {
  if (num_rows == 0) table = out;        // (every row is zeros: the kernel reads a row that exists and drops it)
  if (row_bytes >= 16) return launch_gather_t<uint4>(table, num_rows, row_bytes, ids, num_ids, out, st);
  if (row_bytes >= 8) return launch_gather_t<uint2>(table, num_rows, row_bytes, ids, num_ids, out, st);
  if (row_bytes >= 4) return launch_gather_t<uint32_t>(table, num_rows, row_bytes, ids, num_ids, out, st);
  return launch_gather_t<uint8_t>(table, num_rows, row_bytes, ids, num_ids, out, st);
}

hipError_t launch_store_slot(SlotConst* at, const SlotConst& value, hipStream_t st) {
  hipLaunchKernelGGL(store_slot_kernel, dim3(1), dim3(64), 0, st, at, value);
  return hipGetLastError();
}

hipError_t launch_fill_i64(long long* p, int64_t n, long long value, hipStream_t st) {
  const unsigned grid = clamp_grid((n + 255) / 256, 8192);
  hipLaunchKernelGGL(fill_i64_kernel, dim3(grid), dim3(256), 0, st, p, n, value);
  return hipGetLastError();
}

}  // namespace gss
