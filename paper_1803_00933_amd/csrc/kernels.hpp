// HIP kernels of the replay memory (gfx950).  Host-side entry points are in apex_replay.hip.
//
// Data layout in HBM
//   payload ring   obs[P][obs_bytes], act[P][act_bytes], ret[P], gacc[P]   (structure of arrays)
//   sum tree       level 0 = one uint64 mass per slot; node i of level l+1 = sum of nodes
//                  [64 i, 64 i + 64) of level l; levels are added until one has at most kExportedTopMax
//                  nodes.  A wavefront reads the 64 children of a node as one coalesced 512-byte row.
//                  If the last of these levels has more than kTopMax nodes, a summit stands above it:
//                  node i = sum of 2^top_log2 of its nodes, the smallest power of two that leaves at
//                  most kSummitMax.  So the level a walk starts from always fits the registers of one wave
//                  (8 nodes per lane, 16 if there are more than 512).  Where every workgroup staged the
//                  whole top in LDS instead, a draw of 4096 from 2^24 slots (4352 nodes) took 16.3 us, now
//                  11.0; the learner steps on 2^18 slots (4096 nodes) 8.8 us per launch, now 5.6.
//                  Between 513 and 1024 nodes no summit: its round trip and its atomics cost more than the
//                  wider read (steps of 512 on 50,000 slots, 782 nodes: 5.6 us with one, 5.2 without).
//                  Not fewer nodes than that: every change of a mass is an atomic on every level, and
//                  atomics of different waves on one cache line take some 6 ns one after the other.
//   device state   head, tail, counters: read by the kernels, so the same launches can be replayed.
// The set of transitions and the sampled indices do not depend on this shape: a sample is
// defined by the cumulative mass in slot order, whatever tree sums it up.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "apex_replay.h"
#include "quantise.hpp"
#include "wave.hpp"

namespace apex {

constexpr uint32_t kFanoutLog2 = 6;
constexpr uint32_t kFanout = 1u << kFanoutLog2;
constexpr uint32_t kExportedTopMax = 4608;  // covers 2^24 + 2^20 slots with three levels
constexpr uint32_t kTopMax = 1024;          // nodes of the level that walks start from ...
constexpr uint32_t kSummitMax = 512;        // ... where that is a summit
constexpr uint32_t kMaxLevels = 8;

struct DeviceState {
  uint64_t head, tail;      // valid keys: head <= key < tail
  uint64_t n_stale, n_clamped;
  uint32_t ticket_add;      // workgroups of the running add launch that are done with tail ...
  uint32_t ticket_evict;    // ... and of the running evict launch that are done with head (the two may overlap)
};

// The launches that move head or tail on read them first: every workgroup takes a ticket once all its threads
// have what they read of the counter (the caller puts a barrier in between), and the one with the last ticket
// writes the counter, so that the launch needs no follow-up launch for it (the ticket is back at 0 afterwards).
// The last lane of the workgroup does it: the ticket's round trip (1.5 - 2 us, like that of every atomic that the
// eight L2 caches have to agree on) then runs beside those of the first wave's atomics on the tree.
// n_wgs: the workgroups that take part.
__device__ __forceinline__ void advance_state(uint32_t *ticket, uint64_t *counter, uint64_t now, uint32_t n_wgs)
{
  if (threadIdx.x == blockDim.x - 1) {
    const uint32_t t = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t == n_wgs - 1) {
      *ticket = 0;
      *counter = now;
    }
  }
}

// Exact floor(n / d) for any n by a multiplication, for a divisor that the host knows at launch time
// (a 64-bit quotient is otherwise a long software division).  Granlund and Montgomery's unsigned division by an
// invariant integer: L = ceil(log2 d), mul = floor(2^64 (2^L - d) / d) + 1, sh1 = min(L, 1), sh2 = max(L - 1, 0).
struct FastDiv {
  uint64_t mul;
  uint32_t sh1, sh2;
};

__device__ __forceinline__ uint64_t fast_div(uint64_t n, const FastDiv &d)
{
  const uint64_t t = __umul64hi(d.mul, n);
  return (t + ((n - t) >> d.sh1)) >> d.sh2;
}

struct TreeView {
  uint64_t *level[kMaxLevels];
  uint32_t nlev;      // level nlev-1 is the top
  uint32_t n_top;     // nodes of the top level: at most kTopMax
  uint32_t top_log2;  // log2 of the top level's fan-out (kFanoutLog2, or less where the top is a summit)
  uint32_t pad;
  uint64_t P;         // ring size
  FastDiv p_div;      // division by P
};

// key mod P
__device__ __forceinline__ uint64_t ring_slot(const TreeView &tv, uint64_t key) { return key - fast_div(key, tv.p_div) * tv.P; }

// Keeps wave-uniform values in scalar registers from here on: the compiler would otherwise fetch a kernel argument only
// where it is first used, behind a wait of its own.  Values named in one call are waited for together.
template <typename T>
__device__ __forceinline__ void fetch_now(T p)
{
  asm volatile("" ::"s"(p));
}
template <typename A, typename B, typename C, typename D>
__device__ __forceinline__ void fetch_now(A a, B b, C c, D d)
{
  asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d));
}

// A barrier for what the workgroup exchanges through LDS (and for scalar loads): vector loads and stores that are under way are
// not waited for.  Whoever lets go of a word behind it, by a ticket, has to see to it that every wave has the word by then:
// fetch_now for a scalar, arrived for a vector.
__device__ __forceinline__ void lds_barrier()
{
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// log2 of the fan-out of level l (l >= 1) over the level below it.
__device__ __forceinline__ uint32_t fanout_log2(const TreeView &tv, uint32_t l)
{
  return l + 1 == tv.nlev ? tv.top_log2 : kFanoutLog2;
}

// Calls f(l) for the levels from kFrom up.  The lowest ones one by one: their addresses are at fixed places of a kernel's
// arguments then and are fetched together, where a loop fetched each behind a wait of its own.
template <uint32_t kFrom, typename F>
__device__ __forceinline__ void for_levels(const TreeView &tv, F f)
{
  constexpr uint32_t kApart = 4;
#pragma unroll
  for (uint32_t l = kFrom; l < kApart; ++l) {
    if (l >= tv.nlev) return;
    f(l);
  }
  for (uint32_t l = kApart; l < tv.nlev; ++l) f(l);
}

// Adds delta (mod 2^64) to every ancestor of `slot` above level 0.
__device__ __forceinline__ void add_to_ancestors(const TreeView &tv, uint64_t slot, uint64_t delta)
{
  uint64_t idx = slot;
  for_levels<1>(tv, [&](uint32_t l) {
    idx >>= fanout_log2(tv, l);
    atomic_add_u64(tv.level[l] + idx, delta);
  });
}

// Where the runs of neighbouring lanes with equal `node` lie that a prefix sum of the lanes' values is cut into.
struct LaneRuns {
  bool ends;        // this lane is the last of its run
  int first;        // the first lane of this lane's run
};

__device__ __forceinline__ LaneRuns lane_runs(uint32_t node)
{
  const int lane = lane_id();
  const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)node, 0x138, 0xf, 0xf, false);  // wave_shr:1
  const uint64_t starts = __ballot(lane == 0 || prev != node);
  LaneRuns r;
  r.ends = lane == kWave - 1 || ((starts >> (lane + 1)) & 1);
  r.first = 63 - __builtin_clzll(starts & (~0ull >> (63 - lane)));  // bit 0 is set
  return r;
}

// Adds to a node of the tree and, if second != 0, to the same node of the copy that lies `second` words behind it.
__device__ __forceinline__ void atomic_add_both(uint64_t *p, uint64_t second, uint64_t v)
{
  atomic_add_u64(p, v);
  if (second) atomic_add_u64(p + second, v);
}

// Same, for a wave whose lanes hold slots in mostly ascending order (the consecutive slots of an add or a FIFO
// eviction, free slots handed out again, drawn keys): on every level each run of neighbouring lanes under one node
// is summed with one prefix sum over the wave and sends one atomic instead of one per lane.  A node that appears
// in several runs receives several atomics.  Sums are modulo 2^64, so a removal passes 0 - mass.  Must be called
// by all 64 lanes; `active` marks the lanes that carry a delta.
// idx: the node of level kFrom - 1 that the delta belongs to (a slot, kFrom = 1).
template <uint32_t kFrom = 1>
__device__ __forceinline__ void add_runs_to_ancestors(const TreeView &tv, bool active, uint32_t idx, uint64_t delta,
                                                      uint64_t second = 0)
{
  const uint64_t incl = wave_inclusive_scan(active ? delta : 0);
  for_levels<kFrom>(tv, [&](uint32_t l) {
    idx >>= fanout_log2(tv, l);
    const LaneRuns run = lane_runs(active ? idx : ~0u);  // lanes without a delta form runs of their own, which send nothing
    const uint64_t before = __shfl(incl, run.first > 0 ? run.first - 1 : 0, kWave);
    if (active && run.ends) atomic_add_both(tv.level[l] + idx, second, incl - (run.first > 0 ? before : 0));
  });
}

// Same, for a workgroup of at most 1024 threads that holds consecutive slots of the ring, one per thread: the waves'
// sums on level 1 (at most three runs a wave: 64 slots that cross one node's border and the ring's end) are
// collected in LDS, and one wave enters them into the levels above, which so receive one atomic per workgroup and
// node instead of one per wave: all waves of a round meet on one or two nodes there (51,200 transitions of 2^24:
// 800 atomics on one address, about 10 ns each; the launch took 8.6 us, now 4.4).  Contains a barrier.  Called by
// every thread.
struct DenseSums {
  uint64_t sum[64];
  uint32_t node[64];
};

__device__ __forceinline__ void add_dense_to_ancestors(const TreeView &tv, bool active, uint64_t slot, uint64_t delta,
                                                       uint64_t second, DenseSums &sh)
{
  if (tv.nlev < 2) {
    __syncthreads();
    return;
  }
  const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
  const uint64_t incl = wave_inclusive_scan(active ? delta : 0);
  const uint32_t node = (uint32_t)slot >> fanout_log2(tv, 1);
  const LaneRuns run = lane_runs(active ? node : ~0u);
  const uint64_t before = __shfl(incl, run.first > 0 ? run.first - 1 : 0, kWave);
  const uint64_t sum = incl - (run.first > 0 ? before : 0);
  const bool sends = active && run.ends;
  const uint64_t senders = __ballot(sends);
  if (sends) atomic_add_both(tv.level[1] + node, second, sum);
  const bool more = tv.nlev > 2;  // levels above (level 1 then has the full fan-out: at most three runs)
  const uint32_t e = 4 * wave + (more ? __popcll(senders & ((1ull << lane) - 1)) : 0);
  if (sends && more) {
    sh.sum[e] = sum;
    sh.node[e] = node;
  }
  // places a wave does not use: zero on its last node (a gap would cut the runs of the second stage), none if idle
  const uint32_t n_sent = __popcll(senders);
  const uint32_t filler = n_sent ? (uint32_t)__shfl(node, 63 - __builtin_clzll(senders | 1), kWave) : ~0u;
  if (lane < 4 && lane >= n_sent) {
    sh.sum[4 * wave + lane] = 0;
    sh.node[4 * wave + lane] = filler;
  }
  __syncthreads();
  if (wave == 0 && more) {
    const uint32_t nd = lane < 4 * (blockDim.x / kWave) ? sh.node[lane] : ~0u;
    add_runs_to_ancestors<2>(tv, nd != ~0u, nd, sh.sum[lane], second);
  }
}

// --------------------------------------------------------------------------------------------
// n-step priorities: one thread per transition (Algorithm 1, ComputePriorities; Sections 3.1, 3.2)
// --------------------------------------------------------------------------------------------
struct NstepArgs {
  uint32_t S, T, n, A;
  FastDiv t_div;                     // division by T
  const float *q_online, *q_target;  // [S, T+n, A]
  const int32_t *action;             // [S, T+n]
  const float *reward, *discount;    // [S, T+n]
};

struct NstepOut {
  float p, R, G;  // priority |delta|, partial return, accumulated discount
};

// argmax_a row[a], the lowest action of several.  Eight values on their way together (one by one, every value was a round
// trip).  Where fewer than eight are left the last one is read again: a value is never above itself.  One or two at the end
// are not worth the seven reads too many.
// n-step priorities of 18,000 transitions of 18 actions 4.5 -> 4.2 us, of 3300 of 40 actions, eleven steps, 9.2 -> 8.1.
__device__ __forceinline__ uint32_t greedy_action(const float *row, uint32_t A)
{
  constexpr uint32_t kAhead = 8;
  uint32_t best = 0, b = 1;
  float vbest = row[0];
  auto take = [&](float v, uint32_t at) {
    const bool above = v > vbest;
    vbest = above ? v : vbest;
    best = above ? at : best;
  };
  for (; b + 2 < A; b += kAhead) {
    float v[kAhead];
#pragma unroll
    for (uint32_t t = 0; t < kAhead; ++t) v[t] = row[min(b + t, A - 1)];
#pragma unroll
    for (uint32_t t = 0; t < kAhead; ++t) take(v[t], b + t);
  }
  for (; b < A; ++b) take(row[b], b);
  return best;
}

// Up to this many steps the rewards and discounts of a transition are read together (3200 transitions of five steps, one
// action: 3.3 -> 2.9 us).
constexpr int kNstepHeld = 8;

// Transition gid = s * T + t of an add round (gid < S * T).
__device__ __forceinline__ NstepOut nstep_one(const NstepArgs &a, uint64_t gid)
{
  const uint32_t T = a.T, n = a.n, A = a.A;
  const uint32_t s = (uint32_t)fast_div(gid, a.t_div), t = (uint32_t)(gid - (uint64_t)s * T);
  const uint64_t row0 = (uint64_t)s * (T + n);  // first row of this stream
  const float *rw = a.reward + row0 + t;
  const float *dc = a.discount + row0 + t;

  // rewards, discounts and the action go out ahead of the Q-values that the greedy action is looked for in: all is on its way
  // before the first wait
  uint32_t at = (uint32_t)a.action[row0 + t];
  float r[kNstepHeld], d[kNstepHeld];
  const bool held = n <= kNstepHeld;
  if (held) {
#pragma unroll
    for (int j = 0; j < kNstepHeld; ++j)
      if ((uint32_t)j < n) r[j] = rw[j], d[j] = dc[j];
  }
  const uint32_t best = greedy_action(a.q_online + (row0 + t + n) * A, A);
  if (at >= A) at = A - 1;  // keeps a corrupt action index inside the row
  const float boot = a.q_target[(row0 + t + n) * A + best], q_at = a.q_online[(row0 + t) * A + at];
  float R = 0.0f, G = 1.0f;
  if (held) {
#pragma unroll
    for (int j = kNstepHeld - 1; j >= 0; --j) R = (uint32_t)j < n ? __builtin_fmaf(d[j], R, r[j]) : R;  // Horner, one rounding per step
#pragma unroll
    for (int j = 0; j < kNstepHeld; ++j) G = (uint32_t)j < n ? G * d[j] : G;
  } else {
    for (int j = (int)n - 1; j >= 0; --j) R = __builtin_fmaf(dc[j], R, rw[j]);
    for (uint32_t j = 0; j < n; ++j) G = G * dc[j];
  }
  const float target = __builtin_fmaf(G, boot, R);
  const float delta = target - q_at;
  return NstepOut{__builtin_fabsf(delta), R, G};
}

__global__ __launch_bounds__(256) void nstep_kernel(NstepArgs a, QuantParams qp, float *__restrict__ prio,
                                                    float *__restrict__ ret, float *__restrict__ gacc,
                                                    uint64_t *__restrict__ prio_fx)
{
  const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (uint64_t)a.S * a.T) return;
  const NstepOut o = nstep_one(a, gid);
  ret[gid] = o.R;
  gacc[gid] = o.G;
  prio[gid] = o.p;
  if (prio_fx) {
    bool c;
    prio_fx[gid] = quantise_priority(o.p, qp, &c);
  }
}

// --------------------------------------------------------------------------------------------
// row copies: payload into the ring (add) and out of it (gather)
// --------------------------------------------------------------------------------------------
// Row i of the source / destination is found through a RowMap: an index array (gather by slot),
// a ring position read from device memory (keys base+i, slot = key mod ring), or the identity.
struct RowMap {
  const uint32_t *index;     // row = index[i]
  const uint64_t *ring_key;  // row = (*ring_key + i) mod ring; with index: row = index[(*ring_key + i) mod ring]
  uint64_t ring;
  FastDiv ring_div;          // division by ring
};

__device__ __forceinline__ uint64_t map_row(const RowMap &m, uint64_t i)
{
  if (m.ring_key) {
    const uint64_t key = *m.ring_key + i;
    i = key - fast_div(key, m.ring_div) * m.ring;
  }
  return m.index ? m.index[i] : i;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));

// The pieces in which a kernel moves a row: Reg in registers, Mem in memory; piece v of a row of n bytes starts at
// byte at(v, n), and a row has count(n) of them.
template <typename Vec>
struct Piece {  // whole pieces, all aligned
  typedef Vec Reg;
  typedef Vec Mem;
  static constexpr bool kWhole = true;
  static __device__ __forceinline__ uint64_t at(uint32_t v, uint64_t) { return (uint64_t)v * sizeof(Vec); }
};
// Rows of at least 16 bytes at any alignment and of any length: pieces of 16 bytes, the last one overlapping the one
// before it (both carry the same bytes there).  The hardware takes unaligned vector accesses; in the widest units that
// length and addresses divide by, rows of odd lengths went byte by byte (999 rows of 5003 bytes: 11.4 us, now 6.1).
struct PieceAny {
  typedef u32x4 Reg;
  typedef u32x4_any Mem;
  static constexpr bool kWhole = false;
  static __device__ __forceinline__ uint64_t at(uint32_t v, uint64_t n) { return min((uint64_t)v * 16, n - 16); }
};
typedef Piece<u32x4> Piece16;
typedef Piece<uint32_t> Piece4;
typedef Piece<uint8_t> Piece1;

template <typename P>
__device__ __forceinline__ typename P::Reg load_piece(const uint8_t *row, uint32_t v, uint64_t n)
{
  return *reinterpret_cast<const typename P::Mem *>(row + P::at(v, n));
}
template <typename P>
__device__ __forceinline__ typename P::Reg load_piece_streaming(const uint8_t *row, uint32_t v, uint64_t n)
{
  return __builtin_nontemporal_load(reinterpret_cast<const typename P::Mem *>(row + P::at(v, n)));
}
template <typename P>
__device__ __forceinline__ void store_piece(uint8_t *row, uint32_t v, uint64_t n, typename P::Reg x)
{
  *reinterpret_cast<typename P::Mem *>(row + P::at(v, n)) = x;
}
template <typename P>
__device__ __forceinline__ void store_piece_streaming(uint8_t *row, uint32_t v, uint64_t n, typename P::Reg x)
{
  __builtin_nontemporal_store(x, reinterpret_cast<typename P::Mem *>(row + P::at(v, n)));
}

// --------------------------------------------------------------------------------------------
// Observations stored through the block codec (Section 4.1: observations are kept compressed in the
// replay memory): shape of an encoded row, and how a lane fetches a 16-byte piece of the raw row
// out of it.  The format is described in codec.inc.hpp: every part has a fixed place, so the three
// loads below depend on nothing but the row's address.
// --------------------------------------------------------------------------------------------
struct CodecShape {
  uint32_t raw_bytes, nb, mask_words;  // raw_bytes == 0: no codec
  uint32_t flat_off, image_off;        // M, M + V
  uint64_t stride;                     // M + V + 64 nb
};

__host__ __device__ inline CodecShape codec_shape(uint32_t raw_bytes)
{
  CodecShape c{};
  c.raw_bytes = raw_bytes;
  c.nb = raw_bytes / 64;
  c.mask_words = (c.nb + 63) / 64;
  const uint32_t M = (8 * c.mask_words + 15) / 16 * 16, V = (c.nb + 15) / 16 * 16;
  c.flat_off = M;
  c.image_off = M + V;
  c.stride = (uint64_t)c.image_off + 64ull * c.nb;
  return c;
}

// What a lane has asked for of piece v (16 bytes) of the raw row: the piece as the image holds it, its
// block's byte, and the word of the mask that says which of the two counts.
struct CodecFetched {
  u32x4 data;
  uint64_t word;
  uint32_t byte, bit;
};

// All three at once (for paths bound by latency: nothing waits for the mask).  v < raw_bytes / 16.
__device__ __forceinline__ CodecFetched codec_fetch_all(const uint8_t *e, const CodecShape &c, uint32_t v)
{
  CodecFetched f;
  const uint32_t b = v / 4;
  f.data = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(e + c.image_off) + v);
  f.byte = e[c.flat_off + b];
  f.word = reinterpret_cast<const uint64_t *>(e)[b / 64];
  f.bit = b & 63;
  return f;
}

// Mask words and block bytes of a whole wave that holds four runs of 64 consecutive pieces, run u from piece v_first[u] on,
// a multiple of 64 (16 blocks: one word of the mask, 16 consecutive block bytes): they come through the scalar data cache
// (read only), which keeps them out of the queue of the vector memory pipeline, and all eight loads are in flight
// together.  e must be 16-byte aligned, the runs must start inside the row.
__device__ __forceinline__ void codec_fetch_wave_scalars(const uint8_t *e, const CodecShape &c, const uint32_t (&v_first)[4],
                                                         uint64_t (&word)[4], u32x4 (&bytes)[4])
{
  const uint64_t pe = (uint64_t)(uintptr_t)e;
  // (the builtin returns a signed int: without the casts the low half would be sign-extended)
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(pe >> 32));
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)pe);
  const uint64_t base = ((uint64_t)hi << 32) | (uint64_t)lo;
  uint64_t p_word[4], p_bytes[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint32_t vf = (uint32_t)__builtin_amdgcn_readfirstlane((int)v_first[u]);
    p_word[u] = base + 8ull * (vf >> 8);
    p_bytes[u] = base + c.flat_off + vf / 4;
  }
  asm volatile("s_load_dwordx2 %0, %8, 0x0\n\ts_load_dwordx2 %1, %9, 0x0\n\t"
               "s_load_dwordx2 %2, %10, 0x0\n\ts_load_dwordx2 %3, %11, 0x0\n\t"
               "s_load_dwordx4 %4, %12, 0x0\n\ts_load_dwordx4 %5, %13, 0x0\n\t"
               "s_load_dwordx4 %6, %14, 0x0\n\ts_load_dwordx4 %7, %15, 0x0\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&s"(word[0]), "=&s"(word[1]), "=&s"(word[2]), "=&s"(word[3]), "=&s"(bytes[0]), "=&s"(bytes[1]),
                 "=&s"(bytes[2]), "=&s"(bytes[3])
               : "s"(p_word[0]), "s"(p_word[1]), "s"(p_word[2]), "s"(p_word[3]), "s"(p_bytes[0]), "s"(p_bytes[1]),
                 "s"(p_bytes[2]), "s"(p_bytes[3])
               : "memory");
}

// The byte of the block of lane `lane`'s piece out of the 16 bytes fetched above.
__device__ __forceinline__ uint32_t codec_wave_byte(const u32x4 &bytes, uint32_t lane)
{
  const uint32_t i = lane / 4;  // block within the wave
  const uint32_t dw = i < 4 ? bytes.x : i < 8 ? bytes.y : i < 12 ? bytes.z : bytes.w;
  return (dw >> (8 * (i & 3))) & 0xffu;
}

__device__ __forceinline__ u32x4 codec_piece(const CodecFetched &f)
{
  const uint32_t x = f.byte * 0x01010101u;
  return (f.word >> f.bit & 1) ? f.data : u32x4{x, x, x, x};
}

// A learner batch (m <= blockDim) handled by one workgroup, beside rows that others copy: duplicates are resolved in an
// LDS hash table keyed by slot (the highest position wins), so no pass over global memory is needed for it, and the old
// mass is fetched while the table is being filled.
constexpr uint32_t kDedupeSlots = 2048;  // >= 2 * 1024 pairs: linear probing stays short

// Learner-side ComputePriorities (Algorithm 2) fused into the write-back: the new priority of a
// sampled transition is recomputed from the partial return and accumulated discount stored with it
// (Appendix "Implementation", "Adding Data") and the Q-values the learner has just evaluated,
//   | ret + gacc * q_target_next[argmax_a q_online_next[a]] - q_taken |     (Section 3.1 target),
// in the same fp32 order as the actor-side kernel.  q_taken == null: priorities are given.
struct QSource {
  const float *q_taken;        // [m]   q(S_t, A_t) of the online network
  const float *q_online_next;  // [m,A] q(S_{t+n}, .) of the online network
  const float *q_target_next;  // [m,A] q(S_{t+n}, .) of the target network
  uint32_t A;
  const float *ret, *gacc;     // columns of the payload ring
  float *prio_out;             // [m] or null: the priorities that were computed (0 for skipped pairs)
};

// What does not depend on the transition's slot: q_target_next of the greedy action, and q_taken.
struct TdInputs {
  float boot, taken;
};

__device__ __forceinline__ TdInputs td_inputs(const QSource &qs, uint32_t i)
{
  const float taken = qs.q_taken[i];
  const uint32_t best = greedy_action(qs.q_online_next + (uint64_t)i * qs.A, qs.A);
  return TdInputs{qs.q_target_next[(uint64_t)i * qs.A + best], taken};
}

__device__ __forceinline__ float td_priority(float ret, float gacc, const TdInputs &in)
{
  return __builtin_fabsf(__builtin_fmaf(gacc, in.boot, ret) - in.taken);
}

struct UpdateArgs {
  TreeView tv;
  DeviceState *st;
  uint32_t m;
  const uint64_t *key;
  const float *prio;
  QuantParams qp;
  // Set by callers that draw a batch and write its priorities back with nothing touching the tree
  // in between: pair i is known to be valid, to live in slot_hint[i] and to weigh mass_hint[i],
  // which saves the two dependent loads key -> slot -> mass.
  const uint32_t *slot_hint;
  const uint64_t *mass_hint;
  QSource qs;
};

// What one lane holds of its pair between the two halves below.
struct UpdateLane {
  uint64_t key, old;
  uint32_t slot;
  float prio;
  uint64_t head, tail;
};

// First half: only loads, so that a caller can put other memory work behind them.
__device__ __forceinline__ UpdateLane update_batch_load(const UpdateArgs &ua)
{
  UpdateLane u{0, 0, 0, 0.0f, 0, ~0ull};
  const uint32_t i = threadIdx.x;
  if (i < ua.m) {
    u.prio = ua.prio[i];
    if (ua.slot_hint) {
      u.slot = ua.slot_hint[i];
      u.old = ua.mass_hint[i];
    } else {
      u.key = ua.key[i];
    }
  }
  if (!ua.slot_hint) {
    u.head = ua.st->head;
    u.tail = ua.st->tail;
  }
  return u;
}

// Second half.  h_slot, h_pos: LDS, kDedupeSlots words each.  Called by every thread of the workgroup.
__device__ __forceinline__ void update_batch_apply(const UpdateArgs &ua, UpdateLane u, uint32_t *h_slot, uint32_t *h_pos)
{
  const TreeView &tv = ua.tv;
  const uint32_t i = threadIdx.x;
  for (uint32_t t = i; t < kDedupeSlots; t += blockDim.x) {
    h_slot[t] = 0xffffffffu;  // no slot has this number: max_slots <= 2^31
    h_pos[t] = 0;
  }
  __syncthreads();
  const bool valid = i < ua.m && u.key >= u.head && u.key < u.tail;
  const bool stale = i < ua.m && !valid;
  bool clamped = false;
  uint32_t slot = u.slot, h = 0;
  uint64_t q = 0, old = u.old;
  if (valid) {
    if (!ua.slot_hint) {
      slot = (uint32_t)ring_slot(tv, u.key);
      old = tv.level[0][slot];  // in flight during the dedupe
    }
    h = (slot * 2654435761u) >> 21;  // top 11 bits
    for (;;) {
      const uint32_t prev = atomicCAS(&h_slot[h], 0xffffffffu, slot);
      if (prev == 0xffffffffu || prev == slot) break;
      h = (h + 1) & (kDedupeSlots - 1);
    }
    atomicMax(&h_pos[h], i + 1);
    q = quantise_priority(u.prio, ua.qp, &clamped);
  }
  __syncthreads();
  const bool wins = valid && h_pos[h] == i + 1;
  if (wins) {
    tv.level[0][slot] = q;
    add_to_ancestors(tv, slot, q - old);
  }
  const uint64_t ns = __popcll(__ballot(stale)), nc = __popcll(__ballot(clamped));
  if (lane_id() == 0) {
    if (ns) atomic_add_u64(&ua.st->n_stale, ns);
    if (nc) atomic_add_u64(&ua.st->n_clamped, nc);
  }
}

// An update of up to kHeld * kUpdateThreads pairs in one launch.  A workgroup writes 64 of them back, those of one of its
// waves; which of several pairs naming one slot is the last, every workgroup finds out for itself, by a table in LDS of all
// keys of the update (the highest position wins).  So nothing has to be settled between workgroups, and what one compute
// unit would take one after the other - scattered masses, rows of Q-values, the atomics on every level - is shared out.
// Bound by its chain: key, slot, mass, atomics, 3.3 us for 16 pairs and 3.9 for 1024 (a launch of nothing: 2.5).  us, drawn
// or random keys, against one workgroup for everything up to 1024 pairs and two launches beyond:
//   512 pairs, 2^18 / 2^24 slots      4.4 - 4.7 / 5.4  -> 3.6 / 3.7
//   1024 pairs, 2^18 / 2^24 slots     5.5 - 6.3 / 7.4 - 8.1 -> 3.9 / 4.1
//   2048 pairs, 2^18 / 2^24 slots     6.2 - 6.8 / 6.2 - 6.9 -> 5.1 / 5.3 - 5.7
//   512 / 1024 pairs from the learner's Q-values, 18 actions, 2^21 slots  7.4 / 15.2 -> 4.3 / 4.5
// With twice instead of four times as many places as pairs 1024 take 4.4 us and 2048 take 6.0 - 7.2 (probing); 4096 pairs
// with four per thread take 8 - 10 us.
// A pair's mass, and from Q-values its columns, are asked for as soon as its key is there, ahead of the table (device time,
// replayed graphs, behind the table / ahead): 32 pairs of 2^24 slots 2.67 / 2.55, from Q-values 3.35 / 3.06, 512 pairs
// 3.01 / 2.93 and 3.71 / 3.47, 2048 4.56 / 4.49 and 5.38 / 4.98; 4096, the kernel below, 5.54 / 5.09 and 6.88 / 5.81.
constexpr uint32_t kUpdateThreads = 1024;       // most threads per workgroup ...
constexpr uint32_t kUpdateMinThreads = 256;     // ... and fewest: one wave alone is slow to clear the table (32 pairs 3.8 us)

template <int kHeld>
__global__ __launch_bounds__(kUpdateThreads) void update_small_kernel(UpdateArgs ua)
{
  constexpr uint32_t kPlaces = 4 * kUpdateThreads * kHeld;
  __shared__ __align__(16) uint32_t h_slot[kPlaces];
  __shared__ __align__(16) uint32_t h_pos[kPlaces];
  const TreeView &tv = ua.tv;
  const uint32_t tid = threadIdx.x, nthr = blockDim.x, per = nthr / kWave;
  uint64_t *const leaves = tv.level[0];
  // the pairs that are written back here: number own_t of those that the lanes of wave own_wave hold
  const uint32_t own_t = kHeld == 1 ? 0 : blockIdx.x / per, own_wave = kHeld == 1 ? blockIdx.x : blockIdx.x - own_t * per;
  const bool own = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / kWave)) == own_wave, from_q = ua.qs.q_taken != nullptr;
  uint64_t key[kHeld];
#pragma unroll
  for (int t = 0; t < kHeld; ++t) key[t] = ua.key[min(t * nthr + tid, ua.m - 1)];
  const uint32_t i = own_t * nthr + tid;
  const uint64_t head = ua.st->head, tail = ua.st->tail;
  for (uint32_t t = tid; t < kPlaces / 4; t += nthr) {
    reinterpret_cast<u32x4 *>(h_slot)[t] = u32x4{~0u, ~0u, ~0u, ~0u};  // no slot has this number: max_slots <= 2^31
    reinterpret_cast<u32x4 *>(h_pos)[t] = u32x4{0, 0, 0, 0};
  }
  // Everything that a pair's mass and priority are made of is on its way before the workgroup first waits for one another:
  // Q-values beside the keys, the transition's mass and columns as soon as the key is there.  (Those of a key that is not valid
  // any more are those of the slot it would have: read, and not used.)
  float prio = 0.f, ret = 0.f, gacc = 0.f;
  TdInputs td{};
  uint64_t old = 0;
  uint32_t slot[kHeld], h[kHeld], prev[kHeld];
  bool valid[kHeld], valid_own = false;
  uint32_t slot_own = 0, h_own = 0;
  if (own) {
    if (from_q) td = td_inputs(ua.qs, min(i, ua.m - 1));
    else prio = ua.prio[min(i, ua.m - 1)];
  }
#pragma unroll
  for (int t = 0; t < kHeld; ++t) {
    slot[t] = (uint32_t)ring_slot(tv, key[t]);
    if (t == (int)own_t) slot_own = slot[t];
  }
  if (own) {
    old = leaves[slot_own];
    if (from_q) ret = ua.qs.ret[slot_own], gacc = ua.qs.gacc[slot_own];
  }
#pragma unroll
  for (int t = 0; t < kHeld; ++t) {
    valid[t] = t * nthr + tid < ua.m && key[t] >= head && key[t] < tail;
    h[t] = (slot[t] * 2654435761u) / (0xffffffffu / kPlaces + 1);
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kHeld; ++t)
    if (valid[t]) prev[t] = atomicCAS(&h_slot[h[t]], 0xffffffffu, slot[t]);
#pragma unroll
  for (int t = 0; t < kHeld; ++t) {
    if (valid[t]) {
      while (prev[t] != 0xffffffffu && prev[t] != slot[t]) {
        h[t] = (h[t] + 1) & (kPlaces - 1);
        prev[t] = atomicCAS(&h_slot[h[t]], 0xffffffffu, slot[t]);
      }
      atomicMax(&h_pos[h[t]], t * nthr + tid + 1);
    }
    if (t == (int)own_t) valid_own = valid[t], h_own = h[t];
  }
  bool clamped = false;
  uint64_t q = 0;
  float p = prio;
  if (own) {
    if (from_q) p = td_priority(ret, gacc, td);
    q = quantise_priority(p, ua.qp, &clamped);
    clamped &= valid_own;
  }
  __syncthreads();
  if (!own) return;
  const bool stale = i < ua.m && !valid_own;
  if (from_q && ua.qs.prio_out && i < ua.m) ua.qs.prio_out[i] = valid_own ? p : 0.0f;
  if (valid_own && h_pos[h_own] == i + 1) {
    leaves[slot_own] = q;
    add_to_ancestors(tv, slot_own, q - old);
  }
  const uint64_t ns = __popcll(__ballot(stale)), nc = __popcll(__ballot(clamped));
  if (lane_id() == 0) {
    if (ns) atomic_add_u64(&ua.st->n_stale, ns);
    if (nc) atomic_add_u64(&ua.st->n_clamped, nc);
  }
}

// The same for more pairs, up to kUpdateOneLaunchMax: a workgroup puts only its own 64 into a table and looks every later
// pair of the update up, first in a map of bits, in which a look-up is one read that depends on none before (64 of 16,384
// bits are set), and only where that says so in the table.  The sums of neighbouring keys go to a node together: without it
// drawn keys are 0.6 - 1.5 us slower.  Against the two launches below, us, drawn / random keys:
//   2049 pairs, 2^18 / 2^24 slots   6.2 / 6.8, 6.2 / 6.9 -> 5.4 / 5.5, 5.5 / 5.6     (2048 in the kernel above 5.1, 5.5)
//   4096 pairs, 2^18 / 2^24 slots   6.2 / 7.3, 6.4 / 7.8 -> 5.7 / 6.0, 5.8 / 6.6     5000: 6.2 / 7.6, 6.5 / 8.3 -> 6.0 / 6.3, 6.1 / 7.0
//   4096 pairs from the learner's Q-values, 18 actions, 2^24 slots   8.6 -> 6.8
// and one launch less on the host.  Beyond, every key is read by too many workgroups (8192 drawn keys 7.1, 6.2 apart).
constexpr uint32_t kUpdateOneLaunchMax = 4096;
constexpr uint32_t kUpdateManyThreads = 1024;
constexpr uint32_t kUpdateManyAhead = 4;       // keys that a thread looks up together
constexpr uint32_t kOwnPlaces = 4 * kWave;     // places of the table
constexpr uint32_t kSeenWords = 512;           // of the map

__global__ __launch_bounds__(kUpdateManyThreads) void update_many_kernel(UpdateArgs ua)
{
  __shared__ unsigned long long own_key[kOwnPlaces];
  __shared__ uint32_t own_last[kOwnPlaces];  // 1 + the last of this workgroup's pairs that names the key; ~0: a later one does
  __shared__ uint32_t seen[kSeenWords];
  const TreeView &tv = ua.tv;
  const uint32_t tid = threadIdx.x;
  const bool first_wave = __builtin_amdgcn_readfirstlane((int)tid) == 0, from_q = ua.qs.q_taken != nullptr;
  uint64_t *const leaves = tv.level[0];
  const uint32_t i = blockIdx.x * kWave + (tid & (kWave - 1)), mine = min(i, ua.m - 1);
  const uint32_t later = min((blockIdx.x + 1) * kWave, ua.m);
  const uint64_t key = ua.key[mine];
  uint64_t ahead[kUpdateManyAhead];
  auto read_ahead = [&](uint32_t j0) {  // (the last pair again and again beyond the end: it is a later one all the same)
#pragma unroll
    for (uint32_t t = 0; t < kUpdateManyAhead; ++t) ahead[t] = ua.key[min(j0 + t * kUpdateManyThreads + tid, ua.m - 1)];
  };
  read_ahead(later);
  const uint64_t head = ua.st->head, tail = ua.st->tail;
  if (tid < kSeenWords) seen[tid] = 0;
  if (tid < kOwnPlaces) {
    own_key[tid] = ~0ull;  // no valid key: tails stay below it
    own_last[tid] = 0;
  }
  auto hash = [](uint64_t k) { return (uint32_t)k * 2654435761u; };
  // as in the kernel above: what the pair's mass and priority are made of goes out before the first wait for one another
  float prio = 0.f, ret = 0.f, gacc = 0.f;
  TdInputs td{};
  uint64_t old = 0, slot = 0;
  uint32_t h = hash(key) >> 24;
  const bool valid = first_wave && i < ua.m && key >= head && key < tail;
  if (first_wave) {
    if (from_q) td = td_inputs(ua.qs, mine);
    else prio = ua.prio[mine];
    slot = ring_slot(tv, key);
    old = leaves[slot];
    if (from_q) ret = ua.qs.ret[slot], gacc = ua.qs.gacc[slot];
  }
  __syncthreads();
  if (valid) {
    for (;;) {
      const uint64_t prev = atomicCAS(&own_key[h], ~0ull, key);
      if (prev == ~0ull || prev == key) break;
      h = (h + 1) & (kOwnPlaces - 1);
    }
    atomicMax(&own_last[h], tid + 1);
    const uint32_t bit = hash(key) >> 18;
    atomicOr(&seen[bit >> 5], 1u << (bit & 31));
  }
  __syncthreads();
  for (uint32_t j0 = later; j0 < ua.m; j0 += kUpdateManyAhead * kUpdateManyThreads) {
    if (j0 != later) read_ahead(j0);
    uint32_t hit = 0;
#pragma unroll
    for (uint32_t t = 0; t < kUpdateManyAhead; ++t) {
      const uint32_t bit = hash(ahead[t]) >> 18;
      hit |= (seen[bit >> 5] >> (bit & 31) & 1) << t;
    }
    if (hit) {
#pragma unroll
      for (uint32_t t = 0; t < kUpdateManyAhead; ++t) {
        if (!(hit >> t & 1)) continue;
        uint32_t p = hash(ahead[t]) >> 24;
        for (uint64_t there; (there = own_key[p]) != ~0ull; p = (p + 1) & (kOwnPlaces - 1)) {
          if (there == ahead[t]) {
            own_last[p] = ~0u;
            break;
          }
        }
      }
    }
  }
  bool clamped = false;
  uint64_t q = 0;
  float p = prio;
  if (first_wave) {
    if (from_q) p = td_priority(ret, gacc, td);
    q = quantise_priority(p, ua.qp, &clamped);
    clamped &= valid;
  }
  __syncthreads();
  if (!first_wave) return;
  const bool stale = i < ua.m && !valid;
  if (from_q && ua.qs.prio_out && i < ua.m) ua.qs.prio_out[i] = valid ? p : 0.0f;
  const bool wins = valid && own_last[h] == tid + 1;
  if (wins) leaves[slot] = q;
  add_runs_to_ancestors(tv, wins, (uint32_t)slot, q - old);  // the keys of a drawn batch ascend: neighbours share their upper nodes
  const uint64_t ns = __popcll(__ballot(stale)), nc = __popcll(__ballot(clamped));
  if (tid == 0) {
    if (ns) atomic_add_u64(&ua.st->n_stale, ns);
    if (nc) atomic_add_u64(&ua.st->n_clamped, nc);
  }
}
static_assert(kOwnPlaces == 1 << 8 && kSeenWords == 1 << (14 - 5));

// Importance-sampling weights of one batch of k samples, by one workgroup:
//   (N P_i)^-beta / max_j (N P_j)^-beta  ==  (min_j mass_j / mass_i)^beta,   P_i = mass_i / total.
// `red` is LDS scratch of blockDim/64 words.
struct WeightArgs {
  const uint64_t *mass;  // [nb,k], written by the descent kernel that ran before
  float *weight_out;     // [nb,k]; null: no weights wanted
  uint32_t k;
  float beta;
};

// fp32 with the library's own power routine (relative error below 1e-6 here): a double-precision pow would cost 70
// registers per lane.
__device__ __forceinline__ float batch_weight(float mass_min, float mass, float beta)
{
  return pow_fixed_sequence(mass_min / mass, beta);
}

// part, nparts: the workgroup writes the weights of samples [part * k / nparts ...) of batch b only
// (every part still finds the minimum over the whole batch).  The masses that a thread writes weights of go out with those it
// looks for the minimum in, the first two of them; the minimum is a float's from the lanes on, by data-parallel primitives
// (the rounding of a smaller mass is no larger, so it is the rounding of the smallest).
__device__ __forceinline__ void batch_weights(const WeightArgs &wa, uint32_t b, float *red, uint32_t part = 0, uint32_t nparts = 1)
{
  constexpr uint32_t kOwn = 2;
  const uint32_t tid = threadIdx.x, nthr = blockDim.x, nwave = nthr / kWave;
  const uint64_t *bm = wa.mass + (uint64_t)b * wa.k;
  const uint32_t per = (wa.k + nparts - 1) / nparts;
  const uint32_t lo = min(part * per, wa.k), hi = min(lo + per, wa.k);
  uint64_t own[kOwn], mn = ~0ull;
#pragma unroll
  for (uint32_t t = 0; t < kOwn; ++t) own[t] = bm[min(lo + t * nthr + tid, wa.k - 1)];
  for (uint32_t i0 = 0; i0 < wa.k; i0 += 8 * nthr) {  // eight loads in flight (one by one, 16,384 masses took 20 us)
    uint64_t m[8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (i0 + t * nthr < wa.k) m[t] = bm[min(i0 + t * nthr + tid, wa.k - 1)];
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (i0 + t * nthr < wa.k) mn = m[t] < mn ? m[t] : mn;
  }
  float smallest = wave_min((float)mn);
  if (nwave > 1) {
    if (lane_id() == 0) red[tid / kWave] = smallest;
    lds_barrier();
    smallest = wave_min(red[lane_id() < (int)nwave ? lane_id() : 0]);
  }
  float *const out = wa.weight_out + (uint64_t)b * wa.k;
#pragma unroll
  for (uint32_t t = 0; t < kOwn; ++t) {
    const uint32_t i = lo + t * nthr + tid;
    if (i < hi) out[i] = batch_weight(smallest, (float)own[t], wa.beta);
  }
  for (uint32_t i = lo + kOwn * nthr + tid; i < hi; i += nthr) out[i] = batch_weight(smallest, (float)bm[i], wa.beta);
}

constexpr int kLongCopyThreads = 1024;  // one workgroup of 16 waves per 28 KB frame stack
constexpr int kLongCopyUnroll = 2;      // 1024 lanes * 2 * 16 B = 32 KB per workgroup

// grid: (batches, parts of a batch).  Bound by its chain: masses, minimum over the workgroup, arithmetic.  A weight per thread:
// behind a draw with its rows, one batch of 4096 / 8192 / 30,000 9.6 / 11.7 / 24.3 us with 256 threads for 512 weights and the
// masses fetched anew behind the minimum, 8.6 / 10.0 / 19.5 so.
constexpr uint32_t kWeightThreads = 512;

__global__ __launch_bounds__(kWeightThreads) void batch_weights_kernel(WeightArgs wa)
{
  __shared__ float red[kWeightThreads / kWave];
  batch_weights(wa, blockIdx.x, red, blockIdx.y, gridDim.y);
}

// Long rows (frame stacks): a workgroup copies kUnroll * blockDim consecutive vectors of one row,
// all loads issued before the first store so that a whole row can be in flight.
// Some workgroups can take a side job that touches none of the copied bytes (its loads issued
// behind the row loads, its work done once the row has been stored), so that a learner step
// needs no launch of its own for it and the grid stays at one workgroup per row (the chip holds
// exactly 512 workgroups of 1024 lanes at a time, the size of a learner batch):
//   kUpdate = 1  workgroup 0 writes a batch of (key, priority) pairs back into the sum tree;
//   kUpdate = 2  the rows are a freshly drawn batch whose own priorities are written back: the
//                workgroup of row i handles pair i (slot and old mass are known from the draw;
//                it wins unless a later sample drew the same slot), which spreads the atomics
//                over the whole chip;
//   kWeights     the first weight_blocks workgroups (after workgroup 0 if kUpdate = 1) write one
//                batch's importance weights each.
template <typename P, int kUnroll, bool kWeights, int kUpdate>
__global__ __launch_bounds__(kLongCopyThreads) void copy_rows_long_kernel(const uint8_t *__restrict__ src, RowMap smap,
                                                                          uint8_t *__restrict__ dst, RowMap dmap,
                                                                          uint32_t vecs_per_row, uint32_t chunks_per_row,
                                                                          uint64_t row_bytes, WeightArgs wa,
                                                                          uint32_t weight_blocks, UpdateArgs ua)
{
  const uint32_t blk = blockIdx.x;
  const uint32_t row = blk / chunks_per_row;
  const uint32_t chunk = blk - row * chunks_per_row;
  const uint8_t *s = src + map_row(smap, row) * row_bytes;
  uint8_t *d = dst + map_row(dmap, row) * row_bytes;
  const uint32_t v0 = chunk * (kUnroll * blockDim.x) + threadIdx.x;
  typename P::Reg tmp[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t v = v0 + u * blockDim.x;
    if (v < vecs_per_row) tmp[u] = load_piece_streaming<P>(s, v, row_bytes);
  }
  // side-job loads go out behind the row loads; the row is stored as soon as it has arrived
  UpdateLane ul{};
  if (kUpdate == 1 && blk == 0) ul = update_batch_load(ua);
  const bool writer = kUpdate == 2 && chunk == 0 && threadIdx.x < kWave;  // first wave of the row's first workgroup
  uint32_t my_slot = 0;
  bool later_dup = false;
  if (writer) {
    my_slot = ua.slot_hint[row];
    for (uint32_t j = row + 1 + threadIdx.x; j < ua.m; j += kWave) later_dup |= ua.slot_hint[j] == my_slot;
    if (threadIdx.x == 0) {
      ul.old = ua.mass_hint[row];
      ul.prio = ua.prio[row];
    }
  }
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t v = v0 + u * blockDim.x;
    if (v < vecs_per_row) store_piece_streaming<P>(d, v, row_bytes, tmp[u]);
  }
  if (kUpdate == 1) {
    __shared__ uint32_t h_slot[kDedupeSlots];
    __shared__ uint32_t h_pos[kDedupeSlots];
    if (blk == 0) update_batch_apply(ua, ul, h_slot, h_pos);
  }
  if (writer) {
    const bool loses = __ballot(later_dup) != 0;  // last occurrence wins, as in a sequential loop
    if (threadIdx.x == 0) {
      bool clamped;
      const uint64_t q = quantise_priority(ul.prio, ua.qp, &clamped);  // counted for losers too
      if (!loses) {
        ua.tv.level[0][my_slot] = q;
        add_to_ancestors(ua.tv, my_slot, q - ul.old);
      }
      if (clamped) atomic_add_u64(&ua.st->n_clamped, 1);
    }
  }
  if (kWeights) {
    __shared__ float red[kLongCopyThreads / kWave];
    const uint32_t first = kUpdate == 1 ? 1 : 0;
    if (blk >= first && blk < first + weight_blocks) batch_weights(wa, blk - first, red);
  }
}

// Long rows from a dense source into the ring (the payload of an add round: row i of the source is its
// i-th run of row_bytes bytes): the copy is cut into runs of kUnroll * blockDim vectors whatever the row
// boundaries, so that every lane carries a full load (a 28,224-byte row fills only 86 % of a workgroup's
// 2048 vector slots); each vector finds its destination row by one division.  (For gathers, whose source
// rows are looked up per row, one workgroup per row is faster.)
template <typename P, int kUnroll>
__global__ __launch_bounds__(kLongCopyThreads) void copy_rows_dense_kernel(const uint8_t *__restrict__ src,
                                                                           uint8_t *__restrict__ dst, RowMap dmap,
                                                                           uint32_t vecs_per_row, uint64_t row_bytes,
                                                                           uint32_t total_vecs)
{
  const uint32_t f0 = blockIdx.x * (kUnroll * blockDim.x) + threadIdx.x;
  typename P::Reg tmp[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t f = f0 + u * blockDim.x;
    if constexpr (P::kWhole) {  // the source is one run of pieces
      if (f < total_vecs) tmp[u] = load_piece_streaming<P>(src, f, 0);
    } else {
      const uint32_t row = f / vecs_per_row, v = f - row * vecs_per_row;
      if (f < total_vecs) tmp[u] = load_piece_streaming<P>(src + row * row_bytes, v, row_bytes);
    }
  }
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t f = f0 + u * blockDim.x;
    if (f < total_vecs) {
      const uint32_t row = f / vecs_per_row, v = f - row * vecs_per_row;
      store_piece_streaming<P>(dst + map_row(dmap, row) * row_bytes, v, row_bytes, tmp[u]);
    }
  }
}

// Long rows looked up through row maps (gathers), packed the same way: a workgroup's run of
// kUnroll * blockDim vectors touches at most kPackedRows rows, whose source and destination offsets its
// first lanes fetch once.  The first weight_blocks workgroups write one batch's importance weights
// each instead of copying.
constexpr uint32_t kPackedRows = 10;  // rows longer than 256 vectors: 2048 / 257 + 2

template <typename P, int kUnroll, bool kWeights>
__global__ __launch_bounds__(kLongCopyThreads) void copy_rows_packed_kernel(const uint8_t *__restrict__ src, RowMap smap,
                                                                            uint8_t *__restrict__ dst, RowMap dmap,
                                                                            uint32_t nrows, uint32_t vecs_per_row,
                                                                            uint64_t row_bytes, uint32_t total_vecs,
                                                                            WeightArgs wa, uint32_t weight_blocks)
{
  if (kWeights && blockIdx.x < weight_blocks) {
    __shared__ float red[kLongCopyThreads / kWave];
    batch_weights(wa, blockIdx.x, red);
    return;
  }
  __shared__ uint64_t src_off[kPackedRows], dst_off[kPackedRows];
  const uint32_t blk = blockIdx.x - (kWeights ? weight_blocks : 0);
  const uint32_t first = blk * (kUnroll * blockDim.x);
  const uint32_t r0 = first / vecs_per_row;
  if (threadIdx.x < kPackedRows && r0 + threadIdx.x < nrows) {
    src_off[threadIdx.x] = map_row(smap, r0 + threadIdx.x) * row_bytes;
    dst_off[threadIdx.x] = map_row(dmap, r0 + threadIdx.x) * row_bytes;
  }
  __syncthreads();
  typename P::Reg tmp[kUnroll];
  uint32_t ri[kUnroll], v[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t f = first + threadIdx.x + u * blockDim.x;
    const uint32_t row = f / vecs_per_row;
    ri[u] = row - r0;
    v[u] = f - row * vecs_per_row;
    if (f < total_vecs) tmp[u] = load_piece_streaming<P>(src + src_off[ri[u]], v[u], row_bytes);
  }
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t f = first + threadIdx.x + u * blockDim.x;
    if (f < total_vecs) store_piece_streaming<P>(dst + dst_off[ri[u]], v[u], row_bytes, tmp[u]);
  }
}

// Short rows: 2^lanes_log2 lanes per row, several rows per workgroup.
struct ShortCopyArgs {
  const uint8_t *src;
  RowMap smap;
  uint8_t *dst;
  RowMap dmap;
  uint64_t nrows;
  uint32_t vecs_per_row, lanes_log2;
  uint64_t row_bytes;
};

template <typename P>
__device__ __forceinline__ void copy_rows_short_block(const ShortCopyArgs &c, uint32_t blk)
{
  const uint32_t rows_per_block = blockDim.x >> c.lanes_log2;
  const uint64_t row = (uint64_t)blk * rows_per_block + (threadIdx.x >> c.lanes_log2);
  const uint32_t v = threadIdx.x & ((1u << c.lanes_log2) - 1);
  if (row >= c.nrows || v >= c.vecs_per_row) return;
  const uint8_t *s = c.src + map_row(c.smap, row) * c.row_bytes;
  store_piece<P>(c.dst + map_row(c.dmap, row) * c.row_bytes, v, c.row_bytes, load_piece<P>(s, v, c.row_bytes));
}

template <typename P>
__global__ __launch_bounds__(256) void copy_rows_short_kernel(ShortCopyArgs c)
{
  copy_rows_short_block<P>(c, blockIdx.x);
}

// All four payload columns of an add round with short observation rows, in one launch: 2^lanes_log2
// lanes per transition copy its observation, its action bytes, and (first lane) its partial
// return and accumulated discount.  act, ret, gacc may be null.
template <typename P>
__global__ __launch_bounds__(256) void add_payload_short_kernel(const uint8_t *__restrict__ obs,
                                                                const uint8_t *__restrict__ act,
                                                                const float *__restrict__ ret,
                                                                const float *__restrict__ gacc,
                                                                uint8_t *__restrict__ obs_ring,
                                                                uint8_t *__restrict__ act_ring,
                                                                float *__restrict__ ret_ring,
                                                                float *__restrict__ gacc_ring, RowMap dmap,
                                                                uint64_t nrows, uint32_t vecs_per_row,
                                                                uint32_t lanes_log2, uint64_t obs_bytes,
                                                                uint32_t act_bytes)
{
  const uint32_t rows_per_block = blockDim.x >> lanes_log2, lanes = 1u << lanes_log2;
  const uint64_t row = (uint64_t)blockIdx.x * rows_per_block + (threadIdx.x >> lanes_log2);
  const uint32_t v = threadIdx.x & (lanes - 1);
  if (row >= nrows) return;
  const uint64_t to = map_row(dmap, row);
  if (v < vecs_per_row)
    store_piece<P>(obs_ring + to * obs_bytes, v, obs_bytes, load_piece<P>(obs + row * obs_bytes, v, obs_bytes));
  if (act)
    for (uint32_t by = v; by < act_bytes; by += lanes) act_ring[to * act_bytes + by] = act[row * act_bytes + by];
  if (v == 0) {
    if (ret) ret_ring[to] = ret[row];
    if (gacc) gacc_ring[to] = gacc[row];
  }
}

// --------------------------------------------------------------------------------------------
// add: masses of the new keys, and their sums into the upper levels
// --------------------------------------------------------------------------------------------
// second: the second copy of the tree is in step with the first, lies that many words behind it and is kept so;
// 0: the first copy alone is written.
struct AddLeavesArgs {
  TreeView tv;
  uint64_t second;
  DeviceState *st;
  uint64_t count;
  const float *prio;  // [count]
  QuantParams qp;
};

// Workgroup blk of n_wgs.
__device__ __forceinline__ void add_leaves_block(const AddLeavesArgs &a, uint32_t blk, uint32_t n_wgs, DenseSums &sh)
{
  const uint64_t i = (uint64_t)blk * blockDim.x + threadIdx.x;
  const bool active = i < a.count;
  const uint64_t tail = a.st->tail;
  const float prio = a.prio[active ? i : 0];
  const uint64_t slot = ring_slot(a.tv, tail + (active ? i : 0));
  bool clamped = false;
  const uint64_t q = quantise_priority(prio, a.qp, &clamped);
  if (active) {
    a.tv.level[0][slot] = q;  // the slot was empty (mass 0): the ring is never over-filled
    if (a.second) a.tv.level[0][slot + a.second] = q;
  }
  add_dense_to_ancestors(a.tv, active, slot, q, a.second, sh);
  advance_state(&a.st->ticket_add, &a.st->tail, tail + a.count, n_wgs);
  const uint64_t nc = __popcll(__ballot(active && clamped));
  if (nc && lane_id() == 0) atomic_add_u64(&a.st->n_clamped, nc);
}

constexpr int kLeavesThreads = 1024;  // most threads per workgroup of add_leaves_kernel and evict_leaves_kernel

// Small payload columns of the transitions that add_leaves_kernel enters (each may be null).
struct AddColumns {
  const uint8_t *act;
  const float *ret, *gacc;
  uint8_t *act_ring;
  float *ret_ring, *gacc_ring;
  uint32_t act_bytes;
};

// Up to this many action bytes a lane of add_leaves_kernel copies a transition's small columns on the way: both launches
// are a few dependent loads and a round trip of atomics, so one of them goes.  More bytes would be strided accesses, one
// cache line per lane, which add_payload_short_kernel shares out over several lanes.
// Actor round of 18,000 frame stacks (n-step, payload, masses, eviction): 178 - 180 us either way, the payload copy bounds it;
// add and eviction of 700 rows of 5000 bytes 14.6 -> 11.1 us, the pieces of any alignment included.
constexpr uint32_t kColumnsInAddBytes = 16;

// The small columns of transition i into slot, by one lane.
__device__ __forceinline__ void add_columns(const AddColumns &c, uint64_t i, uint64_t slot)
{
  if (c.ret) c.ret_ring[slot] = c.ret[i];
  if (c.gacc) c.gacc_ring[slot] = c.gacc[i];
  if (!c.act) return;
  const uint8_t *const s = c.act + i * c.act_bytes;
  uint8_t *const d = c.act_ring + slot * c.act_bytes;
  if (c.act_bytes < 4) {
    for (uint32_t at = 0; at < c.act_bytes; ++at) d[at] = s[at];
  } else {
    for (uint32_t at = 0; at < c.act_bytes; at += 4) {  // the last piece overlaps the one before it
      const uint32_t p = min(at, c.act_bytes - 4);
      *reinterpret_cast<u32_any *>(d + p) = *reinterpret_cast<const u32_any *>(s + p);
    }
  }
}

__global__ __launch_bounds__(kLeavesThreads) void add_leaves_kernel(AddLeavesArgs a, AddColumns c)
{
  __shared__ DenseSums sh;
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < a.count && (c.act || c.ret || c.gacc))  // (the tail moves on only after a barrier of add_leaves_block)
    add_columns(c, i, ring_slot(a.tv, a.st->tail + i));
  add_leaves_block(a, blockIdx.x, gridDim.x, sh);
}

// A whole add of short observation rows in one launch: a workgroup copies the rows of as many transitions as it has
// threads, 2^lanes_log2 lanes per row, then each of its threads has the small columns and the mass of one.  The two launches
// that it replaces are each a few dependent loads; the atomics on the upper levels ask for large workgroups, the rows for
// many.  Add and eviction, us, as two launches / with 256 / 512 / 1024 threads:
//    3000 rows of  32 B of 2^20 slots  10.0 /  8.0 /  8.1 /  8.5      51,200   11.3 / 10.6 /  9.5 /  9.5
//    3000 rows of 256 B of 2^20 slots  10.0 /  9.1 /  9.6 / 12.2      51,200   14.5 / 12.8 / 12.6 / 14.9
//    3000 rows of 128 B of 2^24 slots  10.4 /  8.8 /  8.9 / 10.7      51,200   12.3 / 12.0 / 11.1 / 12.1
//     400 rows of 500 B of 2^20 slots   8.7 /  9.2 /  9.7 /  9.8      18,000   13.6 / 12.2 / 13.1 / 17.6
// and with 512 / 1024, whole calls, of 2^22 slots:
//    300,000 rows of 16 B  18.9 / 18.7 / 16.5    64 B  24.2 / 22.9 / 20.3    256 B  43.2 / 33.3 / 37.1
//    400,000               22.2 / 23.4 / 18.2          29.3 / 28.7 / 22.4           53.6 / 42.1 / 46.7
constexpr uint32_t kAddRowsInOneBytes = 256;

constexpr uint32_t add_rows_threads(uint64_t count, uint64_t obs_bytes)
{
  return count > 16384 ? (count > 200000 && obs_bytes <= 64 ? 1024 : 512) : 256;
}

template <typename P>
__global__ __launch_bounds__(kLeavesThreads) void add_rows_kernel(AddLeavesArgs a, AddColumns c, const uint8_t *__restrict__ obs,
                                                                  uint8_t *__restrict__ obs_ring, uint32_t vecs_per_row,
                                                                  uint32_t lanes_log2, uint64_t obs_bytes)
{
  constexpr uint32_t kAhead = 8;  // pieces per lane in flight
  __shared__ DenseSums sh;
  const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x;
  const uint32_t n = (uint32_t)min((uint64_t)blockDim.x, a.count - i0), rows = blockDim.x >> lanes_log2;  // per pass
  const uint32_t v = threadIdx.x & ((1u << lanes_log2) - 1);
  const uint64_t first = ring_slot(a.tv, a.st->tail + i0);
  auto slot_of = [&](uint32_t r) { return first + r < a.tv.P ? first + r : first + r - a.tv.P; };
  if (v < vecs_per_row) {
    for (uint32_t r0 = threadIdx.x >> lanes_log2; r0 < n; r0 += kAhead * rows) {
      typename P::Reg t[kAhead];
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u)
        if (r0 + u * rows < n) t[u] = load_piece<P>(obs + (i0 + r0 + u * rows) * obs_bytes, v, obs_bytes);
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u)
        if (r0 + u * rows < n) store_piece<P>(obs_ring + slot_of(r0 + u * rows) * obs_bytes, v, obs_bytes, t[u]);
    }
  }
  if (threadIdx.x < n) add_columns(c, i0 + threadIdx.x, slot_of(threadIdx.x));
  add_leaves_block(a, blockIdx.x, gridDim.x, sh);
}

// A small add round in one launch (Algorithm 1: ComputePriorities, replay.Add): 2^lanes_log2 lanes
// per transition copy its payload row into the ring; the first of them computes the n-step
// priority, stores the partial return and the accumulated discount, and enters the mass into the
// tree; the last workgroup to finish moves the tail on.  act may be null.
// The masses of a workgroup's transitions are collected in LDS and entered into the upper levels by
// whole waves of 64 neighbouring transitions, so that a node receives one atomic per 64 of them.
constexpr int kAddRoundThreads = 1024;

struct AddRoundArgs {
  NstepArgs ns;
  TreeView tv;
  uint64_t second;  // as in AddLeavesArgs
  DeviceState *st;
  QuantParams qp;
  const uint8_t *obs, *act;  // [S*T, obs_bytes], [S*T, act_bytes] (act may be null)
  uint8_t *obs_ring, *act_ring;
  float *ret_ring, *gacc_ring;
  uint32_t vecs_per_row, lanes_log2;
  uint64_t obs_bytes;
  uint32_t act_bytes;
};

// Workgroup blk of n_wgs of such a round; sh_slot, sh_q: blockDim words of LDS each.
template <typename P>
__device__ __forceinline__ void add_round_small_block(const AddRoundArgs &a, uint32_t blk, uint32_t n_wgs,
                                                      uint64_t *sh_slot, uint64_t *sh_q)
{
  const uint32_t rows_per_block = blockDim.x >> a.lanes_log2, lanes = 1u << a.lanes_log2;
  const uint32_t r = threadIdx.x >> a.lanes_log2;  // row of this workgroup
  const uint64_t i = (uint64_t)blk * rows_per_block + r;
  const uint32_t v = threadIdx.x & (lanes - 1);
  const uint64_t count = (uint64_t)a.ns.S * a.ns.T;
  const bool in_range = i < count;
  bool clamped = false;
  const uint64_t tail = a.st->tail;
  if (in_range) {
    const uint64_t slot = ring_slot(a.tv, tail + i);
    for (uint32_t vv = v; vv < a.vecs_per_row; vv += lanes)
      store_piece<P>(a.obs_ring + slot * a.obs_bytes, vv, a.obs_bytes,
                     load_piece<P>(a.obs + i * a.obs_bytes, vv, a.obs_bytes));
    if (a.act)
      for (uint32_t by = v; by < a.act_bytes; by += lanes)
        a.act_ring[slot * a.act_bytes + by] = a.act[i * a.act_bytes + by];
    if (v == 0) {
      const NstepOut o = nstep_one(a.ns, i);
      a.ret_ring[slot] = o.R;
      a.gacc_ring[slot] = o.G;
      const uint64_t q = quantise_priority(o.p, a.qp, &clamped);
      a.tv.level[0][slot] = q;  // the slot was empty (mass 0): the ring is never over-filled
      if (a.second) a.tv.level[0][slot + a.second] = q;
      sh_slot[r] = slot;
      sh_q[r] = q;
    }
  }
  const uint64_t nc = __popcll(__ballot(clamped));
  if (nc && lane_id() == 0) atomic_add_u64(&a.st->n_clamped, nc);
  __syncthreads();
  if (threadIdx.x < ((rows_per_block + kWave - 1) & ~(uint32_t)(kWave - 1))) {  // whole waves
    const uint32_t e = threadIdx.x;
    const bool active = e < rows_per_block && (uint64_t)blk * rows_per_block + e < count;
    add_runs_to_ancestors(a.tv, active, active ? sh_slot[e] : 0, active ? sh_q[e] : 0, a.second);
  }
  advance_state(&a.st->ticket_add, &a.st->tail, tail + count, n_wgs);
}

template <typename P>
__global__ __launch_bounds__(kAddRoundThreads) void add_round_small_kernel(AddRoundArgs a)
{
  __shared__ uint64_t sh_slot[kAddRoundThreads], sh_q[kAddRoundThreads];
  add_round_small_block<P>(a, blockIdx.x, gridDim.x, sh_slot, sh_q);
}

// evict: zero the masses of the e oldest keys and take them out of the upper levels
struct EvictLeavesArgs {
  TreeView tv;
  uint64_t second;  // as in AddLeavesArgs
  DeviceState *st;
  uint64_t e;
};

__global__ __launch_bounds__(kLeavesThreads) void evict_leaves_kernel(EvictLeavesArgs a)
{
  __shared__ DenseSums sh;
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool active = i < a.e;
  const uint64_t head = a.st->head;
  const uint64_t slot = ring_slot(a.tv, head + (active ? i : 0));
  const uint64_t old = a.tv.level[0][slot];
  if (active) {
    a.tv.level[0][slot] = 0;
    if (a.second) a.tv.level[0][slot + a.second] = 0;
  }
  add_dense_to_ancestors(a.tv, active, slot, 0 - old, a.second, sh);
  advance_state(&a.st->ticket_evict, &a.st->head, head + a.e, gridDim.x);
}

// --------------------------------------------------------------------------------------------
// update: two passes so that, of several pairs naming one key, the last one wins
// --------------------------------------------------------------------------------------------
// pass 1: every valid pair bids its position for the slot (highest position wins)
struct ClaimArgs {
  uint64_t P;
  FastDiv p_div;
  DeviceState *st;
  uint32_t m;           // 0: nothing to claim
  const uint64_t *key;
  uint32_t *claim;
};

__device__ __forceinline__ void update_claim_block(const ClaimArgs &c, uint32_t blk)
{
  const uint32_t i = blk * blockDim.x + threadIdx.x;
  bool stale = false;
  if (i < c.m) {
    const uint64_t k = c.key[i];
    if (k >= c.st->head && k < c.st->tail)
      __hip_atomic_fetch_max(c.claim + (k - fast_div(k, c.p_div) * c.P), i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      stale = true;
  }
  const uint64_t ns = __popcll(__ballot(stale));
  if (ns && lane_id() == 0) atomic_add_u64(&c.st->n_stale, ns);
}

__global__ __launch_bounds__(256) void update_claim_kernel(ClaimArgs c) { update_claim_block(c, blockIdx.x); }

// Everything that only needs the results of a draw of short rows, in one launch: the gather of the rows,
// the importance weights, and the first pass of a priority update of the drawn keys.  Workgroups
// [0, copy_blocks) copy, the next batches * weight_parts write weights, the rest claim.
template <typename P>
__global__ __launch_bounds__(kWeightThreads) void finish_short_kernel(ShortCopyArgs c, uint32_t copy_blocks, WeightArgs wa,
                                                           uint32_t batches, uint32_t weight_parts, ClaimArgs cl)
{
  __shared__ float red[kWeightThreads / kWave];
  const uint32_t blk = blockIdx.x, weight_blocks = batches * weight_parts;
  if (blk < copy_blocks) {
    copy_rows_short_block<P>(c, blk);
  } else if (blk < copy_blocks + weight_blocks) {
    const uint32_t wb = blk - copy_blocks;
    batch_weights(wa, wb / weight_parts, red, wb % weight_parts, weight_parts);
  } else {
    update_claim_block(cl, blk - copy_blocks - weight_blocks);
  }
}

__global__ __launch_bounds__(256) void update_apply_kernel(TreeView tv, DeviceState *__restrict__ st, uint32_t m,
                                                           const uint64_t *__restrict__ key,
                                                           const float *__restrict__ prio, QuantParams qp,
                                                           uint32_t *__restrict__ claim, QSource qs)
{
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  bool clamped = false, wins = false;
  uint64_t slot = 0, delta = 0;
  if (i < m) {
    const uint64_t k = key[i];
    const TdInputs td = qs.q_taken ? td_inputs(qs, i) : TdInputs{};
    if (k >= st->head && k < st->tail) {
      slot = ring_slot(tv, k);
      const float p = qs.q_taken ? td_priority(qs.ret[slot], qs.gacc[slot], td) : prio[i];
      if (qs.q_taken && qs.prio_out) qs.prio_out[i] = p;
      const uint64_t q = quantise_priority(p, qp, &clamped);
      if (claim[slot] == i + 1) {
        wins = true;
        delta = q - tv.level[0][slot];
        tv.level[0][slot] = q;
        claim[slot] = 0;
      }
    } else if (qs.q_taken && qs.prio_out) {
      qs.prio_out[i] = 0.0f;
    }
  }
  add_runs_to_ancestors(tv, wins, slot, delta);  // the keys of a drawn batch ascend: neighbours share their upper nodes
  const uint64_t nc = __popcll(__ballot(clamped));
  if (nc && lane_id() == 0) atomic_add_u64(&st->n_clamped, nc);
}

// --------------------------------------------------------------------------------------------
// sample: stratified descent, four samples per wavefront (sample_kernel), and in the same launch whatever of
// replay.Sample the caller wants there.  The importance weights need the smallest mass of a whole batch, which the
// workgroups of a batch settle through a ticket; where another launch follows anyway (the gather of long rows), or the
// batch is too large for one workgroup's registers, that launch writes them (batch_weights).
// --------------------------------------------------------------------------------------------
// What every draw needs, and no more: the step kernel has these among its arguments, and with 8 bytes more in them its
// launches took 0.2 us longer.
struct DrawArgs {
  TreeView tv;
  const DeviceState *st;
  uint32_t k;                // samples per batch
  const uint64_t *rnd;       // [nb,k]
  uint64_t *key_out;         // [nb,k] or null
  uint32_t *slot_out;        // [nb,k]
  uint64_t *mass;            // [nb,k]: mass of each drawn transition, for the weights
};

// The payload columns of a transition and where a gather writes them (each output may be null).
struct GatherArgs {
  const uint8_t *act;
  uint32_t act_bytes;
  const float *ret, *gacc;
  uint8_t *act_out;
  float *ret_out, *gacc_out;
  const uint8_t *obs;
  uint64_t obs_bytes;
  uint8_t *obs_out;
};

struct SampleArgs : DrawArgs {
  const uint64_t *top;       // the level that the walks start from (its address at a fixed place of the arguments)
  const uint64_t *k_dev;     // not null: the number of samples is read here, on the device (waves beyond it idle)
  FastDiv k_div;             // division by k (unused with k_dev)
  const uint32_t *gen;       // not null: keys are (generation of the slot << 32) | slot instead of ring keys
  GatherArgs g;              // obs_out null: the rows are gathered by another launch (copy_rows_*)
  float *weight_out;         // null: no weights, or written by another launch (batch_weights)
  float beta;
  uint32_t *ticket;          // with weight_out: words that lie kTicketStride apart, 0 before and after: one per batch ...
  uint32_t *ticket_ahead;    // the words that a launch to come will use, at most this many: cleared by this launch
  uint32_t ticket_lines;
  uint32_t *board;           // sample_rows_kernel: as `ticket`, a word per sample; null: tickets
  uint32_t *board_ahead;
  uint32_t board_words;
  uint32_t *claim;           // not null: the first pass of an update of the drawn keys (update_claim_block) as well
};

constexpr uint32_t kTicketStride = 16;
constexpr uint32_t kTicketSets = 4;  // a power of two

// Where word i of the board lies: 64 of every 256 bytes are used, so that the words are spread over more of the memory's
// channels (64 samples 4.4 -> 4.2 us, 256 5.4 -> 5.2).  A batch's words start at an even one.
__host__ __device__ constexpr uint32_t board_place(uint32_t i) { return i / 16 * 64 + i % 16; }
__host__ __device__ constexpr uint32_t board_stride(uint32_t k) { return (k + 1) & ~1u; }
constexpr uint32_t kBoardWordsMax = 4096;  // of a launch

// The words that launches to come will use are cleared by the n threads that call this.
__device__ __forceinline__ void clear_ahead(const SampleArgs &a, uint32_t thread, uint32_t n)
{
  for (uint32_t i = thread; i < a.ticket_lines; i += n) a.ticket_ahead[i * kTicketStride] = 0;
  for (uint32_t i = thread; i < a.board_words; i += n) a.board_ahead[board_place(i)] = 0;
}

// Waits until every load (and store) that this wave has issued is through.
__device__ __forceinline__ void wait_for_all_loads()
{
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0); the other counters at their maxima (not waited for)
}

struct Drawn {
  uint64_t slot, mass;
  uint64_t x;  // where in the slot's interval of cumulative mass the point fell: 0 <= x < mass
};

// Where a walk stands after the top level: node idx of that level, whose interval of cumulative mass
// holds the point; x is the point's offset inside the interval, mass the node's mass.
struct TopHit {
  uint64_t idx, x, mass;
};

__device__ __forceinline__ uint32_t read_lane_u32(uint32_t v, uint32_t l)
{
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}
__device__ __forceinline__ uint64_t read_lane_u64(uint64_t v, uint32_t l)
{
  return ((uint64_t)read_lane_u32((uint32_t)(v >> 32), l) << 32) | read_lane_u32((uint32_t)v, l);
}

typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

// The top level in the registers of one wave: lane l holds the masses v[0..8) of nodes 8l .. 8l+7, and, of a level of
// more than 512 nodes, w[0..8) of nodes 512 + 8l .. 512 + 8l+7.  Lanes beyond the level hold its first nodes again, count
// as empty in the sums and are never found: their prefix sum is the level's.  (No load sits in a branch: what other loads
// the wave has in flight would be waited for behind it.)  load() only issues the loads (16 bytes wide), scan() waits for
// them.
// kMayBeWide: levels of more than 512 nodes are provided for.
template <bool kMayBeWide>
struct TopLevel {
  uint64_t v[8], w[8];
  uint64_t before, before_w;  // sum of all nodes before this lane's (before_w: of the whole level if there are none)
  bool wide;                  // the same for all lanes
  bool in, in_w;              // this lane's nodes v, w belong to the level

  static __device__ __forceinline__ void load_8(uint64_t (&r)[8], const uint64_t *top, uint32_t i0, uint32_t n_pad)
  {
    const uint64_t *const at = top + (i0 < n_pad ? i0 : 0);
#pragma unroll
    for (int t = 0; t < 8; t += 2) {
      const u64x2 v2 = *reinterpret_cast<const u64x2 *>(at + t);
      r[t] = v2.x, r[t + 1] = v2.y;
    }
  }

  __device__ __forceinline__ void load(const uint64_t *top, uint32_t n_top)
  {
    const uint32_t i0 = 8 * (uint32_t)lane_id();
    const uint32_t n_pad = (n_top + kFanout - 1) & ~(kFanout - 1);  // the level is zero-padded to this in memory
    wide = kMayBeWide && n_top > 512;
    in = i0 < n_pad, in_w = 512 + i0 < n_pad;
    load_8(v, top, i0, n_pad);
    if (wide) load_8(w, top, 512 + i0, n_pad);
  }

  static __device__ __forceinline__ uint64_t sum_8(const uint64_t (&r)[8])
  {
    uint64_t sum = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) sum += r[t];
    return sum;
  }

  // Returns the sum of the whole level.  (All loads of the wave that come before in the source are on their way by then: the
  // statement in assembly, which names the values, keeps them from being moved behind it, or into a branch on `in`.)
  __device__ __forceinline__ uint64_t scan()
  {
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]));
    const uint64_t mine = in ? sum_8(v) : 0, incl = wave_inclusive_scan(mine);
    before = incl - mine;
    uint64_t total = read_lane_u64(incl, kWave - 1);
    before_w = total;
    if (wide) {
      const uint64_t mine_w = in_w ? sum_8(w) : 0, incl_w = wave_inclusive_scan(mine_w);
      before_w = total + incl_w - mine_w;
      total += read_lane_u64(incl_w, kWave - 1);
    }
    return total;
  }

  // The group of eight nodes (one lane's v or w) that holds x: the last one whose prefix sum is <= x.
  __device__ __forceinline__ uint32_t find_group(uint64_t x) const
  {
    // lane 0 has before = 0 <= x; without w the second ballot is empty, x being below the level's sum
    const uint32_t l = __popcll(__ballot(before <= x)) - 1;
    return kMayBeWide ? l + __popcll(__ballot(before_w <= x)) : l;
  }

  static __device__ __forceinline__ TopHit find_in(const uint64_t (&r)[8], uint64_t before_r, uint32_t group, uint64_t x)
  {
    const uint32_t l = group & (kWave - 1);
    uint64_t p = before_r, p_hit = before_r, v_hit = r[0];
    uint32_t t_hit = 0;
#pragma unroll
    for (int t = 1; t < 8; ++t) {
      p += r[t - 1];
      const bool le = p <= x;  // true for the first few t only: the prefix sums do not decrease
      t_hit = le ? t : t_hit;
      p_hit = le ? p : p_hit;
      v_hit = le ? r[t] : v_hit;
    }
    return TopHit{8ull * group + read_lane_u32(t_hit, l), x - read_lane_u64(p_hit, l), read_lane_u64(v_hit, l)};
  }

  // The last node whose prefix sum is <= x: the group by ballots, the node inside it by eight comparisons that every
  // lane makes for itself, the winner's values by lane reads.
  __device__ __forceinline__ TopHit find(uint64_t x) const
  {
    const uint32_t group = find_group(x);
    return !kMayBeWide || group < kWave ? find_in(v, before, group, x) : find_in(w, before_w, group, x);
  }
};

// One wavefront walks from its place in the top level down to the slot whose cumulative-mass interval holds the point.
// Called by all 64 lanes.
// between(): called once, when the loads of the first level below the top are on their way (right away if
// the tree has no such level): arithmetic that does not depend on the walk costs nothing there.
template <typename Between>
__device__ __forceinline__ Drawn walk_down(const TreeView &tv, const TopHit &top, Between between)
{
  const uint32_t lane = lane_id();
  // the lowest levels' addresses are at fixed places of the arguments: fetched with them, not on the way down
  const uint64_t *const low0 = tv.level[0], *const low1 = tv.level[1];
  uint64_t x = top.x, idx = top.idx, mass = top.mass;
  // up to 64 children per step, prefix sum across the wave, first child whose running sum exceeds the remainder
  auto select = [&](uint64_t c, uint32_t fl) {
    const uint64_t sc = wave_inclusive_scan(c);
    const uint64_t hit = __ballot(sc > x);
    const uint32_t sel = hit ? __ffsll((unsigned long long)hit) - 1 : (1u << fl) - 1;
    mass = read_lane_u64(c, sel);
    x -= read_lane_u64(sc, sel) - mass;
    idx = (idx << fl) + sel;
  };
  auto level = [&](int l) { return l == 0 ? low0 : l == 1 ? low1 : tv.level[l]; };
  int l = (int)tv.nlev - 2;
  if (l < 0) {
    between();
  } else {
    const uint32_t fl = tv.top_log2;  // a summit's node has fewer children than the wave has lanes
    const uint64_t c = level(l)[(idx << fl) + (lane & ((1u << fl) - 1))];
    between();
    select(lane >> fl ? 0 : c, fl);
    for (--l; l >= 0; --l) select(level(l)[idx * kFanout + lane], kFanoutLog2);
  }
  return Drawn{idx, mass, x};
}

// The ring key of a drawn slot: head + its distance from the head's slot around the ring.
// head_slot = head mod P.
__device__ __forceinline__ uint64_t ring_key(uint64_t slot, uint64_t head, uint64_t head_slot, uint64_t P)
{
  return head + (slot >= head_slot ? slot - head_slot : slot + P - head_slot);
}

// The walk of four samples at once, one per 16-lane row of the wave (every lane of a row holds its sample's values):
// a lane takes four neighbouring children, so that a level costs four steps of a prefix sum for four samples
// instead of six for one.  With a whole wave per sample the arithmetic of the scans, not memory, was what a call
// of many samples took (replay.Sample of 16 x 512 from 2^21 slots: 13.6 us, now 9.1; an eviction of 65,536 in three
// rounds: 115, now 55); a call of few is bound by its chain of round trips (256 from 2^20 slots, alone: 7.0 us, now 6.1).
struct RowWalk {
  uint64_t idx, x, mass;
};

// c ? a : b without a branch (which the compiler makes of a choice between 64-bit values, and moves loads into).
__device__ __forceinline__ uint64_t pick(bool c, uint64_t a, uint64_t b)
{
  const uint32_t lo = c ? (uint32_t)a : (uint32_t)b, hi = c ? (uint32_t)(a >> 32) : (uint32_t)(b >> 32);
  return ((uint64_t)hi << 32) | lo;
}

// The lane of the row that holds the first running sum above x has found the child: its values go to the whole row.
// kMass: the child's mass is wanted.
template <bool kMass>
__device__ __forceinline__ void row_descend(RowWalk &w, const uint64_t *lv, uint32_t fl)
{
  const uint32_t lane = lane_id(), gl = lane & 15, child0 = 4 * gl;
  const uint32_t f = 1u << fl;
  const uint64_t base = w.idx << fl;
  // lanes beyond the node's children read its first ones again and count as empty; a node of two children (16-byte
  // aligned all the same) is read together with its neighbour, or with what follows the level in the tree region
  const uint64_t *c = lv + base + (child0 < f ? child0 : 0);
  const u64x2 lo = *reinterpret_cast<const u64x2 *>(c), hi = *reinterpret_cast<const u64x2 *>(c + 2);
  const bool in = child0 < f, in2 = child0 + 2 < f;
  const uint64_t c0 = in ? lo.x : 0, c1 = in ? lo.y : 0, c2 = in2 ? hi.x : 0, c3 = in2 ? hi.y : 0;
  const uint64_t p1 = c0 + c1, p2 = p1 + c2, sum = p2 + c3;
  const uint64_t incl = row_inclusive_scan(sum);
  const uint32_t hits = (uint32_t)(__ballot(incl > w.x) >> (lane & 48)) & 0xffffu;
  const uint32_t src = (lane & 48) + (hits ? __ffs(hits) - 1 : 15);
  const uint64_t r = w.x - (incl - sum);  // of use in the lane that has the hit
  const bool ge0 = r >= c0, ge1 = r >= p1, ge2 = r >= p2;
  const uint32_t t = (uint32_t)ge0 + (uint32_t)ge1 + (uint32_t)ge2;
  const uint64_t below = pick(ge2, p2, pick(ge1, p1, pick(ge0, c0, 0)));
  w.idx = base + __shfl(child0 + t, src, kWave);
  w.x = __shfl(r - below, src, kWave);
  if (kMass) w.mass = __shfl(pick(ge2, c3, pick(ge1, c2, pick(ge0, c1, c0))), src, kWave);
}

// Tells the compiler that a loaded value has arrived, where a wait for all loads has just been made: it would wait for the
// value where that is used, and then for every store that the wave has issued in between as well.
template <typename T>
__device__ __forceinline__ void arrived(T &x)
{
  asm volatile("" : "+v"(x));
}

// An observation row by one 16-lane row of a wave.  Everything that the wave has issued before is through when the
// first piece is stored; loaded() is called there.
template <typename Loaded>
__device__ __forceinline__ void copy_row_by_16(uint8_t *__restrict__ d, const uint8_t *__restrict__ s, uint32_t bytes, Loaded loaded)
{
  constexpr int kUnroll = 8;  // pieces per lane in flight: 2 KB of the row
  const uint32_t gl = lane_id() & 15;
  if (bytes < 16) {
    const uint8_t t = s[min(gl, bytes - 1)];
    wait_for_all_loads();
    loaded();
    if (gl < bytes) d[gl] = t;
    return;
  }
  const uint32_t n = (bytes + 15) / 16, last = bytes - 16;
  auto pass = [&](uint32_t v0, auto between) {
    u32x4_any t[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (v0 + 16 * u < n) t[u] = *reinterpret_cast<const u32x4_any *>(s + min(16 * (v0 + 16 * u + gl), last));
    wait_for_all_loads();
    between();
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (v0 + 16 * u < n) *reinterpret_cast<u32x4_any *>(d + min(16 * (v0 + 16 * u + gl), last)) = t[u];
  };
  pass(0, loaded);  // (inside the loop, the values that `loaded` names would be waited for ahead of it)
  for (uint32_t v0 = 16 * kUnroll; v0 < n; v0 += 16 * kUnroll) pass(v0, [] {});
}

// The walks of four samples, one per 16-lane row, from points (every lane of a row holds its sample's) down to the slots.
// between(): called when the walk has left the top level.
template <bool kWide, typename Between>
__device__ __forceinline__ RowWalk walk_four(const TreeView &tv, const TopLevel<kWide> &top, const uint64_t *top_level,
                                             uint64_t point, Between between)
{
  const uint32_t lane = lane_id();
  // top level: the lane that holds the node by a ballot per sample, then its eight nodes anew (they are in the
  // first cache), as if they were the children of a node
  uint32_t l = 0;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const uint32_t ls = top.find_group(read_lane_u64(point, 16 * s));
    l = lane / 16 == (uint32_t)s ? ls : l;
  }
  uint64_t before = __shfl(top.before, l & (kWave - 1), kWave);
  if (top.wide) {
    const uint64_t before_w = __shfl(top.before_w, l & (kWave - 1), kWave);
    before = l < kWave ? before : before_w;
  }
  RowWalk walk;
  walk.x = point - before;
  walk.idx = l;
  const uint64_t *const low0 = tv.level[0], *const low1 = tv.level[1], *const low2 = tv.level[2];
  const uint32_t nlev = tv.nlev;
  uint32_t fl = tv.top_log2;
  fetch_now(low0, low1, low2, fl);
  if (nlev == 1) {
    row_descend<true>(walk, top_level, 3);
    between();
    return walk;
  }
  row_descend<false>(walk, top_level, 3);
  between();
  for (int lv = (int)nlev - 2; lv > 0; --lv) {
    row_descend<false>(walk, lv == 1 ? low1 : lv == 2 ? low2 : tv.level[lv], fl);
    fl = kFanoutLog2;
  }
  row_descend<true>(walk, low0, fl);
  return walk;
}

// Transition `slot` into place o of the outputs, by one 16-lane row of a wave.  Everything that the wave has issued before
// is through when the first output is stored; loaded() is called there.  No store waits for another one (where the small outputs
// each did, 32,768 samples of 1 KB rows took 22.5 us, and 20.2 so, 512 of 32 bytes with their weights 6.9 and 6.6).
template <typename Loaded>
__device__ __forceinline__ void gather_by_16(const GatherArgs &a, uint64_t slot, uint64_t o, Loaded loaded)
{
  // the small columns' loads go out with those of the observation row: partial return, accumulated discount, and the first
  // 64 action bytes (four per lane; fewer than four in all: one per lane)
  const uint32_t gl = lane_id() & 15;
  const uint8_t *const act = a.act + slot * a.act_bytes;
  uint8_t *const act_out = a.act_out + o * a.act_bytes;
  const bool whole_words = a.act_bytes >= 4;
  const uint32_t act_last = a.act_bytes - (whole_words ? 4 : 1), act_at = min(whole_words ? 4 * gl : gl, act_last);
  float col = 0.f;
  uint32_t act_piece = 0;
  const bool ret_lane = gl == 1 && a.ret_out, gacc_lane = gl == 2 && a.gacc_out;
  if (ret_lane) col = a.ret[slot];
  if (gacc_lane) col = a.gacc[slot];
  if (a.act_out) {
    if (whole_words) act_piece = *reinterpret_cast<const u32_any *>(act + act_at);
    else act_piece = act[act_at];
  }
  const auto all_loaded = [&] {
    arrived(col), arrived(act_piece);
    loaded();
  };
  if (a.obs_out) {
    copy_row_by_16(a.obs_out + o * a.obs_bytes, a.obs + slot * a.obs_bytes, (uint32_t)a.obs_bytes, all_loaded);
  } else {
    wait_for_all_loads();
    all_loaded();
  }
  if (a.act_out) {
    if (whole_words) *reinterpret_cast<u32_any *>(act_out + act_at) = act_piece;
    else act_out[act_at] = (uint8_t)act_piece;
    for (uint32_t at = 64 + 4 * gl; at < a.act_bytes; at += 64) {
      const uint32_t p = min(at, act_last);
      *reinterpret_cast<u32_any *>(act_out + p) = *reinterpret_cast<const u32_any *>(act + p);
    }
  }
  if (ret_lane) a.ret_out[o] = col;
  if (gacc_lane) a.gacc_out[o] = col;
}

// Observation rows up to here ride in the draw's launch.  Together / apart, us of device time for one batch of 1500, 4 of 512,
// 16 of 512 and one of 4096 from 2^18 slots (fewer: sample_by_rows, and one batch of more with shorter rows:
// kGatherApartAboveK).  A launch less is 2.4 us on the host, not counted, which decides where a call with its update is bound by
// the host, at some 12 us; one batch of 4096 rows of 4096 bytes is not, and would be 1.3 us shorter apart: the line goes by the
// row alone.
//   rows of  268 B   7.0 /  6.7    6.3 /  6.9    7.7 /  9.2
//           1024 B   8.0 /  8.0    7.5 /  8.2    9.2 / 11.4
//           2048 B   8.6 /  8.5    8.2 /  8.9   11.9 / 14.2   10.8 / 11.7
//           4096 B   9.8 /  9.5   10.0 / 10.7   19.3 / 19.5   16.0 / 14.7
//           5003 B  12.5 / 10.0   12.8 / 12.1   23.8 / 24.5   17.5 / 16.8
constexpr uint32_t kGatherInDrawBytes = 4096;

// Most samples of a batch whose weights the draw's launch can write: its last workgroup writes them all (16,384 of them
// took that launch 21.6 us instead of 8.2 without, where a launch of its own takes 5).
constexpr uint32_t kWeightsInDrawMaxK = 4096;

// One batch of more samples than kGatherApartAboveK of rows up to kGatherApartBytes is gathered by a launch of its own after all,
// which writes the weights as well (a weight per thread, finish_short_kernel): with the draw, the last workgroup's weights are the
// tail of the launch.  (Above kWeightsInDrawMaxK they have a launch of their own either way.)  Us of device time, with / apart,
// from 2^18 slots:
//                    2561          3300          4096
//    rows of   32 B   7.6 / 6.8     8.0 / 7.0     8.6 / 7.0
//             268 B   7.9 / 7.4     8.3 / 7.8     9.0 / 8.3
//            1024 B   8.7 / 8.5     9.1 / 8.8     9.8 / 9.4
// (With 256 threads for 512 weights, apart, 4096: 7.6, 8.8 and 9.9.)  Up to 2560 the 0.2 to 0.7 us are less than the launch more
// costs the host (2.4); beyond, a call with its update is 13 us on the device and 12 on the host.
constexpr uint32_t kGatherApartAboveK = 2560;
constexpr uint64_t kGatherApartBytes = 1024;

// Threads per workgroup.  16 samples (256 threads) spread the draws best over the chip; a batch of at most 32 goes into
// one workgroup, whose waves agree on the smallest mass through LDS (32 samples: 5.7 instead of 6.5 us through tickets
// and memory; with 64 the sixteen waves of the workgroup slow one another down, 8.8 us); a large one has fewer tickets to
// take and more threads for its weights with 32 samples than with 16 (4096 samples 9.9 and 12.1 us, 3000 9.1 and 10.7,
// 2048 8.5 and 8.6, 1500 8.2 and 7.9, 512 7.7 and 6.8).
constexpr uint32_t kSampleMaxThreads = 512;
constexpr int kHeldMasses = 8;  // masses per thread of the workgroup that writes a batch's weights

__host__ __device__ constexpr uint32_t sample_threads(uint32_t k, bool weights)
{
  if (!weights) return 256;
  return k <= 32 ? (k + 3) / 4 * kWave : k > 2048 ? kSampleMaxThreads : 256;
}
static_assert(kHeldMasses * sample_threads(2048, true) >= 2048 && sample_threads(32, true) <= kSampleMaxThreads &&
              kHeldMasses * sample_threads(kWeightsInDrawMaxK, true) >= kWeightsInDrawMaxK);

// Four consecutive samples of a batch per wave: the walks, and with them whatever of replay.Sample the caller wants in
// the same launch: the gather of short observation rows, the importance weights, the first pass of an update.
// The weights need the smallest mass of the whole batch: every workgroup writes its masses through to memory (agent
// scope), takes the batch's ticket, and the one with the last ticket reads all of them back and writes the batch's
// weights.  Only these words cross between workgroups, so no cache has to be written back or invalidated for it.
// A launch leaves its ticket words at 0.  Launches take turns on kTicketSets words per batch, and each also clears the
// words that the launch two turns on will use: whatever left a word at another value (calls that overlapped although
// they must be ordered), the calls after it find their last workgroups again.
// Bound by a chain of round trips (top level, its eight nodes again, a row of children per level, the payload row, with
// weights the ticket and the masses).  Against a wave per sample and a second launch for gather and weights: 16 x 512 rows
// of 64 bytes from 2^21 slots 13.6 -> 9.1 us, 4096 of 128 bytes from 2^24 16.2 -> 11.0, 256 of 268 bytes from 2^20
// 7.3 -> 6.7, each with one launch (3 us on the host) less.  (Both halves' times: kGatherInDrawBytes.)
// kWide: the top level has more than 512 nodes.  (With the branch in the kernel 256 samples from 2^20 slots and their
// update took 11.76 us, without 11.55.)
template <bool kWide>
__global__ __launch_bounds__(kSampleMaxThreads) void sample_kernel(SampleArgs a)
{
  __shared__ float red[kSampleMaxThreads / kWave];
  __shared__ uint32_t sh_ticket;
  const TreeView &tv = a.tv;
  const uint32_t lane = lane_id(), gl = lane & 15, b = blockIdx.y;
  const uint32_t nthr = blockDim.x;
  const uint32_t j0 = (blockIdx.x * (nthr / kWave) + threadIdx.x / kWave) * 4;
  const uint32_t k = a.k_dev ? (uint32_t)*a.k_dev : a.k;
  const uint32_t j = j0 + lane / 16;
  uint64_t my_mass = ~0ull;
  if (j0 < k) {
    const uint64_t o = (uint64_t)b * k + min(j, k - 1);  // a row without a sample repeats the last one and writes nothing
    const uint64_t *const top_level = a.top;
    fetch_now(top_level, tv.n_top, a.rnd, a.st);
    TopLevel<kWide> top;
    top.load(top_level, tv.n_top);
    const uint64_t u = a.rnd[o], head = a.st->head;
    const uint64_t total = top.scan();
    const uint64_t w = a.k_dev ? total / k : fast_div(total, a.k_div);  // stratum width
    const uint64_t point = (uint64_t)min(j, k - 1) * w + __umul64hi(u, w);  // inside stratum j
    uint64_t head_slot = 0;
    const RowWalk walk = walk_four(tv, top, top_level, point, [&] { head_slot = ring_slot(tv, head); });
    if (j < k) {
      const uint64_t slot = walk.idx;
      my_mass = walk.mass;
      uint32_t gen = 0;
      if (gl == 0) {
        __hip_atomic_store(a.mass + o, walk.mass, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a.slot_out[o] = (uint32_t)slot;
        if (a.claim) __hip_atomic_fetch_max(a.claim + slot, (uint32_t)o + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (a.gen) gen = a.gen[slot];
      }
      gather_by_16(a.g, slot, o, [&] { arrived(gen); });  // (this wave's masses are in memory from here on)
      if (gl == 0 && a.key_out)
        a.key_out[o] = a.gen ? ((uint64_t)gen << 32) | slot : ring_key(slot, head, head_slot, tv.P);
    }
  }
  if (!a.weight_out) return;

  const uint32_t wave = threadIdx.x / kWave, nwave = nthr / kWave;
  // The smallest of the waves' masses; as floats, which round alike.  Called by every thread.
  const auto smallest_of = [&](float mine) {
    const float of_wave = wave_min(mine);
    if (lane == 0) red[wave] = of_wave;
    lds_barrier();
    return wave_min(red[lane < nwave ? lane : 0]);
  };
  if (gridDim.x == 1) {  // the whole batch is here
    const float mass = (float)my_mass, smallest = smallest_of(mass);
    if (gl == 0 && j < k) a.weight_out[(uint64_t)b * k + j] = batch_weight(smallest, mass, a.beta);
    return;
  }
  __syncthreads();
  uint32_t *const ticket = a.ticket + (uint64_t)b * kTicketStride;
  if (threadIdx.x == 0) sh_ticket = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (blockIdx.x == 0 && b == 0) clear_ahead(a, threadIdx.x, nthr);
  if (sh_ticket != gridDim.x - 1) return;
  if (threadIdx.x == 0) *ticket = 0;
  const uint64_t *const bm = a.mass + (uint64_t)b * k;
  float *const bw = a.weight_out + (uint64_t)b * k;
  // every mass of the batch in a register of this workgroup: all loads on their way together
  uint64_t held[kHeldMasses];
#pragma unroll
  for (int t = 0; t < kHeldMasses; ++t)
    held[t] = __hip_atomic_load(bm + min(threadIdx.x + t * nthr, k - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  float m[kHeldMasses], mn = __builtin_inff();
#pragma unroll
  for (int t = 0; t < kHeldMasses; ++t) m[t] = (float)held[t], mn = fminf(mn, m[t]);
  const float smallest = smallest_of(mn);
#pragma unroll
  for (int t = 0; t < kHeldMasses; ++t) {
    const uint32_t i = threadIdx.x + t * nthr;
    if (i < k) bw[i] = batch_weight(smallest, m[t], a.beta);
  }
}

// replay.Sample in one launch with a workgroup per sample: its first wave draws the sample, the others wait for the slot
// and copy the row, the last of them the small columns.  For rows too long for 16 lanes, and for few samples, where it spreads
// the draws over more of the chip and the weights' chain runs beside the copies.
//
// The weights need the smallest mass of the batch.  Every workgroup puts its sample's mass, as the float that the weights
// are made of, on a board (a word per sample, 0 before the launch), waits until it is there, and reads the whole batch's
// words: the one that does so last, if not others before it, finds all of them and writes the weights.  (Word written
// through at agent scope, wait for it, words read at agent scope: the order that sequential consistency asks for.)  Several
// may find them all; they write the same weights, and clear the words.  That is two round trips (where keys hold the slot's
// generation three: its load is waited for with the word, the key's store behind it); a ticket to be the last
// workgroup by, in two steps because atomics on one address take turns of some 14 ns, was four: of the 4.3 us of 32 samples
// 1.2 were spent behind the draw, of the 5.8 of 256 2.0.  Weights by all waves of the workgroup, which are as many as the rows
// want, and at least a wave more than there are whole waves of samples, up to four: one took 0.6 us
// for 512 and 1.3 for 1024.  Launches of more than kBoardSamplesMax samples in batches of more than kBoardSmallK keep the
// tickets: words written through wait behind too many reads of the same board (3 x 500 rows of 2 KB 7.6 us by tickets, 8.9).
//
// Within a wave everything that does not depend on the slot is fetched before it, all loads of a pass are on their way
// before the first is waited for (as first written a lane's second piece waited for its first, and the small columns one by
// one for the row), and a wave has one streaming store in flight at a time (512 frame stacks 8.7 us with both at once, 8.5
// so).  Rows below kStreamingBytes are stored through the cache: streaming, the partial lines at their ends cost 268-byte
// rows 0.3 us.  The barrier in between does not wait for stores.
//
// us by tickets, one wave for the weights -> so (device time, replayed graphs):
//                     1 x 32       1 x 64       1 x 256      1 x 512      3 x 333      1 x 1000     2 x 200
//      32 B, 268 B   4.4 -> 3.9   4.9 -> 3.9   5.9 -> 4.5
//      1 KB, 4 KB                 5.2 -> 4.2 (128)           6.5 -> 5.3
//      5003 B                                                             7.8 -> 6.7
//      8 KB                                                                            9.4 -> 8.1
//      16 KB                                                 7.7 -> 6.6
//      28,224 B                                7.0 -> 6.2    9.5 -> 8.6
//      40,000 B                                                                                     10.0 -> 10.0
// A workgroup holds 30 KB of a row with two pieces per lane and 60 with four; what is longer takes passes that wait for one
// another, where two launches give every 32 KB a workgroup (65,536 bytes, 512 samples 18.0 us and 18.8 in two launches, 1024
// 32.1 and 29.9; 131,072 bytes, 16 samples 10.8 and 9.2).  Rows of up to 32 KB stay with two launches where the chip does not
// hold all their workgroups at once, unless the batches are small (28,688 bytes, 768 at once: 1024 samples 17.7 us apart and
// 19.2, 2 x 700 21.8 and 23.6, 12 x 100 20.1 and 18.7; 20,000 bytes, 1280 at once: 3 x 512 18.0 and 18.9).
constexpr uint32_t kTicketGroup = 32;
constexpr uint32_t kSampleRowsMaxK = 1024;
constexpr uint32_t kSampleRowsMax = 1536;   // samples of a call: beyond, long rows are bound by memory either way
constexpr uint32_t kBoardSamplesMax = 1024, kBoardSmallK = 128;
constexpr uint32_t kWeightWaves = 4;
constexpr uint64_t kStreamingBytes = 2048;
constexpr uint32_t kChipCus = 256, kChipWaves = 8192;  // compute units of the chip, waves that it holds at once
constexpr uint64_t kSampleRowsMaxBytes = 96 << 10, kSampleRowsMaxBytesOfMany = 52 << 10;  // longest rows: up to 512 samples, beyond
constexpr uint64_t kCopyRowBytes = 32 << 10;  // what a workgroup of copy_rows_long_kernel moves
static_assert(kSampleRowsMax + APEX_MAX_BATCHES_PER_CALL <= kBoardWordsMax);

// Whether all words of a batch of k samples are on the board, from word `first` on; the masses go to sh_mass, the smallest to
// *smallest.  By one wave.
__device__ __forceinline__ bool board_complete(const uint32_t *board, uint32_t first, uint32_t k, float *sh_mass, float *smallest)
{
  constexpr uint32_t kPairs = kSampleRowsMaxK / (2 * kWave);
  const uint32_t lane = lane_id();
  uint64_t m[kPairs];
#pragma unroll
  for (uint32_t t = 0; t < kPairs; ++t)
    if (t * 2 * kWave < k)
      m[t] = __hip_atomic_load(reinterpret_cast<const uint64_t *>(board + board_place(first + min(2 * (t * kWave + lane), (k - 1) & ~1u))),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  bool all = true;
  float mn = __builtin_inff();
#pragma unroll
  for (uint32_t t = 0; t < kPairs; ++t) {
    if (t * 2 * kWave >= k) break;
    const uint32_t i = min(2 * (t * kWave + lane), (k - 1) & ~1u);
    const uint32_t m0 = (uint32_t)m[t], m1 = i + 1 < k ? (uint32_t)(m[t] >> 32) : m0;
    all &= m0 != 0 && m1 != 0;
    mn = fminf(mn, fminf(__uint_as_float(m0), __uint_as_float(m1)));
    sh_mass[i] = __uint_as_float(m0), sh_mass[i + 1] = __uint_as_float(m1);
  }
  *smallest = wave_min(mn);
  return __ballot(!all) == 0;
}

// The same by tickets, a word per kTicketGroup samples and then the batch's own, from the masses as the draws left them.
__device__ __forceinline__ bool last_by_tickets(const SampleArgs &a, uint32_t b, uint32_t j, uint32_t k, float *sh_mass, float *smallest)
{
  const uint32_t lane = lane_id();
  auto last_of = [&](uint32_t line, uint32_t n) {
    uint32_t *const t = a.ticket + (uint64_t)line * kTicketStride;
    uint32_t taken = 0;
    if (lane == 0) taken = __hip_atomic_fetch_add(t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = read_lane_u32(taken, 0) == n - 1;
    if (last && lane == 0) *t = 0;
    return last;
  };
  const uint32_t groups = (k + kTicketGroup - 1) / kTicketGroup, g = j / kTicketGroup;
  if (groups > 1 && !last_of(gridDim.y + b * groups + g, min(kTicketGroup, k - g * kTicketGroup))) return false;
  if (!last_of(b, groups > 1 ? groups : k)) return false;
  const uint64_t *const bm = a.mass + (uint64_t)b * k;
  float mn = __builtin_inff();
#pragma unroll 1
  for (uint32_t i0 = 0; i0 < k; i0 += 8 * kWave) {  // eight loads in flight
    uint64_t m[8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
      m[t] = __hip_atomic_load(bm + min(i0 + t * kWave + lane, k - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float mass = (float)m[t];
      mn = fminf(mn, mass);
      sh_mass[min(i0 + t * kWave + lane, k - 1)] = mass;
    }
  }
  *smallest = wave_min(mn);
  return true;
}

template <int kUnroll, bool kWide, bool kStreaming>
__global__ __launch_bounds__(1024) void sample_rows_kernel(SampleArgs a, uint32_t vecs_per_row)
{
  __shared__ uint32_t sh_slot;
  __shared__ float sh_min;                         // smallest mass of the batch; 0: the weights are not written here
  __shared__ float sh_mass[kSampleRowsMaxK + 1];
  const TreeView &tv = a.tv;
  const uint32_t tid = threadIdx.x, lane = lane_id(), j = blockIdx.x, b = blockIdx.y, k = a.k;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / kWave));
  const uint64_t o = (uint64_t)b * k + j;
  float *const weight_out = a.weight_out;

  if (wave == 0) {
    __builtin_amdgcn_s_setprio(2);
    uint64_t *const mass_out = a.mass, *const key_out = a.key_out;
    uint32_t *const slot_out = a.slot_out, *const board = a.board;
    const uint32_t *const gen = a.gen;
    fetch_now(a.top, tv.n_top, a.rnd, a.st);
    fetch_now(a.k_div.mul, a.k_div.sh1, a.k_div.sh2, tv.nlev);
    fetch_now(tv.level[0], tv.level[1], tv.top_log2, tv.P);
    fetch_now(tv.p_div.mul, tv.p_div.sh1, tv.p_div.sh2, gen);
    fetch_now(mass_out, slot_out, key_out, board);
    fetch_now(weight_out);
    TopLevel<kWide> top;
    top.load(a.top, tv.n_top);
    const uint64_t u = a.rnd[o], head = a.st->head;
    const uint64_t w = fast_div(top.scan(), a.k_div);  // stratum width
    uint64_t head_slot = 0;
    const Drawn drawn = walk_down(tv, top.find((uint64_t)j * w + __umul64hi(u, w)), [&] { head_slot = ring_slot(tv, head); });
    if (lane == 0) sh_slot = (uint32_t)drawn.slot;
    lds_barrier();
    const uint32_t first = b * board_stride(k);
    if (lane == 0) {
      if (board) {  // (a mass is at least 1; one drawn from an empty tree counts as there, too)
        __hip_atomic_store(board + board_place(first + j), max(__float_as_uint((float)drawn.mass), 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        mass_out[o] = drawn.mass;
      } else {
        __hip_atomic_store(mass_out + o, drawn.mass, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      slot_out[o] = (uint32_t)drawn.slot;
      if (key_out) key_out[o] = gen ? ((uint64_t)gen[drawn.slot] << 32) | drawn.slot : ring_key(drawn.slot, head, head_slot, tv.P);
    }
    __builtin_amdgcn_s_setprio(0);
    if (weight_out) {
      wait_for_all_loads();  // this sample's mass is in memory from here on
      asm volatile("" ::: "memory");
      if (j == 0 && b == 0) clear_ahead(a, lane, kWave);
      float smallest = 0.f;
      const bool writes = board ? board_complete(board, first, k, sh_mass, &smallest) : last_by_tickets(a, b, j, k, sh_mass, &smallest);
      if (lane == 0) sh_min = writes ? smallest : 0.f;
      if (writes && board)
        for (uint32_t i = lane; i < k; i += kWave) board[board_place(first + i)] = 0;
    }
  } else {
    const uint8_t *const obs = a.g.obs, *const act = a.g.act;
    const float *const ret = a.g.ret, *const gacc = a.g.gacc;
    uint8_t *const obs_out = a.g.obs_out, *const act_out = a.g.act_out;
    float *const ret_out = a.g.ret_out, *const gacc_out = a.g.gacc_out;
    const uint64_t row_bytes = a.g.obs_bytes;
    const uint32_t act_bytes = a.g.act_bytes;
    fetch_now(obs, obs_out, row_bytes, vecs_per_row);
    fetch_now(act, act_out, act_bytes, ret);
    fetch_now(gacc, ret_out, gacc_out, weight_out);
    const uint32_t copiers = blockDim.x - kWave, c0 = tid - kWave, c_wave = (wave - 1) * kWave, v_last = vecs_per_row - 1;
    uint8_t *const d = obs_out + o * row_bytes;
    const bool columns = wave == blockDim.x / kWave - 1, words = act_bytes >= 4;
    const uint32_t act_last = act_bytes - (words ? 4 : 1), act_at = min(words ? 4 * lane : lane, act_last);
    lds_barrier();
    const uint32_t slot = read_lane_u32(sh_slot, 0);
    const uint8_t *const s = obs + slot * row_bytes;
    const auto store = [&](uint32_t v, PieceAny::Reg x) {
      if (kStreaming) store_piece_streaming<PieceAny>(d, v, row_bytes, x);
      else store_piece<PieceAny>(d, v, row_bytes, x);
    };
    // no load sits in a branch that the lanes of a wave take apart: indices are clamped
    PieceAny::Reg t[kUnroll];
    float col_r = 0.f, col_g = 0.f;
    uint32_t act_piece = 0;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      if (c_wave + u * copiers >= vecs_per_row) break;
      t[u] = load_piece_streaming<PieceAny>(s, min(u * copiers + c0, v_last), row_bytes);
    }
    if (columns) {
      col_r = ret[slot], col_g = gacc[slot];
      const uint8_t *const act_row = act + (uint64_t)slot * act_bytes + act_at;
      if (words) act_piece = *reinterpret_cast<const u32_any *>(act_row);
      else act_piece = *act_row;
    }
    wait_for_all_loads();
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t v = u * copiers + c0;
      if (u > 0) wait_for_all_loads();
      if (v < vecs_per_row) store(v, t[u]);
    }
    if (columns) {
      if (ret_out && lane == 0) ret_out[o] = col_r;
      if (gacc_out && lane == 0) gacc_out[o] = col_g;
      if (act_out) {
        uint8_t *const act_to = act_out + o * act_bytes;
        if (words) *reinterpret_cast<u32_any *>(act_to + act_at) = act_piece;
        else act_to[act_at] = (uint8_t)act_piece;
        for (uint32_t at = 4 * (kWave + lane); at < act_bytes; at += 4 * kWave) {  // the last piece overlaps the one before it
          const uint32_t p = min(at, act_last);
          *reinterpret_cast<u32_any *>(act_to + p) = *reinterpret_cast<const u32_any *>(act + (uint64_t)slot * act_bytes + p);
        }
      }
    }
    for (uint32_t v0 = copiers * kUnroll; v0 < vecs_per_row; v0 += copiers * kUnroll) {
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) t[u] = load_piece_streaming<PieceAny>(s, min(v0 + u * copiers + c0, v_last), row_bytes);
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const uint32_t v = v0 + u * copiers + c0;
        if (v < vecs_per_row) store(v, t[u]);
      }
    }
  }

  if (!weight_out) return;
  lds_barrier();
  const float smallest = sh_min;
  if (smallest == 0.f) return;
  float *const bw = weight_out + (uint64_t)b * k;
#pragma unroll 1
  for (uint32_t i = tid; i < k; i += blockDim.x) bw[i] = batch_weight(smallest, sh_mass[i], a.beta);
}

// --------------------------------------------------------------------------------------------
// One launch per learner step (Algorithm 2: replay.Sample, replay.SetPriority in strict order):
// the gather of batch i, its importance weights, and the draw of batch i+1 together with the
// write-back of batch i+1's new priorities (which are an argument of the call), so that the next
// launch finds a tree that is up to date.
//
// A draw may not read a tree that other workgroups of the same launch are writing, so the memory
// keeps two copies of the sum tree.  Launch i reads copy R, which holds every write-back up to
// batch i, and writes copy W, which holds those up to batch i-1: workgroup j adds the change of
// pair j of batch i (known from the launch before) and of pair j of batch i+1 (which it has just
// drawn) to W with atomics.  The next launch reads W and writes R: every change is applied twice,
// once to each copy, in consecutive launches.  The first batch of a sequence is drawn by a launch
// of the same kernel that has nothing to gather yet (slot == null, one wave per workgroup), which
// needs both copies equal when it starts.
//
// Within a batch the drawn slots do not decrease (the strata are ordered), so the pairs that
// share a slot are neighbours and the last of them is the one that counts: the wave that draws
// sample j also computes the point of sample j+1 and sees whether it still lies inside the slot's
// interval of cumulative mass.
// --------------------------------------------------------------------------------------------
__device__ __forceinline__ void add_delta(const TreeView &tv, uint32_t slot, uint64_t delta)
{
  if (!delta) return;
  atomic_add_u64(tv.level[0] + slot, delta);
  add_to_ancestors(tv, slot, delta);
}

// Workgroups of 8 waves, 4 vectors per lane: as fast as 16 waves x 2 when the kernel runs alone, and the
// chip then holds the whole batch in half of its wave slots, which leaves room for the workgroups of
// an add round's payload copy on the other stream (measured: 16.9 instead of 18.4 us per step there).
constexpr int kStepThreads = 512;
constexpr int kStepUnroll = 4;
constexpr uint32_t kStepMaxK = 1024;    // pairs per batch that the fused step handles (size of its scratch rows)

struct StepArgs {
  // gather of batch i: row j of dst = row slot[j] of src; the small columns likewise
  const uint8_t *src;
  uint8_t *dst;
  uint32_t vecs_per_row;  // pieces per row
  uint64_t row_bytes;
  const uint8_t *act;
  uint32_t act_bytes;
  const float *ret, *gacc;
  uint8_t *act_out;
  float *ret_out, *gacc_out;
  uint32_t k;             // <= kStepMaxK
  const uint32_t *slot;   // [k] batch i as it was drawn
  const uint64_t *dq;     // [k] its changes: new mass - mass as drawn; null: nothing is written back in this sequence
  TreeView wr;            // the copy that is written
  WeightArgs wa;          // weights of batch i
  DrawArgs next;          // draw of batch i+1 from next.tv, the copy that is read; next.rnd == null: none
  const uint64_t *next_top;  // the top level of next.tv (its address at a fixed place of the arguments)
  FastDiv next_k_div;        // division by next.k
  const float *next_prio; // [k] new priorities of batch i+1 (null: none) ...
  uint64_t *next_dq;      // ... the changes they bring, kept for the next launch
  QuantParams qp;
  DeviceState *st;
  // What the workgroups beyond the first k of the launch carry out (gridDim.x == k: nothing): a small
  // add round (add_round_small_block) or the masses of a round whose payload is in place
  // (add_leaves_block).  Only in a launch that draws nothing: what a round adds to the tree commutes
  // with the write-back of this batch, not with a draw.
  AddRoundArgs add;
  AddLeavesArgs leaves;
  // Rows stored through the block codec (kCodec launches only): row_bytes is then the stride of the
  // encoded rows in src, the rows written to dst are codec.raw_bytes long, and vecs_per_row counts their
  // 16-byte pieces.
  CodecShape codec;
};

enum StepRider { kNoRider = 0, kRoundRides = 1, kLeavesRide = 2 };

// The draw of sample `row` of the next batch by the first wave of a workgroup, with no barrier and no LDS: the
// top level in registers, the walk down, outputs, and the change that the sample's new priority brings.
// The wave's path through memory is the launch's critical path, so it holds exactly one round trip per
// tree level and as little else as can be:
//  - the top-level loads are the first instructions to go out, the sample's random number, new priority
//    and the ring's head follow them and are used after them (a wave's loads return in the order of issue);
//  - the stratum width is an exact division by multiplication (StepArgs::next_k_div);
//  - what does not depend on the walk (priority -> mass, head % P, the addresses of everything written at
//    the end) is computed or fetched while the first row of children is on its way.
__device__ __forceinline__ void draw_in_first_wave(const StepArgs &a, uint32_t row)
{
  const TreeView &rd = a.next.tv;
  const uint32_t lane = lane_id();
  const bool second = a.next_prio && row + 1 < a.next.k;              // a next sample to compare slots with
  __builtin_amdgcn_s_setprio(2);
  TopLevel<true> top;
  top.load(a.next_top, rd.n_top);
  // no load below is conditional: a branch around a load would make the wave wait for it there
  const uint64_t un0 = a.next.rnd[row], un1 = a.next.rnd[second ? row + 1 : row];
  const float prio_next = *(a.next_prio ? a.next_prio + row : reinterpret_cast<const float *>(a.next.rnd + row));
  const uint64_t head = a.next.st->head;

  // Within a batch the points do not decrease, so the pairs that share a slot are neighbours and the last of
  // them is the one that counts: pair `row` loses to pair row + 1 exactly if the next point still lies in the
  // interval of cumulative mass of the slot drawn here, which needs no second walk: both points are known
  // from the start, and the walk ends with the place of its point inside the slot's interval.
  const uint64_t total = top.scan();
  const uint64_t w = fast_div(total, a.next_k_div);
  const uint64_t point = (uint64_t)row * w + __umul64hi(un0, w), next_point = (uint64_t)(row + 1) * w + __umul64hi(un1, w);
  const TopHit hit = top.find(point);

  bool clamped = false;
  uint64_t q_next = 0, head_slot = 0;
  uint32_t *const slot_out = a.next.slot_out;
  uint64_t *const key_out = a.next.key_out, *const mass_out = a.next.mass, *const dq_out = a.next_dq;
  uint64_t *const wr0 = a.wr.level[0], *const wr1 = a.wr.level[1], *const wr2 = a.wr.level[2];
  // (the two copies of the tree have one shape, which the walk has fetched)
  auto add_to_written_copy = [&](uint64_t slot, uint64_t delta) {  // one lane
    if (!delta) return;
    atomic_add_u64(wr0 + slot, delta);
    uint64_t idx = slot;
    if (rd.nlev > 1) atomic_add_u64(wr1 + (idx >>= fanout_log2(rd, 1)), delta);
    if (rd.nlev > 2) atomic_add_u64(wr2 + (idx >>= fanout_log2(rd, 2)), delta);
    for (uint32_t l = 3; l < rd.nlev; ++l) {
      idx >>= fanout_log2(rd, l);
      atomic_add_u64(a.wr.level[l] + idx, delta);
    }
  };
  auto between = [&] {
    fetch_now(slot_out), fetch_now(key_out), fetch_now(mass_out), fetch_now(dq_out);
    fetch_now(wr0), fetch_now(wr1), fetch_now(wr2);
    if (a.next_prio) q_next = quantise_priority(prio_next, a.qp, &clamped);
    head_slot = ring_slot(rd, head);
  };
  const Drawn drawn = walk_down(rd, hit, between);
  const bool next_has_same_slot = second && next_point - point < drawn.mass - drawn.x;
  // Outputs first, atomics last: nothing that the compiler makes wait for an atomic's completion follows them.
  // (The small payload columns of the drawn batch are gathered by the launch that copies its rows.)
  if (lane == 0) {
    const uint64_t slot = drawn.slot;
    slot_out[row] = (uint32_t)slot;
    if (key_out) key_out[row] = ring_key(slot, head, head_slot, rd.P);
    mass_out[row] = drawn.mass;
    if (a.next_prio) {
      // the change this pair brings: none if the next pair has the same slot (the later one counts)
      const uint64_t delta = next_has_same_slot ? 0 : q_next - drawn.mass;
      dq_out[row] = delta;
      add_to_written_copy(slot, delta);
      if (clamped) atomic_add_u64(&a.st->n_clamped, 1);
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

// No barrier anywhere in the first k workgroups (one per row of the batch): their waves run independently.
//   wave 0       draws sample `row` of the next batch and writes its change into the written copy;
//                copies too only when the other waves cannot hold the whole row (its dependent
//                loads would queue behind the row loads)
//   wave 1       lane 0 carries the change of pair `row` of this batch into the written copy;
//                lanes 1, 2 gather ret and gacc of the row
//   wave 2       gathers the action bytes of the row
//   wave 3       in the first ceil(k / 64) workgroups: importance weights of 64 samples
// kRider: what the workgroups beyond the first k carry (StepArgs::add or ::leaves).
// kCodec: the rows are decoded on their way out (StepArgs::codec; the pieces are Piece16).
template <typename P, int kThreads, int kUnroll, int kRider, bool kCodec = false>
__global__ __launch_bounds__(kThreads) void learner_step_kernel(StepArgs a)
{
  const uint32_t row = blockIdx.x, tid = threadIdx.x, nthr = blockDim.x;
  if constexpr (kRider == kRoundRides) {
    if (row >= a.k) {
      __shared__ uint64_t sh_slot[kThreads], sh_q[kThreads];
      add_round_small_block<P>(a.add, row - a.k, gridDim.x - a.k, sh_slot, sh_q);
      return;
    }
  }
  if constexpr (kRider == kLeavesRide) {
    if (row >= a.k) {
      __shared__ DenseSums sh;
      add_leaves_block(a.leaves, row - a.k, gridDim.x - a.k, sh);
      return;
    }
  }
  const uint32_t wave = tid / kWave, lane = lane_id();
  const bool write_back = a.dq != nullptr, draw = a.next.rnd != nullptr;
  if (!a.slot) {  // the first draw of a sequence (one wave per workgroup): no batch to gather yet
    if (draw && wave == 0) draw_in_first_wave(a, row);
    return;
  }
  const uint32_t first = (draw && a.vecs_per_row <= (nthr - kWave) * kUnroll) ? kWave : 0;
  if (draw && wave == 0) {
    draw_in_first_wave(a, row);
    if (first) return;
  }
  // The compiler places its waits for memory by counting loads in flight; it can count them only along
  // straight-line code, and where a load sits in a branch, or loads and stores are in flight together, it
  // waits for everything.  As first written this part had the row loads wait for every small load, the
  // weights' eight loads wait for one another, and each of the row's stores wait for the one before it to
  // be acknowledged (read in the kernel's own ISA; the waves with a side job ended 1 - 2 us after the
  // others, and the launch with them).  So: the slot is waited for at once (everything depends on it),
  // no load below sits in a divergent branch (indices are clamped, unused lanes read an address of their
  // own workgroup that is always valid), the row is waited for once, and the side jobs' stores and
  // atomics follow the row's.
  const uint32_t my_slot = a.slot[row];
  wait_for_all_loads();

  // ---- small loads, ahead of the row so that they return ahead of it
  // the change that pair `row` brings (0 if a later pair of the batch has the same slot), carried into the
  // written copy by one lane: behind the row's stores in a launch that draws (its end is set by the drawing
  // wave's own atomics, and ahead of the stores this wave's part of the row would wait for them); as soon as
  // it has arrived in a launch that draws nothing (these atomics are then the last thing to finish)
  const bool carrier = write_back && tid == kWave;
  uint64_t pc_dq = 0;
  if (write_back) pc_dq = a.dq[row];  // by every lane: the same for all, and no address that the whole grid shares
  const bool ret_lane = tid == kWave + 1 && a.ret_out, gacc_lane = tid == kWave + 2 && a.gacc_out;
  const float small = *(ret_lane    ? a.ret + my_slot
                        : gacc_lane ? a.gacc + my_slot
                                    : reinterpret_cast<const float *>(a.slot + row));
  const bool weigher = wave == 3 && a.wa.weight_out && row * kWave < a.k;
  uint8_t act_byte[4] = {0, 0, 0, 0};
  const bool act_early = wave == 2 && a.act_out && a.act_bytes <= 4 * kWave;
  if (act_early) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      act_byte[t] = a.act[(uint64_t)my_slot * a.act_bytes + min(t * kWave + lane, a.act_bytes - 1)];
  }

  if (!draw) {  // the same for the whole launch: in a launch that draws, nothing here waits for the change
    if (carrier) add_delta(a.wr, my_slot, pc_dq);
  }

  // ---- the row
  const uint32_t copiers = nthr - first;
  const uint64_t out_bytes = kCodec ? (uint64_t)a.codec.raw_bytes : a.row_bytes;
  const uint8_t *s = a.src + (uint64_t)my_slot * a.row_bytes;
  uint8_t *d = a.dst + (uint64_t)row * out_bytes;
  const uint32_t v_last = a.vecs_per_row - 1;
  // piece of this wave's first lane: a wave loads nothing where the row has no pieces for it.  (Clamped loads keep the
  // memory pipelines of the compute unit as busy as others do: a learner step of 512 rows of 60 bytes 6.0 us, now 5.6; of
  // 1028 bytes 6.1 and 5.7.  Decoded rows are long, and the branch cost their launch 0.2 us.)
  const uint32_t v_wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid - first));
  typename P::Reg tmp[kUnroll];
  CodecFetched fetched[kCodec ? kUnroll : 1] = {};
  // Decoded rows: the first half of a wave's pieces is asked for at once, as the pieces of a plain row are, the other half
  // when the mask has arrived and only where it says that the image counts (other lanes read the row's first bytes, a line
  // that has just been fetched).  All of them at once reads every image whole, all of them behind the mask costs rows
  // without flat blocks a round trip.  Us per launch at 28,224 raw bytes, 512 rows with 0 / 80 % flat blocks: all at once
  // 8.87 / 8.82, half 8.56 / 8.02, none 9.05 / 7.67; 1024 rows: 15.96 / 15.90, 15.91 / 14.43, 17.05 / 14.35; 128 rows of
  // either kind 6.6, half 5.9; 1024 rows of 1 KB 7.07, half 6.83.
  constexpr int kCodecEarly = 2;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    if (!kCodec && v_wave + u * copiers >= a.vecs_per_row) break;
    const uint32_t v = min(tid - first + u * copiers, v_last);
    if constexpr (kCodec) {  // the pieces as the image holds them
      if (u < kCodecEarly) fetched[u].data = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(s + a.codec.image_off) + v);
    } else {
      tmp[u] = load_piece_streaming<P>(s, v, a.row_bytes);
    }
  }
  if constexpr (kCodec) {
    static_assert(kUnroll == 4, "a wave holds four runs of pieces");
    if (v_wave < a.vecs_per_row) {  // the same for all lanes of the wave
      uint32_t v_first[4];          // the wave's 64 pieces start there
      uint64_t word[4];
      u32x4 bytes[4];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) v_first[u] = min(v_wave + u * copiers, v_last & ~(kWave - 1));
      codec_fetch_wave_scalars(s, a.codec, v_first, word, bytes);
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        fetched[u].word = word[u];
        fetched[u].byte = codec_wave_byte(bytes[u], lane);
        fetched[u].bit = ((v_first[u] + lane) / 4) & 63;
        if (u < kCodecEarly) continue;
        if (v_wave + u * copiers >= a.vecs_per_row) break;
        const uint32_t v = min(tid - first + u * copiers, v_last);
        const bool kept = fetched[u].word >> fetched[u].bit & 1;
        fetched[u].data = __builtin_nontemporal_load(
            reinterpret_cast<const u32x4 *>(s + (kept ? a.codec.image_off + 16 * v : 0u)));
      }
    }
  }
  // the weights' loads go out behind the row's (ahead of them, the wave's part of the row would leave a
  // round trip or two late): smallest mass of the batch, eight loads per lane in flight
  uint64_t mass_min = ~0ull, mass_mine = 1;
  if (weigher) {
    mass_mine = a.wa.mass[min(row * kWave + lane, a.k - 1)];
    for (uint32_t j0 = 0; j0 < a.k; j0 += 8 * kWave) {
      uint64_t wm[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) wm[t] = a.wa.mass[min(j0 + t * kWave + lane, a.k - 1)];
#pragma unroll
      for (int t = 0; t < 8; ++t) mass_min = wm[t] < mass_min ? wm[t] : mass_min;
    }
  }

  wait_for_all_loads();
  if constexpr (kCodec) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      tmp[u] = codec_piece(fetched[u]);
    }
  }
  // One store at a time per wave (a wave waits for its last store before it issues the next): with a wave's
  // four stores in flight together the launch took 0.3 - 0.8 us longer, and with every piece stored as soon
  // as it had arrived (the row's writes beside the rest of its reads) 0.2 - 0.5 us longer (each measured
  // against this on one box).  Ordinary stores, streaming loads: streaming stores, which such a wave waits
  // for longer, cost 0.4 us per launch; ordinary loads of the rows cost 1.5.  Decoded rows, which read less, go out two
  // stores at a time.
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t v = tid - first + u * copiers;
    if (u > 0 && (!kCodec || u == 2) && v - lane < a.vecs_per_row) wait_for_all_loads();  // the same for all lanes of the wave
    if (v < a.vecs_per_row) store_piece<P>(d, v, out_bytes, tmp[u]);
  }

  // ---- what the side jobs write
  if (carrier && draw) add_delta(a.wr, my_slot, pc_dq);
  if (ret_lane) a.ret_out[row] = small;
  if (gacc_lane) a.gacc_out[row] = small;
  if (act_early) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t by = t * kWave + lane;
      if (by < a.act_bytes) a.act_out[(uint64_t)row * a.act_bytes + by] = act_byte[t];
    }
  }
  if (weigher) {
    const float weight = batch_weight(wave_min((float)mass_min), (float)mass_mine, a.wa.beta);
    if (row * kWave + lane < a.k) a.wa.weight_out[row * kWave + lane] = weight;
  }

  // rows longer than one pass of the workgroup (more than 32 KB, or narrow vectors)
  for (uint32_t base = copiers * kUnroll; base < a.vecs_per_row; base += copiers * kUnroll) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t v = min(base + tid - first + u * copiers, v_last);
      if constexpr (kCodec) {
        tmp[u] = codec_piece(codec_fetch_all(s, a.codec, v));
      } else {
        tmp[u] = load_piece_streaming<P>(s, v, a.row_bytes);
      }
    }
    wait_for_all_loads();
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t v = base + tid - first + u * copiers;
      if (v < a.vecs_per_row) store_piece_streaming<P>(d, v, out_bytes, tmp[u]);
    }
  }
  if (wave == 2 && a.act_out && !act_early)  // long action rows: after the row, which they would hold up
    for (uint32_t by = lane; by < a.act_bytes; by += kWave)
      a.act_out[(uint64_t)row * a.act_bytes + by] = a.act[(uint64_t)my_slot * a.act_bytes + by];
}

// --------------------------------------------------------------------------------------------
// The same for steps of several batches, or of one large one, of short rows (four samples per wave): launch i gathers the
// batches of step i, writes their weights, draws those of step i+1 from the copy of the tree that holds every write-back up
// to step i, and adds the changes of both steps to the other copy.  All batches of a step are drawn from the same state.
//
// Of all pairs of a step that share a slot the last one counts.  The wave that draws a sample can tell from the uniforms
// alone: a batch has a point in the slot's interval of cumulative mass only if it has one in a stratum that the interval
// meets, and it has one for certain where the interval covers a stratum.  So a later batch has drawn the slot exactly if
// its point in the sample's own stratum, or in the one below or above it, lies in the interval (were the interval to reach
// further, it would cover the neighbour): three points per later batch, one batch per lane of the sample's row.  In the
// sample's own batch it is the point above.
// As two launches per step (sample_kernel with the first pass of the update, update_apply_kernel) and so, us per step of
// rows of 32 bytes, calls of eight steps:
//                 16 x 512       8 x 512       2 x 512       1 x 4096      1 x 16,384     64 x 64       128 x 64
//   2^14 slots   12.4 ->  8.0   11.1 -> 6.6   10.7 -> 5.8   13.7 -> 6.2   20.7 -> 15.7   11.7 -> 8.0   14.2 -> 11.7
//   2^19         13.3 -> 11.0   11.9 -> 8.0   12.1 -> 7.0   14.5 -> 7.7   (two launches) 12.8 -> 8.6   15.4 -> 12.9
//   2^21         13.6 ->  7.7   12.1 -> 6.7   11.4 -> 6.2   15.0 -> 7.7   20.7 -> 14.3   12.9 -> 8.5   15.7 -> 13.0
//   2^23         15.2 ->  9.4   13.6 -> 8.1   12.0 -> 7.3   16.5 -> 8.9   23.0 -> 15.5   14.7 -> 10.0  17.4 -> 14.5
// --------------------------------------------------------------------------------------------
struct MultiStepArgs {
  // workgroups: first those that draw, per batch of step i+1; those from gather_first and weight_first on gather step i and
  // write its weights, weight_wgs_per_batch to a batch
  uint32_t draw_wgs, draw_wgs_per_batch, gather_first, weight_first, weight_wgs, weight_wgs_per_batch;
  GatherArgs g;           // step i: row o of the outputs = row slot[o]
  uint32_t samples;       // of a step
  const uint32_t *slot;
  const uint64_t *dq;     // its changes: new mass - mass as drawn
  WeightArgs wa;
  TreeView wr;            // the copy that is written
  DrawArgs next;          // step i+1, from the copy that is read
  FastDiv next_k_div;
  uint32_t batches;
  const float *next_prio; // its new priorities ...
  uint64_t *next_dq;      // ... and the changes they bring
  QuantParams qp;
  DeviceState *st;
};

// Adds four changes, one per 16-lane row of the wave (every lane of a row holds its row's), to a copy of the tree.  kMerge:
// above the leaves neighbouring rows under one node send one atomic.  The four are uniform values then, no lane has to ask
// another one.  Atomics on one cache line take turns of some 11 ns, so this is worth its 0.2 us only where many meet: see
// kMergePerTopNode.
template <bool kMerge>
__device__ __forceinline__ void add_four(const TreeView &tv, uint32_t slot, uint64_t delta)
{
  const uint32_t lane = lane_id(), row = lane / 16;
  const bool first = (lane & 15) == 0;
  if constexpr (!kMerge) {
    if (first) add_delta(tv, slot, delta);
    return;
  }
  uint32_t node[4];
  uint64_t d[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) node[r] = read_lane_u32(slot, 16 * r), d[r] = read_lane_u64(delta, 16 * r);
  if (first && delta) atomic_add_u64(tv.level[0] + slot, delta);
  for (uint32_t l = 1; l < tv.nlev; ++l) {
    const uint32_t shift = fanout_log2(tv, l);
#pragma unroll
    for (int r = 0; r < 4; ++r) node[r] >>= shift;
    const uint64_t s3 = d[3], s2 = d[2] + (node[2] == node[3] ? s3 : 0), s1 = d[1] + (node[1] == node[2] ? s2 : 0),
                   s0 = d[0] + (node[0] == node[1] ? s1 : 0);
    const uint32_t at = row == 0 ? node[0] : row == 1 ? node[1] : row == 2 ? node[2] : node[3];
    const uint64_t sum = row == 0 ? s0
                         : row == 1 ? (node[1] != node[0] ? s1 : 0)
                         : row == 2 ? (node[2] != node[1] ? s2 : 0)
                                    : (node[3] != node[2] ? s3 : 0);
    if (first && sum) atomic_add_u64(tv.level[l] + at, sum);
  }
}

constexpr int kMultiStepThreads = 256;
constexpr uint32_t kMultiStepRows = kMultiStepThreads / 16;  // samples per workgroup

template <bool kWide, bool kMerge>
__global__ __launch_bounds__(kMultiStepThreads) void multi_step_kernel(MultiStepArgs a)
{
  __shared__ float red[kMultiStepThreads / kWave];
  const uint32_t lane = lane_id(), gl = lane & 15, blk = blockIdx.x;
  if (blk >= a.weight_first && blk - a.weight_first < a.weight_wgs) {
    const uint32_t b = (blk - a.weight_first) / a.weight_wgs_per_batch, part = blk - a.weight_first - b * a.weight_wgs_per_batch;
    batch_weights(a.wa, b, red, part, a.weight_wgs_per_batch);
    return;
  }
  if (blk >= a.gather_first) {
    const uint32_t o = (blk - a.gather_first) * kMultiStepRows + threadIdx.x / 16, at = min(o, a.samples - 1);
    const uint32_t slot = a.slot[at];
    const uint64_t dq = a.dq[at];
    add_four<kMerge>(a.wr, slot, o < a.samples ? dq : 0);
    if (o < a.samples) gather_by_16(a.g, slot, o, [] {});
    return;
  }
  const TreeView &rd = a.next.tv;
  const uint32_t k = a.next.k, b = blk / a.draw_wgs_per_batch;
  const uint32_t j0 = (blk - b * a.draw_wgs_per_batch) * kMultiStepRows + threadIdx.x / kWave * 4;
  if (j0 >= k) return;
  const bool in = j0 + lane / 16 < k;
  const uint32_t j = min(j0 + lane / 16, k - 1);  // a row without a sample repeats the last one and writes nothing
  const uint32_t o = b * k + j;
  TopLevel<kWide> top;
  const uint64_t *const top_level = rd.level[rd.nlev - 1];
  top.load(top_level, rd.n_top);
  const uint64_t u = a.next.rnd[o];
  const uint32_t below = max(j, 1u) - 1, above = min(j + 1, k - 1);
  const uint64_t *const mine = a.next.rnd + (uint64_t)min(b + gl, a.batches - 1) * k;  // batch b + gl is this lane's
  uint64_t u_below = mine[below], u_same = mine[j], u_above = mine[above];
  const float prio = a.next_prio[o];
  const uint64_t head = a.next.st->head;
  const uint64_t w = fast_div(top.scan(), a.next_k_div);  // stratum width
  const uint64_t base = (uint64_t)j * w, point = base + __umul64hi(u, w);
  uint64_t head_slot = 0, q = 0;
  bool clamped = false;
  const RowWalk walk = walk_four(rd, top, top_level, point, [&] {
    head_slot = ring_slot(rd, head);
    q = quantise_priority(prio, a.qp, &clamped);
  });
  const uint64_t lo = point - walk.x, hi = lo + walk.mass;
  bool later = false;
  for (uint32_t c0 = b;;) {
    const uint32_t c = c0 + gl;
    if (c < a.batches) {
      later |= j + 1 < k && base + w + __umul64hi(u_above, w) < hi;
      if (c != b) {
        const uint64_t p = base + __umul64hi(u_same, w);
        later |= (p >= lo && p < hi) || (j > 0 && base - w + __umul64hi(u_below, w) >= lo);
      }
    }
    c0 += 16;
    if (c0 >= a.batches) break;
    const uint64_t *const r = a.next.rnd + (uint64_t)min(c0 + gl, a.batches - 1) * k;
    u_below = r[below], u_same = r[j], u_above = r[above];
  }
  const bool loses = (uint32_t)(__ballot(later) >> (lane & 48)) & 0xffffu;
  const uint64_t delta = loses ? 0 : q - walk.mass;
  if (in && gl == 0) {
    a.next.slot_out[o] = (uint32_t)walk.idx;
    if (a.next.key_out) a.next.key_out[o] = ring_key(walk.idx, head, head_slot, rd.P);
    a.next.mass[o] = walk.mass;
    a.next_dq[o] = delta;
  }
  add_four<kMerge>(a.wr, (uint32_t)walk.idx, in ? delta : 0);
  const uint64_t nc = __popcll(__ballot(in && gl == 0 && clamped));
  if (nc && lane == 0) atomic_add_u64(&a.st->n_clamped, nc);
}

// dst[i] = src[i]: brings the second copy of the tree up to date
__global__ __launch_bounds__(256) void copy_words_kernel(uint64_t *__restrict__ dst, const uint64_t *__restrict__ src,
                                                         uint64_t n)
{
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

// zero fill (hipMemset is avoided so that the library's launches stay replayable)
__global__ __launch_bounds__(256) void fill_zero_kernel(uint64_t *p, uint64_t n)
{
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

}  // namespace apex
