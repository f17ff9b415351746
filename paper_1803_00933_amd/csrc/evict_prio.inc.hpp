// apex_pe_*: a replay memory whose eviction is proportional prioritized sampling with its own
// exponent (Appendix "Continuous Control: Additional Details": alpha_evict = -0.4) instead of oldest
// first.  Included by apex_replay.hip (one translation unit).
//
// Two sum trees of the same shape over the same slots: sampling masses Q(p; alpha) and eviction
// masses Q(p; alpha_evict).  Slots freed by evictions go into a ring of free slots and are re-used
// by later adds in the order in which they were freed; a key is (generation of the slot << 32) |
// slot.  Evicting e transitions without replacement takes rounds: draw as many stratified points
// as are still to go on the eviction tree (the sampling kernel, pointed at that tree), drop
// repeats (they are neighbours, the points being ordered), remove the rest in the order of their
// points (the count of those before each gives its place in the free ring), repeat.

namespace apex {

struct PeState {
  DeviceState base;  // head = evicted so far, tail = inserted so far, and the two counters
  uint64_t free_head, free_tail;   // the free ring holds slots free_ring[free_head .. free_tail) mod P
  uint64_t remaining;              // evictions still to go in the current call
  uint64_t round_done;             // workgroups of the running removal that are done, and what they removed
  // Workgroups of the running pe_add_rows_kernel that have the counters.  On a line of its own: every wave of such a launch reads
  // the counters, and every ticket takes their line out of the caches.
  alignas(128) uint32_t ticket_rows;
};

struct PeView {
  TreeView ts, te;  // sampling masses, eviction masses
  uint32_t *gen;
  uint32_t *free_ring;
  QuantParams qs, qe;
};

__device__ __forceinline__ bool pe_key_valid(const PeView &v, uint64_t key, uint32_t *slot_out)
{
  const uint64_t slot = key & 0xffffffffu;
  if (slot >= v.ts.P) return false;
  *slot_out = (uint32_t)slot;
  return v.gen[slot] == (uint32_t)(key >> 32) && v.ts.level[0][slot] != 0;
}

// add_runs_to_ancestors for both trees: the runs lie alike, so they are found once.
__device__ __forceinline__ void pe_add_runs(const PeView &v, bool active, uint32_t slot, uint64_t d1, uint64_t d2)
{
  const uint64_t incl1 = wave_inclusive_scan(active ? d1 : 0), incl2 = wave_inclusive_scan(active ? d2 : 0);
  uint32_t idx = slot;
  for_levels<1>(v.ts, [&](uint32_t l) {
    idx >>= fanout_log2(v.ts, l);
    const LaneRuns run = lane_runs(active ? idx : ~0u);
    const int lane_before = run.first > 0 ? run.first - 1 : 0;
    const uint64_t before1 = __shfl(incl1, lane_before, kWave), before2 = __shfl(incl2, lane_before, kWave);
    if (active && run.ends) {
      atomic_add_u64(v.ts.level[l] + idx, incl1 - (run.first > 0 ? before1 : 0));
      atomic_add_u64(v.te.level[l] + idx, incl2 - (run.first > 0 ? before2 : 0));
    }
  });
}

// Counts the masses that had to be clamped, c1 and c2 one of a lane's each.  By the whole wave.
__device__ __forceinline__ void pe_count_clamped(PeState *st, bool c1, bool c2)
{
  const uint64_t nc = __popcll(__ballot(c1)) + __popcll(__ballot(c2));
  if (nc && lane_id() == 0) atomic_add_u64(&st->base.n_clamped, nc);
}

__global__ __launch_bounds__(256) void pe_add_kernel(PeView v, PeState *__restrict__ st, uint64_t count,
                                                     const float *__restrict__ prio)
{
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t slot = 0;
  uint64_t q1 = 0, q2 = 0;
  bool c1 = false, c2 = false;
  if (i < count) {
    slot = v.free_ring[ring_slot(v.ts, st->free_head + i)];
    v.gen[slot] += 1;
    const float p = prio[i];
    q1 = quantise_priority(p, v.qs, &c1), q2 = quantise_priority(p, v.qe, &c2);
    v.ts.level[0][slot] = q1;  // a free slot weighs nothing in either tree
    v.te.level[0][slot] = q2;
  }
  pe_add_runs(v, i < count, slot, q1, q2);
  pe_count_clamped(st, c1, c2);
  // the last workgroup to finish moves the free ring's head and the insertion count on
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t t = __hip_atomic_fetch_add(&st->base.ticket_add, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t == gridDim.x - 1) {
      st->base.ticket_add = 0;
      st->free_head += count;
      st->base.tail += count;
    }
  }
}

// The same with the payload of short observation rows in the same launch, in workgroups of kPeAddThreads lanes:
// 2^lanes_log2 lanes per transition copy its observation and action bytes into the next free slot; the first waves, a lane per
// transition, find its priority as well - given (prio), or the n-step priority of an actor round (ns.S != 0: Algorithm 1,
// ComputePriorities; the partial return and accumulated discount are then the computed ones) - and enter the masses, whole
// waves of neighbouring transitions together (add_runs_to_ancestors).  act, ret, gacc may be null.
// Bound by its chain: arguments, the free ring's head, the free slot, generation and atomics.  Rows, action bytes and n-step
// inputs do not depend on the slot and are fetched beside it; a lane that enters a mass looks its slot up by itself, so nothing
// goes through LDS.  Rounds of 3200 rows of 256 bytes, five steps: 5.4 us in the trace when rows came first, 4.8 so.
// The workgroups are as large as they can be, for the sake of the atomics on the top levels: rounds of 3200 rows of 256
// bytes 4.7 us with 1024 threads, 5.1 with 512 and 6.4 with 256, of 7700 rows of 1000 bytes 11.7, 18.3 and 34.1.  (64
// transitions per workgroup whatever the rows, in several passes, when rows came first: 6.2 and 18, where these were 5.5 and 13.)
// Rounds of more workgroups than the chip holds go by what a workgroup costs.  Two are resident per compute unit (64 registers);
// the ticket is away from the counters' line, which 16 waves a workgroup read; n-step inputs, two trips one behind the other,
// are ahead of the row, and the first waves read those of their workgroup's transitions only.  Rounds of 15,000 rows of 1000
// bytes 26.2 us with 66 registers, the ticket beside the counters and rows ahead, 17.8 so (19.8 when rows came first), of
// 18,000 of 4096 bytes 163, 62 and 66, of 7700 of 1000 13.4, 11.8 and 12.6.
constexpr uint32_t kPeAddThreads = 1024;

template <typename P>
__global__ __launch_bounds__(kPeAddThreads, 8) void pe_add_rows_kernel(PeView v, PeState *__restrict__ st, uint64_t count,
                                                                       NstepArgs ns, const float *__restrict__ prio,
                                                                       const uint8_t *__restrict__ obs,
                                                                       const uint8_t *__restrict__ act,
                                                                       const float *__restrict__ ret,
                                                                       const float *__restrict__ gacc,
                                                                       uint8_t *__restrict__ obs_ring,
                                                                       uint8_t *__restrict__ act_ring,
                                                                       float *__restrict__ ret_ring,
                                                                       float *__restrict__ gacc_ring, uint32_t vecs_per_row,
                                                                       uint32_t lanes_log2, uint64_t obs_bytes,
                                                                       uint32_t act_bytes)
{
  const uint32_t rows_per_block = blockDim.x >> lanes_log2, lanes = 1u << lanes_log2;
  fetch_now(st, v.free_ring, v.ts.P, v.ts.p_div.mul);
  fetch_now(v.ts.p_div.sh1, v.ts.p_div.sh2, obs, act);
  fetch_now(obs_bytes, act_bytes, vecs_per_row, count);
  fetch_now(ns.q_online, ns.q_target, ns.action, ns.reward);
  fetch_now(ns.discount, ns.t_div.mul, ns.t_div.sh1, ns.t_div.sh2);
  fetch_now(ns.S, ns.T, ns.n, ns.A);
  const uint64_t free_head = st->free_head, tail = st->base.tail, last = count - 1;
  // what this thread copies: piece vv of transition i, and its action bytes from the one numbered vv on, four at a time
  const uint64_t i = (uint64_t)blockIdx.x * rows_per_block + (threadIdx.x >> lanes_log2), i_at = min(i, last);
  const uint32_t vv = threadIdx.x & (lanes - 1);
  const uint32_t unit = act_bytes >= 4 ? 4 : 1, act_last = act_bytes - unit;
  // the transition whose masses it enters, if it is one of the first rows_per_block
  const uint64_t e = (uint64_t)blockIdx.x * rows_per_block + min(threadIdx.x, rows_per_block - 1), e_at = min(e, last);
  const bool mass_wave = threadIdx.x < ((rows_per_block + kWave - 1) & ~(uint32_t)(kWave - 1));  // the same for a whole wave
  const bool active = threadIdx.x < rows_per_block && e < count;
  const uint32_t slot = v.free_ring[ring_slot(v.ts, free_head + i_at)];
  uint32_t slot_e = 0, act_piece = 0;
  if (mass_wave) slot_e = v.free_ring[ring_slot(v.ts, free_head + e_at)];
  float p = 0.f, r_in = 0.f, g_in = 0.f;
  if (mass_wave && ns.S) {
    const NstepOut o = nstep_one(ns, e_at);
    r_in = o.R, g_in = o.G, p = o.p;
  }
  const typename P::Reg piece = load_piece<P>(obs + i_at * obs_bytes, min(vv, vecs_per_row - 1), obs_bytes);
  if (act) {
    const uint8_t *const from = act + i_at * act_bytes + min(unit * vv, act_last);
    if (unit == 4) act_piece = *reinterpret_cast<const u32_any *>(from);
    else act_piece = *from;
  }
  if (mass_wave && !ns.S) {
    p = prio[e_at];
    if (ret) r_in = ret[e_at];
    if (gacc) g_in = gacc[e_at];
  }
  if (i < count) {
    if (vv < vecs_per_row) store_piece<P>(obs_ring + (uint64_t)slot * obs_bytes, vv, obs_bytes, piece);
    if (act) {
      uint8_t *const to = act_ring + (uint64_t)slot * act_bytes;
      const uint32_t at = min(unit * vv, act_last);
      if (unit == 4) *reinterpret_cast<u32_any *>(to + at) = act_piece;
      else to[at] = (uint8_t)act_piece;
      for (uint32_t by = unit * (vv + lanes); by < act_bytes; by += unit * lanes) {  // the last piece overlaps the one before it
        const uint32_t q = min(by, act_last);
        if (unit == 4) *reinterpret_cast<u32_any *>(to + q) = *reinterpret_cast<const u32_any *>(act + i * act_bytes + q);
        else to[q] = act[i * act_bytes + q];
      }
    }
  }
  uint64_t *const leaf1 = v.ts.level[0], *const leaf2 = v.te.level[0];
  fetch_now(leaf1, leaf2, v.ts.nlev, v.ts.top_log2);
  fetch_now(v.ts.level[1], v.te.level[1], v.ts.level[2], v.te.level[2]);
  fetch_now(v.qs.alpha, v.qs.eps, v.qs.frac_bits, v.qs.qmax);
  fetch_now(v.qe.alpha, v.qe.eps, v.qe.frac_bits, v.qe.qmax);
  // the last workgroup to have read the free ring's head moves it and the insertion count on (by its last lane: the
  // ticket's round trip then runs beside those of the first wave; at the end of the launch it took 0.5 us more; every wave has
  // looked its slots up by the head, so it has the head)
  lds_barrier();
  if (threadIdx.x == blockDim.x - 1) {
    const uint32_t t = __hip_atomic_fetch_add(&st->ticket_rows, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t == gridDim.x - 1) {
      st->ticket_rows = 0;
      st->free_head = free_head + count;
      st->base.tail = tail + count;
    }
  }
  if (!mass_wave) return;
  bool c1 = false, c2 = false;
  uint64_t q1 = 0, q2 = 0;
  if (active) {
    v.gen[slot_e] += 1;
    if (ns.S || ret) ret_ring[slot_e] = r_in;
    if (ns.S || gacc) gacc_ring[slot_e] = g_in;
    q1 = quantise_priority(p, v.qs, &c1);
    q2 = quantise_priority(p, v.qe, &c2);
    leaf1[slot_e] = q1;  // a free slot weighs nothing in either tree
    leaf2[slot_e] = q2;
  }
  pe_add_runs(v, active, slot_e, q1, q2);
  pe_count_clamped(st, c1, c2);
}

// A learner batch of at most 1024 pairs in one workgroup of at least that many lanes: pairs naming one slot are
// resolved in an LDS hash table (the highest position wins), so the two passes below shrink to one launch.
// h_slot, h_pos: kDedupeSlots words of LDS each.  Called by every thread of the workgroup.
// A pair's masses are on their way during the look-ups (the loads are in before the barrier, the stores behind it): 512 pairs
// 5.9 us with the loads behind the barrier, 5.3 so, 1024 10.1 and 8.3.
__device__ __forceinline__ void pe_update_small_block(const PeView &v, PeState *__restrict__ st, uint32_t m,
                                                      const uint64_t *__restrict__ key,
                                                      const float *__restrict__ prio, uint32_t *h_slot, uint32_t *h_pos)
{
  const uint32_t i = threadIdx.x;
  for (uint32_t t = i; t < kDedupeSlots; t += blockDim.x) {
    h_slot[t] = 0xffffffffu;
    h_pos[t] = 0;
  }
  __syncthreads();
  uint32_t slot = 0, h = 0;
  uint64_t q1 = 0, q2 = 0, old1 = 0, old2 = 0;
  bool c1 = false, c2 = false;
  const bool valid = i < m && pe_key_valid(v, key[i], &slot);
  const bool stale = i < m && !valid;
  if (valid) {
    old1 = v.ts.level[0][slot], old2 = v.te.level[0][slot];  // on their way during the look-ups
    h = (slot * 2654435761u) >> 21;  // top 11 bits
    for (;;) {
      const uint32_t prev = atomicCAS(&h_slot[h], 0xffffffffu, slot);
      if (prev == 0xffffffffu || prev == slot) break;
      h = (h + 1) & (kDedupeSlots - 1);
    }
    atomicMax(&h_pos[h], i + 1);
    const float p = prio[i];
    q1 = quantise_priority(p, v.qs, &c1);
    q2 = quantise_priority(p, v.qe, &c2);
  }
  __syncthreads();
  const bool wins = valid && h_pos[h] == i + 1;
  if (wins) {
    v.ts.level[0][slot] = q1;
    v.te.level[0][slot] = q2;
  }
  pe_add_runs(v, wins, slot, q1 - old1, q2 - old2);  // the keys of a drawn batch ascend: neighbours share their ancestors
  const uint64_t ns = __popcll(__ballot(stale));
  if (ns && lane_id() == 0) atomic_add_u64(&st->base.n_stale, ns);
  pe_count_clamped(st, c1, c2);
}

__global__ __launch_bounds__(1024) void pe_update_small_kernel(PeView v, PeState *__restrict__ st, uint32_t m,
                                                               const uint64_t *__restrict__ key,
                                                               const float *__restrict__ prio)
{
  __shared__ uint32_t h_slot[kDedupeSlots];
  __shared__ uint32_t h_pos[kDedupeSlots];
  pe_update_small_block(v, st, m, key, prio, h_slot, h_pos);
}

// The write-back of the batch that the launch before has drawn, nothing having touched the trees since: pair i
// is valid, lives in slot[i] and weighs mass[i] in the sampling tree, so the loads key -> generation -> mass and
// the hash table are not needed; the drawn slots do not decrease (the strata ascend), so pairs naming one slot
// are neighbours and the last of them is the one that stands.  Lane i % 64 of one wave has pair i.
__device__ __forceinline__ void pe_writeback_wave(const PeView &v, PeState *__restrict__ st, uint32_t m, uint32_t i,
                                                  const uint32_t *__restrict__ slot, const uint64_t *__restrict__ mass,
                                                  const float *__restrict__ prio)
{
  uint64_t *const leaf1 = v.ts.level[0], *const leaf2 = v.te.level[0];
  fetch_now(leaf1, leaf2, v.ts.nlev, v.ts.top_log2);
  fetch_now(v.ts.level[1], v.te.level[1], v.ts.level[2], v.te.level[2]);
  fetch_now(v.qs.alpha, v.qs.eps, v.qs.frac_bits, v.qs.qmax);
  fetch_now(v.qe.alpha, v.qe.eps, v.qe.frac_bits, v.qe.qmax);
  const bool in = i < m;
  const uint32_t at = min(i, m - 1);
  uint32_t s = slot[at], s_next = slot[min(i + 1, m - 1)];
  uint64_t drawn = mass[at];
  float p = prio[at];
  arrived(s), arrived(s_next), arrived(drawn), arrived(p);
  const bool wins = in && (i + 1 == m || s != s_next);
  uint64_t old2 = leaf2[s];  // on its way during the arithmetic
  bool c1, c2;
  const uint64_t q1 = quantise_priority(p, v.qs, &c1), q2 = quantise_priority(p, v.qe, &c2);
  arrived(old2);
  const uint64_t d1 = wins ? q1 - drawn : 0, d2 = wins ? q2 - old2 : 0;
  if (wins) {
    leaf1[s] = q1;
    leaf2[s] = q2;
  }
  pe_add_runs(v, wins, s, d1, d2);
  pe_count_clamped(st, in && c1, in && c2);  // of pairs that lose too, as when they are applied one by one
}

// What follows the draw and gather of one batch whose new priorities are known: the first half of the workgroups (one wave
// each) write the new priorities of 64 pairs back (m = k <= 1024 pairs in all), the others the weights of as many samples.
// One workgroup for all pairs is one compute unit that reads the scattered eviction masses and sends every atomic: draw
// and this, 512 pairs of 1,114,112 slots 11.0 us, 8.9 so; 1024 pairs 14.1 and 8.9.  Bound by the chain arguments, slot, eviction
// mass, atomics; with the arguments fetched together and the eviction mass ahead of the arithmetic 0.2 us less.
__global__ __launch_bounds__(kWave) void pe_finish_update_kernel(WeightArgs wa, PeView v, PeState *__restrict__ st,
                                                                 uint32_t m, const uint32_t *__restrict__ slot,
                                                                 const float *__restrict__ prio)
{
  __shared__ float red[1];
  const uint32_t shares = (m + kWave - 1) / kWave;
  if (blockIdx.x < shares)
    pe_writeback_wave(v, st, m, blockIdx.x * kWave + threadIdx.x, slot, wa.mass, prio);
  else
    batch_weights(wa, 0, red, blockIdx.x - shares, shares);
}

__global__ __launch_bounds__(256) void pe_update_claim_kernel(PeView v, PeState *__restrict__ st, uint32_t m,
                                                              const uint64_t *__restrict__ key,
                                                              uint32_t *__restrict__ claim)
{
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  bool stale = false;
  if (i < m) {
    uint32_t slot;
    if (pe_key_valid(v, key[i], &slot))
      __hip_atomic_fetch_max(claim + slot, i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      stale = true;
  }
  const uint64_t ns = __popcll(__ballot(stale));
  if (ns && lane_id() == 0) atomic_add_u64(&st->base.n_stale, ns);
}

__global__ __launch_bounds__(256) void pe_update_apply_kernel(PeView v, PeState *__restrict__ st, uint32_t m,
                                                              const uint64_t *__restrict__ key,
                                                              const float *__restrict__ prio,
                                                              uint32_t *__restrict__ claim)
{
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t slot = 0;
  bool wins = false, c1 = false, c2 = false;
  uint64_t d1 = 0, d2 = 0;
  if (i < m && pe_key_valid(v, key[i], &slot)) {  // a winner only ever writes non-zero masses, so this cannot flip
    const float p = prio[i];
    const uint64_t q1 = quantise_priority(p, v.qs, &c1), q2 = quantise_priority(p, v.qe, &c2);
    if (claim[slot] == i + 1) {
      wins = true;
      d1 = q1 - v.ts.level[0][slot], d2 = q2 - v.te.level[0][slot];
      v.ts.level[0][slot] = q1;
      v.te.level[0][slot] = q2;
      claim[slot] = 0;
    }
  }
  pe_add_runs(v, wins, slot, d1, d2);  // the keys of a drawn batch ascend: neighbours share their ancestors
  pe_count_clamped(st, c1, c2);
}

constexpr uint32_t kPeScanThreads = 1024;

// Threads of a workgroup of pe_remove_kernel that counts for itself: smaller ones start and end sooner and spread over more
// compute units, but there are more of them to read what lies before.  An add and an eviction of 1000 in three rounds, with
// workgroups of 1024 / 512 / 256: 39.1 / 34.9 / 33.3 us; of 8000 40.1 / 36.3 / 36.5; of 32,000 50.6 / 47.3 / 49.2; of 65,000
// 60.1 / 58.3 / 64.1.
constexpr uint32_t kPeRecountThreads = 512;

// Candidates of a round up to which pe_remove_kernel counts for itself (see there).  An add and an eviction of 32,000 in three
// rounds 47.2 us so, 53.8 with the launch that counts; of 50,000 52.7 and 58.0, of 65,000 58.1 and 60.8, of 98,000 69.0 and 68.2,
// of 131,000 81.2 and 76.2.
constexpr uint64_t kPeRecountMax = 65536;

// A drawn candidate counts if it is the first of its run of equal slots.
__device__ __forceinline__ bool pe_counts(const uint32_t *cand, uint64_t j, uint64_t rem)
{
  return j < rem && (j == 0 || cand[j] != cand[j - 1]);
}

// How many candidates of each workgroup of pe_remove_kernel count, for rounds of more than kPeRecountMax.
__global__ __launch_bounds__(kPeScanThreads) void pe_count_kernel(const uint32_t *__restrict__ cand, uint64_t first_rem,
                                                                  const PeState *__restrict__ st,
                                                                  uint32_t *__restrict__ block_sums)
{
  __shared__ uint32_t wave_tot[kPeScanThreads / kWave];
  const uint64_t rem = first_rem ? first_rem : st->remaining;
  const uint64_t mask = __ballot(pe_counts(cand, (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, rem));
  if (lane_id() == 0) wave_tot[threadIdx.x / kWave] = __popcll(mask);
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t total = 0;
    for (uint32_t w = 0; w < kPeScanThreads / kWave; ++w) total += wave_tot[w];
    block_sums[blockIdx.x] = total;
  }
}

// Removes the candidates that count, in the order of their points.  first_rem: evictions asked for in the first round
// of a call, 0 in the later ones (what the round before has left to do is in st).
// A workgroup's place in the free ring is the number of candidates before it that count.  Up to kPeRecountMax
// candidates every workgroup counts them itself (block_sums null): four candidates per lane and load, four loads ahead of the
// first wait, all of them in the second cache; above, a launch of its own has counted them (block_sums), because the repeated
// reading grows with the square of the round.  What bounds it is its chain of memory trips: counters, candidate, masses, the
// candidates before, atomics.  The masses are asked for ahead of the count so that nothing is loaded behind the barrier (as
// compiled they are in before the count's first load goes out).
// Waves beyond the round's candidates, most of them in the rounds after the first, load none, and the counters come as scalars:
// vector loads of every wave queue for a line that every ticket takes out of the caches.  Rounds 1 / 2 / 3 of an eviction of
// 32,000 8.6 / 3.4 / 3.4 us in the trace, where lanes beyond the round loaded its last candidate and counters came as vectors
// 9.0 / 4.1 / 4.0; of 98,000 9.4 / 4.5 / 4.3 and 9.5 / 4.9 / 5.0.
// An eviction of 32,000 in three rounds is six launches instead of ten (count and removal apart, a launch ahead of them
// that set the number): ten add rounds, ten learner steps and the eviction 243.5 -> 238.6 us.
__global__ __launch_bounds__(kPeScanThreads) void pe_remove_kernel(PeView v, PeState *__restrict__ st,
                                                                   uint64_t first_rem,
                                                                   const uint32_t *__restrict__ cand,
                                                                   const uint32_t *__restrict__ block_sums)
{
  __shared__ uint32_t wave_before[kPeScanThreads / kWave], wave_own[kPeScanThreads / kWave];
  const uint32_t t = threadIdx.x, wave = t / kWave, nthr = blockDim.x, lane = lane_id();
  uint64_t *const leaf1 = v.ts.level[0], *const leaf2 = v.te.level[0];
  const uint64_t rem_before = st->remaining, head = st->base.head, free_tail = st->free_tail;
  fetch_now(cand, leaf1, leaf2, rem_before);
  fetch_now(v.ts.P, v.ts.p_div.mul, v.ts.p_div.sh1, v.ts.p_div.sh2);
  fetch_now(v.ts.level[1], v.te.level[1], v.ts.level[2], v.te.level[2]);
  const uint64_t rem = first_rem ? first_rem : rem_before;  // at most 2^20
  const uint64_t j0 = (uint64_t)blockIdx.x * nthr, j = j0 + t;
  // this thread's candidate and its masses (a lane beyond the round's reads the round's last)
  uint32_t slot = 0, slot_prev = 0;
  uint64_t o1 = 0, o2 = 0;
  const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)rem);
  if ((uint32_t)j0 + (uint32_t)__builtin_amdgcn_readfirstlane((int)wave) * kWave < n) {
    const uint32_t at = min((uint32_t)j, n - 1);
    slot = cand[at], slot_prev = cand[max(at, 1u) - 1];
    o1 = leaf1[slot], o2 = leaf2[slot];
  }
  const bool counts = j < rem && (j == 0 || slot != slot_prev);
  uint32_t before = 0;
  if (block_sums) {
    if (t < blockIdx.x) before = block_sums[t];  // at most kPeScanThreads workgroups of as many threads: one per lane
  } else if (j0 < rem) {  // (then every candidate before j0 belongs to the round)
    const u32x4 *const cand4 = reinterpret_cast<const u32x4 *>(cand);
    const uint32_t n4 = (uint32_t)j0 / 4;
    constexpr uint32_t kAhead = 4;
    for (uint32_t i0 = t; i0 < n4 + t; i0 += kAhead * nthr) {  // the same number of turns for all threads
      u32x4 c[kAhead];
      uint32_t prev[kAhead];
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u) {
        const uint32_t i = min(i0 + u * nthr, n4 - 1);
        c[u] = cand4[i], prev[u] = cand[max(4 * i, 1u) - 1];
      }
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u) {
        const uint32_t i = i0 + u * nthr;
        const uint32_t runs = (uint32_t)(i == 0 || c[u].x != prev[u]) + (uint32_t)(c[u].y != c[u].x) + (uint32_t)(c[u].z != c[u].y) +
                              (uint32_t)(c[u].w != c[u].z);
        before += i < n4 ? runs : 0;
      }
    }
  }
  const uint64_t mask = __ballot(counts);
  const uint32_t wave_total = read_lane_u32((uint32_t)wave_inclusive_scan(before), kWave - 1);
  if (lane == 0) {
    wave_before[wave] = wave_total;
    wave_own[wave] = __popcll(mask);
  }
  fetch_now(head), fetch_now(free_tail);  // every wave has them before its workgroup's ticket lets another one overwrite them
  lds_barrier();
  uint32_t place = __popcll(mask & ((1ull << lane) - 1)), own = 0;
  for (uint32_t w = 0; w < nthr / kWave; ++w) {
    place += wave_before[w] + (w < wave ? wave_own[w] : 0);
    own += wave_own[w];
  }
  // the last workgroup to have read the round's counters closes the round: its ticket comes with what the others
  // remove (ticket in the low word, removals in the high one); the round trip runs beside those of the other lanes
  if (t == nthr - 1) {
    const uint64_t tk = __hip_atomic_fetch_add(&st->round_done, ((uint64_t)own << 32) | 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint32_t)tk == gridDim.x - 1) {
      const uint64_t removed = (tk >> 32) + own;
      st->round_done = 0;
      st->free_tail = free_tail + removed;
      st->base.head = head + removed;
      st->remaining = rem - removed;
    }
  }
  if (counts) {
    leaf1[slot] = 0;
    leaf2[slot] = 0;
    v.free_ring[ring_slot(v.ts, free_tail + place)] = slot;
  }
  pe_add_runs(v, counts, slot, 0 - o1, 0 - o2);  // the candidates ascend: neighbours share their ancestors
}

__global__ __launch_bounds__(256) void pe_init_free_ring_kernel(uint32_t *ring, uint64_t P, PeState *st)
{
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P) ring[i] = (uint32_t)i;
  if (i == 0) {
    st->free_head = 0;
    st->free_tail = P;
  }
}

}  // namespace apex

namespace {

struct PeGeometry {
  uint64_t obs_off, act_off, ret_off, gacc_off, storage_bytes;
  uint32_t nlev, exported_nlev, top_log2;  // as in Geometry
  uint64_t level_off[kMaxLevels], level_size[kMaxLevels], tree_words;  // of one tree; the second follows it
  uint64_t state_off, ticket_off, mass_off, cand_off, sums_off, gen_off, ring_off, claim_off, board_off, scratch_bytes;
};

int pe_validate(const apex_pe_config_t *c)
{
  if (!c) return APEX_ERR_INVALID_ARG;
  if (c->capacity == 0 || c->max_slots < c->capacity || c->max_slots > (1ull << 31)) return APEX_ERR_INVALID_ARG;
  if (c->obs_bytes == 0 || c->act_bytes == 0 || c->frac_bits > 32) return APEX_ERR_INVALID_ARG;
  if (!(c->alpha >= -1.0f && c->alpha <= 1.0f) || !(c->alpha_evict >= -1.0f && c->alpha_evict <= 1.0f))
    return APEX_ERR_INVALID_ARG;
  if (!(c->eps >= 0.0f) || !(c->eps < 1e30f)) return APEX_ERR_INVALID_ARG;
  return APEX_OK;
}

int pe_geometry(const apex_pe_config_t *c, PeGeometry *g)
{
  apex_replay_config_t rc{};
  rc.capacity = c->capacity;
  rc.max_slots = c->max_slots;
  rc.obs_bytes = c->obs_bytes;
  rc.act_bytes = c->act_bytes;
  Geometry base;
  const int rv = geometry(&rc, &base);
  if (rv != APEX_OK) return rv;
  g->obs_off = base.obs_off;
  g->act_off = base.act_off;
  g->ret_off = base.ret_off;
  g->gacc_off = base.gacc_off;
  g->storage_bytes = base.storage_bytes;
  g->nlev = base.nlev;
  g->exported_nlev = base.exported_nlev;
  g->top_log2 = base.top_log2;
  for (uint32_t l = 0; l < kMaxLevels; ++l) {
    g->level_off[l] = base.level_off[l];
    g->level_size[l] = base.level_size[l];
  }
  g->tree_words = base.tree_words;
  const uint64_t P = c->max_slots;
  g->state_off = 0;
  static_assert(sizeof(PeState) <= 256);
  g->ticket_off = 256;
  g->mass_off = g->ticket_off + kTicketBytes;
  g->cand_off = g->mass_off + (uint64_t)APEX_PE_MAX_EVICT_PER_CALL * 8;  // also holds the masses of a sample call
  g->sums_off = g->cand_off + (uint64_t)APEX_PE_MAX_EVICT_PER_CALL * 4;
  g->gen_off = g->sums_off + round_up(kPeScanThreads * 4, 256);
  g->ring_off = g->gen_off + round_up(P * 4, 256);
  g->claim_off = g->ring_off + round_up(P * 4, 256);
  g->board_off = g->claim_off + round_up(P * 4, 256);
  g->scratch_bytes = g->board_off + kBoardBytes;
  return APEX_OK;
}

}  // namespace

struct apex_pe_replay {
  apex_pe_config_t cfg;
  PeGeometry geo;
  uint8_t *storage;
  uint64_t *tree;
  uint8_t *scratch;
  // Host mirror.  `evicted` is what the host takes to have been evicted: exact after calls that report back
  // (apex_pe_evict, apex_pe_stats); after apex_pe_evict_enqueue it assumes that the eviction removed all it was
  // asked to, until the snapshot of the device's counters that the call left behind says otherwise.
  uint64_t inserted, evicted;
  uint64_t evicted_confirmed = 0;  // the last value read back from the device: evicted >= evicted_confirmed
  bool pending = false;            // a snapshot has been requested and not looked at yet
  uint64_t pending_claim = 0;      // what `evicted` was taken to be when it was requested
  TicketUse ticket_use;
  PeState *snap = nullptr;         // pinned host memory that the snapshot lands in
  hipEvent_t snap_ev = nullptr;    // recorded behind the snapshot's copy
  PeView v;

  PeState *state() const { return reinterpret_cast<PeState *>(scratch + geo.state_off); }
  uint32_t *tickets() const { return reinterpret_cast<uint32_t *>(scratch + geo.ticket_off); }
  uint64_t *mass() const { return reinterpret_cast<uint64_t *>(scratch + geo.mass_off); }
  uint32_t *cand() const { return reinterpret_cast<uint32_t *>(scratch + geo.cand_off); }
  uint32_t *sums() const { return reinterpret_cast<uint32_t *>(scratch + geo.sums_off); }
  uint32_t *claim() const { return reinterpret_cast<uint32_t *>(scratch + geo.claim_off); }
  uint32_t *board() const { return reinterpret_cast<uint32_t *>(scratch + geo.board_off); }
  uint8_t *obs() const { return storage + geo.obs_off; }
  uint8_t *act() const { return storage + geo.act_off; }
  float *ret() const { return reinterpret_cast<float *>(storage + geo.ret_off); }
  float *gacc() const { return reinterpret_cast<float *>(storage + geo.gacc_off); }
  uint64_t size() const { return inserted - evicted; }
};

namespace {

// Looks at the snapshot that apex_pe_evict_enqueue requested, if it has arrived (wait: blocks until it has),
// and corrects the mirror if that eviction fell short of what it was asked for.
int pe_resolve(apex_pe_replay *r, bool wait)
{
  if (!r->pending) return APEX_OK;
  if (wait) {
    APEX_HIP(hipEventSynchronize(r->snap_ev));
  } else {
    const hipError_t e = hipEventQuery(r->snap_ev);
    if (e == hipErrorNotReady) {
      (void)hipGetLastError();  // not an error: nothing to report later
      return APEX_OK;
    }
    if (hip_failed(e)) return APEX_ERR_HIP;
  }
  r->pending = false;
  const uint64_t head = r->snap->base.head;
  r->evicted_confirmed = head;
  if (head < r->pending_claim) r->evicted -= r->pending_claim - head;  // the rounds ran out: fewer are gone
  return APEX_OK;
}

// Room for `count` more?  Decided from the mirror; where the mirror rests on an eviction that has not been
// confirmed and the answer depends on it, the confirmation is waited for.
int pe_check_room(apex_pe_replay *r, uint64_t count)
{
  APEX_TRY(pe_resolve(r, false));
  if (r->pending && r->inserted - r->evicted_confirmed + count > r->cfg.max_slots) APEX_TRY(pe_resolve(r, true));
  return r->size() + count > r->cfg.max_slots ? APEX_ERR_FULL : APEX_OK;
}

// The launches of an eviction of e transitions in `rounds` rounds.
int pe_enqueue_eviction(apex_pe_replay *r, uint64_t e, uint32_t rounds, const uint64_t *rnd, hipStream_t stream)
{
  PeState *st = r->state();
  SampleArgs a{};
  a.tv = r->v.te;
  a.st = &st->base;
  a.k = (uint32_t)e;
  a.gen = nullptr;
  a.key_out = nullptr;
  a.slot_out = r->cand();
  a.mass = r->mass();
  a.g.act = nullptr;
  a.g.act_bytes = 0;
  a.g.ret = a.g.gacc = nullptr;
  a.g.act_out = nullptr;
  a.g.ret_out = a.g.gacc_out = nullptr;
  uint32_t *const sums = e > kPeRecountMax ? r->sums() : nullptr;
  const uint32_t threads = sums ? kPeScanThreads : kPeRecountThreads;
  const dim3 grid(blocks_for(e, threads)), block(threads);  // <= 1024 workgroups with sums since e <= 2^20
  for (uint32_t rd = 0; rd < rounds; ++rd) {
    const uint64_t first_rem = rd == 0 ? e : 0;
    a.k_dev = rd == 0 ? nullptr : &st->remaining;
    a.rnd = rnd + (uint64_t)rd * e;
    APEX_TRY(launch_sample(a, 1, stream));
    if (sums) pe_count_kernel<<<grid, block, 0, stream>>>(r->cand(), first_rem, st, sums);
    pe_remove_kernel<<<grid, block, 0, stream>>>(r->v, st, first_rem, r->cand(), sums);
  }
  APEX_HIP(hipGetLastError());
  return APEX_OK;
}

// The arguments of a draw with the small payload columns.
SampleArgs pe_sample_args(apex_pe_replay *r, uint32_t k, const uint64_t *rnd, uint64_t *key_out, uint32_t *slot_out,
                          void *act_out, float *ret_out, float *gacc_out)
{
  SampleArgs a{};
  a.tv = r->v.ts;
  a.st = &r->state()->base;
  a.k = k;
  a.gen = r->v.gen;
  a.rnd = rnd;
  a.key_out = key_out;
  a.slot_out = slot_out;
  a.mass = r->mass();
  a.g.act = r->act();
  a.g.act_bytes = r->cfg.act_bytes;
  a.g.ret = r->ret();
  a.g.gacc = r->gacc();
  a.g.act_out = static_cast<uint8_t *>(act_out);
  a.g.ret_out = ret_out;
  a.g.gacc_out = gacc_out;
  a.g.obs = r->obs();
  a.g.obs_bytes = r->cfg.obs_bytes;
  a.ticket = r->tickets();
  a.board = r->board();
  return a;
}

// The fused calls take rows of at most 256 of the widest aligned units (16, 4 or 1 bytes) that the row length and both
// addresses divide by: a limit of the interface.
bool pe_rows_too_long(const apex_pe_replay *r, const void *rows)
{
  const uintptr_t mis = (uintptr_t)rows | (uintptr_t)r->obs() | (uintptr_t)r->cfg.obs_bytes;
  return r->cfg.obs_bytes / ((mis & 15) == 0 ? 16 : (mis & 3) == 0 ? 4 : 1) > 256;
}

void pe_free(apex_pe_replay *r)
{
  if (r->snap_ev) (void)hipEventDestroy(r->snap_ev);
  if (r->snap) (void)hipHostFree(r->snap);
  delete r;
}

}  // namespace

extern "C" {

int apex_pe_workspace_bytes(const apex_pe_config_t *cfg, size_t *storage_bytes, size_t *tree_bytes,
                            size_t *scratch_bytes)
{
  int rc = pe_validate(cfg);
  if (rc != APEX_OK) return rc;
  PeGeometry g;
  rc = pe_geometry(cfg, &g);
  if (rc != APEX_OK) return rc;
  if (storage_bytes) *storage_bytes = g.storage_bytes;
  if (tree_bytes) *tree_bytes = 2 * g.tree_words * 8;
  if (scratch_bytes) *scratch_bytes = g.scratch_bytes;
  return APEX_OK;
}

int apex_pe_create(const apex_pe_config_t *cfg, void *d_storage, void *d_tree, void *d_scratch, apex_pe_replay_t **out)
{
  int rc = pe_validate(cfg);
  if (rc != APEX_OK) return rc;
  if (!d_storage || !d_tree || !d_scratch || !out) return APEX_ERR_INVALID_ARG;
  if (((uintptr_t)d_storage | (uintptr_t)d_tree | (uintptr_t)d_scratch) & 255) return APEX_ERR_INVALID_ARG;
  apex_pe_replay *r = new (std::nothrow) apex_pe_replay();
  if (!r) return APEX_ERR_INVALID_ARG;
  r->cfg = *cfg;
  rc = pe_geometry(cfg, &r->geo);
  if (rc != APEX_OK) {
    delete r;
    return rc;
  }
  r->storage = static_cast<uint8_t *>(d_storage);
  r->tree = static_cast<uint64_t *>(d_tree);
  r->scratch = static_cast<uint8_t *>(d_scratch);
  r->inserted = r->evicted = 0;
  const uint64_t qmax = qmax_for(cfg->max_slots);
  r->v.qs = QuantParams{cfg->alpha, cfg->eps, cfg->frac_bits, qmax};
  r->v.qe = QuantParams{cfg->alpha_evict, cfg->eps, cfg->frac_bits, qmax};
  for (TreeView *tv : {&r->v.ts, &r->v.te}) {
    tv->nlev = r->geo.nlev;
    tv->n_top = (uint32_t)r->geo.level_size[r->geo.nlev - 1];
    tv->top_log2 = r->geo.top_log2;
    tv->P = cfg->max_slots;
    tv->p_div = make_fast_div((uint32_t)cfg->max_slots);
    uint64_t *base = r->tree + (tv == &r->v.te ? r->geo.tree_words : 0);
    for (uint32_t l = 0; l < kMaxLevels; ++l) tv->level[l] = l < r->geo.nlev ? base + r->geo.level_off[l] : nullptr;
  }
  r->v.gen = reinterpret_cast<uint32_t *>(r->scratch + r->geo.gen_off);
  r->v.free_ring = reinterpret_cast<uint32_t *>(r->scratch + r->geo.ring_off);
  // (host memory and an event for apex_pe_evict_enqueue's snapshots: no device memory is allocated)
  if (hip_failed(hipHostMalloc(reinterpret_cast<void **>(&r->snap), sizeof(PeState), hipHostMallocDefault)) ||
      hip_failed(hipEventCreateWithFlags(&r->snap_ev, hipEventDisableTiming))) {
    pe_free(r);
    return APEX_ERR_HIP;
  }
  fill_zero_kernel<<<dim3(1024), dim3(256), 0, nullptr>>>(r->tree, 2 * r->geo.tree_words);
  fill_zero_kernel<<<dim3(1024), dim3(256), 0, nullptr>>>(reinterpret_cast<uint64_t *>(r->scratch),
                                                          r->geo.scratch_bytes / 8);
  pe_init_free_ring_kernel<<<dim3(blocks_for(cfg->max_slots, 256)), dim3(256), 0, nullptr>>>(
      r->v.free_ring, cfg->max_slots, r->state());
  if (hip_failed(hipGetLastError()) || hip_failed(hipDeviceSynchronize())) {
    pe_free(r);
    return APEX_ERR_HIP;
  }
  *out = r;
  return APEX_OK;
}

int apex_pe_destroy(apex_pe_replay_t *r)
{
  if (!r) return APEX_ERR_INVALID_ARG;
  if (r->pending) (void)hipEventSynchronize(r->snap_ev);  // the snapshot's copy still names r->snap
  pe_free(r);
  return APEX_OK;
}

int apex_pe_layout(const apex_pe_replay_t *r, apex_pe_layout_t *out)
{
  if (!r || !out) return APEX_ERR_INVALID_ARG;
  out->obs_offset = r->geo.obs_off;
  out->act_offset = r->geo.act_off;
  out->ret_offset = r->geo.ret_off;
  out->gacc_offset = r->geo.gacc_off;
  out->tree_levels = r->geo.exported_nlev;
  out->tree_fanout = kFanout;
  for (uint32_t l = 0; l < APEX_TREE_MAX_LEVELS; ++l) {
    out->level_offset[l] = l < r->geo.exported_nlev ? r->geo.level_off[l] : 0;
    out->level_size[l] = l < r->geo.exported_nlev ? r->geo.level_size[l] : 0;
  }
  out->evict_tree_offset = r->geo.tree_words;
  out->gen_offset = r->geo.gen_off;
  out->free_ring_offset = r->geo.ring_off;
  return APEX_OK;
}

int apex_pe_add(apex_pe_replay_t *r, uint64_t count, const void *obs, const void *act, const float *ret,
                const float *gacc, const float *prio, void *hip_stream)
{
  if (!r || (count && !prio)) return APEX_ERR_INVALID_ARG;
  APEX_TRY(pe_check_room(r, count));
  if (count == 0) return APEX_OK;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const RowMap freed{r->v.free_ring, &r->state()->free_head, r->cfg.max_slots, r->v.ts.p_div};  // the next free slots, in order
  const PayloadRing pr{r->obs(), r->act(), r->ret(), r->gacc(), r->cfg.obs_bytes, r->cfg.act_bytes};
  const RowPieces rp = row_pieces((uintptr_t)obs | (uintptr_t)r->obs(), r->cfg.obs_bytes);
  const uint32_t vpr = (uint32_t)pieces_per_row(rp, r->cfg.obs_bytes);
  if (obs && vpr <= 256) {  // short rows: payload and masses in one launch
    uint32_t lanes_log2 = 0;
    while ((1u << lanes_log2) < vpr) ++lanes_log2;
    const uint64_t rows_per_block = kPeAddThreads >> lanes_log2;
    const uint64_t blocks = (count + rows_per_block - 1) / rows_per_block;
    if (blocks > 0x7fffffffull) return APEX_ERR_TOO_LARGE;
    const dim3 grid((uint32_t)blocks), block(kPeAddThreads);
    const uint8_t *o8 = static_cast<const uint8_t *>(obs), *a8 = static_cast<const uint8_t *>(act);
    with_pieces(rp, [&](auto p) {
      pe_add_rows_kernel<decltype(p)><<<grid, block, 0, stream>>>(r->v, r->state(), count, NstepArgs{}, prio, o8, a8, ret,
                                                                  gacc, pr.obs, pr.act, pr.ret, pr.gacc, vpr, lanes_log2,
                                                                  pr.obs_bytes, pr.act_bytes);
    });
  } else {
    const int rc = add_payload_rows(pr, count, obs, act, ret, gacc, freed, stream);
    if (rc != APEX_OK) return rc;
    pe_add_kernel<<<dim3(blocks_for(count, 256)), dim3(256), 0, stream>>>(r->v, r->state(), count, prio);
  }
  APEX_HIP(hipGetLastError());
  r->inserted += count;
  return APEX_OK;
}

int apex_pe_sample(apex_pe_replay_t *r, uint32_t num_batches, uint32_t k, float beta, const uint64_t *rnd,
                   uint64_t *key_out, uint32_t *slot_out, float *weight_out, void *obs_out, void *act_out,
                   float *ret_out, float *gacc_out, void *hip_stream)
{
  if (!r || !num_batches || !k || !rnd || !slot_out || !(beta >= 0.0f) || !(beta <= 1.0f)) return APEX_ERR_INVALID_ARG;
  if (num_batches > APEX_MAX_BATCHES_PER_CALL || (uint64_t)num_batches * k > APEX_MAX_SAMPLES_PER_CALL)
    return APEX_ERR_TOO_LARGE;
  if (r->size() == 0) return APEX_ERR_EMPTY;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  SampleArgs a = pe_sample_args(r, k, rnd, key_out, slot_out, act_out, ret_out, gacc_out);
  SideJobs jobs;
  jobs.wa = WeightArgs{r->mass(), weight_out, k, beta};
  const bool by_rows = obs_out && sample_by_rows(r->cfg.obs_bytes, num_batches, k);
  const bool gather = obs_out && (by_rows || r->cfg.obs_bytes <= kGatherInDrawBytes);
  if (gather) a.g.obs_out = static_cast<uint8_t *>(obs_out);
  if ((gather || !obs_out) && k <= kWeightsInDrawMaxK) {
    a.weight_out = weight_out;
    a.beta = beta;
    jobs.wa.weight_out = nullptr;
  }
  if (by_rows) return launch_sample_rows(a, num_batches, stream, &r->ticket_use);
  APEX_TRY(launch_sample(a, num_batches, stream, &r->ticket_use));
  if (obs_out && !gather) {
    const RowMap by_slot{slot_out, nullptr, 0, {}};
    const RowMap ident{nullptr, nullptr, 0, {}};
    APEX_TRY(launch_copy(r->obs(), by_slot, obs_out, ident, (uint64_t)num_batches * k, r->cfg.obs_bytes, stream, &jobs));
  }
  return jobs.wa.weight_out ? launch_weights(jobs.wa, num_batches, stream) : APEX_OK;
}

int apex_pe_update_priorities(apex_pe_replay_t *r, uint64_t m, const uint64_t *key, const float *prio,
                              void *hip_stream)
{
  if (!r || (m && (!key || !prio))) return APEX_ERR_INVALID_ARG;
  if (m >= 0xffffffffull) return APEX_ERR_TOO_LARGE;
  if (m == 0) return APEX_OK;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (m <= 1024) {
    pe_update_small_kernel<<<dim3(1), dim3((uint32_t)round_up(m, kWave)), 0, stream>>>(r->v, r->state(), (uint32_t)m, key, prio);
    APEX_HIP(hipGetLastError());
    return APEX_OK;
  }
  const dim3 grid(blocks_for(m, 256)), block(256);
  pe_update_claim_kernel<<<grid, block, 0, stream>>>(r->v, r->state(), (uint32_t)m, key, r->claim());
  pe_update_apply_kernel<<<grid, block, 0, stream>>>(r->v, r->state(), (uint32_t)m, key, prio, r->claim());
  APEX_HIP(hipGetLastError());
  return APEX_OK;
}

int apex_pe_evict(apex_pe_replay_t *r, uint32_t rounds, const uint64_t *rnd, uint64_t *evicted_out, void *hip_stream)
{
  if (!r) return APEX_ERR_INVALID_ARG;
  APEX_TRY(pe_resolve(r, true));  // this call reports back anyway: start from exact counts
  const uint64_t size = r->size();
  const uint64_t e = size > r->cfg.capacity ? size - r->cfg.capacity : 0;
  if (evicted_out) *evicted_out = 0;
  if (e == 0) return APEX_OK;
  if (!rnd || rounds == 0) return APEX_ERR_INVALID_ARG;
  if (e > APEX_PE_MAX_EVICT_PER_CALL) return APEX_ERR_TOO_LARGE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  APEX_TRY(pe_enqueue_eviction(r, e, rounds, rnd, stream));
  PeState h;
  APEX_HIP(hipMemcpyAsync(&h, r->state(), sizeof h, hipMemcpyDeviceToHost, stream));
  APEX_HIP(hipStreamSynchronize(stream));
  r->evicted = r->evicted_confirmed = h.base.head;
  if (evicted_out) *evicted_out = e - h.remaining;
  return APEX_OK;
}

int apex_pe_evict_enqueue(apex_pe_replay_t *r, uint32_t rounds, const uint64_t *rnd, uint64_t *requested_out,
                          void *hip_stream)
{
  if (!r) return APEX_ERR_INVALID_ARG;
  APEX_TRY(pe_resolve(r, true));  // the snapshot of the eviction before this one (long done by now) frees r->snap
  const uint64_t size = r->size();
  const uint64_t e = size > r->cfg.capacity ? size - r->cfg.capacity : 0;
  if (requested_out) *requested_out = e;
  if (e == 0) return APEX_OK;
  if (!rnd || rounds == 0) return APEX_ERR_INVALID_ARG;
  if (e > APEX_PE_MAX_EVICT_PER_CALL) return APEX_ERR_TOO_LARGE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  APEX_TRY(pe_enqueue_eviction(r, e, rounds, rnd, stream));
  APEX_HIP(hipMemcpyAsync(r->snap, r->state(), sizeof(PeState), hipMemcpyDeviceToHost, stream));
  APEX_HIP(hipEventRecord(r->snap_ev, stream));
  r->evicted += e;
  r->pending = true;
  r->pending_claim = r->evicted;
  return APEX_OK;
}

int apex_pe_add_round(apex_pe_replay_t *r, uint32_t S, uint32_t T, uint32_t n, uint32_t A, const float *q_online,
                      const float *q_target, const int32_t *action, const float *reward, const float *discount,
                      const void *obs, const void *act, void *hip_stream)
{
  if (!r || !S || !T || !n || !A || !q_online || !q_target || !action || !reward || !discount || !obs)
    return APEX_ERR_INVALID_ARG;
  const uint64_t count = (uint64_t)S * T;
  if ((uint64_t)T + n > 0xffffffffull) return APEX_ERR_TOO_LARGE;
  if (pe_rows_too_long(r, obs)) return APEX_ERR_TOO_LARGE;  // apex_nstep_priorities + apex_pe_add take them
  const RowPieces rp = row_pieces((uintptr_t)obs | (uintptr_t)r->obs(), r->cfg.obs_bytes);
  const uint32_t vpr = (uint32_t)pieces_per_row(rp, r->cfg.obs_bytes);
  APEX_TRY(pe_check_room(r, count));
  uint32_t lanes_log2 = 0;
  while ((1u << lanes_log2) < vpr) ++lanes_log2;
  const uint64_t rows_per_block = kPeAddThreads >> lanes_log2;
  const uint64_t blocks = (count + rows_per_block - 1) / rows_per_block;
  if (blocks > 0x7fffffffull) return APEX_ERR_TOO_LARGE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const NstepArgs ns{S, T, n, A, make_fast_div(T), q_online, q_target, action, reward, discount};
  const dim3 grid((uint32_t)blocks), block(kPeAddThreads);
  const uint8_t *o8 = static_cast<const uint8_t *>(obs), *a8 = static_cast<const uint8_t *>(act);
  with_pieces(rp, [&](auto p) {
    pe_add_rows_kernel<decltype(p)><<<grid, block, 0, stream>>>(r->v, r->state(), count, ns, nullptr, o8, a8, nullptr,
                                                                nullptr, r->obs(), r->act(), r->ret(), r->gacc(), vpr,
                                                                lanes_log2, r->cfg.obs_bytes, r->cfg.act_bytes);
  });
  APEX_HIP(hipGetLastError());
  r->inserted += count;
  return APEX_OK;
}

int apex_pe_sample_update(apex_pe_replay_t *r, uint32_t k, float beta, const uint64_t *rnd, const float *new_prio,
                          uint64_t *key_out, uint32_t *slot_out, float *weight_out, void *obs_out, void *act_out,
                          float *ret_out, float *gacc_out, void *hip_stream)
{
  if (!r || !k || !rnd || !new_prio || !key_out || !slot_out || !(beta >= 0.0f) || !(beta <= 1.0f))
    return APEX_ERR_INVALID_ARG;
  if (k > 1024) return APEX_ERR_TOO_LARGE;
  if (obs_out && pe_rows_too_long(r, obs_out)) return APEX_ERR_TOO_LARGE;  // apex_pe_sample + apex_pe_update_priorities
  if (r->size() == 0) return APEX_ERR_EMPTY;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  SampleArgs a = pe_sample_args(r, k, rnd, key_out, slot_out, act_out, ret_out, gacc_out);
  a.g.obs_out = static_cast<uint8_t *>(obs_out);
  // The draw and the rows by a workgroup per sample, whatever the size: without weights nothing is settled between workgroups.
  // Both launches, us, with 16 lanes per sample / so, k of 1, 32, 128, 512 and 1000:
  //     16 bytes  5.9 / 5.4   7.0 / 6.5   7.6 / 6.8    7.8 / 7.3    7.9 / 7.6
  //     64        5.8 / 5.3   7.2 / 6.1   7.4 / 6.4    7.4 / 6.7    7.6 / 7.3
  //    256        5.9 / 5.4   7.1 / 6.4   7.6 / 6.8    7.9 / 7.3    8.4 / 7.7
  //   1000        5.8 / 5.2   7.3 / 6.5   7.8 / 6.8    8.0 / 7.3    8.9 / 7.9
  //   4096        6.6 / 5.6   9.1 / 6.8   9.4 / 7.1   11.0 / 7.5   11.2 / 8.3
  if (obs_out && r->cfg.obs_bytes >= 16) APEX_TRY(launch_sample_rows(a, 1, stream, nullptr));
  else APEX_TRY(launch_sample(a, 1, stream));
  // weights and the write-back of the batch just drawn: one launch
  const WeightArgs wa{r->mass(), weight_out, k, beta};
  const dim3 grid(blocks_for(k, kWave) * (weight_out ? 2 : 1));
  pe_finish_update_kernel<<<grid, dim3(kWave), 0, stream>>>(wa, r->v, r->state(), k, slot_out, new_prio);
  APEX_HIP(hipGetLastError());
  return APEX_OK;
}

int apex_pe_stats(apex_pe_replay_t *r, apex_pe_stats_t *out, void *hip_stream)
{
  if (!r || !out) return APEX_ERR_INVALID_ARG;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  PeState h;
  static thread_local uint64_t top[2][kTopMax];
  const uint32_t n_top = r->v.ts.n_top;
  APEX_HIP(hipMemcpyAsync(&h, r->state(), sizeof h, hipMemcpyDeviceToHost, stream));
  APEX_HIP(hipMemcpyAsync(top[0], r->v.ts.level[r->v.ts.nlev - 1], (size_t)n_top * 8, hipMemcpyDeviceToHost, stream));
  APEX_HIP(hipMemcpyAsync(top[1], r->v.te.level[r->v.te.nlev - 1], (size_t)n_top * 8, hipMemcpyDeviceToHost, stream));
  APEX_HIP(hipStreamSynchronize(stream));
  uint64_t root[2] = {0, 0};
  for (int t = 0; t < 2; ++t)
    for (uint32_t i = 0; i < n_top; ++i) root[t] += top[t][i];
  if (r->pending) APEX_TRY(pe_resolve(r, true));  // (an enqueued eviction's snapshot precedes this read on the stream
                                                  // only if it was enqueued on hip_stream; else it is simply waited for)
  out->size = h.base.tail - h.base.head;
  out->inserted = h.base.tail;
  out->evicted = h.base.head;
  out->root = root[0];
  out->root_evict = root[1];
  out->free_head = h.free_head;
  out->free_tail = h.free_tail;
  out->n_stale_dropped = h.base.n_stale;
  out->n_clamped = h.base.n_clamped;
  return APEX_OK;
}

}  // extern "C"
