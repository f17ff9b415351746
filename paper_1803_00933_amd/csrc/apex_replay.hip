// Host side of the C ABI declared in include/apex_replay.h: argument checks, host mirror of
// head/tail, and the kernel launches.  Every entry point only enqueues work on the caller's
// stream; nothing here allocates device memory.
#include "apex_replay.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "kernels.hpp"

using namespace apex;

// Scratch of apex_replay_sample_noalloc: the masses of the drawn transitions between the descent
// and the weights.  One copy per GPU, held until the process ends.  In host code this name is only
// a handle for hipGetSymbolAddress: the device address it yields (static_scratch_ptr) is what goes
// into kernel arguments.
static __device__ __align__(256) uint64_t scratch[APEX_NOALLOC_MAX_SAMPLES];

namespace {

thread_local int g_last_hip_error = 0;

inline bool hip_failed(hipError_t e)
{
  if (e == hipSuccess) return false;
  g_last_hip_error = (int)e;
  return true;
}

#define APEX_HIP(call)                         \
  do {                                         \
    if (hip_failed((call))) return APEX_ERR_HIP; \
  } while (0)

// The device address of `scratch` on the GPU that is current in the calling thread: looked up once per
// device (each GPU holds its own copy of the array at its own address) and kept.  Null, with the
// error recorded, if the lookup fails.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
uint64_t *g_scratch_ptr[kMaxDevices] = {};

uint64_t *static_scratch_ptr()
{
  int dev = -1;
  if (hip_failed(hipGetDevice(&dev)) || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    if (hip_failed(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) || !ptr) return nullptr;
    g_scratch_ptr[dev] = static_cast<uint64_t *>(ptr);
  }
  return g_scratch_ptr[dev];
}

inline uint64_t round_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }
inline uint32_t blocks_for(uint64_t n, uint32_t per) { return (uint32_t)((n + per - 1) / per); }

uint32_t ceil_log2(uint64_t v)
{
  uint32_t l = 0;
  while ((1ull << l) < v) ++l;
  return l;
}

// The constants of fast_div for the divisor d >= 1.
FastDiv make_fast_div(uint32_t d)
{
  if (d == 0) d = 1;
  uint32_t L = 0;
  while (L < 32 && (1ull << L) < d) ++L;
  const unsigned __int128 num = ((unsigned __int128)((1ull << L) - d)) << 64;
  return FastDiv{(uint64_t)(num / d) + 1, L < 1 ? L : 1, L > 0 ? L - 1 : 0};
}

uint64_t qmax_for(uint64_t max_slots) { return max_slots ? 1ull << (62 - ceil_log2(max_slots)) : 1ull << 62; }

constexpr uint64_t kTicketBytes = (uint64_t)APEX_MAX_BATCHES_PER_CALL * kTicketStride * 4;
constexpr uint64_t kBoardSetWords = board_place(kBoardWordsMax), kBoardBytes = 4 * kTicketSets * kBoardSetWords;
constexpr uint32_t kStepSets = 64;  // buffer sets a sequence of fused steps can cycle through

struct Geometry {
  uint64_t obs_off, act_off, ret_off, gacc_off, storage_bytes;
  uint32_t nlev;            // levels in the tree, ...
  uint32_t exported_nlev;   // ... of which apex_replay_layout shows these (a summit is not shown)
  uint32_t top_log2;        // fan-out of the last level over the one below it
  uint64_t level_off[kMaxLevels], level_size[kMaxLevels], tree_words;
  // scratch: DeviceState | tickets of sample calls | mass | claim | new masses of the batches of fused steps | board of sample calls
  uint64_t state_off, ticket_off, mass_off, claim_off, stepq_off, board_off, scratch_bytes;
};

int validate(const apex_replay_config_t *c)
{
  if (!c) return APEX_ERR_INVALID_ARG;
  if (c->capacity == 0 || c->max_slots < c->capacity || c->max_slots > (1ull << 31)) return APEX_ERR_INVALID_ARG;
  if (c->obs_bytes == 0 || c->act_bytes == 0 || c->frac_bits > 32 || c->reserved != 0) return APEX_ERR_INVALID_ARG;
  if (!(c->alpha >= -1.0f && c->alpha <= 1.0f) || !(c->eps >= 0.0f) || !(c->eps < 1e30f)) return APEX_ERR_INVALID_ARG;
  return APEX_OK;
}

int geometry(const apex_replay_config_t *c, Geometry *g)
{
  const uint64_t P = c->max_slots;
  g->obs_off = 0;
  g->act_off = g->obs_off + round_up(P * c->obs_bytes, 256);
  g->ret_off = g->act_off + round_up(P * c->act_bytes, 256);
  g->gacc_off = g->ret_off + round_up(P * 4, 256);
  g->storage_bytes = g->gacc_off + round_up(P * 4, 256);

  uint64_t n = P, off = 0;
  uint32_t l = 0;
  for (;;) {
    if (l + 1 >= kMaxLevels) return APEX_ERR_INVALID_ARG;  // one place is kept for the summit
    g->level_off[l] = off;
    g->level_size[l] = n;
    off += round_up(n, kFanout);
    ++l;
    if (n <= kExportedTopMax) break;
    n = (n + kFanout - 1) / kFanout;
  }
  g->exported_nlev = g->nlev = l;
  g->top_log2 = kFanoutLog2;
  if (n > kTopMax) {  // the summit
    g->top_log2 = 0;
    while (((n - 1) >> g->top_log2) + 1 > kSummitMax) ++g->top_log2;
    g->level_off[l] = off;
    g->level_size[l] = ((n - 1) >> g->top_log2) + 1;
    off += round_up(g->level_size[l], kFanout);
    ++g->nlev;
  }
  g->tree_words = off;

  g->state_off = 0;
  g->ticket_off = 256;
  g->mass_off = g->ticket_off + kTicketBytes;
  g->claim_off = g->mass_off + (uint64_t)APEX_MAX_SAMPLES_PER_CALL * 8;
  g->stepq_off = g->claim_off + round_up(P * 4, 256);
  g->board_off = g->stepq_off + (uint64_t)kStepSets * kStepMaxK * 8;
  g->scratch_bytes = g->board_off + kBoardBytes;
  return APEX_OK;
}

// The sample launches on one memory that have used tickets or a board (see sample_kernel, sample_rows_kernel), and the most
// words one of them used.
struct TicketUse {
  uint32_t launches = 0, lines = 0, board_words = 0;
};

}  // namespace

struct apex_replay {
  apex_replay_config_t cfg;
  Geometry geo;
  uint8_t *storage;
  uint64_t *tree;
  uint8_t *scratch;
  uint64_t head, tail;  // host mirror of the device state
  TicketUse ticket_use;
  QuantParams qp;
  TreeView tv;
  // Second copy of the tree, behind the first in the tree region: used by sequences of fused learner
  // steps only.  It equals the first while tree_version == second_version; every entry point that
  // changes the first copy moves tree_version on.
  TreeView tv2;
  uint64_t tree_version = 1, second_version = 0;

  // Words from the first copy to the second while the two are equal, else 0 (see AddLeavesArgs).
  uint64_t second_words() const { return second_version == tree_version ? geo.tree_words : 0; }
  // What a launch that has written to both copies (or, second == 0, to the first alone) leaves behind.
  void tree_changed(uint64_t second)
  {
    ++tree_version;
    if (second) second_version = tree_version;
  }

  DeviceState *state() const { return reinterpret_cast<DeviceState *>(scratch + geo.state_off); }
  uint32_t *tickets() const { return reinterpret_cast<uint32_t *>(scratch + geo.ticket_off); }
  uint64_t *mass() const { return reinterpret_cast<uint64_t *>(scratch + geo.mass_off); }
  uint32_t *claim() const { return reinterpret_cast<uint32_t *>(scratch + geo.claim_off); }
  uint32_t *board() const { return reinterpret_cast<uint32_t *>(scratch + geo.board_off); }
  uint64_t *stepq(uint32_t set) const { return reinterpret_cast<uint64_t *>(scratch + geo.stepq_off) + (uint64_t)set * kStepMaxK; }
  uint8_t *obs() const { return storage + geo.obs_off; }
  uint8_t *act() const { return storage + geo.act_off; }
  float *ret() const { return reinterpret_cast<float *>(storage + geo.ret_off); }
  float *gacc() const { return reinterpret_cast<float *>(storage + geo.gacc_off); }
};

namespace {

// How rows of row_bytes bytes at addresses whose bits are or-ed into mis are moved (see Piece): in aligned 16-byte
// pieces, in 16-byte pieces at any alignment, or, rows shorter than that, in aligned words or bytes.
enum RowPieces { kPieces16, kPiecesAny, kPieces4, kPieces1 };

RowPieces row_pieces(uintptr_t mis, uint64_t row_bytes)
{
  mis |= (uintptr_t)row_bytes;
  if (row_bytes >= 16) return (mis & 15) == 0 ? kPieces16 : kPiecesAny;
  return (mis & 3) == 0 ? kPieces4 : kPieces1;
}

uint64_t pieces_per_row(RowPieces rp, uint64_t row_bytes)
{
  return rp == kPieces1 ? row_bytes : rp == kPieces4 ? row_bytes / 4 : (row_bytes + 15) / 16;
}

// Calls f with the piece type that rp names.
template <typename F>
auto with_pieces(RowPieces rp, F f)
{
  switch (rp) {
    case kPieces16: return f(Piece16{});
    case kPiecesAny: return f(PieceAny{});
    case kPieces4: return f(Piece4{});
    default: return f(Piece1{});
  }
}

// Copies nrows rows of row_bytes bytes with the long- or short-row kernel.
// Side jobs a long-row copy can take along in leading workgroups (see copy_rows_long_kernel).
// A field is cleared once a kernel has taken the job on; what is left needs launches of its own.
struct SideJobs {
  WeightArgs wa{nullptr, nullptr, 1, 0.f};  // wa.weight_out != null: importance weights wanted
  UpdateArgs ua{};                          // ua.m != 0: a priority update of at most 1024 pairs
  ClaimArgs claim{};                        // claim.m != 0: first pass of a larger update (short rows only)
};

// The write-back of a batch that has just been drawn, spread over the workgroups that copy its rows (kUpdate = 2 of
// copy_rows_long_kernel), up to this many pairs (every pair looks through those behind it for its slot) ...
constexpr uint64_t kSpreadWritebackMax = 1024;
// ... and for rows above this length.  (Steps of 1024 on 2^20 slots, rows of 1028 bytes: 16.1 us so, 22.8 with the update
// in one workgroup of a launch of its own; 2 x 512 of 4092 bytes 15.9 and 22.8; 8 x 128 of 1028 bytes from 20,000 slots, where
// it gains least, 15.5 and 15.0.)
constexpr uint64_t kSpreadWritebackAbove = 1024;

template <typename Vec>
int launch_copy_t(const uint8_t *src, const RowMap &smap, uint8_t *dst, const RowMap &dmap, uint64_t nrows,
                  uint64_t row_bytes, uint32_t vpr, hipStream_t stream, SideJobs *jobs)
{
  constexpr int kUnroll = kLongCopyUnroll, kThreads = kLongCopyThreads;
  const bool spread = jobs && jobs->ua.m && jobs->ua.slot_hint && jobs->ua.m <= kSpreadWritebackMax &&
                      row_bytes > kSpreadWritebackAbove;
  if (vpr > 256 || spread) {
    const uint32_t cpr = (vpr + kThreads * kUnroll - 1) / (kThreads * kUnroll);
    if (nrows * cpr > 0x7ffffff0ull) return APEX_ERR_TOO_LARGE;
    const uint32_t blocks = (uint32_t)(nrows * cpr);
    bool w = jobs && jobs->wa.weight_out, u = jobs && jobs->ua.m;
    uint32_t nb = w ? (uint32_t)(nrows / jobs->wa.k) : 0;  // one workgroup per batch takes its weights along
    if (blocks < nb + (u ? 1u : 0u)) w = u = false, nb = 0;    // too few workgroups to carry the side jobs
    const WeightArgs wa = w ? jobs->wa : WeightArgs{nullptr, nullptr, 1, 0.f};
    const UpdateArgs ua = u ? jobs->ua : UpdateArgs{};
    const dim3 grid(blocks), block(kThreads);
    if (!jobs && !smap.index && !smap.ring_key && !dmap.index && nrows * vpr < 0xfffff000ull && nrows >= 1024) {
      // dense source, many rows (the payload of an add round): workgroups packed with vectors
      const uint32_t total = (uint32_t)(nrows * vpr);
      copy_rows_dense_kernel<Vec, kUnroll><<<dim3(blocks_for(total, kThreads * kUnroll)), block, 0, stream>>>(
          src, dst, dmap, vpr, row_bytes, total);
      return hip_failed(hipGetLastError()) ? APEX_ERR_HIP : APEX_OK;
    }
    if (!u && vpr <= kThreads * kUnroll / 2 && nrows * vpr < 0xfffff000ull && nrows < 0xffffffffull) {
      // rows that would fill at most half of a workgroup (4 to 16 KB), no write-back riding along:
      // workgroups packed with vectors.  (For longer rows one workgroup per row measured a little faster.)
      const uint32_t total = (uint32_t)(nrows * vpr);
      const dim3 pgrid(blocks_for(total, kThreads * kUnroll) + nb);
      if (w)
        copy_rows_packed_kernel<Vec, kUnroll, true><<<pgrid, block, 0, stream>>>(src, smap, dst, dmap, (uint32_t)nrows, vpr,
                                                                             row_bytes, total, wa, nb);
      else
        copy_rows_packed_kernel<Vec, kUnroll, false><<<pgrid, block, 0, stream>>>(src, smap, dst, dmap, (uint32_t)nrows,
                                                                              vpr, row_bytes, total, wa, 0);
      if (w) jobs->wa.weight_out = nullptr;
      return hip_failed(hipGetLastError()) ? APEX_ERR_HIP : APEX_OK;
    }
    // a same-batch write-back (slot/mass known) has one pair per copied row: spread it over the rows
    const int umode = !u ? 0 : (ua.slot_hint && ua.m == nrows) ? 2 : 1;
#define APEX_LAUNCH_COPY(W, U) \
  copy_rows_long_kernel<Vec, kUnroll, W, U><<<grid, block, 0, stream>>>(src, smap, dst, dmap, vpr, cpr, row_bytes, wa, nb, ua)
    if (w && umode == 2) APEX_LAUNCH_COPY(true, 2);
    else if (w && umode == 1) APEX_LAUNCH_COPY(true, 1);
    else if (w) APEX_LAUNCH_COPY(true, 0);
    else if (umode == 2) APEX_LAUNCH_COPY(false, 2);
    else if (umode == 1) APEX_LAUNCH_COPY(false, 1);
    else APEX_LAUNCH_COPY(false, 0);
#undef APEX_LAUNCH_COPY
    if (w) jobs->wa.weight_out = nullptr;
    if (u) jobs->ua.m = 0;
  } else {
    uint32_t lanes_log2 = 0;
    while ((1u << lanes_log2) < vpr) ++lanes_log2;
    const bool w = jobs && jobs->wa.weight_out, cl = jobs && jobs->claim.m;
    const uint32_t threads = w && jobs->wa.k > 256 ? kWeightThreads : 256;  // powers of two: whole rows
    const uint64_t rows_per_block = threads >> lanes_log2;
    const uint64_t blocks = (nrows + rows_per_block - 1) / rows_per_block;
    if (blocks > 0x7ffffff0ull) return APEX_ERR_TOO_LARGE;
    const ShortCopyArgs c{src, smap, dst, dmap, nrows, vpr, lanes_log2, row_bytes};
    if (w || cl) {
      // the importance weights and the claim pass of a large update ride along
      const uint32_t batches = w ? (uint32_t)(nrows / jobs->wa.k) : 0, parts = w ? blocks_for(jobs->wa.k, kWeightThreads) : 0;
      const uint32_t claim_blocks = cl ? blocks_for(jobs->claim.m, threads) : 0;
      finish_short_kernel<Vec><<<dim3((uint32_t)blocks + batches * parts + claim_blocks), dim3(threads), 0, stream>>>(
          c, (uint32_t)blocks, w ? jobs->wa : WeightArgs{nullptr, nullptr, 1, 0.f}, batches, parts,
          cl ? jobs->claim : ClaimArgs{});
      if (w) jobs->wa.weight_out = nullptr;
      if (cl) jobs->claim.m = 0;
    } else {
      copy_rows_short_kernel<Vec><<<dim3((uint32_t)blocks), dim3(256), 0, stream>>>(c);
    }
  }
  return hip_failed(hipGetLastError()) ? APEX_ERR_HIP : APEX_OK;
}

int launch_copy(const void *src, const RowMap &smap, void *dst, const RowMap &dmap, uint64_t nrows, uint64_t row_bytes,
                hipStream_t stream, SideJobs *jobs = nullptr)
{
  if (nrows == 0) return APEX_OK;
  const RowPieces rp = row_pieces((uintptr_t)src | (uintptr_t)dst, row_bytes);
  const uint32_t vpr = (uint32_t)pieces_per_row(rp, row_bytes);
  return with_pieces(rp, [&](auto p) {
    return launch_copy_t<decltype(p)>(static_cast<const uint8_t *>(src), smap, static_cast<uint8_t *>(dst), dmap, nrows,
                                      row_bytes, vpr, stream, jobs);
  });
}

// One launch of the fused learner step (see learner_step_kernel).
// Steps whose rows are decoded on their way out (aligned 16-byte pieces; riders: none, or the masses of an add round).
void launch_step_codec(const StepArgs &a, uint32_t wgs, uint32_t threads, int rider, hipStream_t stream)
{
  const dim3 grid(wgs), block(threads);
  if (rider == kLeavesRide)
    learner_step_kernel<Piece16, kStepThreads, kStepUnroll, kLeavesRide, true><<<grid, block, 0, stream>>>(a);
  else
    learner_step_kernel<Piece16, kStepThreads, kStepUnroll, kNoRider, true><<<grid, block, 0, stream>>>(a);
}

template <typename Vec>
void launch_step_t(const StepArgs &a, uint32_t wgs, uint32_t threads, int rider, hipStream_t stream)
{
  const dim3 grid(wgs), block(threads);
  if (rider == kRoundRides)  // further workgroups carry part of an add round (such a launch draws nothing)
    learner_step_kernel<Vec, kStepThreads, kStepUnroll, kRoundRides><<<grid, block, 0, stream>>>(a);
  else if (rider == kLeavesRide)
    learner_step_kernel<Vec, kStepThreads, kStepUnroll, kLeavesRide><<<grid, block, 0, stream>>>(a);
  else
    learner_step_kernel<Vec, kStepThreads, kStepUnroll, kNoRider><<<grid, block, 0, stream>>>(a);
}

// A small add round (observations of at most 1 KB per row) as one launch: n-step priorities, payload,
// masses.  Same effect as apex_nstep_priorities + apex_replay_add.

// Arguments of such a round for workgroups of `threads` lanes and pieces of the kind rp;
// *blocks: the workgroups it takes.
int add_round_args(const apex_replay *r, const NstepArgs &ns, const void *obs, const void *act, RowPieces rp,
                   uint32_t threads, AddRoundArgs *out, uint32_t *blocks)
{
  const uint64_t count = (uint64_t)ns.S * ns.T;
  const uint32_t vpr = (uint32_t)pieces_per_row(rp, r->cfg.obs_bytes);
  uint32_t lanes_log2 = 0;
  while ((1u << lanes_log2) < vpr && lanes_log2 < 6) ++lanes_log2;  // at most one wave per row
  const uint64_t rows_per_block = threads >> lanes_log2;
  const uint64_t nb = (count + rows_per_block - 1) / rows_per_block;
  if (nb > 0x7ffffff0ull) return APEX_ERR_TOO_LARGE;
  *blocks = (uint32_t)nb;
  *out = AddRoundArgs{ns, r->tv, r->second_words(), r->state(), r->qp, static_cast<const uint8_t *>(obs),
                      static_cast<const uint8_t *>(act), r->obs(), r->act(), r->ret(), r->gacc(), vpr, lanes_log2,
                      r->cfg.obs_bytes, r->cfg.act_bytes};
  return APEX_OK;
}

// Whether a round can go that way, and how its rows are moved.
bool add_round_small_fits(const apex_replay *r, const NstepArgs &ns, const void *obs, RowPieces *rp)
{
  if (!obs || r->cfg.obs_bytes > 1024 || (uint64_t)ns.S * ns.T == 0) return false;
  *rp = row_pieces((uintptr_t)obs | (uintptr_t)r->obs(), r->cfg.obs_bytes);
  return true;
}

// Host-side bookkeeping of a round that has been enqueued.
void add_round_published(apex_replay *r, uint64_t count, uint64_t second, uint64_t *first_key_out)
{
  r->tree_changed(second);
  if (first_key_out) *first_key_out = r->tail;
  r->tail += count;
}

// APEX_ERR_NOT_READY - with nothing enqueued - when the rows are too long for the single launch.
int add_round_small(apex_replay *r, const NstepArgs &ns, const void *obs, const void *act, uint64_t *first_key_out,
                    hipStream_t stream)
{
  const uint64_t count = (uint64_t)ns.S * ns.T;
  RowPieces rp = kPieces1;
  uint32_t blocks = 0;
  if (!add_round_small_fits(r, ns, obs, &rp)) return APEX_ERR_NOT_READY;
  if ((r->tail - r->head) + count > r->cfg.max_slots) return APEX_ERR_FULL;
  const uint64_t second = r->second_words();
  AddRoundArgs a;
  const int rc = add_round_args(r, ns, obs, act, rp, kAddRoundThreads, &a, &blocks);
  if (rc != APEX_OK) return rc;
  const dim3 grid(blocks), block(kAddRoundThreads);
  with_pieces(rp, [&](auto p) { add_round_small_kernel<decltype(p)><<<grid, block, 0, stream>>>(a); });
  APEX_HIP(hipGetLastError());
  add_round_published(r, count, second, first_key_out);
  return APEX_OK;
}

// Short observation rows: the whole payload of an add round in one launch.  APEX_ERR_NOT_READY - with
// nothing enqueued - when the rows are long (the column-by-column copies take over).
struct PayloadRing {
  uint8_t *obs, *act;
  float *ret, *gacc;
  uint64_t obs_bytes;
  uint32_t act_bytes;
};

template <typename Vec>
int add_payload_short_t(const PayloadRing &pr, uint64_t count, const void *obs, const void *act, const float *ret,
                        const float *gacc, const RowMap &to, uint32_t vpr, hipStream_t stream)
{
  uint32_t lanes_log2 = 0;
  while ((1u << lanes_log2) < vpr) ++lanes_log2;
  const uint64_t rows_per_block = 256u >> lanes_log2;
  const uint64_t blocks = (count + rows_per_block - 1) / rows_per_block;
  if (blocks > 0x7fffffffull) return APEX_ERR_TOO_LARGE;
  add_payload_short_kernel<Vec><<<dim3((uint32_t)blocks), dim3(256), 0, stream>>>(
      static_cast<const uint8_t *>(obs), static_cast<const uint8_t *>(act), ret, gacc, pr.obs, pr.act, pr.ret, pr.gacc,
      to, count, vpr, lanes_log2, pr.obs_bytes, pr.act_bytes);
  return hip_failed(hipGetLastError()) ? APEX_ERR_HIP : APEX_OK;
}

// Whether rows like these are added by add_payload_short_kernel.
bool short_rows(const PayloadRing &pr, const void *obs)
{
  return pieces_per_row(row_pieces((uintptr_t)obs | (uintptr_t)pr.obs, pr.obs_bytes), pr.obs_bytes) <= 256;
}

int add_payload_short(const PayloadRing &pr, uint64_t count, const void *obs, const void *act, const float *ret,
                      const float *gacc, const RowMap &to, hipStream_t stream)
{
  const RowPieces rp = row_pieces((uintptr_t)obs | (uintptr_t)pr.obs, pr.obs_bytes);
  const uint64_t vpr = pieces_per_row(rp, pr.obs_bytes);
  return with_pieces(rp, [&](auto p) {
    return add_payload_short_t<decltype(p)>(pr, count, obs, act, ret, gacc, to, (uint32_t)vpr, stream);
  });
}

// The three small columns (action bytes, partial return, accumulated discount) in one launch:
// 2^lanes_log2 lanes per transition share the action bytes.
int add_small_columns(const PayloadRing &pr, uint64_t count, const void *act, const float *ret, const float *gacc,
                      const RowMap &to, hipStream_t stream)
{
  uint32_t lanes_log2 = 0;
  while ((4u << lanes_log2) < pr.act_bytes && lanes_log2 < 6) ++lanes_log2;
  const uint64_t rows_per_block = 256u >> lanes_log2;
  const uint64_t blocks = (count + rows_per_block - 1) / rows_per_block;
  if (blocks > 0x7fffffffull) return APEX_ERR_TOO_LARGE;
  add_payload_short_kernel<Piece1><<<dim3((uint32_t)blocks), dim3(256), 0, stream>>>(
      nullptr, static_cast<const uint8_t *>(act), ret, gacc, pr.obs, pr.act, pr.ret, pr.gacc, to, count,
      /*vecs_per_row=*/0, lanes_log2, pr.obs_bytes, pr.act_bytes);
  return hip_failed(hipGetLastError()) ? APEX_ERR_HIP : APEX_OK;
}

// obs, act, ret, gacc (any may be null) of `count` transitions into the rows that `to` names.
int add_payload_rows(const PayloadRing &pr, uint64_t count, const void *obs, const void *act, const float *ret,
                     const float *gacc, const RowMap &to, hipStream_t stream)
{
  const RowMap ident{nullptr, nullptr, 0, {}};
  int rc;
  if (obs && short_rows(pr, obs)) return add_payload_short(pr, count, obs, act, ret, gacc, to, stream);
  if (obs && (rc = launch_copy(obs, ident, pr.obs, to, count, pr.obs_bytes, stream)) != APEX_OK) return rc;
  if (act || ret || gacc) return add_small_columns(pr, count, act, ret, gacc, to, stream);
  return APEX_OK;
}

}  // namespace

extern "C" {

int apex_last_hip_error(void) { return g_last_hip_error; }

int apex_replay_workspace_bytes(const apex_replay_config_t *cfg, size_t *storage_bytes, size_t *tree_bytes,
                                size_t *scratch_bytes)
{
  int rc = validate(cfg);
  if (rc != APEX_OK) return rc;
  Geometry g;
  rc = geometry(cfg, &g);
  if (rc != APEX_OK) return rc;
  if (storage_bytes) *storage_bytes = g.storage_bytes;
  if (tree_bytes) *tree_bytes = 2 * g.tree_words * 8;  // two copies, see learner_step_kernel
  if (scratch_bytes) *scratch_bytes = g.scratch_bytes;
  return APEX_OK;
}

int apex_replay_create(const apex_replay_config_t *cfg, void *d_storage, void *d_tree, void *d_scratch,
                       apex_replay_t **out)
{
  int rc = validate(cfg);
  if (rc != APEX_OK) return rc;
  if (!d_storage || !d_tree || !d_scratch || !out) return APEX_ERR_INVALID_ARG;
  if (((uintptr_t)d_storage | (uintptr_t)d_tree | (uintptr_t)d_scratch) & 255) return APEX_ERR_INVALID_ARG;
  apex_replay *r = new (std::nothrow) apex_replay();
  if (!r) return APEX_ERR_INVALID_ARG;
  r->cfg = *cfg;
  rc = geometry(cfg, &r->geo);
  if (rc != APEX_OK) {
    delete r;
    return rc;
  }
  r->storage = static_cast<uint8_t *>(d_storage);
  r->tree = static_cast<uint64_t *>(d_tree);
  r->scratch = static_cast<uint8_t *>(d_scratch);
  r->head = r->tail = 0;
  r->qp = QuantParams{cfg->alpha, cfg->eps, cfg->frac_bits, qmax_for(cfg->max_slots)};
  r->tv.nlev = r->geo.nlev;
  r->tv.n_top = (uint32_t)r->geo.level_size[r->geo.nlev - 1];
  r->tv.top_log2 = r->geo.top_log2;
  r->tv.P = cfg->max_slots;
  r->tv.p_div = make_fast_div((uint32_t)cfg->max_slots);
  for (uint32_t l = 0; l < kMaxLevels; ++l) r->tv.level[l] = l < r->geo.nlev ? r->tree + r->geo.level_off[l] : nullptr;
  r->tv2 = r->tv;
  for (uint32_t l = 0; l < r->geo.nlev; ++l) r->tv2.level[l] = r->tv.level[l] + r->geo.tree_words;

  // set-up for apex_replay_sample_noalloc on this GPU, so that the call itself has nothing left to look up
  if (!static_scratch_ptr()) {
    delete r;
    return APEX_ERR_HIP;
  }
  fill_zero_kernel<<<dim3(1024), dim3(256), 0, nullptr>>>(r->tree, 2 * r->geo.tree_words);
  fill_zero_kernel<<<dim3(1024), dim3(256), 0, nullptr>>>(reinterpret_cast<uint64_t *>(r->scratch),
                                                          r->geo.scratch_bytes / 8);
  if (hip_failed(hipGetLastError()) || hip_failed(hipDeviceSynchronize())) {
    delete r;
    return APEX_ERR_HIP;
  }
  *out = r;
  return APEX_OK;
}

int apex_replay_destroy(apex_replay_t *r)
{
  if (!r) return APEX_ERR_INVALID_ARG;
  delete r;
  return APEX_OK;
}

int apex_replay_layout(const apex_replay_t *r, apex_replay_layout_t *out)
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
  return APEX_OK;
}

int apex_nstep_priorities(uint32_t S, uint32_t T, uint32_t n, uint32_t A, const float *q_online,
                          const float *q_target, const int32_t *action, const float *reward,
                          const float *discount, float alpha, float eps, uint32_t frac_bits,
                          uint64_t max_slots, float *prio, float *ret, float *gacc, uint64_t *prio_fx,
                          void *hip_stream)
{
  if (!S || !T || !n || !A) return APEX_ERR_INVALID_ARG;
  if (!q_online || !q_target || !action || !reward || !discount || !prio || !ret || !gacc) return APEX_ERR_INVALID_ARG;
  if (frac_bits > 32 || !(alpha >= -1.0f && alpha <= 1.0f) || !(eps >= 0.0f) || max_slots > (1ull << 31))
    return APEX_ERR_INVALID_ARG;
  const uint64_t total = (uint64_t)S * T;
  if (total > 0x7fffffffull * 256 || (uint64_t)T + n > 0xffffffffull) return APEX_ERR_TOO_LARGE;
  const QuantParams qp{alpha, eps, frac_bits, qmax_for(max_slots)};
  const NstepArgs ns{S, T, n, A, make_fast_div(T), q_online, q_target, action, reward, discount};
  nstep_kernel<<<dim3(blocks_for(total, 256)), dim3(256), 0, static_cast<hipStream_t>(hip_stream)>>>(ns, qp, prio, ret,
                                                                                                 gacc, prio_fx);
  APEX_HIP(hipGetLastError());
  return APEX_OK;
}

}  // extern "C"

namespace {

// Threads per workgroup of add_leaves_kernel and evict_leaves_kernel for `count` transitions: no more than there is work
// for (add and eviction of 1 to 130 transitions of 2^20 slots 9.2 - 9.8 us, 8.5 - 9.2 so), but two waves, so that the
// ticket's round trip runs beside those of the first wave's atomics.
uint32_t leaves_threads(uint64_t count)
{
  return (uint32_t)std::clamp<uint64_t>(round_up(count, kWave), 2 * kWave, kLeavesThreads);
}

// Enters `count` transitions under the next keys: launch(arguments) enqueues the launch that does it.
template <typename F>
int publish_with(apex_replay_t *r, uint64_t count, const float *prio, uint64_t *first_key_out, F launch)
{
  if ((r->tail - r->head) + count > r->cfg.max_slots) return APEX_ERR_FULL;
  if (count) {
    const uint64_t second = r->second_words();
    r->tree_changed(second);
    launch(AddLeavesArgs{r->tv, second, r->state(), count, prio, r->qp});
    APEX_HIP(hipGetLastError());
  }
  if (first_key_out) *first_key_out = r->tail;
  r->tail += count;
  return APEX_OK;
}

// columns: as far as the small columns are to be copied too.
int publish(apex_replay_t *r, uint64_t count, const float *prio, const AddColumns &columns, uint64_t *first_key_out,
            void *hip_stream)
{
  if (!r || (count && !prio)) return APEX_ERR_INVALID_ARG;
  return publish_with(r, count, prio, first_key_out, [&](const AddLeavesArgs &a) {
    const uint32_t threads = leaves_threads(count);
    add_leaves_kernel<<<dim3(blocks_for(count, threads)), dim3(threads), 0, static_cast<hipStream_t>(hip_stream)>>>(a, columns);
  });
}

}  // namespace

extern "C" {

int apex_replay_add_payload(apex_replay_t *r, uint64_t count, const void *obs, const void *act, const float *ret,
                            const float *gacc, void *hip_stream)
{
  if (!r) return APEX_ERR_INVALID_ARG;
  if ((r->tail - r->head) + count > r->cfg.max_slots) return APEX_ERR_FULL;
  if (count == 0) return APEX_OK;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const RowMap ring{nullptr, &r->state()->tail, r->cfg.max_slots, r->tv.p_div};
  const PayloadRing pr{r->obs(), r->act(), r->ret(), r->gacc(), r->cfg.obs_bytes, r->cfg.act_bytes};
  return add_payload_rows(pr, count, obs, act, ret, gacc, ring, stream);
}

int apex_replay_add_publish(apex_replay_t *r, uint64_t count, const float *prio, uint64_t *first_key_out,
                            void *hip_stream)
{
  return publish(r, count, prio, AddColumns{}, first_key_out, hip_stream);
}

int apex_replay_add(apex_replay_t *r, uint64_t count, const void *obs, const void *act, const float *ret,
                    const float *gacc, const float *prio, uint64_t *first_key_out, void *hip_stream)
{
  if (!r || (count && !prio)) return APEX_ERR_INVALID_ARG;
  const PayloadRing pr{r->obs(), r->act(), r->ret(), r->gacc(), r->cfg.obs_bytes, r->cfg.act_bytes};
  const AddColumns columns{static_cast<const uint8_t *>(act), ret, gacc, r->act(), r->ret(), r->gacc(), r->cfg.act_bytes};
  if (obs && r->cfg.obs_bytes <= kAddRowsInOneBytes && r->cfg.act_bytes <= kColumnsInAddBytes) {
    const RowPieces rp = row_pieces((uintptr_t)obs | (uintptr_t)r->obs(), r->cfg.obs_bytes);
    const uint32_t vpr = (uint32_t)pieces_per_row(rp, r->cfg.obs_bytes), lanes_log2 = ceil_log2(vpr);
    const uint32_t threads = std::min(leaves_threads(count), add_rows_threads(count, r->cfg.obs_bytes));
    return publish_with(r, count, prio, first_key_out, [&](const AddLeavesArgs &a) {
      with_pieces(rp, [&](auto p) {
        add_rows_kernel<decltype(p)><<<dim3(blocks_for(count, threads)), dim3(threads), 0, static_cast<hipStream_t>(hip_stream)>>>(
            a, columns, static_cast<const uint8_t *>(obs), r->obs(), vpr, lanes_log2, r->cfg.obs_bytes);
      });
    });
  }
  if ((obs && short_rows(pr, obs)) || r->cfg.act_bytes > kColumnsInAddBytes) {
    const int rc = apex_replay_add_payload(r, count, obs, act, ret, gacc, hip_stream);
    return rc != APEX_OK ? rc : apex_replay_add_publish(r, count, prio, first_key_out, hip_stream);
  }
  const int rc = apex_replay_add_payload(r, count, obs, nullptr, nullptr, nullptr, hip_stream);
  return rc != APEX_OK ? rc : publish(r, count, prio, columns, first_key_out, hip_stream);
}

namespace {

// Importance weights in a launch of their own.
int launch_weights(const WeightArgs &wa, uint32_t num_batches, hipStream_t stream)
{
  const uint32_t threads = (uint32_t)std::clamp<uint64_t>(round_up(wa.k, kWave), kWave, kWeightThreads);
  batch_weights_kernel<<<dim3(num_batches, blocks_for(wa.k, threads)), dim3(threads), 0, stream>>>(wa);
  return hip_failed(hipGetLastError()) ? APEX_ERR_HIP : APEX_OK;
}

// Gives a launch that takes tickets, or uses a board (a.board then names its region), its set of words.
void take_tickets(SampleArgs &a, uint32_t lines, uint32_t board_words, TicketUse *tickets)
{
  const uint32_t set = tickets->launches++ & (kTicketSets - 1), ahead = (set + 2) & (kTicketSets - 1);
  tickets->lines = std::max(tickets->lines, lines);
  tickets->board_words = std::max(tickets->board_words, board_words);
  a.ticket_ahead = a.ticket + ahead;
  a.ticket += set;
  a.ticket_lines = tickets->lines;
  a.board_ahead = a.board + ahead * kBoardSetWords;
  a.board = board_words ? a.board + set * kBoardSetWords : nullptr;
  a.board_words = tickets->board_words;
}

// Waves of a workgroup of sample_rows_kernel whose lanes hold `pieces` pieces of a row of vpr (a row that it does not hold
// takes further passes), and how many such workgroups the chip has room for: a workgroup's waves are on one compute unit.
uint32_t sample_rows_waves(uint32_t vpr, uint32_t pieces) { return std::min(1 + blocks_for(vpr, pieces * kWave), 1024u / kWave); }
uint32_t sample_rows_at_once(uint32_t waves) { return kChipCus * (kChipWaves / kChipCus / waves); }

// Whether such a launch finds its batches' smallest masses by the board.
bool sample_uses_board(uint32_t num_batches, uint32_t k) { return num_batches * k <= kBoardSamplesMax || k <= kBoardSmallK; }

// Whether num_batches x k samples with rows of obs_bytes go into sample_rows_kernel rather than sample_kernel (rows of up to
// kGatherInDrawBytes) or two launches.  (The times on both sides of the lines of long rows are at the kernel.)  Short rows, us,
// sample_kernel / sample_rows_kernel, device time from 2^18 to 2^20 slots:
//               1 x 512    1 x 700    1 x 800    1 x 900    1 x 1024   2 x 512    12 x 100   40 x 32    3 x 500    2 x 768
//     32 bytes  5.7 / 5.1  5.9 / 5.8  6.1 / 6.3  6.1 / 6.7  6.3 / 6.8  5.7 / 5.6  5.8 / 6.4  5.4 / 5.6  5.8 / 6.3  6.0 / 6.8
//    128        5.7 / 5.1  6.0 / 5.8  6.2 / 6.2  6.2 / 6.7  6.4 / 6.7  5.8 / 5.6  6.2 / 6.3  5.7 / 5.6  5.9 / 6.4  6.1 / 6.9
//    268        5.8 / 5.1  6.1 / 5.9  6.3 / 6.3  6.4 / 6.7  6.7 / 6.9  6.2 / 5.7  6.5 / 6.3  6.1 / 5.6  6.6 / 6.5  6.7 / 7.1
//   1024        6.1 / 5.1  6.8 / 6.1  7.0 / 6.6  7.2 / 7.3  7.4 / 7.8  7.0 / 6.5  6.9 / 6.6  6.5 / 6.0  7.2 / 6.8  7.3 / 7.4
//   1500        7.0 / 5.3  7.2 / 6.3  7.4 / 7.0  7.5 / 7.7  7.7 / 7.9  7.3 / 6.7  7.2 / 6.5  6.8 / 6.1  7.5 / 7.0  7.7 / 7.5
//   2048        6.9 / 5.2  7.4 / 5.9  7.7 / 6.4  7.7 / 6.9  7.9 / 7.1  7.6 / 5.8  7.4 / 6.6  7.1 / 5.7  7.7 / 6.8  7.9 / 7.5
//   4096        8.3 / 5.3  8.5 / 6.2  8.7 / 6.7  8.8 / 7.3  8.9 / 7.4  8.6 / 6.1  8.5 / 6.8  8.9 / 6.2  9.0 / 7.6  9.3 / 8.3
// (3 x 500 and 2 x 768 by tickets.  From 256 to 2047 bytes the two are too close there, and on either side, for a line.)
bool sample_by_rows(uint64_t obs_bytes, uint32_t num_batches, uint32_t k)
{
  const uint64_t samples = (uint64_t)num_batches * k;
  if (obs_bytes < 16 || k > kSampleRowsMaxK || samples > kSampleRowsMax) return false;
  if (obs_bytes <= kGatherInDrawBytes) {
    if (obs_bytes < 2048 && k > (obs_bytes < 1024 ? 768u : 832u)) return false;
    if (samples <= kBoardSamplesMax) return true;
    return k <= kBoardSmallK ? obs_bytes >= 256 : obs_bytes >= 2048 && k <= obs_bytes / 4;
  }
  if (obs_bytes > (samples <= 512 ? kSampleRowsMaxBytes : kSampleRowsMaxBytesOfMany)) return false;
  // not where workgroups that copy a row in one pass come in more than one round, their batches' weights in the last one
  return obs_bytes > kCopyRowBytes || k <= 384 ||
         samples <= sample_rows_at_once(sample_rows_waves((uint32_t)((obs_bytes + 15) / 16), 4));
}

// a.k samples of each of num_batches batches, as sample_by_rows has it.  Two pieces per lane as long as the chip then holds
// all workgroups at once, else four (28,224 bytes: 256 samples 7.3 us with two and 8.2 with four, 999 samples 16.4 and 14.0;
// 896 samples of 16 KB, 9 waves to a workgroup with two, 13.6 and 11.1).
int launch_sample_rows(SampleArgs &a, uint32_t num_batches, hipStream_t stream, TicketUse *tickets)
{
  a.k_div = make_fast_div(a.k);
  a.top = a.tv.level[a.tv.nlev - 1];
  uint32_t weight_waves = 0;
  if (a.weight_out) {
    const uint32_t groups = blocks_for(a.k, kTicketGroup);
    if (sample_uses_board(num_batches, a.k)) take_tickets(a, 0, num_batches * board_stride(a.k), tickets);
    else take_tickets(a, num_batches * (groups > 1 ? 1 + groups : 1), 0, tickets);
    weight_waves = std::min(kWeightWaves, 1 + a.k / kWave);
  } else {
    a.board = nullptr;
  }
  const uint32_t vpr = (uint32_t)((a.g.obs_bytes + 15) / 16);
  const bool two = num_batches * a.k <= sample_rows_at_once(sample_rows_waves(vpr, 2)), wide = a.tv.n_top > 512;
  const dim3 grid(a.k, num_batches), block(std::max(weight_waves, sample_rows_waves(vpr, two ? 2 : 4)) * kWave);
  const auto launch = [&](auto unroll, auto streaming) {
    if (wide) sample_rows_kernel<unroll.value, true, streaming.value><<<grid, block, 0, stream>>>(a, vpr);
    else sample_rows_kernel<unroll.value, false, streaming.value><<<grid, block, 0, stream>>>(a, vpr);
  };
  typedef std::integral_constant<int, 2> Two;
  typedef std::integral_constant<int, 4> Four;
  if (a.g.obs_bytes < kStreamingBytes) launch(Two{}, std::false_type{});
  else if (two) launch(Two{}, std::true_type{});
  else launch(Four{}, std::true_type{});
  return hip_failed(hipGetLastError()) ? APEX_ERR_HIP : APEX_OK;
}

// a.k samples of each of num_batches batches (with a.k_dev: at most a.k).  tickets may be null where a.weight_out is.
int launch_sample(SampleArgs &a, uint32_t num_batches, hipStream_t stream, TicketUse *tickets = nullptr)
{
  a.k_div = make_fast_div(a.k);
  a.top = a.tv.level[a.tv.nlev - 1];
  const uint32_t threads = sample_threads(a.k, a.weight_out != nullptr), wgs = blocks_for(a.k, threads / 16);
  if (a.weight_out && wgs > 1) take_tickets(a, num_batches, 0, tickets);
  const dim3 grid(wgs, num_batches), block(threads);
  if (a.tv.n_top > 512)
    sample_kernel<true><<<grid, block, 0, stream>>>(a);
  else
    sample_kernel<false><<<grid, block, 0, stream>>>(a);
  return hip_failed(hipGetLastError()) ? APEX_ERR_HIP : APEX_OK;
}

// Checks, and the arguments of a draw with the small payload columns (no weights, no observation rows).
int sample_args(apex_replay *r, uint32_t num_batches, uint32_t k, const uint64_t *rnd, uint64_t *key_out,
                uint32_t *slot_out, uint64_t *mass_out, void *act_out, float *ret_out, float *gacc_out, SampleArgs *out)
{
  if (!r || !num_batches || !k || !rnd || !slot_out || !mass_out) return APEX_ERR_INVALID_ARG;
  if (num_batches > APEX_MAX_BATCHES_PER_CALL || (uint64_t)num_batches * k > APEX_MAX_SAMPLES_PER_CALL)
    return APEX_ERR_TOO_LARGE;
  const uint64_t size = r->tail - r->head;
  if (size < r->cfg.min_size_to_sample) return APEX_ERR_NOT_READY;
  if (size == 0) return APEX_ERR_EMPTY;
  SampleArgs &a = *out;
  a = SampleArgs{};
  a.tv = r->tv;
  a.st = r->state();
  a.k = k;
  a.rnd = rnd;
  a.key_out = key_out;
  a.slot_out = slot_out;
  a.mass = mass_out;
  a.g.act = r->act();
  a.g.act_bytes = r->cfg.act_bytes;
  a.g.ret = r->ret();
  a.g.gacc = r->gacc();
  a.g.act_out = static_cast<uint8_t *>(act_out);
  a.g.ret_out = ret_out;
  a.g.gacc_out = gacc_out;
  return APEX_OK;
}

int sample_begin_impl(apex_replay *r, uint32_t num_batches, uint32_t k, const uint64_t *rnd, uint64_t *key_out,
                      uint32_t *slot_out, uint64_t *mass_out, void *act_out, float *ret_out, float *gacc_out,
                      hipStream_t stream)
{
  SampleArgs a;
  const int rc = sample_args(r, num_batches, k, rnd, key_out, slot_out, mass_out, act_out, ret_out, gacc_out, &a);
  return rc != APEX_OK ? rc : launch_sample(a, num_batches, stream);
}

// Whether a batch of `per` samples goes that way when its own priorities are written back.
bool writeback_spreads(const apex_replay *r, uint64_t per)
{
  return per <= kSpreadWritebackMax && r->cfg.obs_bytes > kSpreadWritebackAbove;
}

// Whether the rows' gather rides in the draw's launch: short rows do (the wave that has drawn a sample copies its row);
// of long ones a workgroup per row moves more bytes per second (copy_rows_long_kernel).
bool gather_in_draw(const apex_replay *r) { return r->cfg.obs_bytes <= kGatherInDrawBytes; }

// apex_replay_sample for rows that gather_in_draw or sample_by_rows: one launch (two for the weights of very large batches).  claim: the
// first pass of an update of all drawn keys rides along.
int sample_in_one(apex_replay *r, uint32_t num_batches, uint32_t k, float beta, const uint64_t *rnd, uint64_t *key_out,
                  uint32_t *slot_out, uint64_t *mass_out, float *weight_out, void *obs_out, void *act_out,
                  float *ret_out, float *gacc_out, bool claim, hipStream_t stream)
{
  SampleArgs a;
  const int rc = sample_args(r, num_batches, k, rnd, key_out, slot_out, mass_out, act_out, ret_out, gacc_out, &a);
  if (rc != APEX_OK) return rc;
  a.g.obs = r->obs();
  a.g.obs_bytes = r->cfg.obs_bytes;
  a.g.obs_out = static_cast<uint8_t *>(obs_out);
  a.weight_out = k <= kWeightsInDrawMaxK ? weight_out : nullptr;
  a.beta = beta;
  a.ticket = r->tickets();
  a.board = r->board();
  a.claim = claim ? r->claim() : nullptr;
  const int rl = !claim && obs_out && sample_by_rows(a.g.obs_bytes, num_batches, k)
                     ? launch_sample_rows(a, num_batches, stream, &r->ticket_use)
                     : launch_sample(a, num_batches, stream, &r->ticket_use);
  return rl != APEX_OK || a.weight_out == weight_out ? rl
                                                     : launch_weights(WeightArgs{mass_out, weight_out, k, beta}, num_batches, stream);
}

}  // namespace

int apex_replay_sample_begin(apex_replay_t *r, uint32_t num_batches, uint32_t k, const uint64_t *rnd,
                             uint64_t *key_out, uint32_t *slot_out, uint64_t *mass_out, void *act_out, float *ret_out,
                             float *gacc_out, void *hip_stream)
{
  return sample_begin_impl(r, num_batches, k, rnd, key_out, slot_out, mass_out, act_out, ret_out, gacc_out,
                           static_cast<hipStream_t>(hip_stream));
}

namespace {

// claimed: the first pass (update_claim) of a large update has already run.
int launch_update(apex_replay *r, uint64_t m, const uint64_t *key, const float *prio, hipStream_t stream,
                  const QSource &qs = QSource{}, bool claimed = false)
{
  ++r->tree_version;
  if (m <= kUpdateOneLaunchMax && !claimed) {
    const UpdateArgs ua{r->tv, r->state(), (uint32_t)m, key, prio, r->qp, nullptr, nullptr, qs};
    const dim3 grid(blocks_for(m, kWave)), block((uint32_t)std::clamp<uint64_t>(round_up(m, kWave), kUpdateMinThreads, kUpdateThreads));
    if (m <= kUpdateThreads)
      update_small_kernel<1><<<grid, block, 0, stream>>>(ua);
    else if (m <= 2 * kUpdateThreads)
      update_small_kernel<2><<<grid, block, 0, stream>>>(ua);
    else
      update_many_kernel<<<grid, dim3(kUpdateManyThreads), 0, stream>>>(ua);
  } else {
    const dim3 grid(blocks_for(m, 256)), block(256);
    if (!claimed)
      update_claim_kernel<<<grid, block, 0, stream>>>(ClaimArgs{r->cfg.max_slots, r->tv.p_div, r->state(), (uint32_t)m, key, r->claim()});
    update_apply_kernel<<<grid, block, 0, stream>>>(r->tv, r->state(), (uint32_t)m, key, prio, r->qp, r->claim(), qs);
  }
  return hip_failed(hipGetLastError()) ? APEX_ERR_HIP : APEX_OK;
}

// gather + importance weights (+ a priority update riding along when it fits one workgroup)
// same_batch: the pairs are the batch being finished (key[i] lives in slot[i] and weighs mass[i]) and
// nothing has touched the tree since it was drawn.
int finish_impl(apex_replay *r, uint32_t num_batches, uint32_t k, float beta, const uint32_t *slot,
                const uint64_t *mass, float *weight_out, void *obs_out, uint64_t m, const uint64_t *key,
                const float *prio, hipStream_t stream, bool same_batch = false)
{
  SideJobs jobs;
  jobs.wa = WeightArgs{mass, weight_out, k, beta};
  const bool hint = same_batch && mass && m == (uint64_t)num_batches * k;
  if (m) ++r->tree_version;
  if (m && (m <= 1024 || hint)) {
    jobs.ua = UpdateArgs{r->tv, r->state(), (uint32_t)m, key, prio, r->qp, hint ? slot : nullptr, hint ? mass : nullptr,
                         QSource{}};
  }
  if (m > 1024) jobs.claim = ClaimArgs{r->cfg.max_slots, r->tv.p_div, r->state(), (uint32_t)m, key, r->claim()};
  if (obs_out) {
    const RowMap by_slot{slot, nullptr, 0, {}};
    const RowMap ident{nullptr, nullptr, 0, {}};
    const int rc = launch_copy(r->obs(), by_slot, obs_out, ident, (uint64_t)num_batches * k, r->cfg.obs_bytes, stream, &jobs);
    if (rc != APEX_OK) return rc;
  }
  if (jobs.wa.weight_out) {  // no gather, or short rows: the weights get a small launch of their own
    const int rc = launch_weights(jobs.wa, num_batches, stream);
    if (rc != APEX_OK) return rc;
  }
  // whatever of the update no launch above has taken (a claim pass that has run leaves the second pass)
  if (m && (jobs.ua.m || !(m <= 1024 || hint)))
    return launch_update(r, m, key, prio, stream, QSource{}, /*claimed=*/m > 1024 && jobs.claim.m == 0);
  return APEX_OK;
}

// n learner steps of one batch of k each, in strict order (draw i, write-back i, draw i+1, ...), as
// one standalone draw, one launch per step, and one small launch at the end: see
// learner_step_kernel.  Batch i goes to sets[(first_set + i) % depth]; kernel i reads the sets of
// batches i-1 and i and writes that of batch i+1, hence depth >= 3.
// Returns APEX_ERR_NOT_READY - with nothing enqueued - when the shapes do not fit the fused launch.
// How the rows of the ring and of the batch buffers are moved.
RowPieces step_pieces(const apex_replay *r, uint32_t depth, const apex_batch_buffers_t *sets)
{
  uintptr_t mis = (uintptr_t)r->obs();
  for (uint32_t i = 0; i < depth; ++i) mis |= (uintptr_t)sets[i].obs;
  return row_pieces(mis, r->cfg.obs_bytes);
}

bool fused_steps_fit(const apex_replay *r, uint32_t num_batches, uint32_t k, uint32_t depth,
                     const apex_batch_buffers_t *sets)
{
  if (num_batches != 1 || k > kStepMaxK || depth < 3 || depth > kStepSets) return false;
  for (uint32_t i = 0; i < depth; ++i)
    if ((uintptr_t)sets[i].slot & 15) return false;
  return true;
}

void launch_step(const StepArgs &args, RowPieces rp, uint32_t wgs, uint32_t threads, hipStream_t stream,
                 int rider = kNoRider)
{
  StepArgs a = args;
  a.next_top = a.next.tv.level[a.next.tv.nlev - 1];
  a.next_k_div = make_fast_div(a.next.k);
  if (a.codec.raw_bytes && a.slot) return launch_step_codec(a, wgs, threads, rider, stream);
  with_pieces(rp, [&](auto p) { launch_step_t<decltype(p)>(a, wgs, threads, rider, stream); });
}

// A step launch that has been prepared but not issued: the last one of a call, held back while a small
// add round is open, because the round can ride in the same launch (see StepArgs::add).
struct HeldStep {
  bool valid = false;
  StepArgs a;
  RowPieces rp;
};

int issue_held_step(HeldStep *h, hipStream_t stream)
{
  if (!h->valid) return APEX_OK;
  h->valid = false;
  launch_step(h->a, h->rp, h->a.k, kStepThreads, stream);
  APEX_HIP(hipGetLastError());
  return APEX_OK;
}

// The held step and a small add round in one launch.  APEX_ERR_NOT_READY - with nothing enqueued - if
// there is no held step or the two do not fit together (the round's rows allow only narrower pieces).
int issue_held_step_with_round(apex_replay *r, HeldStep *h, const NstepArgs &ns, const void *obs, const void *act,
                               uint64_t *first_key_out, hipStream_t stream)
{
  const uint64_t count = (uint64_t)ns.S * ns.T;
  RowPieces rp = kPieces1;
  uint32_t blocks = 0;
  if (!h->valid || h->a.codec.raw_bytes || !add_round_small_fits(r, ns, obs, &rp) || rp > h->rp)
    return APEX_ERR_NOT_READY;
  if ((r->tail - r->head) + count > r->cfg.max_slots) return APEX_ERR_FULL;
  const uint64_t second = r->second_words();
  const int rc = add_round_args(r, ns, obs, act, h->rp, kStepThreads, &h->a.add, &blocks);
  if (rc != APEX_OK) return rc;
  h->valid = false;
  launch_step(h->a, h->rp, h->a.k + blocks, kStepThreads, stream, kRoundRides);
  APEX_HIP(hipGetLastError());
  add_round_published(r, count, second, first_key_out);
  return APEX_OK;
}

// The held step and the masses of `count` new keys whose payload is in place (apex_replay_add_publish)
// in one launch.  APEX_ERR_NOT_READY - with nothing enqueued - if there is no held step.
int issue_held_step_with_leaves(apex_replay *r, HeldStep *h, uint64_t count, const float *prio,
                                uint64_t *first_key_out, hipStream_t stream)
{
  if (!h->valid || !count || !prio) return APEX_ERR_NOT_READY;
  if ((r->tail - r->head) + count > r->cfg.max_slots) return APEX_ERR_FULL;
  const uint64_t second = r->second_words();
  h->a.leaves = AddLeavesArgs{r->tv, second, r->state(), count, prio, r->qp};
  h->valid = false;
  launch_step(h->a, h->rp, h->a.k + blocks_for(count, kStepThreads), kStepThreads, stream, kLeavesRide);
  APEX_HIP(hipGetLastError());
  add_round_published(r, count, second, first_key_out);
  return APEX_OK;
}

int fused_steps(apex_replay *r, uint32_t n, uint32_t k, float beta, const uint64_t *rnd, const float *new_prio,
                const apex_batch_buffers_t *sets, uint32_t depth, uint32_t first_set, HeldStep *hold,
                uint32_t codec_raw_bytes, hipStream_t stream)
{
  // The same gate as apex_replay_sample, from the host mirror and before anything is enqueued: a draw from an
  // empty tree has no defined result (every stratum has width 0), and the learner waits for a minimum fill.
  const uint64_t size = r->tail - r->head;
  if (size < r->cfg.min_size_to_sample) return APEX_ERR_NOT_READY;
  if (size == 0) return APEX_ERR_EMPTY;
  const auto idx = [&](uint32_t i) { return (first_set + i) % depth; };
  const auto set = [&](uint32_t i) -> const apex_batch_buffers_t & { return sets[idx(i)]; };
  const apex_batch_buffers_t &b0 = set(0);
  const RowPieces rp = step_pieces(r, depth, sets);
  if (new_prio) {
    // Launch i reads one copy of the tree and writes the other; the first draw is launch "-1" of that
    // scheme (it reads the first copy and writes the first batch's changes into the second), so both
    // copies have to be equal before it.
    if (r->second_version != r->tree_version)
      copy_words_kernel<<<dim3(2048), dim3(256), 0, stream>>>(r->tv2.level[0], r->tv.level[0], r->geo.tree_words);
    StepArgs a{};
    a.k = k;
    a.qp = r->qp;
    a.st = r->state();
    a.wr = r->tv2;
    a.next.tv = r->tv;
    a.next.st = r->state();
    a.next.k = k;
    a.next.rnd = rnd;
    a.next.key_out = b0.key;
    a.next.slot_out = b0.slot;
    a.next.mass = b0.mass;
    a.next_prio = new_prio;
    a.next_dq = r->stepq(idx(0));
    launch_step(a, rp, k, kWave, stream);
    APEX_HIP(hipGetLastError());
  } else {
    const int rc = sample_begin_impl(r, 1, k, rnd, b0.key, b0.slot, b0.mass, nullptr, nullptr, nullptr, stream);
    if (rc != APEX_OK) return rc;
  }
  for (uint32_t i = 0; i < n; ++i) {
    const apex_batch_buffers_t &b = set(i);
    const TreeView &rd = (new_prio && !(i & 1)) ? r->tv2 : r->tv;
    const TreeView &wr = (new_prio && !(i & 1)) ? r->tv : r->tv2;
    StepArgs a{};
    a.src = r->obs();
    a.dst = static_cast<uint8_t *>(b.obs);
    a.row_bytes = r->cfg.obs_bytes;
    a.vecs_per_row = (uint32_t)pieces_per_row(rp, a.row_bytes);
    if (codec_raw_bytes) {  // rows decoded on their way out: the set's obs buffer is [k, raw bytes]
      a.codec = codec_shape(codec_raw_bytes);
      a.vecs_per_row = codec_raw_bytes / 16;
    }
    a.act = r->act();
    a.act_bytes = r->cfg.act_bytes;
    a.ret = r->ret();
    a.gacc = r->gacc();
    a.act_out = static_cast<uint8_t *>(b.act);
    a.ret_out = b.ret;
    a.gacc_out = b.gacc;
    a.k = k;
    a.slot = b.slot;
    a.dq = new_prio ? r->stepq(idx(i)) : nullptr;
    a.qp = r->qp;
    a.wr = wr;
    a.st = r->state();
    a.wa = WeightArgs{b.mass, b.weight, k, beta};
    a.next.tv = rd;
    a.next.st = r->state();
    a.next.k = k;
    if (i + 1 < n) {
      const apex_batch_buffers_t &nb = set(i + 1);
      a.next.rnd = rnd + (uint64_t)(i + 1) * k;
      a.next.key_out = nb.key;
      a.next.slot_out = nb.slot;
      a.next.mass = nb.mass;
      // the small columns of batch i+1 are gathered by the launch that copies its rows
      if (new_prio) {
        a.next_prio = new_prio + (uint64_t)(i + 1) * k;
        a.next_dq = r->stepq(idx(i + 1));
      }
    }
    if (hold && i + 1 == n) {  // issued by the caller's next call, perhaps together with an add round
      hold->valid = true;
      hold->a = a;
      hold->rp = rp;
    } else {
      launch_step(a, rp, k, kStepThreads, stream);
    }
  }
  // (every change has now been applied to both copies)
  if (new_prio) r->second_version = ++r->tree_version;
  APEX_HIP(hipGetLastError());
  return APEX_OK;
}

// Whether n steps of num_batches x k samples go that way: several batches, or one that is too large for a workgroup per
// sample, of rows that sample_kernel gathers, with room for their changes in the scratch region, and
//   - up to kMultiStepMaxBatches: a drawn sample is held against those of every later batch.  Two launches per step / one,
//     us per step, 2^21 slots: 128 x 64 15.7 / 13.0, 160 x 32 13.1 / 11.9, 192 x 32 13.6 / 13.8, 256 x 32 14.3 / 17.3,
//     1024 x 32 30.2 / 106;
//   - up to kMultiStepMaxPerTopNode samples per node of the top level: every sample adds to it twice, and up to four
//     neighbours together, where two launches add up whole waves of 64.  8192 samples (16 x 512) on 74 nodes 13.7 / 14.8,
//     on 128 13.3 / 11.0, 16,384 (32 x 512) on 128 16.3 / 19.3, on 256 14.9 / 12.6, on 512 16.3 / 12.2.
// Neighbours are added up (add_four) from kMergePerTopNode samples per top node on: without it 4 x 512 on 74 nodes take 12.4
// us per step, so 7.2; 16 x 512 on 512 nodes 8.4 and 7.7; 2 x 512 on 512 6.2, and 6.6 with it.  (All of them before prefix sums
// took two instructions a step: one launch is 0.4 to 0.8 us shorter since, 16 x 512 on 512 nodes 7.1, 2 x 512 5.4.)
constexpr uint32_t kMultiStepMaxBatches = 160, kMultiStepMaxPerTopNode = 64, kMergePerTopNode = 8;

// The second copy of the tree may have to be brought up to date first, at some 5 TB/s.  A call that finds it behind does so
// where its steps win that back.  n steps, join, update_priorities of 64, fork, two launches per step / refresh and one launch,
// us (2 x 512): 2^20 slots n = 1 46 / 51; 2^21 n = 4 75 / 65; 2^22 n = 4 76 / 70; 2^23 n = 8 134 / 110; 2^24 n = 8 134 / 134.
// By ratios the line stands where calls of four steps (2^22 - 2^23) and of eight (2^24) break even.  Calls of one or two
// steps that alternate with plain updates break even at 2^18 and 2^21 already and lose up to 10 % between there and the line
// (2^21, 2^22): they are let through because declining would last.  Two launches per step leave the copy behind, so a learner
// that makes one plain update and then single steps only would never come back; let through, it refreshes the copy once.
constexpr uint64_t kTreeWordsPerStep = 2u << 20;

bool multi_steps_fit(const apex_replay *r, uint32_t n, uint32_t num_batches, uint32_t k, uint32_t depth)
{
  const uint64_t samples = (uint64_t)num_batches * k;
  if ((num_batches == 1 && k <= kStepMaxK) || depth < 2 || depth * samples > (uint64_t)kStepSets * kStepMaxK) return false;
  if (num_batches > kMultiStepMaxBatches || samples > (uint64_t)kMultiStepMaxPerTopNode * r->tv.n_top) return false;
  if (r->second_version != r->tree_version && (n + 1) * kTreeWordsPerStep < 2 * r->geo.tree_words) return false;
  return gather_in_draw(r);
}

// n learner steps of num_batches x k each whose new priorities are known, in strict order, as one launch per step and one
// for the first draw: see multi_step_kernel.
int multi_steps(apex_replay *r, uint32_t n, uint32_t num_batches, uint32_t k, float beta, const uint64_t *rnd,
                const float *new_prio, const apex_batch_buffers_t *sets, uint32_t depth, uint32_t first_set,
                hipStream_t stream)
{
  const uint64_t size = r->tail - r->head;  // the gate of apex_replay_sample, before anything is enqueued
  if (size < r->cfg.min_size_to_sample) return APEX_ERR_NOT_READY;
  if (size == 0) return APEX_ERR_EMPTY;
  const uint32_t samples = num_batches * k;
  if (r->second_version != r->tree_version)
    copy_words_kernel<<<dim3(2048), dim3(256), 0, stream>>>(r->tv2.level[0], r->tv.level[0], r->geo.tree_words);
  const auto changes = [&](uint32_t set) { return r->stepq(0) + (uint64_t)set * samples; };
  for (uint32_t i = 0; i <= n; ++i) {  // launch i gathers step i - 1 and draws step i
    MultiStepArgs a{};
    a.samples = samples;
    a.batches = num_batches;
    a.qp = r->qp;
    a.st = r->state();
    a.wr = i & 1 ? r->tv : r->tv2;
    uint32_t gather_wgs = 0;
    if (i > 0) {
      const uint32_t set = (first_set + i - 1) % depth;
      const apex_batch_buffers_t &b = sets[set];
      a.g = GatherArgs{r->act(), r->cfg.act_bytes, r->ret(), r->gacc(), static_cast<uint8_t *>(b.act), b.ret, b.gacc,
                       r->obs(), r->cfg.obs_bytes, static_cast<uint8_t *>(b.obs)};
      a.slot = b.slot;
      a.dq = changes(set);
      a.wa = WeightArgs{b.mass, b.weight, k, beta};
      gather_wgs = blocks_for(samples, kMultiStepRows);
      a.weight_wgs_per_batch = blocks_for(k, 512);
      a.weight_wgs = num_batches * a.weight_wgs_per_batch;
    }
    if (i < n) {
      const uint32_t set = (first_set + i) % depth;
      const apex_batch_buffers_t &b = sets[set];
      a.next.tv = i & 1 ? r->tv2 : r->tv;
      a.next.st = r->state();
      a.next.k = k;
      a.next.rnd = rnd + (uint64_t)i * samples;
      a.next.key_out = b.key;
      a.next.slot_out = b.slot;
      a.next.mass = b.mass;
      a.next_k_div = make_fast_div(k);
      a.next_prio = new_prio + (uint64_t)i * samples;
      a.next_dq = changes(set);
      a.draw_wgs_per_batch = blocks_for(k, kMultiStepRows);
      a.draw_wgs = num_batches * a.draw_wgs_per_batch;
    }
    // The weights of large batches take longer than a gather and go ahead of it, 512 to a workgroup: one batch of 4096 of 2^21
    // slots 9.8 us per step with one workgroup behind the gather, 7.7 so, of 16,384 38 and 14.  (Those of many small ones
    // would hold the gather up: 128 x 16 of 2^20 9.3 us, and 9.9 with them ahead.)
    const bool ahead = a.weight_wgs_per_batch > 1;
    a.gather_first = a.draw_wgs + (ahead ? a.weight_wgs : 0);
    a.weight_first = a.draw_wgs + (ahead ? 0 : gather_wgs);
    const dim3 grid(a.draw_wgs + gather_wgs + a.weight_wgs), block(kMultiStepThreads);
    const bool wide = r->tv.n_top > 512, merge = samples > kMergePerTopNode * r->tv.n_top;
    if (wide && merge) multi_step_kernel<true, true><<<grid, block, 0, stream>>>(a);
    else if (wide) multi_step_kernel<true, false><<<grid, block, 0, stream>>>(a);
    else if (merge) multi_step_kernel<false, true><<<grid, block, 0, stream>>>(a);
    else multi_step_kernel<false, false><<<grid, block, 0, stream>>>(a);
  }
  r->second_version = ++r->tree_version;  // every change is in both copies
  APEX_HIP(hipGetLastError());
  return APEX_OK;
}

int check_finish_args(const apex_replay *r, uint32_t num_batches, uint32_t k, float beta, const uint32_t *slot,
                      const uint64_t *mass, const float *weight_out)
{
  if (!r || !num_batches || !k || !slot || !(beta >= 0.0f) || !(beta <= 1.0f)) return APEX_ERR_INVALID_ARG;
  if (weight_out && !mass) return APEX_ERR_INVALID_ARG;
  if (num_batches > APEX_MAX_BATCHES_PER_CALL || (uint64_t)num_batches * k > APEX_MAX_SAMPLES_PER_CALL)
    return APEX_ERR_TOO_LARGE;
  return APEX_OK;
}

}  // namespace

int apex_replay_sample_finish(apex_replay_t *r, uint32_t num_batches, uint32_t k, float beta, const uint32_t *slot,
                              const uint64_t *mass, float *weight_out, void *obs_out, void *hip_stream)
{
  const int rc = check_finish_args(r, num_batches, k, beta, slot, mass, weight_out);
  if (rc != APEX_OK) return rc;
  return finish_impl(r, num_batches, k, beta, slot, mass, weight_out, obs_out, 0, nullptr, nullptr,
                     static_cast<hipStream_t>(hip_stream));
}

int apex_replay_sample_finish_update(apex_replay_t *r, uint32_t num_batches, uint32_t k, float beta,
                                     const uint32_t *slot, const uint64_t *mass, float *weight_out, void *obs_out,
                                     uint64_t m, const uint64_t *key, const float *prio, void *hip_stream)
{
  const int rc = check_finish_args(r, num_batches, k, beta, slot, mass, weight_out);
  if (rc != APEX_OK) return rc;
  if (m && !prio) return APEX_ERR_INVALID_ARG;
  if (m >= 0xffffffffull) return APEX_ERR_TOO_LARGE;
  if (m && !key) return APEX_ERR_INVALID_ARG;
  return finish_impl(r, num_batches, k, beta, slot, mass, weight_out, obs_out, m, key, prio,
                     static_cast<hipStream_t>(hip_stream));
}

int apex_replay_sample_finish_writeback(apex_replay_t *r, uint32_t num_batches, uint32_t k, float beta,
                                        const uint64_t *key, const uint32_t *slot, const uint64_t *mass,
                                        float *weight_out, void *obs_out, const float *prio, void *hip_stream)
{
  const int rc = check_finish_args(r, num_batches, k, beta, slot, mass, weight_out);
  if (rc != APEX_OK) return rc;
  if (!key || !mass || !prio) return APEX_ERR_INVALID_ARG;
  return finish_impl(r, num_batches, k, beta, slot, mass, weight_out, obs_out, (uint64_t)num_batches * k, key, prio,
                     static_cast<hipStream_t>(hip_stream), /*same_batch=*/true);
}

int apex_replay_sample(apex_replay_t *r, uint32_t num_batches, uint32_t k, float beta, const uint64_t *rnd,
                       uint64_t *key_out, uint32_t *slot_out, float *weight_out, void *obs_out, void *act_out,
                       float *ret_out, float *gacc_out, void *hip_stream)
{
  if (!r || !(beta >= 0.0f) || !(beta <= 1.0f)) return APEX_ERR_INVALID_ARG;
  const bool apart = obs_out && weight_out && num_batches == 1 && k > kGatherApartAboveK && k <= kWeightsInDrawMaxK &&
                     r->cfg.obs_bytes <= kGatherApartBytes;
  if (!obs_out || (gather_in_draw(r) && !apart) || sample_by_rows(r->cfg.obs_bytes, num_batches, k))
    return sample_in_one(r, num_batches, k, beta, rnd, key_out, slot_out, r->mass(), weight_out, obs_out, act_out, ret_out,
                         gacc_out, /*claim=*/false, static_cast<hipStream_t>(hip_stream));
  const int rc = apex_replay_sample_begin(r, num_batches, k, rnd, key_out, slot_out, r->mass(), act_out, ret_out,
                                          gacc_out, hip_stream);
  if (rc != APEX_OK) return rc;
  if (!weight_out && !obs_out) return APEX_OK;
  return apex_replay_sample_finish(r, num_batches, k, beta, slot_out, r->mass(), weight_out, obs_out, hip_stream);
}

int apex_replay_sample_noalloc(apex_replay_t *r, uint32_t num_batches, uint32_t k, float beta, const uint64_t *rnd,
                               uint64_t *key_out, uint32_t *slot_out, float *weight_out, void *obs_out, void *act_out,
                               float *ret_out, float *gacc_out, void *hip_stream)
{
  if (!r || !(beta >= 0.0f) || !(beta <= 1.0f)) return APEX_ERR_INVALID_ARG;
  if (num_batches && k && (uint64_t)num_batches * k > APEX_NOALLOC_MAX_SAMPLES) return APEX_ERR_TOO_LARGE;
  uint64_t *const mass = static_scratch_ptr();  // this GPU's copy; every entry the weights read is written by the draw
  if (!mass) return APEX_ERR_HIP;
  const int rc = apex_replay_sample_begin(r, num_batches, k, rnd, key_out, slot_out, mass, act_out, ret_out, gacc_out,
                                          hip_stream);
  if (rc != APEX_OK) return rc;
  if (!weight_out && !obs_out) return APEX_OK;
  return apex_replay_sample_finish(r, num_batches, k, beta, slot_out, mass, weight_out, obs_out, hip_stream);
}

int apex_replay_gather(apex_replay_t *r, uint64_t count, const uint32_t *slot, void *obs_out, void *act_out,
                       float *ret_out, float *gacc_out, void *hip_stream)
{
  if (!r || (count && !slot)) return APEX_ERR_INVALID_ARG;
  if (count > APEX_MAX_SAMPLES_PER_CALL) return APEX_ERR_TOO_LARGE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const RowMap by_slot{slot, nullptr, 0, {}};
  const RowMap ident{nullptr, nullptr, 0, {}};
  int rc;
  if (obs_out && (rc = launch_copy(r->obs(), by_slot, obs_out, ident, count, r->cfg.obs_bytes, stream)) != APEX_OK) return rc;
  if (act_out && (rc = launch_copy(r->act(), by_slot, act_out, ident, count, r->cfg.act_bytes, stream)) != APEX_OK) return rc;
  if (ret_out && (rc = launch_copy(r->ret(), by_slot, ret_out, ident, count, 4, stream)) != APEX_OK) return rc;
  if (gacc_out && (rc = launch_copy(r->gacc(), by_slot, gacc_out, ident, count, 4, stream)) != APEX_OK) return rc;
  return APEX_OK;
}

int apex_replay_update_priorities(apex_replay_t *r, uint64_t m, const uint64_t *key, const float *prio,
                                  void *hip_stream)
{
  if (!r || (m && (!key || !prio))) return APEX_ERR_INVALID_ARG;
  if (m >= 0xffffffffull) return APEX_ERR_TOO_LARGE;
  if (m == 0) return APEX_OK;
  return launch_update(r, m, key, prio, static_cast<hipStream_t>(hip_stream));
}

int apex_replay_update_from_q(apex_replay_t *r, uint64_t m, const uint64_t *key, uint32_t A, const float *q_taken,
                              const float *q_online_next, const float *q_target_next, float *prio_out,
                              void *hip_stream)
{
  if (!r || !A || (m && (!key || !q_taken || !q_online_next || !q_target_next))) return APEX_ERR_INVALID_ARG;
  if (m >= 0xffffffffull) return APEX_ERR_TOO_LARGE;
  if (m == 0) return APEX_OK;
  const QSource qs{q_taken, q_online_next, q_target_next, A, r->ret(), r->gacc(), prio_out};
  return launch_update(r, m, key, nullptr, static_cast<hipStream_t>(hip_stream), qs);
}

int apex_replay_evict(apex_replay_t *r, uint64_t *evicted_out, void *hip_stream)
{
  if (!r) return APEX_ERR_INVALID_ARG;
  const uint64_t size = r->tail - r->head;
  const uint64_t e = size > r->cfg.capacity ? size - r->cfg.capacity : 0;
  if (evicted_out) *evicted_out = e;
  if (e == 0) return APEX_OK;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const uint64_t second = r->second_words();
  r->tree_changed(second);
  const uint32_t threads = leaves_threads(e);
  evict_leaves_kernel<<<dim3(blocks_for(e, threads)), dim3(threads), 0, stream>>>(EvictLeavesArgs{r->tv, second, r->state(), e});
  APEX_HIP(hipGetLastError());
  r->head += e;
  return APEX_OK;
}

int apex_replay_resync(apex_replay_t *r, void *hip_stream)
{
  if (!r) return APEX_ERR_INVALID_ARG;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  DeviceState st;
  APEX_HIP(hipMemcpyAsync(&st, r->state(), sizeof st, hipMemcpyDeviceToHost, stream));
  APEX_HIP(hipStreamSynchronize(stream));
  r->head = st.head;
  r->tail = st.tail;
  return APEX_OK;
}

int apex_replay_stats(apex_replay_t *r, apex_replay_stats_t *out, void *hip_stream)
{
  if (!r || !out) return APEX_ERR_INVALID_ARG;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  DeviceState st;
  APEX_HIP(hipMemcpyAsync(&st, r->state(), sizeof st, hipMemcpyDeviceToHost, stream));
  // root = sum of the top level (at most kTopMax words)
  static thread_local uint64_t top[kTopMax];
  APEX_HIP(hipMemcpyAsync(top, r->tv.level[r->tv.nlev - 1], (size_t)r->tv.n_top * 8, hipMemcpyDeviceToHost, stream));
  APEX_HIP(hipStreamSynchronize(stream));
  uint64_t root = 0;
  for (uint32_t i = 0; i < r->tv.n_top; ++i) root += top[i];
  out->size = st.tail - st.head;
  out->head = st.head;
  out->tail = st.tail;
  out->root = root;
  out->n_stale_dropped = st.n_stale;
  out->n_clamped = st.n_clamped;
  return APEX_OK;
}

}  // extern "C"

#include "pipeline.inc.hpp"
#include "evict_prio.inc.hpp"
#include "codec.inc.hpp"
