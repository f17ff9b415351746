// Lossless block codec of stored observations (Section 4.1: observations are kept compressed in the
// replay memory and decompressed as batches are fetched): encode on the way into the ring, decode on
// the way out.  Included by apex_replay.hip (one translation unit), after the plain entry points.
//
// A row of raw_bytes = 64 * nb bytes is cut into nb blocks of 64 bytes.  A block whose bytes are all
// equal is kept as that byte, any other block as it is, and every part has a fixed place, so that
// nothing has to be looked up before it can be fetched.  Encoded row, little-endian:
//   0        mask, bit b set iff block b is kept as it is: ceil(nb/64) u64 words, zero-padded to 16 bytes (M)
//   M        one byte per block: the byte of block b if it is not kept as it is (else unspecified); nb bytes,
//            rounded up to a multiple of 16 (V)
//   M + V    the image of the row: bytes [64 b, 64 b + 64) hold block b if it is kept as it is (else unspecified)
// The stride of the store (obs_bytes of the memory) must be at least M + V + 64 * nb.  An encoder writes,
// and a decoder that looks at the mask first reads, only the parts that carry data.

namespace apex {

constexpr uint32_t kCodecThreads = 512;
constexpr uint32_t kCodecUnroll = 4;

// The value of the lane that kPerm, a permutation of the four lanes of a quad, names.
template <int kPerm>
__device__ __forceinline__ uint32_t quad_swap(uint32_t x)
{
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kPerm, 0xf, 0xf, true);
}

// Run `run` (64 pieces of 16 bytes, one per lane of the wave) of a row goes into the encoded row d; nothing does of a run
// beyond its end.  The four lanes of a block agree on whether it is flat with two exchanges and a ballot; every fourth bit
// of it is 16 bits of the mask.
__device__ __forceinline__ void encode_run(uint8_t *d, const CodecShape &c, uint32_t run, const u32x4 &t)
{
  const uint32_t lane = lane_id(), nvec = c.raw_bytes / 16, v = run * kWave + lane, x = t.x;
  // a block is flat if each of its four lanes holds one byte throughout, the same as two of the others hold
  const bool even = x == (x & 0xffu) * 0x01010101u && t.y == x && t.z == x && t.w == x;
  const bool same = quad_swap<0xb1>(x) == x && quad_swap<0x4e>(x) == x;
  uint64_t flat = __ballot(even && same);
  flat &= flat >> 1;
  flat &= flat >> 2;
  const uint64_t kept = ~flat & __ballot(v < nvec) & 0x1111111111111111ull;  // one bit per block, at every fourth place
  uint64_t bits = kept;
  bits = (bits | bits >> 3) & 0x0303030303030303ull;
  bits = (bits | bits >> 6) & 0x000f000f000f000full;
  bits = (bits | bits >> 12) & 0x000000ff000000ffull;
  bits = (bits | bits >> 24) & 0xffffull;
  if (lane == 0 && v < nvec) reinterpret_cast<uint16_t *>(d)[run] = (uint16_t)bits;
  if (kept >> (lane & ~3u) & 1)
    __builtin_nontemporal_store(t, reinterpret_cast<u32x4 *>(d + c.image_off) + v);
  else if (v < nvec && (v & 3) == 0)
    d[c.flat_off + v / 4] = (uint8_t)x;
}

// One workgroup per row, a lane per 16-byte piece, in row order (loads and stores as a plain copy makes them).  No LDS,
// no barrier.  18,000 rows of 28,224 bytes, 80 % of the blocks flat: 125 us (4.9 TB/s).
__global__ __launch_bounds__(kCodecThreads) void codec_encode_rows_kernel(const uint8_t *__restrict__ src,
                                                                         uint8_t *__restrict__ ring, RowMap to,
                                                                         uint64_t ring_stride, CodecShape c)
{
  const uint64_t i = blockIdx.x;
  const u32x4 *s = reinterpret_cast<const u32x4 *>(src + i * c.raw_bytes);
  uint8_t *d = ring + map_row(to, i) * ring_stride;
  const uint32_t tid = threadIdx.x, nvec = c.raw_bytes / 16;
  const uint32_t runs = (nvec + kWave - 1) / kWave;  // 16-bit pieces of the mask that hold blocks
  for (uint32_t g = runs + tid; g < c.flat_off / 2; g += kCodecThreads) reinterpret_cast<uint16_t *>(d)[g] = 0;
  for (uint32_t v0 = 0; v0 < nvec; v0 += kCodecUnroll * kCodecThreads) {
    u32x4 t[kCodecUnroll];
#pragma unroll
    for (int u = 0; u < (int)kCodecUnroll; ++u) {
      const uint32_t v = v0 + u * kCodecThreads + tid;
      t[u] = v < nvec ? __builtin_nontemporal_load(s + v) : u32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int u = 0; u < (int)kCodecUnroll; ++u) {
      // a run beyond the row writes nothing (a branch around it cost 1 - 2 %)
      encode_run(d, c, (v0 + u * kCodecThreads + tid) / kWave, t[u]);
    }
  }
}

// Short rows: a workgroup takes 8 consecutive runs, whatever rows they belong to, a wave two of them.  A workgroup per row
// is mostly idle lanes there (18,000 rows of 640 bytes, 80 % flat: 51 us, so 8; 3,000 of 4,160 bytes 12.4 and 7.5; 18,000 of
// 6,400 bytes 55 and 31).
constexpr uint32_t kEncodeWaves = 4, kEncodeRuns = 2, kEncodeRunsPerWorkgroup = kEncodeWaves * kEncodeRuns;
__global__ __launch_bounds__(kEncodeWaves * kWave) void codec_encode_runs_kernel(const uint8_t *__restrict__ src,
                                                                                uint8_t *__restrict__ ring, RowMap to,
                                                                                uint64_t ring_stride, CodecShape c,
                                                                                uint32_t runs_per_row, uint32_t total_runs)
{
  const uint32_t lane = lane_id(), nvec = c.raw_bytes / 16;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const uint32_t first = blockIdx.x * kEncodeRunsPerWorkgroup + wave * kEncodeRuns;
  if (first >= total_runs) return;
  uint32_t row[kEncodeRuns], run[kEncodeRuns];
  u32x4 t[kEncodeRuns];
#pragma unroll
  for (int u = 0; u < (int)kEncodeRuns; ++u) {
    const uint32_t r = min(first + u, total_runs - 1);  // a run beyond the last is read as the last, and not written
    row[u] = r / runs_per_row;
    run[u] = r - row[u] * runs_per_row;
    t[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + (uint64_t)row[u] * c.raw_bytes) +
                                      min(run[u] * kWave + lane, nvec - 1));
  }
#pragma unroll
  for (int u = 0; u < (int)kEncodeRuns; ++u) {
    if (first + u >= total_runs) return;
    uint8_t *const d = ring + map_row(to, row[u]) * ring_stride;
    encode_run(d, c, run[u], t[u]);
    if (run[u] + 1 == runs_per_row && runs_per_row + lane < c.flat_off / 2)  // the rest of the mask (at most 7 pieces)
      reinterpret_cast<uint16_t *>(d)[runs_per_row + lane] = 0;
  }
}

// One workgroup per output row, a lane per 16-byte piece, in row order.  The word of the mask first (the 64
// lanes of a wave share it), then only what carries data is read: the piece, or its block's byte.
__global__ __launch_bounds__(kCodecThreads) void codec_decode_rows_kernel(const uint8_t *__restrict__ ring,
                                                                         const uint32_t *__restrict__ slot,
                                                                         uint64_t ring_stride,
                                                                         uint8_t *__restrict__ out, CodecShape c)
{
  const uint64_t i = blockIdx.x;
  const uint8_t *e = ring + (uint64_t)slot[i] * ring_stride;
  const uint64_t *mask = reinterpret_cast<const uint64_t *>(e);
  u32x4 *o = reinterpret_cast<u32x4 *>(out + i * c.raw_bytes);
  const uint32_t tid = threadIdx.x, nvec = c.raw_bytes / 16;
  for (uint32_t v0 = 0; v0 < nvec; v0 += kCodecUnroll * kCodecThreads) {
    uint64_t word[kCodecUnroll];
#pragma unroll
    for (int u = 0; u < (int)kCodecUnroll; ++u) {
      const uint32_t v = v0 + u * kCodecThreads + tid;
      word[u] = v < nvec ? mask[v >> 8] : 0;
    }
    u32x4 t[kCodecUnroll];
    uint32_t byte[kCodecUnroll];
#pragma unroll
    for (int u = 0; u < (int)kCodecUnroll; ++u) {
      const uint32_t v = v0 + u * kCodecThreads + tid, b = v / 4;
      t[u] = u32x4{0, 0, 0, 0};
      byte[u] = 0;
      if (v < nvec) {
        if (word[u] >> (b & 63) & 1)
          t[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(e + c.image_off) + v);
        else
          byte[u] = e[c.flat_off + b];
      }
    }
#pragma unroll
    for (int u = 0; u < (int)kCodecUnroll; ++u) {
      const uint32_t v = v0 + u * kCodecThreads + tid, b = v / 4;
      if (v < nvec) {
        const uint32_t x = byte[u] * 0x01010101u;
        __builtin_nontemporal_store((word[u] >> (b & 63) & 1) ? t[u] : u32x4{x, x, x, x}, o + v);
      }
    }
  }
}

}  // namespace apex

extern "C" {

size_t apex_codec_row_bytes(uint32_t raw_bytes)
{
  if (raw_bytes == 0 || raw_bytes % 64) return 0;
  return (size_t)codec_shape(raw_bytes).stride;
}

int apex_replay_add_payload_encoded(apex_replay_t *r, uint64_t count, const void *raw_obs, uint32_t raw_bytes,
                                    const void *act, const float *ret, const float *gacc, void *hip_stream)
{
  if (!r || (count && !raw_obs)) return APEX_ERR_INVALID_ARG;
  const size_t stride = apex_codec_row_bytes(raw_bytes);
  if (!stride || ((uintptr_t)raw_obs & 15) || (r->cfg.obs_bytes & 15)) return APEX_ERR_INVALID_ARG;
  if (stride > r->cfg.obs_bytes) return APEX_ERR_TOO_LARGE;
  if ((r->tail - r->head) + count > r->cfg.max_slots) return APEX_ERR_FULL;
  if (count == 0) return APEX_OK;
  if (count > 0x7ffffff0ull) return APEX_ERR_TOO_LARGE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const RowMap ring{nullptr, &r->state()->tail, r->cfg.max_slots, r->tv.p_div};
  const CodecShape shape = codec_shape(raw_bytes);
  const uint8_t *const src = static_cast<const uint8_t *>(raw_obs);
  const uint32_t runs_per_row = (raw_bytes / 16 + kWave - 1) / kWave;
  const uint64_t runs = count * runs_per_row, blocks = (runs + kEncodeRunsPerWorkgroup - 1) / kEncodeRunsPerWorkgroup;
  // Rows shorter than the runs of a workgroup go packed.  Longer ones are faster that way as well while nothing else runs
  // (18,000 of 28,224 bytes 125 us, packed 117), but beside learner steps they hold these up: 25 steps with such a round,
  // twice, 662 us, packed 683; with rows of 8,192 bytes 449 and 484, with 6,400 bytes 425 and 405, with 3,200 418 and 379.
  // (The grid's lanes are counted in 32 bits.)
  if (runs_per_row < kEncodeRunsPerWorkgroup && blocks * kEncodeWaves * kWave <= 0xffffffffull)
    codec_encode_runs_kernel<<<dim3((uint32_t)blocks), dim3(kEncodeWaves * kWave), 0, stream>>>(
        src, r->obs(), ring, r->cfg.obs_bytes, shape, runs_per_row, (uint32_t)runs);
  else
    codec_encode_rows_kernel<<<dim3((uint32_t)count), dim3(kCodecThreads), 0, stream>>>(src, r->obs(), ring,
                                                                                       r->cfg.obs_bytes, shape);
  APEX_HIP(hipGetLastError());
  if (act || ret || gacc) {
    const PayloadRing pr{r->obs(), r->act(), r->ret(), r->gacc(), r->cfg.obs_bytes, r->cfg.act_bytes};
    return add_small_columns(pr, count, act, ret, gacc, ring, stream);
  }
  return APEX_OK;
}

int apex_replay_gather_decoded(apex_replay_t *r, uint64_t count, const uint32_t *slot, uint32_t raw_bytes,
                               void *obs_out, void *act_out, float *ret_out, float *gacc_out, void *hip_stream)
{
  if (!r || (count && !slot)) return APEX_ERR_INVALID_ARG;
  const size_t stride = apex_codec_row_bytes(raw_bytes);
  if (!stride || ((uintptr_t)obs_out & 15) || (r->cfg.obs_bytes & 15)) return APEX_ERR_INVALID_ARG;
  if (stride > r->cfg.obs_bytes || count > APEX_MAX_SAMPLES_PER_CALL) return APEX_ERR_TOO_LARGE;
  if (count == 0) return APEX_OK;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (obs_out) {
    codec_decode_rows_kernel<<<dim3((uint32_t)count), dim3(kCodecThreads), 0, stream>>>(
        r->obs(), slot, r->cfg.obs_bytes, static_cast<uint8_t *>(obs_out), codec_shape(raw_bytes));
    APEX_HIP(hipGetLastError());
  }
  return apex_replay_gather(r, count, slot, nullptr, act_out, ret_out, gacc_out, hip_stream);
}

}  // extern "C"
