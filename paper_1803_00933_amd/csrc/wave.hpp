// Wavefront-wide helpers for gfx950 (64 lanes).  All kernels in this library launch 1-D blocks
// whose size is a multiple of 64, so lane = threadIdx.x & 63.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace apex {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Prefix sums with data-parallel primitives (no LDS traffic): in every step a lane adds the value that the DPP control routes to
// it, or 0 where it routes none.  In assembly because the two halves of a 64-bit sum can take their operand through the control
// themselves, with the carry between them: two instructions a step and a wait, where the compiler moves both halves through the
// control first, into registers that it has cleared, and adds twice (six and a wait).
// The waits, which nobody adds to assembly, are the compiler's own on this target: two wait states between an instruction that
// writes vcc and one that reads it, the carry included, and two between the write of a register and its read through a DPP
// control.  The first keeps a step's halves apart and brings the second with it; those at both ends are for what the compiler
// puts before and behind.
#define APEX_SCAN_STEP(ctrl)                             \
  "v_add_co_u32_dpp %0, vcc, %0, %0 " ctrl "\n\t"        \
  "s_nop 1\n\t"                                          \
  "v_addc_co_u32_dpp %1, vcc, %1, %1, vcc " ctrl "\n\t"
#define APEX_SCAN_ROW                                                       \
  "s_nop 1\n\t"                                                             \
  APEX_SCAN_STEP("row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0")       \
  APEX_SCAN_STEP("row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:0")       \
  APEX_SCAN_STEP("row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:0")       \
  APEX_SCAN_STEP("row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:0")

// Inclusive prefix sum inside each 16-lane row of the wave, modulo 2^64.  Called by all 64 lanes.
__device__ __forceinline__ uint64_t row_inclusive_scan(uint64_t v)
{
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  asm volatile(APEX_SCAN_ROW "s_nop 1" : "+v"(lo), "+v"(hi) : : "vcc");
  return ((uint64_t)hi << 32) | lo;
}

// Inclusive prefix sum of one uint64 per lane over the wave: inside the rows, then the last lane of row 0 (2) is added to row 1
// (3), then lane 31 to rows 2 and 3.  Called by all 64 lanes.
__device__ __forceinline__ uint64_t wave_inclusive_scan(uint64_t v)
{
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  asm volatile(APEX_SCAN_ROW
               APEX_SCAN_STEP("row_bcast:15 row_mask:0xa bank_mask:0xf")
               APEX_SCAN_STEP("row_bcast:31 row_mask:0xc bank_mask:0xf")
               "s_nop 1"
               : "+v"(lo), "+v"(hi)
               :
               : "vcc");
  return ((uint64_t)hi << 32) | lo;
}
#undef APEX_SCAN_ROW
#undef APEX_SCAN_STEP

// One step of a minimum with data-parallel primitives: lanes to which the DPP control word routes no value keep theirs.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ float dpp_min_step(float v)
{
  const int x = (int)__float_as_uint(v);
  return fminf(v, __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(x, x, kCtrl, kRowMask, 0xf, false)));
}

// Minimum over the wave, the same in every lane.  The minimum of no NaN.
__device__ __forceinline__ float wave_min(float v)
{
  v = dpp_min_step<0x111, 0xf>(v);  // row_shr:1, the steps of wave_inclusive_scan
  v = dpp_min_step<0x112, 0xf>(v);
  v = dpp_min_step<0x114, 0xf>(v);
  v = dpp_min_step<0x118, 0xf>(v);
  v = dpp_min_step<0x142, 0xa>(v);
  v = dpp_min_step<0x143, 0xc>(v);
  return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), kWave - 1));
}

// Device-scope atomics on the tree.  The eight XCDs of the chip have separate L2 caches, so
// these must be (and are) performed at agent scope.
__device__ __forceinline__ void atomic_add_u64(uint64_t *p, uint64_t v)
{
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace apex
