// Pieces shared by the bf16 decode (decode.hip) and the fp32 decode and
// prefill (decode_f32.hip, prefill_f32.hip).
#pragma once

#include "bros_device.h"
#include "bros_kernels.h"

#include <math.h>

namespace bros {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kTileElems = kBlockSize * kHeadDim;   // one (block, KV head) tile
constexpr float kRescaleSlack = 8.0f;               // log2 units: weights stay <= 2^8
constexpr float kNoMax = -1.0e30f;                  // finite "no score yet" reference
constexpr int kMaxRowsLds = 4096;                   // rows whose prefix fits in LDS

typedef unsigned v4u_t __attribute__((ext_vector_type(4)));

// Lane id through an asm the compiler cannot hoist: values derived from it are
// recomputed where they are used instead of being held in registers.
__device__ __forceinline__ int lane_id_here() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {   // round to nearest even
  typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f2_t;
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 b2_t;
  const f2_t f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, b2_t));
}

// Decode row r is sequence r and sees its whole context.
__device__ __forceinline__ void resolve_row(const DecodeArgs& a, int row, int& s, int& ctx) {
  s = row;
  ctx = min(a.ctx_lens[s], a.max_ctx);
  ctx = min(ctx, a.max_blocks_per_seq * kBlockSize);
}

hipError_t launch_decode_f32(const DecodeArgs& a, int group, hipStream_t stream);
// Folds the split partials of every row whose context took more than one split of a.split_blocks blocks.
hipError_t launch_f32_merge(const DecodeArgs& a, hipStream_t stream);

}  // namespace bros
