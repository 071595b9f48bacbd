// bros_attn_prefill_chunk (bf16) launch on the matrix cores: the unit kernel
// and the merge of split units. The device code (and what it computes) is in
// prefill_device.h.
#include "prefill_device.h"

#include <algorithm>

namespace bros {
namespace pf {

template <int G, bool kOff32, bool kRing>
__global__ __launch_bounds__(kThreads, 2) void prefill_mfma_kernel(PrefillArgs a) {
  BROS_PREFILL_UNIT_LDS
  prefill_unit<G, kOff32, kRing>(a, paired_id(a, blockIdx.x, gridDim.x), s_kring, s_vring, &s_first_bad, s_tbl, s_dir);
}

// Fold the pieces of split units, from the list the prefill grid's first
// workgroup wrote: one workgroup per (split item, KV head, 32 of its 128 rows),
// so that the few units of a call that splits still spread over the chip. Per
// row, with M = max_p m_p (log2 units): o = sum_p 2^(m_p - M) O_p / sum_p
// 2^(m_p - M) l_p. Wave w folds dims 32 w .. 32 w + 31 in the order the pieces
// left them (lane l: row l % 32, four float4 of its dims per piece). Rows of
// unsplit units were written by the prefill kernel itself.
template <int G>
__global__ __launch_bounds__(kThreads) void prefill_merge_kernel(PrefillArgs a) {
  constexpr int QT = kRows / G;
  const int Hkv = a.num_kv_heads;
  const int rg = blockIdx.x & 3;
  const int j = (int)(blockIdx.x >> 2) / Hkv, g = (int)(blockIdx.x >> 2) % Hkv;
  if (j >= load_uniform(a.ws_list, 0)) return;
  const int item = load_uniform(a.ws_list, 1 + 3 * j);
  const int parts = load_uniform(a.ws_list, 2 + 3 * j);
  const int slot0 = load_uniform(a.ws_list, 3 + 3 * j);
  const int tps = a.tiles_per_seq;
  const int s = item / tps, t = item % tps;
  const int q_begin = load_uniform(a.cu_q, s);
  const int n = load_uniform(a.cu_q, s + 1) - q_begin;
  if (q_begin < 0 || n <= 0 || q_begin + n > a.num_q_tokens || t * QT >= n) return;   // (never split)
  const int dt = wave_id_uniform();
  const int lane = threadIdx.x & (kWave - 1);
  const int r = 32 * rg + (lane & 31);
  const size_t row0 = ((size_t)slot0 * Hkv + g) * kRows;   // workspace row of part 0, unit row 0
  const size_t pstride = (size_t)Hkv * kRows;              // workspace rows from one part to the next
  const float2* ml = reinterpret_cast<const float2*>(a.ws_ml) + row0 + r;
  const float4* po = reinterpret_cast<const float4*>(a.ws_o + (row0 + 32 * rg) * kHeadDim) + 4 * dt * kWave + lane;
  float m = -INFINITY;
#pragma unroll 4
  for (int p = 0; p < parts; ++p) m = fmaxf(m, ml[p * pstride].x);
  float l = 0.0f;
  float4 acc[4];
#pragma unroll
  for (int jq = 0; jq < 4; ++jq) acc[jq] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 4
  for (int p = 0; p < parts; ++p) {
    const float2 x = ml[p * pstride];
    const float w = fast_exp2(x.x - m);
    l = fmaf(x.y, w, l);
#pragma unroll
    for (int jq = 0; jq < 4; ++jq) {
      const float4 v = po[p * pstride * (kHeadDim / 4) + jq * kWave];
      acc[jq].x = fmaf(v.x, w, acc[jq].x);
      acc[jq].y = fmaf(v.y, w, acc[jq].y);
      acc[jq].z = fmaf(v.z, w, acc[jq].z);
      acc[jq].w = fmaf(v.w, w, acc[jq].w);
    }
  }
  const int qrow = t * QT + r % QT;
  if (qrow >= n) return;
  const float inv = l > 0.0f ? 1.0f / l : 0.0f;
  uint16_t* out = static_cast<uint16_t*>(a.out) + ((size_t)(q_begin + qrow) * a.num_q_heads + g * G + r / QT) * kHeadDim;
#pragma unroll
  for (int jq = 0; jq < 4; ++jq) {
    uint2 o2;
    o2.x = pack2_bf16(acc[jq].x * inv, acc[jq].y * inv);
    o2.y = pack2_bf16(acc[jq].z * inv, acc[jq].w * inv);
    *reinterpret_cast<uint2*>(out + 32 * dt + 8 * jq + 4 * (lane >> 5)) = o2;
  }
}

// Compute units a split plan spreads over, at most; the workspace holds
// 2 x this many (split piece, KV head) partials.
constexpr int kMaxPrefillCus = 512;

// The longest context of a call does not fit the LDS copy of a whole table.
bool prefill_needs_ring(int32_t max_ctx, int32_t max_blocks_per_seq) {
  return max_ctx > kPrefillWholeTableCtx && max_blocks_per_seq > kMaxTableLds;
}

template <int G>
hipError_t launch_group(PrefillArgs a, int num_units, hipStream_t stream) {
  // Split only when the units leave compute units idle: with a unit or more
  // per compute unit, splitting measured no faster (1000 rows on 4000 tokens,
  // 256 units: 96 us whole, 100 split).
  a.num_cus = 0;
  if (a.ws_o != nullptr && num_units / a.num_kv_heads <= kMaxRankItems) {
    int cus = stream_compute_units(stream);
    cus = cus < kMaxPrefillCus ? cus : kMaxPrefillCus;
    // Splitting takes about (1 - units / compute units) off the longest unit
    // (the mean work of a compute unit is what remains), more where units
    // differ; it costs a longer plan, the partials and the merge's launch,
    // 8 us or 16 tiles in all. From 48 tiles on it may save that much however
    // many units there are. 512 rows on 0 / 500 / 1000 / 4000 / 16000 cached
    // tokens, 128 units: whole 17.0 / 25.6 / 33.1 / 79 / 265 us, split 19.7 /
    // 26.1 / 30.3 / 55.6 / 150 us. Over 620 calls with fewer units than compute
    // units (1 to 6 chunks, 0 to 20000 cached tokens, 64 / 8 to 8 / 1 heads)
    // splitting by this rule is 1.58 times as fast as none, 5 % faster than
    // asking the device plan every time, and slower than none, by up to 20 %, in 47
    // (units of unlike length near 48 to 100 tiles).
    const int longest = std::min(a.max_ctx, a.max_blocks_per_seq * kBlockSize) / kKeys;
    if (num_units < cus && (longest >= 48 || (int64_t)longest * (cus - num_units) >= 16 * (int64_t)cus)) a.num_cus = cus;
  }
  // Placement of the first round (two workgroups per compute unit): known
  // when the stream has the whole chip, so unsplit units are paired by work.
  a.xcd_cus = 0;
  if (a.num_cus == 0) {
    const int cus = stream_compute_units(stream);
    if (cus == stream_compute_units(nullptr) && cus % kXcds == 0) a.xcd_cus = cus / kXcds;
  }
  // ranks beyond the units: at most 2 num_cus / Hkv more pieces than items
  const long long grid = (long long)num_units + 2 * a.num_cus;
  // (block, KV head) rows of 4 KiB: 32-bit offsets reach them all below 2^20 rows
  const bool off32 = (int64_t)a.num_blocks * a.num_kv_heads <= (int64_t)1 << 20;
  const dim3 g((unsigned)grid), b(kThreads);
  if (prefill_needs_ring(a.max_ctx, a.max_blocks_per_seq)) {
    if (off32)
      hipLaunchKernelGGL((prefill_mfma_kernel<G, true, true>), g, b, 0, stream, a);
    else
      hipLaunchKernelGGL((prefill_mfma_kernel<G, false, true>), g, b, 0, stream, a);
  } else {
    if (off32)
      hipLaunchKernelGGL((prefill_mfma_kernel<G, true, false>), g, b, 0, stream, a);
    else
      hipLaunchKernelGGL((prefill_mfma_kernel<G, false, false>), g, b, 0, stream, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.num_cus == 0) return e;
  // four workgroups per split (item, KV head); split items x Hkv <= num_units
  hipLaunchKernelGGL(prefill_merge_kernel<G>, dim3((unsigned)(4 * num_units)), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace pf

using pf::kMaxPrefillCus;
using pf::kMaxRankItems;
using pf::kRows;
using pf::launch_group;

int prefill_positions_per_tile(int group) { return kRows / group; }

constexpr size_t kSlotBytes = (size_t)kRows * (kHeadDim + 2) * sizeof(float);   // one partial: rows, their max and sum
constexpr size_t kListBytes = (1 + 3 * (size_t)kMaxRankItems) * sizeof(int32_t);
constexpr int kMaxSlots = 2 * kMaxPrefillCus;

size_t prefill_workspace_bytes() {
  return (kMaxSlots * kSlotBytes + kListBytes + 255) & ~(size_t)255;
}

void set_prefill_workspace(PrefillArgs& a, void* ws, size_t bytes, bool whole) {
  a.num_cus = 0;
  a.ws_slots = 0;
  a.ws_o = nullptr;
  a.ws_ml = nullptr;
  a.ws_list = nullptr;
  if (ws == nullptr || bytes < (whole ? prefill_workspace_bytes() : kListBytes)) return;   // no splitting
  const size_t slots = (bytes - kListBytes) / kSlotBytes;
  a.ws_slots = slots < kMaxSlots ? (int32_t)slots : kMaxSlots;
  const size_t rows = (size_t)a.ws_slots * kRows;
  a.ws_o = static_cast<float*>(ws);
  a.ws_ml = a.ws_o + rows * kHeadDim;
  a.ws_list = reinterpret_cast<int32_t*>(a.ws_ml + rows * 2);
}

hipError_t launch_prefill_mfma(PrefillArgs a, int group, int num_tiles_total, hipStream_t stream) {
  if (num_tiles_total <= 0) return hipSuccess;
  switch (group) {
    case 1: return launch_group<1>(a, num_tiles_total, stream);
    case 2: return launch_group<2>(a, num_tiles_total, stream);
    case 4: return launch_group<4>(a, num_tiles_total, stream);
    case 8: return launch_group<8>(a, num_tiles_total, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bros
