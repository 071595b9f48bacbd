// bros_attn_decode (bf16) launch: the decode kernel and the merge of cut
// segments. The device code (and what it computes) is in decode_device.h.
#include "decode_device.h"

#include <atomic>
#include <mutex>
#include <type_traits>

namespace bros {
namespace dm {

template <int G>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void decode_mfma_kernel(DecodeArgs a) {
  __shared__ int s_pre[kMaxRowsLds + 1];
  __shared__ int s_scan[kWaves];

  const int chunk = (a.num_rows + kMaxRowsLds - 1) / kMaxRowsLds;
  const int nch = (a.num_rows + chunk - 1) / chunk;
  const int total = build_tile_prefix(a, s_pre, s_scan, chunk, nch);

  // Workgroup 0 records the shares for the merge. While there are fewer
  // workers than waves, they spread over the workgroups.
  const Shares shares(a, total);
  const int workers = shares.workers;
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) a.ws_wstart[0] = workers;
    for (int w = threadIdx.x; w <= workers; w += kThreads) a.ws_wstart[1 + w] = shares.start(w);
  }
  const int wave = wave_id_uniform();
  const int wid = workers < a.num_workers ? wave * gridDim.x + blockIdx.x : blockIdx.x * kWaves + wave;
  if (wid >= workers) {
    if ((threadIdx.x & (kWave - 1)) == 0) a.ws_cut[2 * wid] = -1;   // idle: nothing to merge
    return;
  }
  // (Kept in vector registers: with the share in scalar ones the compiler packs
  // the kernel into 149 registers with scalar spills and its waves get slower,
  // 169 us against 166 on 64 rows, 37 against 30 on one row of 8000 tokens.)
  int t0 = shares.start(wid), t1 = shares.start(wid + 1);
  asm volatile("" : "+v"(t0), "+v"(t1));
  decode_worker<G>(a, s_pre, chunk, nch, wid, t0, t1 - t0, &shares);
}

// Segments cut between workers: o = sum_w 2^(m_w - M) acc_w / sum_w 2^(m_w -
// M) l_w over the partials of workers w0 .. w1. The decode kernel's worker
// w0 (the one that started the segment and left it unfinished) named the
// segment in its entry of the cut list, with w1 when its shares are the even
// split (then every worker has tiles and the merge reads nothing else before
// the partials); every other entry is -1, so the merge grid has one wave per
// worker and most waves return after one load. Segments
// a single worker covered were written directly, and rows without context
// were written as zeros by that worker (a worker that sees no tile of a row
// never runs for it: rows without context have no tiles, so they are written
// here). The G heads of the segment share the wave: 64 / G lanes per head,
// each folding 2 G of its head's dims, eight partials in flight. A segment of
// more than kAlone partials (few rows, long contexts) is folded by the four
// waves of the workgroup together, a fourth of the partials each. (Merging
// inside the decode kernel instead would need device-scope release/acquire
// between workgroups, which on this chip writes back and invalidates a whole
// L2 per segment; the kernel boundary is far cheaper.)
constexpr int kMergeWaves = 4;
// Partials that a wave folds by itself, in two rounds. (With one round alone, 8,
// the longest contexts of 64 rows go to the whole workgroup after its own
// segments: 6.0 us a merge against 5.4.)
constexpr int kAlone = 16;
static_assert(kMergeWaves * kWave == kThreads, "the merge's workgroup");

template <int G>
__global__ __launch_bounds__(kMergeWaves * kWave) void decode_mfma_merge_kernel(DecodeArgs a) {
  constexpr int L = kWave / G;          // lanes per head
  constexpr int DPL = kHeadDim / L;     // dims per lane (2 G)
  __shared__ float s_acc[kMergeWaves][DPL][kWave], s_m[kMergeWaves][kWave], s_l[kMergeWaves][kWave];
  __shared__ int s_last[kMergeWaves];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_id_uniform();
  const int item = blockIdx.x * kMergeWaves + wave;
  // Rows without context have no tiles, so no worker saw them: zeros.
  if (item < a.num_rows) {
    int s0, ctx0;
    resolve_row(a, item, s0, ctx0);
    if (ctx0 <= 0) {
      uint32_t* z = reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(a.out) + (size_t)item * a.num_q_heads * kHeadDim);
      for (int i = lane; i < a.num_q_heads * kHeadDim / 2; i += kWave) z[i] = 0u;
    }
  }
  const int nkv = a.num_kv_heads;
  // the decode grid's partition of the tiles: workers W, worker w's tiles
  // start at starts[w] (starts[W] = all tiles); a worker may have none, but
  // not where the entry names the last worker
  const int32_t* starts = a.ws_wstart + 1;
  // The cut-list entries of the workgroup's workers, on every wave (every
  // worker of the grid wrote its entry, idle ones -1; num_workers is a multiple
  // of the four): segment and last worker.
  if (blockIdx.x * kMergeWaves >= a.num_workers) return;
  int codes[kMergeWaves], lasts[kMergeWaves];
#pragma unroll
  for (int e = 0; e < kMergeWaves; ++e) {
    codes[e] = load_uniform(a.ws_cut, 2 * (blockIdx.x * kMergeWaves + e));
    lasts[e] = load_uniform(a.ws_cut, 2 * (blockIdx.x * kMergeWaves + e) + 1);
  }
  const int2 own = reinterpret_cast<const int2*>(a.ws_cut)[item];
  const int code = __builtin_amdgcn_readfirstlane(own.x);
  int w1 = __builtin_amdgcn_readfirstlane(own.y);
  const bool known = w1 >= 0;
  if (code >= 0 && !known) {
    // w1: the worker holding the segment's last tile (the last worker whose
    // share starts at or before it), found 64 workers per step
    const int workers = a.ws_wstart[0];
    const int row = code / nkv, g = code - row * nkv;
    int s, ctx;
    resolve_row(a, row, s, ctx);
    const int nblk = (ctx + kBlockSize - 1) / kBlockSize;
    const int64_t last_tile = (int64_t)a.ws_rows[row] + (int64_t)g * nblk + nblk - 1;
    w1 = item;
    for (int base = item + 1; base < workers; base += kWave) {
      const int w = base + lane;
      const bool before = w < workers && starts[w] <= last_tile;
      const uint64_t m = __builtin_amdgcn_ballot_w64(before);
      w1 = base + __builtin_popcountll(m) - 1;
      if (m != ~0ull) break;
    }
    w1 = __builtin_amdgcn_readfirstlane(max(w1, item));
  }
  // Last workers that had to be found (a fused launch) go to the other waves, so
  // that these share long segments too: two prompts beside 32 rows of 100 to 1500
  // tokens 79 us a merge with the wave alone, 28 shared.
  bool given[kMergeWaves], found = false;
#pragma unroll
  for (int e = 0; e < kMergeWaves; ++e) {
    given[e] = lasts[e] >= 0;
    found |= codes[e] >= 0 && !given[e];
  }
  if (found) {   // uniform over the workgroup
    if (lane == 0) s_last[wave] = w1;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kMergeWaves; ++e) lasts[e] = given[e] ? lasts[e] : s_last[e];
  }

  const int hl = lane / L, sub = lane % L;
  float Lsum, M;
  float acc[DPL];
  // Partials of workers [c0, c1] of segment `seg` folded into (M, Lsum, acc);
  // M and acc of the head in every lane, Lsum spread over the head's lanes.
  auto fold = [&](size_t seg, int c0, int c1, bool even) __attribute__((always_inline)) {
    // a worker with no tiles wrote no partial
    auto has_tiles = [&](int w) -> bool { return even || starts[w + 1] > starts[w]; };
    M = kNoMax;
    Lsum = 0.0f;
#pragma unroll
    for (int d = 0; d < DPL; ++d) acc[d] = 0.0f;
    // up to eight partials a round, their sums requested together with their maxima
    for (int c = c0; c <= c1; c += 8) {
      const int cnt = min(8, c1 - c + 1);
      float2 v[8][DPL / 2];
#pragma unroll
      for (int u = 0; u < 8; ++u) {   // indices clamped in range
        const float2* src = reinterpret_cast<const float2*>(a.ws_acc + ((seg + c + min(u, cnt - 1)) * G + hl) * kHeadDim + sub * DPL);
#pragma unroll
        for (int q = 0; q < DPL / 2; ++q) v[u][q] = src[q];
      }
      // lane `sub` of the head holds partial c + sub's maximum and sum
      const int ok = sub < cnt && has_tiles(c + sub);
      float m_l = kNoMax, l_l = 0.0f;
      if (ok) {
        const size_t slot = (seg + c + sub) * G + hl;
        m_l = a.ws_ml[2 * slot];
        l_l = a.ws_ml[2 * slot + 1];
      }
      float Mn = fmaxf(M, m_l);
#pragma unroll
      for (int o = L / 2; o >= 1; o >>= 1) Mn = fmaxf(Mn, __shfl_xor(Mn, o));
      if (c > c0) {
        const float alpha = fast_exp2(M - Mn);
        Lsum *= alpha;
#pragma unroll
        for (int d = 0; d < DPL; ++d) acc[d] *= alpha;
      }
      M = Mn;
      float wt = 0.0f;
      if (ok) {
        wt = fast_exp2(m_l - M);
        Lsum = fmaf(l_l, wt, Lsum);
      }
      // Padding and partials of workers without tiles add zero by selection:
      // their slots may hold anything.
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = min(u, cnt - 1);
        const float w = __shfl(wt, hl * L + j);
        const bool use = u < cnt && __shfl(ok, hl * L + j) != 0;
        const float wu = use ? w : 0.0f;
#pragma unroll
        for (int q = 0; q < DPL / 2; ++q) {
          const float2 x = use ? v[u][q] : make_float2(0.0f, 0.0f);
          acc[2 * q] = fmaf(x.x, wu, acc[2 * q]);
          acc[2 * q + 1] = fmaf(x.y, wu, acc[2 * q + 1]);
        }
      }
    }
#pragma unroll
    for (int o = L / 2; o >= 1; o >>= 1) Lsum += __shfl_xor(Lsum, o);
  };
  auto write = [&](int seg) __attribute__((always_inline)) {
    const int row = seg / nkv, g = seg - row * nkv;
    const float inv = Lsum > 0.0f ? 1.0f / Lsum : 0.0f;
    uint32_t* out = reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(a.out) +
                                                ((size_t)row * a.num_q_heads + g * G + hl) * kHeadDim + sub * DPL);
#pragma unroll
    for (int d = 0; d < DPL; d += 2) out[d / 2] = pack2_bf16(acc[d] * inv, acc[d + 1] * inv);
  };

  // Up to kAlone partials (nearly every segment of a large batch): the wave alone.
  if (code >= 0 && w1 - item < kAlone) {
    fold((size_t)code, item, w1, known);
    write(code);
  }
  // More (long contexts of few rows): the workgroup's waves take a part of them
  // each and fold their results through LDS.
#pragma unroll
  for (int e = 0; e < kMergeWaves; ++e) {
    const int seg = codes[e], c0 = blockIdx.x * kMergeWaves + e, c1 = lasts[e];
    if (seg < 0 || c1 - c0 < kAlone) continue;   // uniform over the workgroup
    const int n = c1 - c0 + 1;
    const int p0 = c0 + n * wave / kMergeWaves, p1 = c0 + n * (wave + 1) / kMergeWaves - 1;   // (n > kAlone: none is empty)
    fold((size_t)seg, p0, p1, given[e]);
    __syncthreads();   // the last segment's results have been read
    s_m[wave][lane] = M;
    s_l[wave][lane] = Lsum;
#pragma unroll
    for (int d = 0; d < DPL; ++d) s_acc[wave][d][lane] = acc[d];
    __syncthreads();
    if (wave == e) {
      float m[kMergeWaves];
      M = kNoMax;
#pragma unroll
      for (int x = 0; x < kMergeWaves; ++x) M = fmaxf(M, m[x] = s_m[x][lane]);
      Lsum = 0.0f;
#pragma unroll
      for (int d = 0; d < DPL; ++d) acc[d] = 0.0f;
#pragma unroll
      for (int x = 0; x < kMergeWaves; ++x) {
        const float wt = fast_exp2(m[x] - M);
        Lsum = fmaf(s_l[x][lane], wt, Lsum);
#pragma unroll
        for (int d = 0; d < DPL; ++d) acc[d] = fmaf(s_acc[x][d][lane], wt, acc[d]);
      }
      write(seg);
    }
  }
}

}  // namespace dm

namespace {

// Compute units enabled for `stream`: the population count of its CU mask, or
// `fallback` when the mask cannot be read.
int stream_cus(hipStream_t stream, int fallback) {
  constexpr int kMaskWords = 32;   // up to 1024 CUs
  uint32_t mask[kMaskWords] = {};
  if (hipExtStreamGetCUMask(stream, kMaskWords, mask) != hipSuccess) {
    (void)hipGetLastError();
    return fallback;
  }
  int n = 0;
  for (int i = 0; i < kMaskWords; ++i) n += __builtin_popcount(mask[i]);
  return (n > 0 && n < fallback) ? n : fallback;
}

}  // namespace

int stream_compute_units(hipStream_t stream) {
  constexpr int kMaxDevices = 64;
  static int cus_cache[kMaxDevices];
  static std::mutex mu;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  int cus = 0;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (cus_cache[dev] == 0) {
      int n = 0;
      if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
      cus_cache[dev] = n;
    }
    cus = cus_cache[dev];
  }
  return stream_cus(stream, cus);
}

int workgroups_per_cu(const void* kernel, int threads, int slot) {
  constexpr int kMaxDevices = 64;
  constexpr int kSlots = 8;
  static int per_cu_cache[kMaxDevices][kSlots];
  static std::mutex mu;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 4;
  int per_cu = 0;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (per_cu_cache[dev][slot] == 0) {
      int n = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, 0) != hipSuccess || n <= 0) n = 4;
      per_cu_cache[dev][slot] = n;
    }
    per_cu = per_cu_cache[dev][slot];
  }
  return per_cu;
}

int resident_workgroups(const void* kernel, int threads, int slot, hipStream_t stream) {
  return workgroups_per_cu(kernel, threads, slot) * stream_compute_units(stream);
}

namespace {

// Workgroups of the bf16 decode grid at most (four workers each): what 256
// compute units hold at four waves per SIMD (the kernel runs two). The
// workspace is sized for it.
constexpr int kMaxDecodeGrid = 1024;
static_assert(kDecodeGroupSlots == kWaves * kMaxDecodeGrid, "the workspace's partials");

// Events recorded around the decode kernel of every bf16 call (a
// benchmark's hook; both null when unused).
std::atomic<hipEvent_t> g_kernel_ev_before{nullptr}, g_kernel_ev_after{nullptr};

template <int G>
hipError_t launch_group(DecodeArgs a, hipStream_t stream, int slot) {
  const hipEvent_t before = g_kernel_ev_before.load(), after = g_kernel_ev_after.load();
  hipError_t e = hipSuccess;
  if (before != nullptr && (e = hipEventRecord(before, stream)) != hipSuccess) return e;
  if (plan_decode_short(a, stream)) return launch_decode_short(a, G, stream, after);
  int grid = resident_workgroups(reinterpret_cast<const void*>(&dm::decode_mfma_kernel<G>), kThreads, slot, stream);
  grid = grid < kMaxDecodeGrid ? grid : kMaxDecodeGrid;
  a.num_workers = grid * kWaves;
  hipLaunchKernelGGL((dm::decode_mfma_kernel<G>), dim3(grid), dim3(kThreads), 0, stream, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (after != nullptr && (e = hipEventRecord(after, stream)) != hipSuccess) return e;
  return launch_decode_merge(a, G, stream);
}

}  // namespace

hipError_t launch_decode_merge(const DecodeArgs& a, int group, hipStream_t stream) {
  // one wave per worker (its cut-list entry) and per row (rows without context)
  const long long items = a.num_workers > a.num_rows ? a.num_workers : a.num_rows;
  const dim3 grid((unsigned)((items + dm::kMergeWaves - 1) / dm::kMergeWaves)), block(dm::kMergeWaves * kWave);
  switch (group) {
    case 1: hipLaunchKernelGGL(dm::decode_mfma_merge_kernel<1>, grid, block, 0, stream, a); break;
    case 2: hipLaunchKernelGGL(dm::decode_mfma_merge_kernel<2>, grid, block, 0, stream, a); break;
    case 4: hipLaunchKernelGGL(dm::decode_mfma_merge_kernel<4>, grid, block, 0, stream, a); break;
    case 8: hipLaunchKernelGGL(dm::decode_mfma_merge_kernel<8>, grid, block, 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

DecodePlan plan_decode(int32_t num_rows, int32_t max_ctx) {
  DecodePlan p;
  const int64_t maxblk = max_ctx > 0 ? ((int64_t)max_ctx + kBlockSize - 1) / kBlockSize : 1;
  int sb = dm::kMaxSplitBlocks;   // 1024 tokens per split by default
  while (sb > 4 && (int64_t)num_rows * ((maxblk + sb - 1) / sb) < 512) sb >>= 1;
  p.split_blocks = sb;
  p.n_split_max = (int32_t)((maxblk + sb - 1) / sb);
  return p;
}

static size_t round_up_256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t decode_workspace_bytes(int32_t num_rows, int32_t num_q_heads, int32_t max_ctx, bool bf16) {
  if (bf16) {
    const int gmax = num_q_heads < 8 ? num_q_heads : 8;
    const size_t slots = (size_t)num_rows * num_q_heads + (size_t)kWaves * kMaxDecodeGrid * gmax;
    return round_up_256(((size_t)num_rows + 1) * sizeof(int32_t)) + round_up_256(slots * kHeadDim * sizeof(float)) +
           round_up_256(slots * 2 * sizeof(float)) + round_up_256((size_t)2 * kWaves * kMaxDecodeGrid * sizeof(int32_t)) +
           round_up_256(((size_t)kWaves * kMaxDecodeGrid + 2) * sizeof(int32_t));
  }
  const DecodePlan p = plan_decode(num_rows, max_ctx);
  if (p.n_split_max <= 1) return 0;
  const size_t slots = (size_t)num_rows * num_q_heads * p.n_split_max;
  return slots * kHeadDim * sizeof(float) + slots * 2 * sizeof(float);
}

void set_decode_workspace(DecodeArgs& a, void* ws, bool bf16) {
  char* base = static_cast<char*>(ws);
  if (bf16) {
    const int gmax = a.num_q_heads < 8 ? a.num_q_heads : 8;
    const size_t slots = (size_t)a.num_rows * a.num_q_heads + (size_t)kWaves * kMaxDecodeGrid * gmax;
    a.ws_rows = reinterpret_cast<int32_t*>(base);
    a.ws_acc = reinterpret_cast<float*>(base + round_up_256(((size_t)a.num_rows + 1) * sizeof(int32_t)));
    a.ws_ml = reinterpret_cast<float*>(reinterpret_cast<char*>(a.ws_acc) + round_up_256(slots * kHeadDim * sizeof(float)));
    a.ws_cut = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(a.ws_ml) + round_up_256(slots * 2 * sizeof(float)));
    a.ws_wstart = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(a.ws_cut) +
                                             round_up_256((size_t)2 * kWaves * kMaxDecodeGrid * sizeof(int32_t)));
    return;
  }
  a.ws_rows = nullptr;
  a.ws_cut = nullptr;
  a.ws_wstart = nullptr;
  a.ws_acc = reinterpret_cast<float*>(base);
  a.ws_ml = base ? a.ws_acc + (size_t)a.num_rows * a.num_q_heads * a.n_split_max * kHeadDim : nullptr;
}

void set_decode_kernel_events(hipEvent_t before, hipEvent_t after) {
  g_kernel_ev_before.store(before);
  g_kernel_ev_after.store(after);
}

hipError_t launch_decode(DecodeArgs a, int group, bool bf16, hipStream_t stream) {
  if (!bf16) return launch_decode_f32(a, group, stream);
  switch (group) {
    case 1: return launch_group<1>(a, stream, 0);
    case 2: return launch_group<2>(a, stream, 1);
    case 4: return launch_group<4>(a, stream, 2);
    case 8: return launch_group<8>(a, stream, 3);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bros
