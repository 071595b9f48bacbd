// bros_attn_decode (bf16) for short contexts and for few (row, KV head)
// segments (the rest: decode.hip, whose device code says what is computed and
// how a tile's operands lie).
//
// decode.hip cuts the tiles evenly over the chip and folds the cut segments in
// a second kernel. Where a wave gets few tiles, the row prefix every workgroup
// builds, the search for its place in it and the walk from there cost more than
// the tiles. Here a workgroup takes a whole segment, or split_blocks blocks of
// it, wave w every fourth block, and folds the waves' results in LDS: no
// prefix, and for whole segments no partials and no second kernel. The loads of
// a wave's next block are requested as its registers are read, with no branch
// around them; four waves per SIMD cover the rest of the latency, which bounds
// it: under 1 us per tile of a wave after 4 us of start-up. Device time in us (32 /
// 8 heads unless said), the even split and this (plan.h says which calls):
//   whole  one row of 200 tokens 10.3 / 5.8, 16 rows of 25 to 200 11.8 / 6.7, 64 of
//          64 to 512 24.7 / 18.8, 512 of 25 to 200 59.4 / 53.6
//   split  one row of 8000 22.6 / 11.1, six of 312 to 2500 19.4 / 14.7, four of 500
//          to 4000 19.3 / 15.1, 64 of 312 to 2500 with 8 / 1 heads 26.4 / 20.7, 8 of
//          1000 to 8000 with 64 / 8 heads 42.3 / 37.5
// (With 8 waves a segment 1 us slower, with 16 up to twice as long: a compute
// unit then reads one segment at its own rate.)
#include "decode_device.h"
#include "plan.h"

#include <algorithm>

namespace bros {
namespace dm {

// Blocks [sp S, (sp + 1) S) of segment seg0 + blockIdx.x, S = split_blocks and
// sp = blockIdx.y: the whole segment when it has no more than S blocks, else a
// partial in slot (segment * n_split_max + sp) * G + head.
template <int G>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void decode_short_kernel(DecodeArgs a, int seg0) {
  __shared__ float s_o[kWaves][G][kHeadDim + 4];
  __shared__ float s_m[kWaves][G], s_l[kWaves][G];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int w = wave_id_uniform();
  const int grp = lane >> 4;
  const int col = lane & 15;
  const bool head_lane = col < G;
  const int nkv = a.num_kv_heads;
  const int Hq = a.num_q_heads;
  const int seg = seg0 + (int)blockIdx.x;
  const int row = seg / nkv, g = seg - row * nkv;
  const int ctx = max(0, min(load_uniform(a.ctx_lens, row), min(a.max_ctx, a.max_blocks_per_seq * kBlockSize)));
  const int nblk = (ctx + kBlockSize - 1) / kBlockSize;
  const int sp = blockIdx.y;
  const int b0 = sp * a.split_blocks, b1 = min(nblk, b0 + a.split_blocks);
  if (sp > 0 && b0 >= nblk) return;
  const int first = b0 + w;                                               // this wave's blocks: first, first + 4, ...
  const int n = b1 > first ? (b1 - first + kWaves - 1) / kWaves : 0;

  v4u_t qf[4], kf[4], vf[4];
  floatx4_t acc[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
  float m_ref = kNoMax, l_part = 0.0f;

  // Pool block of this wave's i-th block: block 0 in place of an invalid entry
  // (masked whole) or past the wave's blocks (not computed), so that the loads
  // need no branch. (The table is not read past the context.)
  auto entry = [&](int i, bool& ok) -> int {
    const int v = load_uniform(a.block_tables, (size_t)row * a.max_blocks_per_seq + min(first + kWaves * i, b1 - 1));
    ok = v >= 0 && v < a.num_blocks;
    return ok ? v : 0;
  };
  auto issue_k = [&](int blk) __attribute__((always_inline)) {
    const size_t base = ((size_t)blk * nkv + g) * kTileElems + (uint32_t)col * kHeadDim + 8 * grp;
#pragma unroll
    for (int k = 0; k < 4; ++k) kf[k] = load_nt(a.k_pool, base + 32 * k);
  };
  auto issue_v = [&](int blk) __attribute__((always_inline)) {
    const size_t base = ((size_t)blk * nkv + g) * kTileElems + (uint32_t)(4 * grp) * kHeadDim + 8 * col;
#pragma unroll
    for (int j = 0; j < 4; ++j) vf[j] = load_nt(a.v_pool, base + (size_t)j * kHeadDim);
  };

  if (n > 0) {
    bool ok;
    int blk = entry(0, ok);
    issue_k(blk);
    {
      const size_t qoff = ((size_t)row * Hq + g * G + min(col, G - 1)) * kHeadDim + 8 * grp;   // (padding columns repeat a head)
#pragma unroll
      for (int k = 0; k < 4; ++k) qf[k] = *reinterpret_cast<const v4u_t*>(static_cast<const uint16_t*>(a.q) + qoff + 32 * k);
    }
    issue_v(blk);
#pragma clang loop unroll(disable)
    for (int i = 0; i < n; ++i) {
      const int b = first + kWaves * i;
      bool next_ok;
      const int next = entry(i + 1, next_ok);
      floatx4_t sc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < 4; ++k)
        sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kf[k]), __builtin_bit_cast(bf16x8_t, qf[k]), sc, 0, 0, 0);
      issue_k(next);   // the K registers are free
      float s[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] = sc[r] * a.scale_log2;
      if (!ok || (b + 1) * kBlockSize > ctx) {   // an invalid entry, or the tail: drop slots past the context
        const int dir = entry_direction(a.dir, a.cls, a.dir_per_entry, a.max_blocks_per_seq, row, b);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (!ok || b * kBlockSize + slot_of_offset(4 * grp + r, dir) >= ctx) {
            s[r] = -INFINITY;
            vf[r] = v4u_t{0u, 0u, 0u, 0u};
          }
        }
      }
      float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
      if (__builtin_amdgcn_ballot_w64(head_lane && mx > m_ref + kRescaleSlack) != 0) {
        // rare: move each head's reference max to the max over its 16 slots
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_ref, mx);
        const float alpha = fast_exp2(m_ref - m_new);
        m_ref = m_new;
        l_part *= alpha;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[t][r] *= alpha;
        }
      }
      float p[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = fast_exp2(s[r] - m_ref);
      l_part += (p[0] + p[1]) + (p[2] + p[3]);
      // The weights as a bf16 and the bf16 of what it leaves: the matrix cores
      // wait for the loads here anyway, and the even split, which this
      // replaces, cut a short context so finely that a good part of its
      // weights were maxima, exactly 1. (Distance from 64 bits, one to six
      // rows: 0.0019-0.0021 there, 0.0022-0.0023 with the first part alone,
      // 0.0017 with both, the output's own rounding; 0.1 us a call.)
      // The first part is taken a little short of the weight, so that the second
      // is positive too: with a part that is 0 or negative, a V value of infinity
      // would become a NaN. (What both leave is below 2^-13 of the weight: the second
      // part, up to 2^-6 + 2^-8 of it, is rounded to 8 bits.)
      constexpr float kShort = 1.0f - 0x1p-6f;
      const uint2 hi2 = {pack2_bf16(kShort * p[0], kShort * p[1]), pack2_bf16(kShort * p[2], kShort * p[3])};
      const uint2 lo2 = {pack2_bf16(p[0] - bf16_lo(hi2.x), p[1] - bf16_hi(hi2.x)),
                         pack2_bf16(p[2] - bf16_lo(hi2.y), p[3] - bf16_hi(hi2.y))};
      const short4_t pb = __builtin_bit_cast(short4_t, hi2), pl = __builtin_bit_cast(short4_t, lo2);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const uint32_t sel = (t & 1) ? 0x07060302u : 0x05040100u;
        const uint32_t lo = __builtin_amdgcn_perm(vf[1][t >> 1], vf[0][t >> 1], sel);
        const uint32_t hi = __builtin_amdgcn_perm(vf[3][t >> 1], vf[2][t >> 1], sel);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4_t, uint2{lo, hi}), pb, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4_t, uint2{lo, hi}), pl, acc[t], 0, 0, 0);
      }
      issue_v(next);   // the V registers are free
      ok = next_ok;
    }
  }

  // The waves' results: lane l holds dims 32 grp + 8 r + t of head col.
  float l_head = l_part;
  l_head += __shfl_xor(l_head, 16);
  l_head += __shfl_xor(l_head, 32);
  if (head_lane) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float* o = &s_o[w][col][32 * grp + 8 * r];
      *reinterpret_cast<floatx4_t*>(o) = floatx4_t{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
      *reinterpret_cast<floatx4_t*>(o + 4) = floatx4_t{acc[4][r], acc[5][r], acc[6][r], acc[7][r]};
    }
    if (grp == 0) {
      s_m[w][col] = m_ref;
      s_l[w][col] = l_head;
    }
  }
  __syncthreads();
  for (int i = tid; i < G * (kHeadDim / 2); i += kThreads) {
    const int h = i / (kHeadDim / 2), d = 2 * (i % (kHeadDim / 2));
    float M = kNoMax;
#pragma unroll
    for (int x = 0; x < kWaves; ++x) M = fmaxf(M, s_m[x][h]);
    float L = 0.0f, A0 = 0.0f, A1 = 0.0f;
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      const float wt = fast_exp2(s_m[x][h] - M);
      const float2 o = *reinterpret_cast<const float2*>(&s_o[x][h][d]);
      L = fmaf(s_l[x][h], wt, L);
      A0 = fmaf(o.x, wt, A0);
      A1 = fmaf(o.y, wt, A1);
    }
    if (nblk > a.split_blocks) {
      const size_t slot = ((size_t)seg * a.n_split_max + sp) * G + h;
      *reinterpret_cast<float2*>(a.ws_acc + slot * kHeadDim + d) = make_float2(A0, A1);
      if (d == 0) {
        a.ws_ml[2 * slot] = M;
        a.ws_ml[2 * slot + 1] = L;
      }
      continue;
    }
    const float inv = L > 0.0f ? 1.0f / L : 0.0f;   // (a row without context is zeros)
    uint32_t* out = reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(a.out) + ((size_t)row * Hq + g * G + h) * kHeadDim + d);
    *out = pack2_bf16(A0 * inv, A1 * inv);
  }
}

constexpr long long kMaxSegmentsPerLaunch = 1 << 23;   // (a launch's threads must stay below 2^32)

// Folds the partials of the segments that were split, a workgroup each: o =
// sum_i 2^(m_i - M) acc_i / sum_i 2^(m_i - M) l_i. Thread t takes two dims of
// one head per pass; the partials' loads do not depend on one another.
template <int G>
__global__ __launch_bounds__(kThreads) void decode_short_merge_kernel(DecodeArgs a) {
  const int seg = blockIdx.x;
  const int nkv = a.num_kv_heads;
  const int row = seg / nkv, g = seg - row * nkv;
  const int ctx = max(0, min(load_uniform(a.ctx_lens, row), min(a.max_ctx, a.max_blocks_per_seq * kBlockSize)));
  const int nblk = (ctx + kBlockSize - 1) / kBlockSize;
  if (nblk <= a.split_blocks) return;   // written by the decode
  const int nsp = (nblk + a.split_blocks - 1) / a.split_blocks;
  const size_t slot0 = (size_t)seg * a.n_split_max * G;
  for (int i = threadIdx.x; i < G * (kHeadDim / 2); i += kThreads) {
    const int h = i / (kHeadDim / 2), d = 2 * (i % (kHeadDim / 2));
    const float2* ml = reinterpret_cast<const float2*>(a.ws_ml) + slot0 + h;
    const float* acc = a.ws_acc + (slot0 + h) * kHeadDim + d;
    float M = kNoMax, L = 0.0f, A0 = 0.0f, A1 = 0.0f;
    for (int c = 0; c < nsp; c += 8) {   // eight partials a round, indices clamped in range
      float2 x[8], v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = min(c + u, nsp - 1);
        x[u] = ml[(size_t)j * G];
        v[u] = *reinterpret_cast<const float2*>(acc + (size_t)j * G * kHeadDim);
      }
      float Mn = M;
#pragma unroll
      for (int u = 0; u < 8; ++u) Mn = fmaxf(Mn, x[u].x);
      const float alpha = fast_exp2(M - Mn);
      L *= alpha;
      A0 *= alpha;
      A1 *= alpha;
      M = Mn;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        // (a round's padding adds zero by selection: the partial it repeats may hold an infinity)
        const bool use = c + u < nsp;
        const float wt = use ? fast_exp2(x[u].x - M) : 0.0f;
        L = fmaf(use ? x[u].y : 0.0f, wt, L);
        A0 = fmaf(use ? v[u].x : 0.0f, wt, A0);
        A1 = fmaf(use ? v[u].y : 0.0f, wt, A1);
      }
    }
    const float inv = L > 0.0f ? 1.0f / L : 0.0f;
    *reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(a.out) + ((size_t)row * a.num_q_heads + g * G + h) * kHeadDim + d) =
        pack2_bf16(A0 * inv, A1 * inv);
  }
}

template <int G>
hipError_t launch_short_group(DecodeArgs a, hipStream_t stream, hipEvent_t between) {
  const int64_t segments = (int64_t)a.num_rows * a.num_kv_heads;
  for (int64_t s0 = 0; s0 < segments; s0 += kMaxSegmentsPerLaunch) {
    const dim3 grid((unsigned)std::min<int64_t>(segments - s0, kMaxSegmentsPerLaunch), (unsigned)a.n_split_max);
    hipLaunchKernelGGL(decode_short_kernel<G>, grid, dim3(kThreads), 0, stream, a, (int)s0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (between != nullptr) {
    const hipError_t e = hipEventRecord(between, stream);
    if (e != hipSuccess) return e;
  }
  if (a.n_split_max <= 1) return hipSuccess;
  hipLaunchKernelGGL(decode_short_merge_kernel<G>, dim3((unsigned)segments), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace dm

bool plan_decode_short(DecodeArgs& a, hipStream_t stream) {
  const int64_t segments = (int64_t)a.num_rows * a.num_kv_heads;
  const int32_t blocks = longest_blocks(a.max_ctx, a.max_blocks_per_seq);
  if (whole_on_any_share(segments, blocks)) {   // (asking for the stream's compute units costs the smallest steps 0.6 us of 16)
    a.split_blocks = blocks;
    a.n_split_max = 1;
    return true;
  }
  // (partials: the workspace has a slot per query row and kDecodeGroupSlots groups more)
  const int64_t slots = (int64_t)a.num_rows * a.num_q_heads + (int64_t)kDecodeGroupSlots * std::min(a.num_q_heads, 8);
  return plan_short_decode(segments, a.num_q_heads / a.num_kv_heads, blocks, stream_compute_units(stream), slots,
                           &a.split_blocks, &a.n_split_max);
}

hipError_t launch_decode_short(const DecodeArgs& a, int group, hipStream_t stream, hipEvent_t between) {
  switch (group) {
    case 1: return dm::launch_short_group<1>(a, stream, between);
    case 2: return dm::launch_short_group<2>(a, stream, between);
    case 4: return dm::launch_short_group<4>(a, stream, between);
    case 8: return dm::launch_short_group<8>(a, stream, between);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bros
