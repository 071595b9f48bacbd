// fp32 prefill chunks over the bidirectional pool, on the fp32 matrix
// instructions (fp32 decode rows: decode_f32.hip; bf16 chunks: prefill.hip).
//
// What it computes (Sec. 2.2 chunked prefill; Sec. 5.1 bidirectional slot
// order; Sec. 6 direction-aware paged kernel): row j of a chunk of n rows of
// sequence s sees the first c0 + j + 1 positions of it, c0 = ctx - n, and for
// query head h in KV group g = h / G,
//     out[j][h] = sum_p softmax_p(scale * q[j][h] . K[p][g]) V[p][g].
// Products, sums, weights and partials are fp32 throughout (the fp32 tolerance
// is 1e-5).
//
// Work. A unit is one (sequence, KV head, 16 / G consecutive positions): 16
// query rows, all G heads. A workgroup takes one unit over a range of its
// 16-slot blocks, its four waves every fourth block each, and folds the waves'
// results in LDS. So a unit's rows share every K and V row they read, and the
// products run on the fp32 matrix instructions (2048 clocks of a SIMD per
// block), which with the vector instructions between them -- the two barely
// overlap -- bound the kernel: 256 rows on 4000 tokens (32 / 8 heads) run at 58
// % of the matrix rate. Run as decode rows, each reading its whole context on
// the vector ALU, chunks of 100 and 200 rows on 500 and 1000 tokens took 195
// us; here 96. (K and V staged in LDS by direct loads: 100 us, so the loads do
// not bound it.)
//
// Per block, as in the bf16 decode: S^T[slot][col] = K q^T, then O^T[dim][col]
// += V^T[dim][slot] P^T[slot][col], both with mfma 16x16x4. Lane l = 16 grp +
// col. The result of the first product puts the weights of slots 4 grp .. 4 grp
// + 3 of column col in lane l, which is the operand layout of the second: its
// step r contracts slots {4 grp + r}, and takes V rows 4 grp + r, dims 4 col
// .. 4 col + 3 and 64 more, as plain loads of 256 bytes side by side (row m of
// output tile t is dim 4 m + t, for t >= 4 dim 60 + 4 m + t). The
// first product contracts dims 16 i + 4 grp + e in step (i, e), so K and q are
// plain 16-byte loads too, 64 bytes of a row side by side.
//
// The next block's loads are requested as this block's registers are read,
// with no branch around them (a wait then counts K and V apart): an invalid
// table entry, or one past the unit, loads pool block 0 and is masked whole. The softmax is online in base 2 with a
// lazily moved reference (weights stay <= 2^8).
//
// Blocks that every row of the unit sees whole need no mask: the order of the
// slots does not matter. In the others each slot's position follows from the
// entry's direction; slots a row does not see are dropped by selection, and V
// rows that no row of the unit sees are zeroed, so a peer's tokens or NaNs
// cannot leak. A V row that some rows see and some do not may hold an infinity
// or a NaN, which a zero weight would spread; such a block (rare) is weighted
// on the vector ALU, each row taking only the V rows it sees.
#include "decode_common.h"
#include "plan.h"

#include <algorithm>

namespace bros {
namespace {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef const int32_t __attribute__((address_space(4)))* scalar_i32_ptr;

constexpr int kCols = 16;   // query rows (columns) of a unit
constexpr int kPad = 4;     // floats between LDS rows: column stride off the bank period

// What the query rows of a unit see. Uniform over the workgroup.
struct Unit {
  int s, g;
  int row0;        // first query row (of 16 / G consecutive ones)
  int rows;        // query rows of the unit (<= 16 / G)
  int see0;        // positions its first row sees; row j sees see0 + j (clamped)
  int cap;         // the clamp: max_ctx and the table's width
};

// The last sequence s with cu_q[s] / kPos + s <= r, 64 sequences per step. Every
// sequence has at least the ranks its tiles need, whatever its rows start at.
template <int kPos>
__device__ __forceinline__ int ranked_sequence(const DecodeArgs& a, int r, int lane) {
  int s = 0;
  for (int base = 0; base < a.num_seqs; base += kWave) {
    const int i = base + lane;
    const uint64_t m = __builtin_amdgcn_ballot_w64(i < a.num_seqs && a.cu_q[min(i, a.num_seqs - 1)] / kPos + i <= r);
    s = max(s, base + __builtin_popcountll(m) - 1);
    if (m != ~0ull) break;
  }
  return __builtin_amdgcn_readfirstlane(s);
}

__device__ __forceinline__ int seen(const Unit& u, int j) { return max(min(u.see0 + j, u.cap), 0); }

// kByRows: how units are ranked (F32ChunkPlan). A variant of its own: with the choice
// made in the kernel, the loop's code came out 2 to 4 % slower.
template <int G, bool kByRows>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void prefill_f32_kernel(DecodeArgs a, int unit0) {
  constexpr int kPos = kCols / G;   // positions of a unit
  __shared__ float s_o[kWaves][kCols][kHeadDim + kPad];
  __shared__ float s_m[kWaves][kCols], s_l[kWaves][kCols];

  const int nkv = a.num_kv_heads;
  const int Hq = a.num_q_heads;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int w = wave_id_uniform();
  const int grp = lane >> 4;
  const int col = lane & 15;

  // The longest units first; all KV heads of a unit on consecutive ids, so
  // that with 8 of them a head stays on one XCD's L2.
  Unit u;
  {
    const int id = unit0 + (int)blockIdx.x;
    const int r = id / nkv;
    u.g = id % nkv;
    int j0;
    if constexpr (!kByRows) {   // every sequence has as many ranks as the longest may need
      u.s = r % a.num_seqs;
      j0 = (a.tiles_per_seq - 1 - r / a.num_seqs) * kPos;
    } else {                    // sequence s has the ranks from cu_q[s] / kPos + s on, its last tile first
      u.s = ranked_sequence<kPos>(a, r, lane);
      j0 = (((scalar_i32_ptr)a.cu_q)[u.s + 1] / kPos + u.s - r) * kPos;
      if (j0 < 0) return;
    }
    const int q0 = ((scalar_i32_ptr)a.cu_q)[u.s], n = ((scalar_i32_ptr)a.cu_q)[u.s + 1] - q0;
    if (q0 < 0 || q0 + n > a.num_rows || j0 >= n) return;
    u.row0 = q0 + j0;
    u.rows = min(kPos, n - j0);
    u.see0 = ((scalar_i32_ptr)a.ctx_lens)[u.s] - n + j0 + 1;
    u.cap = min(a.max_ctx, a.max_blocks_per_seq * kBlockSize);
  }
  const int kmin = seen(u, 0), kmax = seen(u, u.rows - 1);
  const int nblk = (kmax + kBlockSize - 1) / kBlockSize;
  const int sp = blockIdx.y;
  const int b0 = sp * a.split_blocks;
  if (sp > 0 && b0 >= nblk) return;
  const int b1 = min(nblk, b0 + a.split_blocks);
  const int first = b0 + w;                                               // this wave's blocks: first, first + 4, ...
  const int nb = b1 > first ? (b1 - first + kWaves - 1) / kWaves : 0;

  const int pj = col / G;                                                 // this column's row
  const bool live = pj < u.rows;
  const int lim = live ? seen(u, pj) : 0;

  f4_t qf[8], kf[8], vf[8];
  f4_t acc[8];
  float m_ref = kNoMax, l_part = 0.0f;
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};

  const float* kpool = static_cast<const float*>(a.k_pool);
  const float* vpool = static_cast<const float*>(a.v_pool);
  const scalar_i32_ptr tbl = (scalar_i32_ptr)(a.block_tables + (size_t)u.s * a.max_blocks_per_seq);
  // Pool block of this wave's i-th block, or -1. (The table is not read past the unit.)
  auto entry = [&](int i) -> int {
    const int v = tbl[max(min(first + kWaves * i, b1 - 1), 0)];
    return i < nb && v >= 0 && v < a.num_blocks ? v : -1;
  };
  auto issue_k = [&](int blk) __attribute__((always_inline)) {
    const float* p = kpool + ((size_t)max(blk, 0) * nkv + u.g) * kTileElems + col * kHeadDim + 4 * grp;
#pragma unroll
    for (int i = 0; i < 8; ++i) kf[i] = *reinterpret_cast<const f4_t*>(p + 16 * i);
  };
  auto issue_v = [&](int blk) __attribute__((always_inline)) {
    const float* p = vpool + ((size_t)max(blk, 0) * nkv + u.g) * kTileElems + 4 * grp * kHeadDim + 4 * col;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      vf[2 * r] = *reinterpret_cast<const f4_t*>(p + r * kHeadDim);
      vf[2 * r + 1] = *reinterpret_cast<const f4_t*>(p + r * kHeadDim + 64);
    }
  };

  int blk = entry(0);
  {
    const float* qp = static_cast<const float*>(a.q) +
                      ((size_t)(u.row0 + min(pj, u.rows - 1)) * Hq + u.g * G + col % G) * kHeadDim + 4 * grp;
#pragma unroll
    for (int i = 0; i < 8; ++i) {   // (columns past the unit's rows repeat its last row and are not written)
      qf[i] = *reinterpret_cast<const f4_t*>(qp + 16 * i);
    }
  }
  issue_k(blk);
  issue_v(blk);

#pragma clang loop unroll(disable)
  for (int i = 0; i < nb; ++i) {
    const int b = first + kWaves * i;
    const int next = entry(i + 1);
    // Raw scores. Sixteen short chains, summed pairwise: one chain of 32 steps
    // would double the result's distance from 64 bits.
    f4_t sc[8], half;
    float s[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        sc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[k][2 * h], qf[k][2 * h], f4_t{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        sc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[k][2 * h + 1], qf[k][2 * h + 1], sc[k], 0, 0, 0);
      const f4_t sum = ((sc[0] + sc[1]) + (sc[2] + sc[3])) + ((sc[4] + sc[5]) + (sc[6] + sc[7]));
      if (h == 0) {
        half = sum;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = half[r] + sum[r];
      }
    }
    issue_k(next);   // the K registers are free

    uint64_t odd = 0;   // lanes with a non-finite V value that only some rows see
    int pos[4];
    if (blk < 0 || (b + 1) * kBlockSize > kmin) {
      const int dir = entry_direction(a.dir, a.cls, a.dir_per_entry, a.max_blocks_per_seq, u.s, b);
      bool bad = false;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pos[r] = blk < 0 ? INT_MAX : b * kBlockSize + slot_of_offset(4 * grp + r, dir);
        s[r] = pos[r] < lim ? s[r] : -INFINITY;
        if (pos[r] >= kmax) vf[2 * r] = vf[2 * r + 1] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
        if (pos[r] >= kmin) {
#pragma unroll
          for (int e = 0; e < 8; ++e) bad |= !(fabsf(vf[2 * r + (e >> 2)][e & 3]) < INFINITY);
        }
      }
      odd = __builtin_amdgcn_ballot_w64(bad);
    }
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * a.scale_log2;   // log2 units
    if (__builtin_amdgcn_ballot_w64(mx > m_ref + kRescaleSlack) != 0) {
      // rare: move each column's reference max to the max over its 16 slots
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m_ref, mx);
      const float alpha = fast_exp2(m_ref - m_new);
      m_ref = m_new;
      l_part *= alpha;
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] *= alpha;
    }
    float p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = fast_exp2(fmaf(s[r], a.scale_log2, -m_ref));
    l_part += (p[0] + p[1]) + (p[2] + p[3]);
    if (odd == 0) {
      // O^T += V^T P^T: the block's four steps in two pairs of their own, so
      // that the sum over a long context takes one rounding per block. (A pair per
      // step, 128 adds a block, is 5 % slower.)
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        f4_t o[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          o[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[4 * h + (t >> 2)][t & 3], p[2 * h], f4_t{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
          o[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[4 * h + 2 + (t >> 2)][t & 3], p[2 * h + 1], o[h], 0, 0, 0);
        }
        acc[t] += o[0] + o[1];
      }
    } else {
      // on the vector ALU, each column with the V rows it sees (acc[t][rr]: dim 16 grp + 4 rr + t, or 64 more)
      const float* vb = vpool + ((size_t)max(blk, 0) * nkv + u.g) * kTileElems + 16 * grp;
#pragma clang loop unroll(disable)
      for (int slot = 0; slot < kBlockSize; ++slot) {
        const int from = kCols * (slot >> 2);
        const int r = slot & 3;
        const int at = __shfl(r < 2 ? (r ? pos[1] : pos[0]) : (r == 2 ? pos[2] : pos[3]), from);
        const float wt = __shfl(r < 2 ? (r ? p[1] : p[0]) : (r == 2 ? p[2] : p[3]), from + col);
        if (at < lim) {
          const f4_t* v = reinterpret_cast<const f4_t*>(vb + slot * kHeadDim);
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) {
            const f4_t lo = v[rr], hi = v[16 + rr];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              acc[e][rr] = fmaf(wt, lo[e], acc[e][rr]);
              acc[4 + e][rr] = fmaf(wt, hi[e], acc[4 + e][rr]);
            }
          }
        }
      }
    }
    issue_v(next);   // the V registers are free
    blk = next;
  }

  // The waves' results: lane l holds dims 16 grp + 4 r + t, and 64 more, of column col.
  float l_col = l_part;
  l_col += __shfl_xor(l_col, 16);
  l_col += __shfl_xor(l_col, 32);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float* o = &s_o[w][col][16 * grp + 4 * r];
    *reinterpret_cast<f4_t*>(o) = f4_t{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
    *reinterpret_cast<f4_t*>(o + 64) = f4_t{acc[4][r], acc[5][r], acc[6][r], acc[7][r]};
  }
  if (grp == 0) {
    s_m[w][col] = m_ref;
    s_l[w][col] = l_col;
  }
  __syncthreads();
  for (int i = tid; i < kCols * (kHeadDim / 4); i += kThreads) {
    const int c = i / (kHeadDim / 4), d = 4 * (i % (kHeadDim / 4));
    const int j = c / G;
    if (j >= u.rows) continue;
    // splits of this row alone (the unit's last rows may reach one more)
    const int nsp = max(1, ((seen(u, j) + kBlockSize - 1) / kBlockSize + a.split_blocks - 1) / a.split_blocks);
    if (sp >= nsp) continue;
    float M = kNoMax;
#pragma unroll
    for (int x = 0; x < kWaves; ++x) M = fmaxf(M, s_m[x][c]);
    float L = 0.0f;
    f4_t A = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      const float wt = fast_exp2(s_m[x][c] - M);
      L = fmaf(s_l[x][c], wt, L);
      const f4_t o = *reinterpret_cast<const f4_t*>(&s_o[x][c][d]);
#pragma unroll
      for (int e = 0; e < 4; ++e) A[e] = fmaf(o[e], wt, A[e]);
    }
    const size_t qh = (size_t)(u.row0 + j) * Hq + u.g * G + c % G;
    if (nsp == 1) {
      f4_t o = {0.0f, 0.0f, 0.0f, 0.0f};
      if (L > 0.0f) {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = A[e] / L;
      }
      *reinterpret_cast<f4_t*>(static_cast<float*>(a.out) + qh * kHeadDim + d) = o;
    } else {
      const size_t slot = qh * a.n_split_max + sp;
      *reinterpret_cast<f4_t*>(a.ws_acc + slot * kHeadDim + d) = A;
      if (d == 0) {
        a.ws_ml[2 * slot] = M;
        a.ws_ml[2 * slot + 1] = L;
      }
    }
  }
}

// Units of one launch (its threads must stay below 2^32).
constexpr long long kMaxUnitsPerLaunch = 1 << 22;

template <int G>
hipError_t launch_group(DecodeArgs a, hipStream_t stream) {
  constexpr int kPos = kCols / G;
  const F32ChunkPlan plan = plan_f32_chunks(a.num_rows, a.num_seqs, a.max_q_len, a.num_kv_heads, kPos,
                                            longest_blocks(a.max_ctx, a.max_blocks_per_seq), a.split_blocks,
                                            stream_compute_units(stream));
  if (plan.units > 0x7fffffffLL) return hipErrorInvalidValue;
  a.tiles_per_seq = plan.tiles_per_seq;
  a.split_blocks = plan.split_blocks;
  for (long long u0 = 0; u0 < plan.units; u0 += kMaxUnitsPerLaunch) {
    const dim3 grid((unsigned)std::min(plan.units - u0, kMaxUnitsPerLaunch), (unsigned)plan.splits);
    if (plan.tiles_per_seq == 0)
      hipLaunchKernelGGL((prefill_f32_kernel<G, true>), grid, dim3(kThreads), 0, stream, a, (int)u0);
    else
      hipLaunchKernelGGL((prefill_f32_kernel<G, false>), grid, dim3(kThreads), 0, stream, a, (int)u0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return plan.splits > 1 ? launch_f32_merge(a, stream) : hipSuccess;
}

}  // namespace

hipError_t launch_prefill_f32(const DecodeArgs& a, int group, hipStream_t stream) {
  switch (group) {
    case 1: return launch_group<1>(a, stream);
    case 2: return launch_group<2>(a, stream);
    case 4: return launch_group<4>(a, stream);
    case 8: return launch_group<8>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bros
