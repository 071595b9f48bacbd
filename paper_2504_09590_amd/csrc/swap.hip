// Lazy checkpointing on gfx950 (Sec. 5.2; the fetch/store kernels of Sec. 6):
// move the K/V rows of a list of slots between the pool and a dense buffer.
//
//   gather:  out[i][h][:] = pool[id_i / 16][h][id_i % 16][:]   (zero row when
//            id_i lies outside the pool)
//   scatter: pool[id_i / 16][h][id_i % 16][:] = in[i][h][:]     (skipped when
//            id_i lies outside the pool)
//
// for every KV head h, on both tensors. The dense side has the layout of a
// step's new tokens, [n][Hkv][D], so a checkpoint is one contiguous buffer
// that an asynchronous copy moves to or from pinned host memory while the
// compute units run attention. Pure byte movement in 16-byte chunks; each
// thread requests all of its chunks before it stores any. A workgroup moves
// whole ids of one tensor, as many as one pass of its threads holds (or one id
// in several passes), so a chunk's place takes 32-bit arithmetic and no
// division; with 64-bit divisions per chunk the index arithmetic took as long
// as the bytes: 4096 slots of 8 KV heads (16.8 MB read, 16.8 MB written) 13.0 us a
// gather and 12.6 a scatter, now 8.8 and 7.6 (3.8 and 4.4 TB/s moved); 64
// slots 7.4 us, now 4.4 and 3.6.
#include "bros_device.h"
#include "bros_kernels.h"

#include <algorithm>

namespace bros {
namespace {

constexpr int kThreads = 256;
constexpr int kIter = 8;   // 16-byte chunks per thread

typedef unsigned v4u_t __attribute__((ext_vector_type(4)));

// ITERS: chunks per thread, kIter, or 1 for a list that one per thread covers (a
// slot or a few: seven rounds of index arithmetic less, a gather 3.8 us -> 3.0).
template <bool GATHER, int ROW_CHUNKS, int ITERS>
__global__ __launch_bounds__(kThreads) void kv_move_kernel(KvMoveArgs a, int ids_per_group, float rcp) {
  const int tid = threadIdx.x;
  const int per_id = a.num_kv_heads * ROW_CHUNKS;          // chunks of an id's rows of one tensor
  const int i0 = blockIdx.x * ids_per_group;
  const int n = min(ids_per_group, a.num_slots - i0) * per_id;
  const int64_t pool_slots = (int64_t)a.num_blocks * kBlockSize;
  const bool v = blockIdx.y != 0;
  uint8_t* pool = static_cast<uint8_t*>(v ? a.v_pool : a.k_pool);
  uint8_t* dense = static_cast<uint8_t*>(v ? a.v_dense : a.k_dense) + (size_t)i0 * per_id * 16;

  for (int base = 0; base < n; base += kThreads * ITERS) {
    v4u_t data[ITERS];
    int64_t at[ITERS];   // byte offset of the chunk in the pool, -1 when its id lies outside
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int c = min(base + it * kThreads + tid, n - 1);
      const int i = div_small(c, per_id, rcp);
      const int rem = c - i * per_id;
      const int h = rem / ROW_CHUNKS, cc = rem % ROW_CHUNKS;   // (shifts)
      const int sid = a.slot_ids[i0 + i];
      at[it] = sid >= 0 && sid < pool_slots
                   ? ((((int64_t)(sid / kBlockSize) * a.num_kv_heads + h) * kBlockSize + sid % kBlockSize) * ROW_CHUNKS + cc) * 16
                   : -1;
      if (!GATHER) data[it] = *reinterpret_cast<const v4u_t*>(dense + (size_t)c * 16);
    }
    if (GATHER) {
#pragma unroll
      for (int it = 0; it < ITERS; ++it) {
        data[it] = v4u_t{0u, 0u, 0u, 0u};
        if (at[it] >= 0) data[it] = *reinterpret_cast<const v4u_t*>(pool + at[it]);
      }
    }
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int c = base + it * kThreads + tid;
      if (c >= n) continue;
      if (GATHER) *reinterpret_cast<v4u_t*>(dense + (size_t)c * 16) = data[it];
      else if (at[it] >= 0) *reinterpret_cast<v4u_t*>(pool + at[it]) = data[it];
    }
  }
}

}  // namespace

template <bool GATHER>
static hipError_t launch_move(const KvMoveArgs& a, hipStream_t stream) {
  const int row_chunks = a.row_bytes / 16;
  const int per_id = a.num_kv_heads * row_chunks;
  const int ids = std::max(1, kThreads * kIter / per_id);   // one pass per workgroup where an id's rows fit one
  const int64_t groups = ((int64_t)a.num_slots + ids - 1) / ids;
  if (groups == 0) return hipSuccess;
  if (groups > 0x7fffffffLL / kThreads) return hipErrorInvalidValue;
  const dim3 grid((unsigned)groups, 2);
  const float rcp = 1.0f / (float)per_id;
  const bool few = (int64_t)a.num_slots * per_id <= kThreads;
  if (row_chunks == kHeadDim * 2 / 16) {
    if (few) hipLaunchKernelGGL((kv_move_kernel<GATHER, kHeadDim * 2 / 16, 1>), grid, dim3(kThreads), 0, stream, a, ids, rcp);
    else hipLaunchKernelGGL((kv_move_kernel<GATHER, kHeadDim * 2 / 16, kIter>), grid, dim3(kThreads), 0, stream, a, ids, rcp);
  } else if (row_chunks == kHeadDim * 4 / 16) {
    if (few) hipLaunchKernelGGL((kv_move_kernel<GATHER, kHeadDim * 4 / 16, 1>), grid, dim3(kThreads), 0, stream, a, ids, rcp);
    else hipLaunchKernelGGL((kv_move_kernel<GATHER, kHeadDim * 4 / 16, kIter>), grid, dim3(kThreads), 0, stream, a, ids, rcp);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_kv_move(const KvMoveArgs& a, bool gather, hipStream_t stream) {
  return gather ? launch_move<true>(a, stream) : launch_move<false>(a, stream);
}

}  // namespace bros
