// Internal launch interface between the C ABI layer (api.cpp) and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace bros {

struct KvWriteArgs {
  const void* k_new;
  const void* v_new;
  void* k_pool;
  void* v_pool;
  const int32_t* block_tables;
  const int8_t* dir;
  const uint8_t* cls;
  const int32_t* pos0;
  const int32_t* cu_new;
  int32_t dir_per_entry;  // dir is [S][max_blocks_per_seq] (else [S])
  int32_t num_new_tokens;
  int32_t num_seqs;
  int32_t num_blocks;
  int32_t max_blocks_per_seq;
  int32_t num_kv_heads;
};

// Decode rows (cu_q == nullptr): row r is sequence r with context ctx_lens[r].
// For the fp32 prefill chunks (cu_q != nullptr): row r belongs to the sequence s
// with cu_q[s] <= r < cu_q[s+1] and sees the first ctx_lens[s] - (cu_q[s+1] -
// r) + 1 positions (causal, diagonal inclusive).
struct DecodeArgs {
  void* out;
  const void* q;
  const void* k_pool;
  const void* v_pool;
  const int32_t* block_tables;
  const int8_t* dir;
  const uint8_t* cls;
  const int32_t* ctx_lens;
  const int32_t* cu_q;
  int32_t dir_per_entry;  // dir is [S][max_blocks_per_seq] (else [S])
  // Partial results. fp32: [rows][Hq][n_split_max] slots. bf16, even split (one
  // worker per wave over an even share of the tiles): slot (row * Hkv + g +
  // worker) * G + head-in-group, for segments cut between workers. bf16, pieces
  // (decode_short.hip): slot ((row * Hkv + g) * n_split_max + piece) * G + head-in-group.
  float* ws_acc;          // [slots][D] unnormalised partial outputs
  float* ws_ml;           // [slots][2] (running max in log2 units, sum)
  int32_t* ws_rows;       // bf16: first tile of each row, [rows + 1]
  int32_t* ws_cut;        // bf16: per worker, [2 w] the (row * Hkv + g) segment it starts and leaves cut, else -1;
                          // [2 w + 1] the worker holding that segment's last tile, or -1 if not computed
  int32_t* ws_wstart;     // bf16: [0] workers W, then [1 + w] first tile of worker w (w <= W)
  int32_t num_workers;    // bf16: waves of the grid (workers beyond the tile count idle)
  int32_t num_rows;
  int32_t num_seqs;
  int32_t num_blocks;
  int32_t max_blocks_per_seq;
  int32_t max_ctx;
  int32_t num_q_heads;
  int32_t num_kv_heads;
  int32_t split_blocks;   // blocks per split: fp32, from the plan's (multiple of 4, <= 64), of which a launch may
                          // take several at once; bf16 whole segments and pieces
  int32_t n_split_max;    // fp32: splits the workspace is laid out for; bf16 pieces: pieces of the longest context
  int32_t max_q_len;      // fp32 chunks: host bound of a sequence's rows
  int32_t tiles_per_seq;  // fp32 chunks: units of a sequence per KV head (set by the launch)
  float scale_log2;       // softmax scale * log2(e)
};

struct PrefillArgs {
  void* out;
  const void* q;
  const int32_t* cu_q;
  const void* k_pool;
  const void* v_pool;
  const int32_t* block_tables;
  const int8_t* dir;
  const uint8_t* cls;
  const int32_t* ctx_lens;
  int32_t dir_per_entry;  // dir is [S][max_blocks_per_seq] (else [S])
  int32_t num_q_tokens;
  int32_t num_seqs;
  int32_t num_blocks;
  int32_t max_blocks_per_seq;
  int32_t max_ctx;
  int32_t num_q_heads;
  int32_t num_kv_heads;
  int32_t tiles_per_seq;  // ceil(max_q_len / positions per tile)
  float scale_log2;
  // Splitting long units into pieces over key ranges (none when num_cus is 0):
  // the compute units the work is spread over, the partials of split units in
  // fp32, [ws_slots] x (ws_o: the unit's 128 x 128 accumulators as its four
  // waves hold them, ws_ml: [128 rows] max and sum), and the list of split units that the merge walks (count, then (item, parts,
  // first slot) triples).
  int32_t num_cus;
  int32_t xcd_cus;        // compute units per XCD when the launch has the whole chip, else 0
  int32_t ws_slots;
  float* ws_o;
  float* ws_ml;
  int32_t* ws_list;
};

// Rows of a list of slots moved between the pool and a dense [n][Hkv][D]
// buffer (gather: pool -> dense, scatter: dense -> pool).
struct KvMoveArgs {
  void* k_pool;           // gather source / scatter destination (only read by the gather)
  void* v_pool;
  void* k_dense;          // gather destination / scatter source (only read by the scatter)
  void* v_dense;
  const int32_t* slot_ids;
  int32_t num_slots;
  int32_t num_blocks;
  int32_t num_kv_heads;
  int32_t row_bytes;      // head_dim * element bytes (a multiple of 16)
};

// Decode planning shared by the launcher and the workspace query.
struct DecodePlan {
  int32_t split_blocks;
  int32_t n_split_max;
};
DecodePlan plan_decode(int32_t num_rows, int32_t max_ctx);
size_t decode_workspace_bytes(int32_t num_rows, int32_t num_q_heads, int32_t max_ctx, bool bf16);
// Points the workspace fields of `a` (num_rows, num_q_heads, n_split_max set)
// into `ws`, laid out as decode_workspace_bytes sized it.
void set_decode_workspace(DecodeArgs& a, void* ws, bool bf16);

hipError_t launch_kv_write(const KvWriteArgs& a, bool bf16, hipStream_t stream);
hipError_t launch_kv_move(const KvMoveArgs& a, bool gather, hipStream_t stream);
hipError_t launch_decode(DecodeArgs a, int group, bool bf16, hipStream_t stream);
hipError_t launch_prefill_f32(const DecodeArgs& a, int group, hipStream_t stream);
// The bf16 decode of short contexts or few segments (decode_short.hip): whether
// it is better on the stream's compute units than the even split and its merge, and if so its
// splits (split_blocks, n_split_max). `between`, if any, is recorded before its merge.
bool plan_decode_short(DecodeArgs& a, hipStream_t stream);
hipError_t launch_decode_short(const DecodeArgs& a, int group, hipStream_t stream, hipEvent_t between);
// Groups of query heads for which the bf16 decode's workspace holds partials
// beyond one per row: the waves of its largest grid.
constexpr int32_t kDecodeGroupSlots = 4096;
// Events the bf16 decode records around its decode kernel (both null: none).
void set_decode_kernel_events(hipEvent_t before, hipEvent_t after);
// Longest context whose block table the matrix-core prefill stages whole in
// LDS; longer ones run its ring variant.
constexpr int32_t kPrefillWholeTableCtx = 32768;
// Compute units enabled for `stream` (a stream made with
// hipExtStreamCreateWithCUMask runs on a subset of the device): the device's
// count is queried once per device, the stream's CU mask read on every call.
int stream_compute_units(hipStream_t stream);
// Workgroups of `kernel` (launched with `threads` threads) that a compute unit
// holds at once, queried once per device and cache slot (0..7: bf16 decode 0..3,
// fp32 decode 4..7), and that those enabled for `stream` do.
int workgroups_per_cu(const void* kernel, int threads, int slot);
int resident_workgroups(const void* kernel, int threads, int slot, hipStream_t stream);

hipError_t launch_prefill_mfma(PrefillArgs a, int group, int num_tiles_total, hipStream_t stream);
// The merge of the bf16 decode's cut segments (after a decode or a fused launch).
hipError_t launch_decode_merge(const DecodeArgs& a, int group, hipStream_t stream);

// Expected times that place the decode work of a fused prefill|decode launch:
// a prefill unit costs unit_fixed_us + unit_tile_us per key tile on its
// workgroup, a decode tile decode_tile_us on one worker (wave). Every worker
// gets decode tiles in proportion to the time its workgroup has left after
// its prefill unit, so that all end together.
struct MixedModel {
  float unit_fixed_us;
  float unit_tile_us;
  float decode_tile_us;
};
// One launch over the concatenated batch (Sec. 6): workgroup b first runs
// prefill unit b of the matrix-core prefill (no splitting), then its waves
// take their share of the bf16 decode tiles; then the decode merge. pa is set
// up as for launch_prefill_mfma (its workspace fields unused), da as for
// launch_decode with its workspace. Returns hipErrorInvalidValue when the
// prefill units (num_units) exceed the grid or their items exceed what the
// planner ranks; the caller then runs the two calls in turn.
hipError_t launch_mixed(PrefillArgs pa, DecodeArgs da, MixedModel mm, int group, int num_units, hipStream_t stream);
int prefill_positions_per_tile(int group);
// Workspace of the matrix-core prefill (optional: without it no unit is split).
// With `whole`, only one of at least prefill_workspace_bytes() is used; else
// any, for as many partials as it holds.
size_t prefill_workspace_bytes();
void set_prefill_workspace(PrefillArgs& a, void* ws, size_t bytes, bool whole);

}  // namespace bros
