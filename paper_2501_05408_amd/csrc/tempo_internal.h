// Internal declarations shared by the translation units of libtempo.
// Nothing here crosses the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tempo.h"

namespace tempo {

// ---- block-store layout ----------------------------------------------------
// Offsets are in elements, inside the tile of one (block, kv head) pair, which
// holds block_size * head_dim elements.

// f32: row-major [slot][d].
__host__ __device__ inline int64_t tile_off_f32(int D, int slot, int d) {
  return (int64_t)slot * D + d;
}

// bf16 keys.  Groups of 32 slots; a group is 2 row-tiles (slots 0..15, 16..31)
// x D/32 contraction steps, each a 1 KiB unit of 64 lanes x 8 elements: lane
// (row + 16*c) holds dims 32*s + 8*c .. +7 of slot `row` of the tile.  That is
// the A-operand image of a 16x16x32 MFMA (rows = slots, contraction = dims).
__host__ __device__ inline int64_t tile_off_k_bf16(int D, int slot, int d) {
  const int grp = slot >> 5, u = slot & 31, tile = u >> 4, row = u & 15;
  const int s = d >> 5, c = (d & 31) >> 3, e = d & 7;
  return (int64_t)grp * 32 * D + (int64_t)(((tile * (D >> 5) + s) * 64) + c * 16 + row) * 8 + e;
}

// bf16 values.  Same groups of 32 slots; a group is D/16 column-tiles, each a
// 1 KiB unit: lane (n + 16*c) holds dim 16*dt + n of the 8 slots
// {4c..4c+3, 16+4c..16+4c+3}.  That is the B-operand image of a 16x16x32 MFMA
// (contraction = slots, columns = dims) whose contraction order matches the
// accumulator image of the two key row-tiles above.
__host__ __device__ inline int64_t tile_off_v_bf16(int D, int slot, int d) {
  const int grp = slot >> 5, u = slot & 31, half = u >> 4, uu = u & 15;
  const int c = uu >> 2, e = (uu & 3) + 4 * half;
  const int dt = d >> 4, n = d & 15;
  return (int64_t)grp * 32 * D + (int64_t)((dt * 64) + c * 16 + n) * 8 + e;
}

__host__ __device__ inline int clamp_block(int phys, int num_blocks) {
  return phys < 0 ? 0 : (phys >= num_blocks ? num_blocks - 1 : phys);
}

// ---- rotary embedding of one (i, i + D/2) pair ---------------------------------
// Every kernel that rotates uses these two expressions, so the fused and the
// separate launches store the same bits: one product, then one fused multiply-add.
__device__ inline float rope_lo(float lo, float hi, float c, float s) { return fmaf(-hi, s, lo * c); }
__device__ inline float rope_hi(float lo, float hi, float c, float s) { return fmaf(lo, s, hi * c); }

// ---- kernel parameter blocks -------------------------------------------------
struct StoreParams {
  void* k_pool;
  void* v_pool;
  const int32_t* block_table;
  const int32_t* t_per_seq;  // may be null
  int32_t t;                 // uniform step / upper bound
  int32_t z_log2;
  int32_t max_blocks_per_seq;
  int32_t tile_mask;         // ring_blocks-1 for a ring store, INT32_MAX otherwise: table column = tile & mask
  int32_t num_blocks;
  int32_t Hkv;
  int32_t batch;
  int32_t count;             // append: consecutive steps per sequence, rows [B][count][Hkv][D]
  int32_t src_steps;         // steps per sequence in the caller's k_new / v_new (>= count; == count normally)
  const int32_t* count_per_seq;  // may be null; sequence b writes only its first count_per_seq[b] rows
  const float* rope_cos;     // bf16 append: non-null = keys arrive unrotated and are turned to their step's
  const float* rope_sin;     //   position on the way into the store ([positions][D/2] tables)
};

// What only the staging of a prompt on a ring store needs (bf16): the groups' images go here,
// [batch][Hkv][stage_groups] groups from that of step t on, not into the pool, which is only read.
struct StageParams : StoreParams {
  void* k_stage;
  void* v_stage;
  int32_t stage_groups;
};

struct AttnParams {
  void* k_pool;              // written only when k_new is set
  void* v_pool;
  const int32_t* block_table;
  const void* q;
  const void* k_new;         // [B][io_steps][Hkv][D]; non-null: the rows of the call's steps, which the attention
                             //   kernel appends (io_steps == 1, or a prompt from step 0 on)
  const void* v_new;
  const int32_t* t_per_seq;  // may be null
  const int32_t* count_per_seq;  // prompt kernel: may be null; sequence b answers only its first count_per_seq[b] steps
  const float* rope_cos;     // [positions][D/2]; non-null: q (and k_new) arrive unrotated and are
  const float* rope_sin;     //   rotated to their step's position inside the kernel
  const int32_t* worklist;   // bf16 decode kernel: may be null; [0] = number of items, then one item per
                             //   workgroup row: sequence in the low 16 bits, split in the high 16
  float* ws_ml;              // [B][C][Hq][S][2]  (running max in log2 units, running sum)
  float* ws_acc;             // [B][C][Hq][S][D]
  void* out;                 // [B][C][Hq][D]
  int32_t t;                 // uniform step / upper bound
  int32_t window;            // 0 = causal
  int32_t z_log2;
  int32_t max_blocks_per_seq;
  int32_t tile_mask;         // as in StoreParams
  int32_t num_blocks;
  int32_t Hkv;
  int32_t Hq;
  int32_t G;                 // Hq / Hkv
  int32_t tps_log2;          // log2(tokens per split); kWholeRange: not split
  int32_t num_splits;        // S: stride of the split axis in the workspace
  int32_t queries;           // C: consecutive query steps per sequence (q, out, workspace rows are [B][C][Hq])
  int32_t io_steps;          // steps per sequence in the caller's q / out ([B][io_steps][Hq][D]); the block is
                             //   `queries` consecutive ones of them (pointers pre-offset); == queries normally
  int32_t pad_t;             // padded baseline: keys up to pad_t are read and masked; 0 = none
  int32_t direct;            // 1: single split, write `out` and skip the combine
  float scale_log2e;         // s * log2(e)
};

// What only prompts need; not in AttnParams, because the decode kernel's launch is sensitive to the
// size of its arguments.
struct PromptParams : AttnParams {
  int32_t block_columns;     // (step, head) columns per workgroup; each block of them splits its own key range
  const void* k_stage;       // may be null; groups stage_first .. are read from here ([batch][Hkv][stage_groups]
  const void* v_stage;       //   group images), earlier ones from the pool
  int32_t stage_first, stage_groups;
  int32_t keep_first;        // k_new set (a prompt from step 0 on): first step that the launch writes to the store
};

// tps_log2 of a key range that is not split: steps are below 2^31, so no range crosses a multiple of it
// (one of 2^30 keys would be cut where it crosses step 2^30, which a ring store reaches).
constexpr int kWholeRange = 31;

// Last key of split `chunk`.
__host__ __device__ inline int split_end(int chunk, int tps_log2) {
  return (int)((((uint32_t)chunk + 1u) << tps_log2) - 1u);
}

// A prompt's (step, head) columns, step by step, are cut into blocks of `columns` (at least G): how many ...
__host__ __device__ inline uint32_t prompt_blocks(int queries, int G, int columns) {
  return ((uint32_t)queries * (uint32_t)G + (uint32_t)columns - 1u) / (uint32_t)columns;  // queries <= 2^24, G <= 128
}
// ... and the most steps one of them touches (a block may begin and end inside a step).
__host__ __device__ inline int prompt_block_span(int G, int columns) {
  return columns % G == 0 ? columns / G : (columns + G - 2) / G + 1;
}

// Keys that some step of a block of query steps sees.
inline int64_t block_keys(int t, int queries, int window) {
  const int64_t all = (int64_t)t + queries, windowed = (int64_t)window + queries - 1;
  return window > 0 && windowed < all ? windowed : all;
}
// Does the stream kernel (attn_stream_bf16.hip) take a bf16 block of more than 16 columns, or the one that shares
// each group among its wavefronts through LDS (attn_block_bf16.hip)?  The stream kernel has one workgroup of 8
// wavefronts per compute unit, so nothing covers its beginning and its merge (one per tile of 32 columns), and
// pairs beyond the 256 units are a second round.  Several workgroups of the other share a unit, and one split of up to
// 256 keys, or as many pairs as fill the part twice (four times up to 32 columns), needs no combine.  So it is a matter of
// how many keys pay for a round: 3684 blocks, from pools in and out of the caches, 0.2% from the faster one on the mean, 22% at
// most, where stream throughout below 65 columns was up to 2.0 times (us a call, LDS / stream, each with its plan, with the
// write: D = 128, 32 columns, 640 pairs, 256 keys 25.8 / 32.3, 257 48.8 / 35.4, 1024 pairs, 256 36.2 / 44.4; 56 columns, 512
// pairs, 150 keys 22.4 / 30.9, 1400 102 / 101; D = 64, 72 columns, 256 pairs, 208 keys 16.8 / 22.9, 290 38.4 / 30.7; 48
// columns, 768 pairs, 153 keys 22.0 / 36.1, 600 47.6 / 48.3).
// Beyond 64 columns at D = 128 registers do not hold a wavefront's accumulators.
inline bool block_streams(int D, int columns, int64_t pairs, int64_t keys) {
  const int tiles = columns <= 32 ? 0 : columns <= 64 ? 1 : 2;
  const bool wide = D == 128;
  if (wide && tiles == 2) return false;
  int64_t most;  // keys up to which the LDS kernel is the faster one
  if (pairs <= 256) {
    if (tiles == 0) most = 32;
    else if (tiles == 1) most = !wide ? 176 : pairs <= 64 ? 192 : 256;
    else most = pairs > 96 ? 256 : 65536 / pairs;
  } else if (pairs < 512) {  // a second round for some units, a combine for the LDS kernel
    if (tiles == 0) most = wide ? 224 : 32;
    else most = tiles == 1 || pairs >= 400 ? 256 : 1024;
  } else {
    const bool two_rounds = pairs == 512;
    if (tiles == 0) most = wide ? (pairs < 1024 ? 256 : 340) : two_rounds ? 32 : pairs < 1024 ? 192 : 272;
    else if (tiles == 2) most = two_rounds ? 1300 : pairs <= 768 ? 2048 : 1800;
    else if (!wide) most = two_rounds ? 640 : pairs <= 768 ? 900 : 1100;
    else most = two_rounds ? 1200 : pairs < 640 ? 1800 : pairs <= 768 ? 1200 : pairs <= 1100 ? 640 : 1000;
  }
  return keys > most;
}

// Visible range and split bookkeeping of one sequence, identical on host and device.
// With a block of C queries (steps t_b .. t_b+C-1) the range is the union of the
// queries' ranges: from the first query's lo to the last query's step.  The padded
// baseline reads on to key pad_t (masked beyond each query's own step).
struct SeqRange {
  int lo, hi, chunk0, nchunks;
};
__host__ __device__ inline SeqRange seq_range(int t_b, int window, int tps_log2, int queries = 1,
                                              int pad_t = 0) {
  SeqRange r;
  r.hi = t_b + queries - 1;
  r.hi = r.hi > pad_t ? r.hi : pad_t;
  r.lo = (window > 0 && t_b - window + 1 > 0) ? t_b - window + 1 : 0;
  r.chunk0 = r.lo >> tps_log2;
  r.nchunks = (r.hi >> tps_log2) - r.chunk0 + 1;
  return r;
}

// Launch and return the launch's own status.  hipGetLastError() is not used: it
// reports the last error of any HIP call on the thread, including benign ones
// left behind by the caller's framework (an event query that was "not ready").
template <typename... Params>
inline hipError_t launch_converted(void (*kernel)(Params...), dim3 grid, dim3 block, size_t lds,
                                   hipStream_t stream, Params... vals) {
  void* argv[] = {(void*)&vals...};
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, argv, lds, stream);
}
template <typename... Params, typename... Args>
inline hipError_t launch(void (*kernel)(Params...), dim3 grid, dim3 block, size_t lds,
                         hipStream_t stream, Args... args) {
  static_assert(sizeof...(Params) == sizeof...(Args), "kernel argument count");
  return launch_converted<Params...>(kernel, grid, block, lds, stream, static_cast<Params>(args)...);
}

// ---- launchers (defined next to their kernels) -------------------------------
hipError_t launch_append(const StoreParams& p, const void* k_new, const void* v_new, int D,
                         int dtype, hipStream_t stream);
hipError_t launch_stage(const StageParams& p, const void* k_new, const void* v_new, int D, hipStream_t stream);
hipError_t launch_gather(const StoreParams& p, void* k_out, void* v_out, int D, int dtype, int j0,
                         int count, hipStream_t stream);
hipError_t launch_partial_bf16(const AttnParams& p, int batch, int D, int grid_splits, int waves,
                               hipStream_t stream);
size_t partial_bf16_lds_bytes(int waves, int columns, int D);      // dynamic LDS of that launch
hipError_t launch_prefill_bf16(const PromptParams& p, int batch, int D, int waves, int grid_splits, hipStream_t stream);
hipError_t launch_prompt_combine(const PromptParams& p, int batch, int D, hipStream_t stream);
hipError_t launch_short_prompt_bf16(const AttnParams& p, int batch, int D, hipStream_t stream);
hipError_t launch_stream_block_bf16(const AttnParams& p, int batch, int D, int grid_splits, hipStream_t stream);
hipError_t launch_block_bf16(const AttnParams& p, int batch, int D, int grid_splits, hipStream_t stream);
hipError_t launch_partial_f32(const AttnParams& p, int batch, int D, int grid_splits, int waves,
                              hipStream_t stream);

hipError_t launch_step_f32(const AttnParams& p, int batch, int D, int grid_splits, int waves, hipStream_t stream);

hipError_t launch_rope_rotate(const float* rope_cos, const float* rope_sin, const void* x, void* y,
                              int dtype, int batch, int heads, int D, int t, const int32_t* t_per_seq,
                              hipStream_t stream);
hipError_t launch_rope_append(const StoreParams& p, const float* rope_cos, const float* rope_sin,
                              const void* k_raw, const void* v_new, int D, int dtype, hipStream_t stream);
hipError_t launch_combine(const AttnParams& p, int batch, int D, int dtype, hipStream_t stream);
hipError_t launch_worklist_build(const int32_t* t_per_seq, int batch, int t_max, int window, int tps_log2,
                                 int num_splits, int32_t* worklist, hipStream_t stream);
hipError_t launch_discounted_sum(const float* r, float* g, int batch, int T, int n, float gamma, hipStream_t stream);
int discounted_sum_max_window();
hipError_t launch_stream_read(const void* src, size_t bytes, void* sink, int workgroups,
                              hipStream_t stream);
hipError_t launch_stream_copy(const void* src, void* dst, size_t bytes, int workgroups,
                              hipStream_t stream);

}  // namespace tempo
