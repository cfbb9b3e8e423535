// Block store: in-place write of one timestep, and slice read-back.
//
// The paper's block store (Section 6) keeps a recurrent tensor in pre-allocated
// block-sized buffers that are written one timestep at a time, in place; its
// "in-place writes" kernel wrapper lets the producer write at index t directly.
// Here step t of sequence b goes to physical block block_table[b][t div Z],
// slot t mod Z (Section 4.3: tile n holds keys [nZ, (n+1)Z)).  An append may
// carry `count` consecutive steps per sequence (rows [B][count][Hkv][D]): row c
// goes to step t + c.
#include <type_traits>

#include "attn_bf16_common.h"

namespace tempo {
namespace {

// Rows of the call that sequence b writes (all of them unless per-sequence counts are given).
__device__ inline int rows_of(const StoreParams& p, int b) {
  if (!p.count_per_seq) return INT32_MAX;
  const int n = p.count_per_seq[b];
  return n < 0 ? 0 : n;
}

__device__ inline int step_of(const StoreParams& p, int b) {
  int t = p.t_per_seq ? p.t_per_seq[b] : p.t;
  t = t > p.t ? p.t : t;  // the host validated p.t; never index past it
  return t < 0 ? 0 : t;
}

// bf16: one thread per (b, c, head, d).  V is written element by element (the
// operand-major value layout interleaves 8 slots per 16-byte unit); the thread
// with d % 8 == 0 also moves the 16-byte key unit that starts at d.
template <int D>
__global__ __launch_bounds__(256) void kv_append_bf16(StoreParams p, const uint16_t* __restrict__ k_new,
                                                      const uint16_t* __restrict__ v_new) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int total = p.batch * p.count * p.Hkv * D;
  if (idx >= total) return;
  const int d = idx % D;
  const int head = (idx / D) % p.Hkv;
  const int c = (idx / (D * p.Hkv)) % p.count;
  const int b = idx / (D * p.Hkv * p.count);
  if (c >= rows_of(p, b)) return;
  const int t = step_of(p, b) + c;
  const int Z = 1 << p.z_log2;
  const int tile = t >> p.z_log2, slot = t & (Z - 1);
  const int phys = clamp_block(p.block_table[(int64_t)b * p.max_blocks_per_seq + (tile & p.tile_mask)], p.num_blocks);
  const int64_t base = ((int64_t)phys * p.Hkv + head) * Z * D;
  uint16_t* vp = static_cast<uint16_t*>(p.v_pool);
  const int64_t src = (((int64_t)b * p.src_steps + c) * p.Hkv + head) * D + d;
  vp[base + tile_off_v_bf16(D, slot, d)] = v_new[src];
  if ((d & 7) == 0) {
    uint16_t* kp = static_cast<uint16_t*>(p.k_pool);
    if (!p.rope_cos) {
      const uint4 unit = *reinterpret_cast<const uint4*>(k_new + src);
      *reinterpret_cast<uint4*>(kp + base + tile_off_k_bf16(D, slot, d)) = unit;
    } else if (d < D / 2) {  // rotary: the piece at d and its partner at d + D/2 are turned together
      u32x4 lo = *reinterpret_cast<const u32x4*>(k_new + src);
      u32x4 hi = *reinterpret_cast<const u32x4*>(k_new + src + D / 2);
      rotate_pieces(p.rope_cos, p.rope_sin, t, D / 2, d, lo, hi);
      *reinterpret_cast<u32x4*>(kp + base + tile_off_k_bf16(D, slot, d)) = lo;
      *reinterpret_cast<u32x4*>(kp + base + tile_off_k_bf16(D, slot, d + D / 2)) = hi;
    }
  }
}

// bf16, by 32-slot groups: one wavefront per (sequence, head, group) turns up to 32
// consecutive rows of k_new / v_new into the group's operand-major image and writes it as
// 1 KiB units.  Keys: every 16-byte piece of a unit is 8 consecutive dims of one row, so it
// is a gather of 16-byte pieces.  Values: a 16-byte piece holds one dim of 8 slots, so the
// 32 x D tile goes through LDS (row stride D + 2 elements, which spreads the four rows a
// column tile's lanes read over different banks).  The call's first and last group may be
// partly covered: their other slots are not written (their values go element by element), as
// another launch may write them at the same time, so one launch writes a prompt that starts or
// ends anywhere.
// StageParams: the images go to the staging area of a prompt on a ring store, the call's first group
// filled up with the history the pool holds.
template <int D, typename Params>
__global__ __launch_bounds__(64) void kv_append_groups_bf16(Params p, const uint16_t* __restrict__ k_new,
                                                            const uint16_t* __restrict__ v_new) {
  constexpr int KS = D / 32, DT = D / 16, LD = D + 2;
  constexpr bool kStage = std::is_same_v<Params, StageParams>;
  __shared__ uint16_t tile[32 * LD];
  const int lane = threadIdx.x;
  const int g = blockIdx.x, head = blockIdx.y, b = blockIdx.z;
  // slots of this group that sequence b writes: lo .. hi-1
  const int rows_b = rows_of(p, b) < p.count ? rows_of(p, b) : p.count;
  const int t0 = ((p.t >> 5) + g) << 5;                 // first step of this group
  const int first_row = t0 - p.t;                       // source row of slot 0 (negative: before the call)
  const int lo = first_row < 0 ? -first_row : 0;
  const int hi = rows_b - first_row < 32 ? rows_b - first_row : 32;
  if (hi <= lo) return;  // uniform over the workgroup
  const int Z = 1 << p.z_log2;
  const int phys = clamp_block(p.block_table[(int64_t)b * p.max_blocks_per_seq + ((t0 >> p.z_log2) & p.tile_mask)],
                               p.num_blocks);
  const int64_t base = (((int64_t)phys * p.Hkv + head) << p.z_log2) * D + (int64_t)(t0 & (Z - 1)) * D;
  uint16_t* const k_from = static_cast<uint16_t*>(p.k_pool) + base;   // what the group's other slots hold
  uint16_t* const v_from = static_cast<uint16_t*>(p.v_pool) + base;
  uint16_t *k_to = k_from, *v_to = v_from;
  if constexpr (kStage) {
    const int64_t staged = (((int64_t)b * p.Hkv + head) * p.stage_groups + g) * 32 * D;
    k_to = static_cast<uint16_t*>(p.k_stage) + staged;
    v_to = static_cast<uint16_t*>(p.v_stage) + staged;
  }
  const int64_t row0 = ((int64_t)b * p.src_steps + first_row) * p.Hkv + head;  // source row of slot 0 (rows are Hkv apart)

  // Rows outside the call are read as its nearest row (and not written), so that all of the group's
  // loads are in flight together: behind a condition each would be waited for by itself (2048 rows of
  // one sequence in 8 heads: 5.1 us with conditions, 4.4 us).
  auto row_at = [&](int slot) { return row0 + (int64_t)(slot < lo ? lo : (slot < hi ? slot : hi - 1)) * p.Hkv; };

  // values -> LDS, 16 bytes per lane and load
#pragma unroll
  for (int i = 0; i < (32 * D / 8) / 64; ++i) {
    const int piece = lane + 64 * i, row = piece / (D / 8), d8 = (piece % (D / 8)) * 8;
    const u32x4 v = *reinterpret_cast<const u32x4*>(v_new + row_at(row) * D + d8);
    uint32_t* dst = reinterpret_cast<uint32_t*>(tile + row * LD + d8);  // 4-byte aligned: LD and d8 are even
    dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
  }
  // keys: lane (row + 16c) of unit (tile, s) = dims 32s + 8c .. +7 of slot 16*tile + row
  {
    const int row = lane & 15, c = lane >> 4;
    u32x4* kp = reinterpret_cast<u32x4*>(k_to) + lane;
    u32x4 k[2][KS];
#pragma unroll
    for (int tl = 0; tl < 2; ++tl) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
        k[tl][s] = *reinterpret_cast<const u32x4*>(k_new + row_at(16 * tl + row) * D + 32 * s + 8 * c);
    }
#pragma unroll
    for (int tl = 0; tl < 2; ++tl) {
      const int slot = 16 * tl + row;
      if (p.rope_cos) {  // dims 32s + 8c .. +7 and the same + D/2: unit s + KS/2
        const int t = t0 + (slot < lo ? lo : (slot < hi ? slot : hi - 1));
#pragma unroll
        for (int s = 0; s < KS / 2; ++s) rotate_pieces(p.rope_cos, p.rope_sin, t, D / 2, 32 * s + 8 * c, k[tl][s], k[tl][s + KS / 2]);
      }
      const bool ours = slot >= lo && slot < hi, history = kStage && slot < lo;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (history) k[tl][s] = reinterpret_cast<const u32x4*>(k_from)[lane + (tl * KS + s) * 64];
        if (ours || history) kp[(tl * KS + s) * 64] = k[tl][s];
      }
    }
  }
  __syncthreads();
  // values: lane (n + 16c) of unit dt = dim 16dt + n of slots {4c..4c+3, 16+4c..16+4c+3}
  {
    const int n = lane & 15, c = lane >> 4;
    u32x4* vp = reinterpret_cast<u32x4*>(v_to) + lane;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const uint16_t* col = tile + 16 * dt + n;
      uint32_t e[8];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        e[r] = col[(4 * c + r) * LD];
        e[4 + r] = col[(16 + 4 * c + r) * LD];
      }
      u32x4 o;
      o.x = e[0] | (e[1] << 16); o.y = e[2] | (e[3] << 16);
      o.z = e[4] | (e[5] << 16); o.w = e[6] | (e[7] << 16);
      if (!kStage && (lo > 0 || hi < 32)) {  // partly covered: this call's slots only
        uint16_t* at = reinterpret_cast<uint16_t*>(vp + dt * 64);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const int slot = r < 4 ? 4 * c + r : 16 + 4 * c + (r - 4);
          if (slot >= lo && slot < hi) at[r] = (uint16_t)e[r];
        }
        continue;
      }
      if (kStage && lo > 0) {  // the history in the group's first slots (nothing is read beyond the call's last step)
        uint32_t m[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          m[r] = 4 * c + r >= lo ? 0xFFFFu : 0u;
          m[4 + r] = 16 + 4 * c + r >= lo ? 0xFFFFu : 0u;
        }
        const u32x4 old = reinterpret_cast<const u32x4*>(v_from)[lane + dt * 64];
        const uint32_t mx = m[0] | (m[1] << 16), my = m[2] | (m[3] << 16);
        const uint32_t mz = m[4] | (m[5] << 16), mw = m[6] | (m[7] << 16);
        o.x = (o.x & mx) | (old.x & ~mx); o.y = (o.y & my) | (old.y & ~my);
        o.z = (o.z & mz) | (old.z & ~mz); o.w = (o.w & mw) | (old.w & ~mw);
      }
      vp[dt * 64] = o;
    }
  }
}

// f32: one thread per float4 of (b, c, head, d..d+3); both pools are row-major.
template <int D>
__global__ __launch_bounds__(256) void kv_append_f32(StoreParams p, const float* __restrict__ k_new,
                                                     const float* __restrict__ v_new) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int total = p.batch * p.count * p.Hkv * (D / 4);
  if (idx >= total) return;
  const int d = (idx % (D / 4)) * 4;
  const int head = (idx / (D / 4)) % p.Hkv;
  const int c = (idx / ((D / 4) * p.Hkv)) % p.count;
  const int b = idx / ((D / 4) * p.Hkv * p.count);
  if (c >= rows_of(p, b)) return;
  const int t = step_of(p, b) + c;
  const int Z = 1 << p.z_log2;
  const int tile = t >> p.z_log2, slot = t & (Z - 1);
  const int phys = clamp_block(p.block_table[(int64_t)b * p.max_blocks_per_seq + (tile & p.tile_mask)], p.num_blocks);
  const int64_t off = ((int64_t)phys * p.Hkv + head) * Z * D + tile_off_f32(D, slot, d);
  const int64_t src = (((int64_t)b * p.src_steps + c) * p.Hkv + head) * D + d;
  *reinterpret_cast<float4*>(static_cast<float*>(p.k_pool) + off) =
      *reinterpret_cast<const float4*>(k_new + src);
  *reinterpret_cast<float4*>(static_cast<float*>(p.v_pool) + off) =
      *reinterpret_cast<const float4*>(v_new + src);
}

// Slice read: out[b][j - j0][head][d] for j in [j0, j0 + count).  One thread per element.
template <typename T, bool kBf16>
__global__ __launch_bounds__(256) void kv_gather(StoreParams p, T* __restrict__ k_out,
                                                 T* __restrict__ v_out, int D, int j0, int count) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)p.batch * count * p.Hkv * D;
  if (idx >= total) return;
  const int d = (int)(idx % D);
  const int head = (int)((idx / D) % p.Hkv);
  const int jj = (int)((idx / ((int64_t)D * p.Hkv)) % count);
  const int b = (int)(idx / ((int64_t)D * p.Hkv * count));
  const int j = j0 + jj;
  const int Z = 1 << p.z_log2;
  const int tile = j >> p.z_log2, slot = j & (Z - 1);
  const int phys = clamp_block(p.block_table[(int64_t)b * p.max_blocks_per_seq + (tile & p.tile_mask)], p.num_blocks);
  const int64_t base = ((int64_t)phys * p.Hkv + head) * Z * D;
  if (k_out) {
    const int64_t off = kBf16 ? tile_off_k_bf16(D, slot, d) : tile_off_f32(D, slot, d);
    k_out[idx] = static_cast<const T*>(p.k_pool)[base + off];
  }
  if (v_out) {
    const int64_t off = kBf16 ? tile_off_v_bf16(D, slot, d) : tile_off_f32(D, slot, d);
    v_out[idx] = static_cast<const T*>(p.v_pool)[base + off];
  }
}

hipError_t launch_elements_bf16(const StoreParams& p, const uint16_t* k, const uint16_t* v, int D, hipStream_t stream) {
  const int threads = 256;
  const int total = p.batch * p.count * p.Hkv * D;
  const dim3 grid((total + threads - 1) / threads);
  if (D == 128) return launch(kv_append_bf16<128>, grid, dim3(threads), 0, stream, p, k, v);
  return launch(kv_append_bf16<64>, grid, dim3(threads), 0, stream, p, k, v);
}

}  // namespace

hipError_t launch_append(const StoreParams& p, const void* k_new, const void* v_new, int D,
                         int dtype, hipStream_t stream) {
  // bf16, uniform first step, at least one whole 32-slot group: the group kernel (4096 rows of 16
  // sequences in 8 heads: 86 us, element-wise 315 us).  Rows that fill no group go element by
  // element, as the group kernel's work for a partly covered group is that of a whole one.
  const int first_whole = (p.t + 31) >> 5, past_whole = (p.t + p.count) >> 5;
  if (dtype == TEMPO_BF16 && !p.t_per_seq && p.count >= 32 && past_whole > first_whole) {
    const int groups = ((p.t + p.count - 1) >> 5) - (p.t >> 5) + 1;
    // A ring whose every slot is written, from the middle of a group on: the last group lies in the
    // same slots as the first.  Its rows go in a launch behind the others.
    const int64_t ring_slots = p.tile_mask == INT32_MAX ? INT64_MAX : ((int64_t)p.tile_mask + 1) << p.z_log2;
    if ((int64_t)groups * 32 > ring_slots) {
      StoreParams rest = p;
      rest.count = p.count - 32;
      hipError_t e = launch_append(rest, k_new, v_new, D, dtype, stream);
      if (e != hipSuccess) return e;
      rest.t = p.t + rest.count;
      rest.count = 32;
      const int64_t skip = (int64_t)(p.count - 32) * p.Hkv * D;
      return launch_elements_bf16(rest, static_cast<const uint16_t*>(k_new) + skip,
                                  static_cast<const uint16_t*>(v_new) + skip, D, stream);
    }
    const dim3 grid(groups, p.Hkv, p.batch);
    const uint16_t* k = static_cast<const uint16_t*>(k_new);
    const uint16_t* v = static_cast<const uint16_t*>(v_new);
    if (D == 128) return launch((kv_append_groups_bf16<128, StoreParams>), grid, dim3(64), 0, stream, p, k, v);
    return launch((kv_append_groups_bf16<64, StoreParams>), grid, dim3(64), 0, stream, p, k, v);
  }
  if (dtype == TEMPO_BF16)
    return launch_elements_bf16(p, static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new), D, stream);
  const int threads = 256;
  const int total = p.batch * p.count * p.Hkv * (D / 4);
  const dim3 grid((total + threads - 1) / threads);
  const float* k = static_cast<const float*>(k_new);
  const float* v = static_cast<const float*>(v_new);
  if (D == 128) return launch(kv_append_f32<128>, grid, dim3(threads), 0, stream, p, k, v);
  return launch(kv_append_f32<64>, grid, dim3(threads), 0, stream, p, k, v);
}

// The rows' group images to p.k_stage / p.v_stage (p.stage_groups groups per sequence and head).
hipError_t launch_stage(const StageParams& p, const void* k_new, const void* v_new, int D, hipStream_t stream) {
  const int groups = ((p.t + p.count - 1) >> 5) - (p.t >> 5) + 1;
  if (groups != p.stage_groups || p.t_per_seq || p.rope_cos) return hipErrorInvalidConfiguration;
  const dim3 grid(groups, p.Hkv, p.batch);
  const uint16_t* k = static_cast<const uint16_t*>(k_new);
  const uint16_t* v = static_cast<const uint16_t*>(v_new);
  if (D == 128) return launch((kv_append_groups_bf16<128, StageParams>), grid, dim3(64), 0, stream, p, k, v);
  return launch((kv_append_groups_bf16<64, StageParams>), grid, dim3(64), 0, stream, p, k, v);
}

hipError_t launch_gather(const StoreParams& p, void* k_out, void* v_out, int D, int dtype, int j0,
                         int count, hipStream_t stream) {
  const int threads = 256;
  const int64_t total = (int64_t)p.batch * count * p.Hkv * D;
  if (total == 0) return hipSuccess;
  const dim3 grid((unsigned)((total + threads - 1) / threads));
  if (dtype == TEMPO_BF16) {
    return launch((kv_gather<uint16_t, true>), grid, dim3(threads), 0, stream, p,
                       static_cast<uint16_t*>(k_out), static_cast<uint16_t*>(v_out), D, j0, count);
  } else {
    return launch((kv_gather<float, false>), grid, dim3(threads), 0, stream, p,
                       static_cast<float*>(k_out), static_cast<float*>(v_out), D, j0, count);
  }
}

}  // namespace tempo
