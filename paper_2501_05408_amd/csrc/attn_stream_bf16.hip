// Blocks against a long history, bf16, MFMA on gfx950: 17 .. 64 columns (D = 64: .. 128) of one or a few
// query steps in front of a long key range.  Computes what the decode kernel computes for each of those
// steps (Section 2, Eq. 1; Section 4.3 index masks).
//
// Mapping.  As the decode kernel: one workgroup = one (sequence, kv head, split); its wavefronts take the
// split's 32-slot groups round-robin and stream keys and values from the store straight into operand
// registers, one register image each, refilled in halves.  But a wavefront has ALL of the block's columns,
// 32 to a tile: logits = K * Q^T and outputs = V^T * P^T as 32x32x16 products, so every key/value is read
// by one wavefront, once, and no copy in LDS, barrier or other wavefront stands between its loads.  Two
// units of the store side by side are such an operand (four runs of 256 bytes per load).  The queries, the
// same for all wavefronts, are read from LDS.  At the end the wavefronts are merged through LDS, tile by tile.
//
// What bounds it.  HBM, then what precedes a workgroup's first group and follows its last one (about 3.4 us; the
// merge area of 134 KiB at D = 128 leaves a compute unit one workgroup, of 8 wavefronts).  21 steps of 3 heads, 16
// sequences, t = 4075: 49.4 us (5.4 TB/s), 53.1 with the combine, where the kernel that shares each group among its
// wavefronts through LDS takes 53.5 and 59.5; over 396 blocks of 18 to 126 columns behind 150 to 8000 keys, with the
// plans of each, 1.32 times as fast on the geometric mean.  Both tiles' logits before the first tile's softmax, which
// frees the key registers earlier, gained nothing (58.3 / 58.6 a call with its write).
#include "attn_bf16_columns32.h"

namespace tempo {
namespace {

constexpr int kTileColumns = 32;

typedef const __attribute__((address_space(1))) char* global_bytes;
typedef const __attribute__((address_space(1))) u32x4* global_u32x4;

template <int D, int TILES, int NW, bool kRope>
__global__ __launch_bounds__(64 * NW, 2) void attn_stream_bf16(AttnParams p) {
  constexpr int KT = D / 16;                  // 16-dim contraction steps of the logits
  constexpr int OT = D / 32;                  // 32-dim tiles of the output
  constexpr int LD = D + 4;                   // row stride of the merge area (columns on different banks)
  extern __shared__ u32x4 lds[];              // queries [TILES][KT][64] x 16 bytes; later the merge area
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5;
  BlockWork work;
  work.hkv = blockIdx.x;
  work.b = blockIdx.y;
  work.c0 = work.skip = 0;
  work.steps = work.all_steps = p.queries;
  work.ncols = p.queries * p.G;
  work.any = true;
  cut_range(p, work, (int)blockIdx.z);
  if (!work.any) return;                       // uniform over the workgroup
  const int b = work.b, hkv = work.hkv, ncols = work.ncols, start = work.start, t_last = work.t_last;

  // Lane (slot & 15) + 16 (2 (s & 1) + half) of unit (slot / 16, s / 2), slot = lane & 31: key operand s.  Lane
  // (dim & 15) + 16 (2 chunk + half) of unit 2 ot + dim / 16, dim = lane & 31: value operand (ot, chunk).
  // (Byte offsets of 32 bits beside an address in scalar registers.)
  const uint32_t k_lane = 16u * (uint32_t)(((lane >> 4) & 1) * (D / 32) * 64 + (lane & 15) + 16 * half);
  const uint32_t v_lane = 16u * (uint32_t)(((lane >> 4) & 1) * 64 + (lane & 15) + 16 * half);
  u32x4 kreg[KT], vreg[2 * OT];
  auto load_k = [&](int64_t base) {
    const global_bytes from = (global_bytes)p.k_pool + 2 * base;
    uint32_t at = k_lane;
    asm volatile("" : "+v"(at));               // (pool + lane's part, kept across the loop, would be two more registers)
#pragma unroll
    for (int s = 0; s < KT; ++s)
      kreg[s] = __builtin_nontemporal_load((global_u32x4)(from + (at + 1024u * (s >> 1) + 512u * (s & 1))));
  };
  auto load_v = [&](int64_t base) {
    const global_bytes from = (global_bytes)p.v_pool + 2 * base;
    uint32_t at = v_lane;
    asm volatile("" : "+v"(at));               // (pool + lane's part, kept across the loop, would be two more registers)
#pragma unroll
    for (int i = 0; i < 2 * OT; ++i)
      vreg[i] = __builtin_nontemporal_load((global_u32x4)(from + (at + 2048u * (i >> 1) + 512u * (i & 1))));
  };
  int grp = work.g_first + wave;
  if (grp <= work.g_last) {
    const int64_t base = group_base<D>(p, b, hkv, grp);
    load_k(base);
    load_v(base);
  }

  // The query operand of this lane's column in each tile (lane half h: dims 16 s + 8 h .. +7) into LDS.
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
    const LaneColumn mine = lane_column(p, work, kTileColumns * i + (lane & 31));
    const uint16_t* qp = static_cast<const uint16_t*>(p.q) +
                         (((int64_t)b * p.io_steps + mine.cq) * p.Hq + (int64_t)hkv * p.G + mine.gq) * D + 8 * half;
    const bool used = kTileColumns * i + (lane & 31) < ncols;
    constexpr u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int s = 0; s < KT / 2; ++s) {
      if ((i * (KT / 2) + s) % NW != wave) continue;
      u32x4 low = *reinterpret_cast<const u32x4*>(qp + 16 * s), high = *reinterpret_cast<const u32x4*>(qp + 16 * s + D / 2);
      if (kRope) rotate_pieces(p.rope_cos, p.rope_sin, mine.step, D / 2, 16 * s + 8 * half, low, high);
      lds[(i * KT + s) * 64 + lane] = used ? low : zero;
      lds[(i * KT + s + KT / 2) * 64 + lane] = used ? high : zero;
    }
  }
  auto meet = [&]() {                          // (not __syncthreads(), which would also wait for the loads in flight)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  meet();

  float m_run[TILES], l_run[TILES], base_run[TILES], limit[TILES];
  f32x16 acc[TILES][OT];                       // dims 32 ot + 8 (r / 4) + 4 h + (r mod 4) of this lane's column
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
    m_run[i] = limit[i] = -INFINITY;
    l_run[i] = base_run[i] = 0.f;
#pragma unroll
    for (int ot = 0; ot < OT; ++ot) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][ot][r] = 0.f;
    }
  }
  // The groups no column's range cuts.
  const int lo_last = (p.window > 0 && t_last - p.window + 1 > start) ? t_last - p.window + 1 : start;
  const int hi_min = work.t_first < work.end ? work.t_first : work.end;
  const int first_whole = (lo_last + 31) >> 5, last_whole = ((hi_min + 1) >> 5) - 1;

  auto group = [&](int nxt, bool more) __attribute__((always_inline)) {  // group grp; `more`: and request group nxt
    const int64_t base_nxt = more ? group_base<D>(p, b, hkv, nxt) : 0;  // scalar loads, off the vector path
    const bool cut = grp < first_whole || grp > last_whole;             // wave-uniform
    u32x4 pa[TILES][2];
#pragma unroll
    for (int i = 0; i < TILES; ++i) {
      f32x16 x;
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = 0.f;
#pragma unroll
      for (int s = 0; s < KT; ++s) {
        x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kreg[s]), as_bf16x8(lds[(i * KT + s) * 64 + lane]), x, 0, 0, 0);
        if (TILES > 1 && (s & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
      if (TILES > 1) __builtin_amdgcn_sched_barrier(0);
      if (i == TILES - 1 && more) load_k(base_nxt);  // the key registers are free again
      if (cut) {  // (the column's range is worked out anew, here: few groups are cut, and registers are what lacks)
        int column = kTileColumns * i + (lane & 31);
        asm volatile("" : "+v"(column));
        const LaneColumn mine = lane_column(p, work, column);
        mask_tile(grp, mine.lo, mine.hi, lane, x);
      }
      softmax_reference<D>(tile_max(x), p.scale_log2e, limit[i], m_run[i], base_run[i], acc[i], l_run[i]);
      float even;
#pragma unroll
      for (int e = 0; e < 16; ++e) softmax_weight(x, p.scale_log2e, base_run[i], e, even, pa[i], l_run[i]);
      asm volatile("" : "+v"(l_run[i]));
      if (TILES > 1) __builtin_amdgcn_sched_barrier(0);  // one tile's logits at a time, or registers run out
    }
    uint32_t keep[2][4] = {{~0u, ~0u, ~0u, ~0u}, {~0u, ~0u, ~0u, ~0u}};
    if (cut) {  // unwritten slots may hold NaN, and 0 * NaN is NaN
#pragma unroll
      for (int chunk = 0; chunk < 2; ++chunk) value_masks(grp, start, t_last, 16 * (2 * chunk + half), keep[chunk]);
    }
#pragma unroll
    for (int chunk = 0; chunk < 2; ++chunk) {
#pragma unroll
      for (int ot = 0; ot < OT; ++ot) {
        u32x4 v = vreg[2 * ot + chunk];        // (masked in a copy, see the decode kernel)
        v.x &= keep[chunk][0]; v.y &= keep[chunk][1]; v.z &= keep[chunk][2]; v.w &= keep[chunk][3];
#pragma unroll
        for (int i = 0; i < TILES; ++i)
          acc[i][ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(v), as_bf16x8(pa[i][chunk]), acc[i][ot], 0, 0, 0);
        if (TILES > 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (more) load_v(base_nxt);                // the value registers are free again
  };
  // (the last group apart: see the decode kernel)
  for (; grp + NW <= work.g_last; grp += NW) group(grp + NW, true);
  if (grp <= work.g_last) group(grp + NW, false);

  // Wavefronts -> LDS -> one merge, tile by tile (same rule as the split combine; a column that saw no key in
  // this split leaves (-inf, 0, 0)).
  float* const sm_m = reinterpret_cast<float*>(lds);        // [NW][32]
  float* const sm_l = sm_m + NW * kTileColumns;              // [NW][32]
  float* const sm_acc = sm_l + NW * kTileColumns;            // [NW][32][LD]
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
    meet();                                    // queries, or the tile before, are read
    const float l_tot = half_sum(l_run[i]);
    if (half == 0) {
      sm_m[wave * kTileColumns + lane] = m_run[i];
      sm_l[wave * kTileColumns + lane] = l_tot;
    }
    float* const row = sm_acc + (wave * kTileColumns + (lane & 31)) * LD + 4 * half;
#pragma unroll
    for (int ot = 0; ot < OT; ++ot) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<f32x4*>(row + 32 * ot + 8 * r) =
            f32x4{acc[i][ot][4 * r], acc[i][ot][4 * r + 1], acc[i][ot][4 * r + 2], acc[i][ot][4 * r + 3]};
    }
    meet();
    const int left = ncols - kTileColumns * i, cols = left < kTileColumns ? left : kTileColumns;
    for (int idx = threadIdx.x; idx < cols * (D / 4); idx += 64 * NW) {
      const int j = idx / (D / 4), d = 4 * (idx - j * (D / 4));
      float mw[NW], lw[NW];
      f32x4 aw[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        mw[w] = sm_m[w * kTileColumns + j];
        lw[w] = sm_l[w * kTileColumns + j];
        aw[w] = *reinterpret_cast<const f32x4*>(sm_acc + (w * kTileColumns + j) * LD + d);
      }
      float M = mw[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) M = fmaxf(M, mw[w]);
      f32x4 num = {0.f, 0.f, 0.f, 0.f};
      float den = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        // saw no key of this column (by the sum: a group with a logit that is NaN leaves the reference at -inf too)
        const bool none = lw[w] == 0.f;
        const float wgt = none ? 0.f : fast_exp2(mw[w] - M);
        num += wgt * (none ? f32x4{0.f, 0.f, 0.f, 0.f} : aw[w]);
        den += none ? 0.f : wgt * lw[w];
      }
      const int column = kTileColumns * i + j, jc = column / p.G, jg = column - jc * p.G;
      if (p.direct) {
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        const float inv = 1.0f / den;
        const bf16x4 o = {(__bf16)(num[0] * inv), (__bf16)(num[1] * inv), (__bf16)(num[2] * inv), (__bf16)(num[3] * inv)};
        const int64_t orow = ((int64_t)b * p.io_steps + jc) * p.Hq + (int64_t)hkv * p.G + jg;
        *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.out) + orow * D + d) = o;
      } else {
        const int64_t part = (((int64_t)b * p.queries + jc) * p.Hq + (int64_t)hkv * p.G + jg) * p.num_splits + work.split;
        *reinterpret_cast<f32x4*>(p.ws_acc + part * D + d) = num;
        if (d == 0) {
          p.ws_ml[part * 2] = M;
          p.ws_ml[part * 2 + 1] = den;
        }
      }
    }
  }
}

template <int D, int TILES, int NW>
hipError_t launch_tiles(const AttnParams& p, int batch, int grid_splits, hipStream_t stream) {
  const dim3 grid(p.Hkv, batch, grid_splits), block(64 * NW);
  const size_t queries = (size_t)TILES * (D / 16) * 1024, merge = (size_t)NW * kTileColumns * (2 + D + 4) * sizeof(float);
  const size_t lds = queries > merge ? queries : merge;
  if (p.rope_cos) return launch((attn_stream_bf16<D, TILES, NW, true>), grid, block, lds, stream, p);
  return launch((attn_stream_bf16<D, TILES, NW, false>), grid, block, lds, stream, p);
}

}  // namespace

hipError_t launch_stream_block_bf16(const AttnParams& p, int batch, int D, int grid_splits, hipStream_t stream) {
  const int columns = p.queries * p.G;
  if (columns > (D == 128 ? 64 : 128) || p.pad_t != 0 || batch > 65535 || grid_splits > 65535) return hipErrorInvalidConfiguration;
  if (D == 128) {
    if (columns <= 32) return launch_tiles<128, 1, 8>(p, batch, grid_splits, stream);
    return launch_tiles<128, 2, 8>(p, batch, grid_splits, stream);
  }
  if (columns <= 32) return launch_tiles<64, 1, 8>(p, batch, grid_splits, stream);
  if (columns <= 64) return launch_tiles<64, 2, 8>(p, batch, grid_splits, stream);
  return launch_tiles<64, 4, 8>(p, batch, grid_splits, stream);
}

}  // namespace tempo
