// Partial attention of one split, fp32 keys/values (row-major block store), on the fp32
// matrix cores of gfx950.
//
// Same quantities as the bf16 kernel (Section 2, Eq. 1 over one split; Section 4.3 masks):
// running max m, running sum l and accumulator acc in fp32, base-2 units.  Every product is a
// full fp32 product with an fp32 sum (v_mfma_f32_16x16x4_f32).
//
// Mapping.  One workgroup = one (sequence, kv head, tile of 16 (step, head) columns, split);
// column = c*G + g as in the bf16 kernel, so the query group and, in a block or a prompt,
// several steps share every key/value read.  Its wavefronts take the tile's 16-key groups
// round-robin and are merged through LDS.  The row-major rows are loaded straight into operand
// registers: a product does not care which dims its contraction steps are, nor which dims the
// rows of its result are, so both orders are chosen to make a lane's data 16-byte pieces:
//   logits  S^T = K (16 keys x 4 dims) * Q^T (4 dims x 16 columns), D/4 steps; step (i, e) is
//           dims 16i + 4c + e, c = lane / 16, so lane (key, c) holds pieces 16i + 4c .. +3
//   output  O^T = V^T (16 dims x 4 keys) * P^T (4 keys x 16 columns), 4 steps per tile; step r
//           is keys 4c + r, which is where the logits' accumulator keeps them, so the weights
//           are the operand as they stand; row n of tile (j, e) is dim 64j + 4n + e, so lane
//           (n, c) holds pieces 64j + 4n .. +3 of key 4c + r
// A lane's logits, weights, sum and accumulators belong to one column.
//
// What bounds it.  A step: HBM.  16 sequences, 24/8 heads of 128, t = 2047 (269 MB): one
// workgroup per query head and 16 lanes per key (shuffles, each head reading the group's keys
// and values) took 117.6 us a step; this kernel 46.8 us.  A prompt of 512 steps, 8/2 heads of 64,
// in blocks of 128 columns 203 us, as one launch of this kernel 11.2 us.  Blocks and prompts: 64 products
// of 32 cycles per group at D = 128, most of them padding when a tile holds few columns: steps and small
// blocks over short ranges go to attn_step_f32.hip.
#include <type_traits>

#include "attn_bf16_common.h"

namespace tempo {
namespace {

template <int D>
struct GroupF32 {
  f32x4 k[D / 16];
  f32x4 v[4][D / 64];
};

// kRows: a prompt from step 0 on sees its own rows only, so they are read from the caller's arrays (k_new /
// v_new), not from the store, and the workgroup of the tile that holds a step's first column writes that
// step's rows to the store: one launch instead of a write and one that waits for it (512 steps, 8/2 heads of
// 64, 16.8 -> 11.5 us; 16 x 64 steps 11.0 -> 6.6; long prompts alike, 16 x 512 steps of 24/8 heads of 128 754 / 749).
template <int D, bool kRows>
__global__ __launch_bounds__(512) void attn_partial_f32(AttnParams p) {
  constexpr int KI = D / 16;   // 16-byte pieces of a key row per lane
  constexpr int VJ = D / 64;   // 16-byte pieces of a value row per lane
  constexpr int LD = D + 4;    // row stride of the merge area (columns on different banks)
  extern __shared__ float smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwaves = blockDim.x >> 6;
  const int n = lane & 15, c = lane >> 4;
  const int all_cols = p.queries * p.G, tiles = (all_cols + 15) >> 4;
  // longest key ranges (the last tiles of a causal prompt) first
  const int hkv = blockIdx.x / tiles, tile = tiles - 1 - (int)(blockIdx.x - hkv * tiles), b = blockIdx.y;
  int t_b = p.t_per_seq ? ((const_i32_ptr)p.t_per_seq)[b] : p.t;
  t_b = t_b > p.t ? p.t : (t_b < 0 ? 0 : t_b);
  const SeqRange rg = seq_range(t_b, p.window, p.tps_log2, p.queries, p.pad_t);
  if ((int)blockIdx.z >= rg.nchunks) return;  // uniform over the workgroup
  const int split = rg.nchunks - 1 - (int)blockIdx.z;  // newest split first, as in the bf16 kernel
  const int chunk = rg.chunk0 + split;
  const int cs = chunk << p.tps_log2, ce = split_end(chunk, p.tps_log2);

  // this tile's columns and the union of their ranges, cut to the split (empty if they do not meet)
  const int col0 = 16 * tile, ncols = all_cols - col0 < 16 ? all_cols - col0 : 16;
  const int t_first = t_b + col0 / p.G, t_last = t_b + (col0 + ncols - 1) / p.G;
  auto lo_of = [&](int t) { return (p.window > 0 && t - p.window + 1 > 0) ? t - p.window + 1 : 0; };
  const int lo = lo_of(t_first), start = lo > cs ? lo : cs, end = t_last < ce ? t_last : ce;
  const int all_lo = lo_of(t_last) > start ? lo_of(t_last) : start, all_hi = t_first < end ? t_first : end;
  // this lane's column (unused ones behave like the tile's last step with q = 0)
  const int cq = (col0 + (n < ncols ? n : ncols - 1)) / p.G, gq = col0 + n - cq * p.G;
  const int step = t_b + cq;
  const int hi_col = step < end ? step : end, lo_col = lo_of(step) > start ? lo_of(step) : start;

  float* kpool = static_cast<float*>(p.k_pool);
  float* vpool = static_cast<float*>(p.v_pool);
  const int Z = 1 << p.z_log2;
  const_i32_ptr table = (const_i32_ptr)p.block_table + (int64_t)b * p.max_blocks_per_seq;
  // Offset of key j's row in either pool; j is inside the range, so its tile exists.
  auto row_of = [&](int j) -> int64_t {
    const int phys = clamp_block(p.block_table[(int64_t)b * p.max_blocks_per_seq + ((j >> p.z_log2) & p.tile_mask)], p.num_blocks);
    return ((((int64_t)phys * p.Hkv + hkv) << p.z_log2) + (j & (Z - 1))) * D;
  };
  auto clamped = [&](int j) { return j < start ? start : (j > end ? end : j); };
  // Fused block-store write (Section 6, "in-place writes"): step t_b's own key/value are taken from
  // k_new / v_new, and the workgroup of the first column tile also stores them for later steps.
  const float* kn = p.k_new ? static_cast<const float*>(p.k_new) + ((int64_t)b * p.Hkv + hkv) * D : nullptr;
  const float* vn = p.k_new ? static_cast<const float*>(p.v_new) + ((int64_t)b * p.Hkv + hkv) * D : nullptr;
  const int grp_new = !kRows && kn != nullptr && split == rg.nchunks - 1 ? t_b >> 4 : -1;
  // kRows: sequence b's rows, new_row from one step's to the next one's
  const int64_t new_row = (int64_t)p.Hkv * D;
  [[maybe_unused]] const float* k_rows = kRows ? static_cast<const float*>(p.k_new) + (int64_t)b * p.io_steps * new_row + (int64_t)hkv * D : nullptr;
  [[maybe_unused]] const float* v_rows = kRows ? static_cast<const float*>(p.v_new) + (int64_t)b * p.io_steps * new_row + (int64_t)hkv * D : nullptr;
  // Sixteen rows that are all in the range: their address is scalar but for a lane's part that never changes.
  auto whole = [&](int grp) { return kRows && (grp << 4) >= start && (grp << 4) + 15 <= end; };
  const uint32_t k_lane = (uint32_t)(n * new_row + 4 * c), v_lane = (uint32_t)(4 * c * new_row + 4 * n);

  GroupF32<D> g;
  // A group of 16 keys lies in one tile if tiles have at least 16 slots: one scalar table entry.
  // Rows outside the range are read as its nearest row and masked.
  auto group_base = [&](int grp) -> int64_t {
    const int phys = clamp_block(table[((grp << 4) >> p.z_log2) & p.tile_mask], p.num_blocks);
    return (((int64_t)phys * p.Hkv + hkv) << p.z_log2) * D;
  };
  auto load_keys = [&](int grp, int64_t base) {
    const int j = (grp << 4) + n, jc = clamped(j);
    const float* src = kpool + 4 * c + (p.z_log2 >= 4 ? base + (int64_t)(jc & (Z - 1)) * D : row_of(jc));
    if constexpr (kRows) src = whole(grp) ? k_rows + (grp << 4) * new_row + k_lane : k_rows + jc * new_row + 4 * c;
    else if (grp == grp_new) src = jc == t_b ? kn + 4 * c : src;  // (its slot in the pool is not read)
#pragma unroll
    for (int i = 0; i < KI; ++i) g.k[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + 16 * i));
  };
  auto load_values = [&](int grp, int64_t base) {
    if constexpr (kRows) {
      if (whole(grp)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float* src = v_rows + ((grp << 4) + r) * new_row + v_lane;
#pragma unroll
          for (int i = 0; i < VJ; ++i) g.v[r][i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + 64 * i));
        }
        return;
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = (grp << 4) + 4 * c + r, jc = clamped(j);
      const float* src = vpool + 4 * n + (p.z_log2 >= 4 ? base + (int64_t)(jc & (Z - 1)) * D : row_of(jc));
      if constexpr (kRows) src = v_rows + jc * new_row + 4 * n;
      else if (grp == grp_new) src = jc == t_b ? vn + 4 * n : src;
#pragma unroll
      for (int i = 0; i < VJ; ++i) g.v[r][i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + 64 * i));
    }
  };

  const int g_last = end >> 4;
  int grp = (start >> 4) + wave;
  const bool any = start <= end;
  int64_t base = 0;
  if (any && grp <= g_last) {
    base = p.z_log2 >= 4 ? group_base(grp) : 0;
    load_keys(grp, base);
    load_values(grp, base);
  }
  // rotary embedding: dim 16i + 4c + e pairs with piece i + D/32 of the same lane
  auto rotate = [&](f32x4* x, int pos) {
    const float* cs_t = p.rope_cos + (int64_t)pos * (D / 2) + 4 * c;
    const float* sn_t = p.rope_sin + (int64_t)pos * (D / 2) + 4 * c;
#pragma unroll
    for (int i = 0; i < KI / 2; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float co = cs_t[16 * i + e], si = sn_t[16 * i + e], a = x[i][e], h = x[i + KI / 2][e];
        x[i][e] = rope_lo(a, h, co, si);
        x[i + KI / 2][e] = rope_hi(a, h, co, si);
      }
    }
  };
  f32x4 qv[KI];
  {
    const float* qp = static_cast<const float*>(p.q) +
                      (((int64_t)b * p.io_steps + cq) * p.Hq + (int64_t)hkv * p.G + (n < ncols ? gq : 0)) * D + 4 * c;
#pragma unroll
    for (int i = 0; i < KI; ++i) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(qp + 16 * i);
      qv[i] = n < ncols ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (p.rope_cos) rotate(qv, step);
  }
  float m = -INFINITY, l = 0.f;
  f32x4 acc[VJ][4];            // acc[j][e][r]: dim 64j + 16c + 4r + e of this lane's column
#pragma unroll
  for (int j = 0; j < VJ; ++j) {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[j][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  auto group = [&](int nxt, bool more) __attribute__((always_inline)) {  // group grp; `more`: and request group nxt
    const int64_t base_nxt = more && p.z_log2 >= 4 ? group_base(nxt) : 0;
    const int j0 = grp << 4;
    if (grp == grp_new) {  // uniform: the group with step t_b's own key, fetched from k_new / v_new
      if (j0 + n == t_b) {
        if (p.rope_cos) rotate(g.k, t_b);
        if (tile == 0) {
          float* dst = kpool + row_of(t_b) + 4 * c;
#pragma unroll
          for (int i = 0; i < KI; ++i) *reinterpret_cast<f32x4*>(dst + 16 * i) = g.k[i];
        }
      }
      if (tile == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (j0 + 4 * c + r == t_b) {
            float* dst = vpool + row_of(t_b) + 4 * n;
#pragma unroll
            for (int i = 0; i < VJ; ++i) *reinterpret_cast<f32x4*>(dst + 64 * i) = g.v[r][i];
          }
        }
      }
    }
    // Chains of two products (8 dims), added pairwise, because one chain over all dims rounds the
    // logits coarsely: error of a step at t = 2047 against 64 bits 3.4e-7 with two chains and the
    // values summed into the running accumulators, 1.9e-7 with these and the groups' own sums below
    // (one workgroup per query head with shuffles: 2.3e-7).
    f32x4 s[KI * 2];
#pragma unroll
    for (int e = 0; e < KI * 2; ++e) s[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KI; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s[4 * (i >> 1) + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.k[i][e], qv[i][e], s[4 * (i >> 1) + e], 0, 0, 0);
    }
    if (more) load_keys(nxt, base_nxt);  // the key registers are free again

#pragma unroll
    for (int h = KI; h >= 1; h /= 2) {
#pragma unroll
      for (int i = 0; i < h; ++i) s[i] += s[i + h];
    }
    float x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = s[0][r] * p.scale_log2e;
    const bool cut = j0 < all_lo || j0 + 15 > all_hi;  // wave-uniform
    if (cut) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = j0 + 4 * c + r;
        x[r] = (j >= lo_col && j <= hi_col) ? x[r] : -INFINITY;
      }
    }
    const float m_new = fmaxf(m, column_max(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]))));
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // a column that has seen no key yet
    const float alpha = exp2f(m - m_ref);                  // exp2f(-inf) = 0 on the first keys
    float w[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = exp2f(x[r] - m_ref);
    l = l * alpha + ((w[0] + w[1]) + (w[2] + w[3]));
    m = m_new;
    // A key that another column of the tile sees and this one does not has weight 0 here, and
    // 0 times a value that is not finite is NaN: such groups go value by value.
    bool plain = true;
    if (cut) {
      float sum = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int j = 0; j < VJ; ++j) {
#pragma unroll
          for (int e = 0; e < 4; ++e) sum = fmaf(0.f, g.v[r][j][e], sum);
        }
      }
      plain = !__any(!(sum == 0.f));
    }
    if (plain) {
      // the group's own sums first, then added to the running ones: shorter chains, and the
      // rescale is part of the addition
#pragma unroll
      for (int j = 0; j < VJ; ++j) {
        f32x4 sum[2][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
          sum[0][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.v[0][j][e], w[0], zero, 0, 0, 0);
          sum[1][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.v[1][j][e], w[1], zero, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sum[0][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.v[2][j][e], w[2], sum[0][e], 0, 0, 0);
          sum[1][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.v[3][j][e], w[3], sum[1][e], 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[j][e][r] = fmaf(acc[j][e][r], alpha, sum[0][e][r] + sum[1][e][r]);
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < VJ; ++j) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] *= alpha;
      }
      for (int k = 0; k < 16; ++k) {  // key j0 + k: its weight sits in lanes (column, k / 4), its value piece j in (n, k / 4)
        const int from = 16 * (k >> 2);
        const float w01 = (k & 1) ? w[1] : w[0], w23 = (k & 1) ? w[3] : w[2];
        const float wk = __shfl((k & 2) ? w23 : w01, from + n);
        const bool seen = j0 + k >= lo_col && j0 + k <= hi_col;
#pragma unroll
        for (int j = 0; j < VJ; ++j) {
          const f32x4 a = (k & 1) ? g.v[1][j] : g.v[0][j], b4 = (k & 1) ? g.v[3][j] : g.v[2][j];
          const f32x4 v4 = (k & 2) ? b4 : a;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float v = __shfl(v4[e], from + 4 * c + r);   // dim 64j + 4 (4c + r) + e
              if (seen) acc[j][e][r] = fmaf(wk, v, acc[j][e][r]);
            }
          }
        }
      }
    }
    if (more) load_values(nxt, base_nxt);
    base = base_nxt;
  };
  // The last group apart, so that a wait for keys is not one for the values requested behind them (see the bf16
  // decode kernel; 16 sequences, 24/8 heads of 128, t = 2047, 48.3 -> 46.8 us a step; D = 64, 100 to 9000 keys of 1 to 64
  // sequences, 94 shapes 4% on the mean, one more than 1% slower: 32/8 heads, 16 of 4096 keys 48.2 -> 48.9).
  if (any) {
    for (; grp + nwaves <= g_last; grp += nwaves) group(grp + nwaves, true);
    if (grp <= g_last) group(grp + nwaves, false);
  }

  // wavefronts -> LDS, then one merge
  const float l_tot = column_sum(l);
  float* sm_m = smem;                     // [nwaves][16]
  float* sm_l = smem + nwaves * 16;       // [nwaves][16]
  float* sm_acc = smem + nwaves * 32;     // [nwaves][ncols][LD]
  if (c == 0) {
    sm_m[wave * 16 + n] = m;
    sm_l[wave * 16 + n] = l_tot;
  }
  if (n < ncols) {
#pragma unroll
    for (int j = 0; j < VJ; ++j) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<f32x4*>(sm_acc + (wave * ncols + n) * LD + 64 * j + 16 * c + 4 * r) =
            f32x4{acc[j][0][r], acc[j][1][r], acc[j][2][r], acc[j][3][r]};
    }
  }
  __syncthreads();

  // All wavefronts' values of an element in one batch of reads: a loop over them is a chain of LDS
  // round trips (24/8 heads of 128, 1 sequence, t = 150, 8 wavefronts: 10.0 us a step with the loop, 9.5 us; a
  // group of 16 heads, t = 15: 7.4 us, 6.2 us).
  auto merge = [&](auto waves) {
    for (int idx = threadIdx.x; idx < ncols * (D / 4); idx += blockDim.x) {
      const int jcol = idx / (D / 4), d = 4 * (idx - jcol * (D / 4));
      constexpr int NW = decltype(waves)::value;
      float mw[NW], lw[NW];
      f32x4 aw[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        mw[w] = sm_m[w * 16 + jcol];
        lw[w] = sm_l[w * 16 + jcol];
        aw[w] = *reinterpret_cast<const f32x4*>(sm_acc + (w * ncols + jcol) * LD + d);
      }
      float M = -INFINITY;
#pragma unroll
      for (int w = 0; w < NW; ++w) M = fmaxf(M, mw[w]);
      f32x4 num = {0.f, 0.f, 0.f, 0.f};
      float den = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        // saw no key of this column (all wavefronts: the partial is (-inf, 0, 0))
        const bool none = mw[w] == -INFINITY;
        const float wgt = none ? 0.f : exp2f(mw[w] - M);
        num += wgt * (none ? f32x4{0.f, 0.f, 0.f, 0.f} : aw[w]);
        den += wgt * (none ? 0.f : lw[w]);
      }
      const int jc = (col0 + jcol) / p.G, jg = col0 + jcol - jc * p.G;
      if (p.direct) {
        const int64_t orow = ((int64_t)b * p.io_steps + jc) * p.Hq + (int64_t)hkv * p.G + jg;
        *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + orow * D + d) = num / den;
      } else {
        const int64_t part = (((int64_t)b * p.queries + jc) * p.Hq + (int64_t)hkv * p.G + jg) * p.num_splits + split;
        *reinterpret_cast<f32x4*>(p.ws_acc + part * D + d) = num;
        if (d == 0) {
          p.ws_ml[part * 2] = M;
          p.ws_ml[part * 2 + 1] = den;
        }
      }
    }
  };
  switch (nwaves) {
    case 1: merge(std::integral_constant<int, 1>{}); break;
    case 2: merge(std::integral_constant<int, 2>{}); break;
    case 4: merge(std::integral_constant<int, 4>{}); break;
    default: merge(std::integral_constant<int, 8>{});
  }

  // The store's rows, read once more (the loop has brought them near): stores before the barrier above
  // would be waited for there (16 x 300 steps, window 100, 24/8 heads of 128: 202 us with them, 179).
  if constexpr (kRows) {
    const int tile_first = (col0 + p.G - 1) / p.G, tile_last = (col0 + ncols + p.G - 1) / p.G - 1;
    const int64_t slots = p.tile_mask == INT32_MAX ? INT32_MAX : ((int64_t)p.tile_mask + 1) << p.z_log2;  // a ring keeps the last ones
    const int kept = p.queries > slots ? p.queries - (int)slots : 0, from_step = tile_first > kept ? tile_first : kept;
    const int first = from_step > cs ? from_step : cs, last = tile_last < ce ? tile_last : ce;  // of this split
    for (int i = threadIdx.x; i < (last - first + 1) * (D / 4); i += blockDim.x) {
      const int j = first + i / (D / 4), d = 4 * (i % (D / 4));
      const int64_t from = j * new_row + d, to = row_of(j) + d;
      const f32x4 key = *reinterpret_cast<const f32x4*>(k_rows + from), value = *reinterpret_cast<const f32x4*>(v_rows + from);
      *reinterpret_cast<f32x4*>(kpool + to) = key;
      *reinterpret_cast<f32x4*>(vpool + to) = value;
    }
  }
}

}  // namespace

hipError_t launch_partial_f32(const AttnParams& p, int batch, int D, int grid_splits, int waves,
                              hipStream_t stream) {
  const int columns = p.queries * p.G, tiles = (columns + 15) / 16;
  if ((int64_t)tiles * p.Hkv > INT32_MAX || batch > 65535 || grid_splits > 65535) return hipErrorInvalidConfiguration;
  const dim3 grid(tiles * p.Hkv, batch, grid_splits);
  const dim3 block(64 * waves);
  const size_t lds = (size_t)waves * (32 + (size_t)(columns < 16 ? columns : 16) * (D + 4)) * sizeof(float);
  if (p.k_new && p.io_steps > 1) {  // (one step a call: [B][Hkv][D] either way)
    if (p.rope_cos || p.t_per_seq || p.t != 0) return hipErrorInvalidConfiguration;
    if (D == 128) return launch((attn_partial_f32<128, true>), grid, block, lds, stream, p);
    return launch((attn_partial_f32<64, true>), grid, block, lds, stream, p);
  }
  if (D == 128) return launch((attn_partial_f32<128, false>), grid, block, lds, stream, p);
  return launch((attn_partial_f32<64, false>), grid, block, lds, stream, p);
}

}  // namespace tempo
