// One or a few fp32 decode steps over a short range, on the vector ALU.
//
// Same quantities as attn_partial_f32.hip (running max m, running sum l and accumulator acc in
// fp32, base-2 units; Section 2, Eq. 1 over one split; Section 4.3 masks).  One workgroup = one
// (sequence, step, QUERY head, split).  A wavefront looks at 4 key positions at a time: 16 lanes per
// position, each lane holding D/16 consecutive dims.  The dot product is a 16-lane butterfly (DPP
// row operations); each 16-lane row keeps its own (m, l, acc) and the rows and wavefronts are
// merged once, through LDS, at the end.
//
// What bounds it: latency.  The matrix-core kernel takes 64 products of 32 cycles for 16 keys at
// D = 128 however few of its 16 columns are used, and wavefronts that share a SIMD wait for each
// other's; here a key costs D/16 fused multiply-adds and a butterfly, and every head has a compute
// unit.  Over long ranges it is the slower one, as every head of a group reads the group's keys and
// values.  Which calls come here, and what both take: f32_on_vector_alu() in tempo_api.hip.
#include "tempo_internal.h"

namespace tempo {
namespace {

// kRows: the steps from 0 on, whose keys/values are read from the caller's rows (k_new / v_new, [B][io_steps][Hkv][D]);
// the workgroup of a step's first query head of the group stores them for later calls.
template <int D, bool kRows>
__global__ __launch_bounds__(512) void attn_step_f32(AttnParams p) {
  constexpr int E = D / 16;  // dims per lane
  extern __shared__ float smem[];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  const int cq = blockIdx.x / p.Hq, hq = blockIdx.x - cq * p.Hq, b = blockIdx.y;  // cq < p.queries
  const int hkv = hq / p.G;
  int t_b = p.t_per_seq ? p.t_per_seq[b] : p.t;
  t_b = t_b > p.t ? p.t : (t_b < 0 ? 0 : t_b);
  const SeqRange rg = seq_range(t_b, p.window, p.tps_log2, p.queries);
  if ((int)blockIdx.z >= rg.nchunks) return;
  const int split = rg.nchunks - 1 - (int)blockIdx.z;  // newest split first, as in the other kernels
  const int chunk = rg.chunk0 + split;
  const int cs = chunk << p.tps_log2, ce = split_end(chunk, p.tps_log2);
  // this step's own range, cut to the split (empty if they do not meet)
  const int t_q = t_b + cq;
  const int lo_q = (p.window > 0 && t_q - p.window + 1 > 0) ? t_q - p.window + 1 : 0;
  const int start = lo_q > cs ? lo_q : cs;
  const int end = t_q < ce ? t_q : ce;

  const int row = lane >> 4, col = lane & 15;
  const int Z = 1 << p.z_log2;
  float* kpool = static_cast<float*>(p.k_pool);
  float* vpool = static_cast<float*>(p.v_pool);
  // Fused block-store write (Section 6, "in-place writes"): step t_b's own key/value are taken from
  // k_new / v_new, and the first query head of the group also stores them for later steps.
  const float* kn = p.k_new ? static_cast<const float*>(p.k_new) + ((int64_t)b * p.Hkv + hkv) * D : nullptr;
  const float* vn = p.k_new ? static_cast<const float*>(p.v_new) + ((int64_t)b * p.Hkv + hkv) * D : nullptr;

  float qv[E];
  {
    const float* qp = static_cast<const float*>(p.q) + (((int64_t)b * p.io_steps + cq) * p.Hq + hq) * D + col * E;
#pragma unroll
    for (int e = 0; e < E; ++e) qv[e] = qp[e];
  }
  // Rotary embedding: dims col*E .. +E-1 pair with those of lane col ^ 8 of the same 16-lane row;
  // table entry (position, i) with i = (col & 7) * E + e.
  auto rotate = [&](float* x, int pos) {
    const float* cs_t = p.rope_cos + (int64_t)pos * (D / 2) + (col & 7) * E;
    const float* sn_t = p.rope_sin + (int64_t)pos * (D / 2) + (col & 7) * E;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const float other = __shfl_xor(x[e], 8);
      x[e] = col < 8 ? rope_lo(x[e], other, cs_t[e], sn_t[e]) : rope_hi(other, x[e], cs_t[e], sn_t[e]);
    }
  };
  if (p.rope_cos) rotate(qv, t_q);
  float m = -INFINITY, l = 0.f, acc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.f;

  // Rows of a wavefront may leave this loop at different trips; the butterfly below only
  // exchanges data inside one 16-lane row, whose lanes share j.
  for (int j = start + 4 * wave + row; j <= end; j += 4 * nwaves) {
    const int tile = j >> p.z_log2, slot = j & (Z - 1);
    const int phys = clamp_block(p.block_table[(int64_t)b * p.max_blocks_per_seq + (tile & p.tile_mask)], p.num_blocks);
    const int64_t off = ((int64_t)phys * p.Hkv + hkv) * Z * D + (int64_t)slot * D + col * E;
    const bool fresh = kn != nullptr && j == t_b;  // uniform over the 16-lane row
    const float* ksrc = fresh ? kn + col * E : kpool + off;
    const float* vsrc = fresh ? vn + col * E : vpool + off;
    if constexpr (kRows) {
      const int64_t from = (((int64_t)b * p.io_steps + j) * p.Hkv + hkv) * D + col * E;
      ksrc = static_cast<const float*>(p.k_new) + from;
      vsrc = static_cast<const float*>(p.v_new) + from;
    }
    float kx[E], vx[E];
#pragma unroll
    for (int e = 0; e < E; e += 4) {
      const float4 k4 = *reinterpret_cast<const float4*>(ksrc + e);
      const float4 v4 = *reinterpret_cast<const float4*>(vsrc + e);
      kx[e] = k4.x; kx[e + 1] = k4.y; kx[e + 2] = k4.z; kx[e + 3] = k4.w;
      vx[e] = v4.x; vx[e + 1] = v4.y; vx[e + 2] = v4.z; vx[e + 3] = v4.w;
    }
    if (kRows ? j == t_q : fresh) {  // all 16 lanes of the row take this branch together
      if (p.rope_cos) rotate(kx, t_b);  // the new key arrives unrotated
      if (hq == hkv * p.G) {
#pragma unroll
        for (int e = 0; e < E; e += 4) {
          *reinterpret_cast<float4*>(kpool + off + e) = float4{kx[e], kx[e + 1], kx[e + 2], kx[e + 3]};
          *reinterpret_cast<float4*>(vpool + off + e) = float4{vx[e], vx[e + 1], vx[e + 2], vx[e + 3]};
        }
      }
    }
    float half[2] = {0.f, 0.f};  // (two short chains round less than a long one, here and in the merge)
#pragma unroll
    for (int e = 0; e < E; ++e) half[e & 1] = fmaf(qv[e], kx[e], half[e & 1]);
    float dot = half[0] + half[1];
    // 16-lane butterfly: every lane of the row ends with the full dot product
    dot += __shfl_xor(dot, 8);
    dot += __shfl_xor(dot, 4);
    dot += __shfl_xor(dot, 2);
    dot += __shfl_xor(dot, 1);
    const float x = dot * p.scale_log2e;
    const float m_new = fmaxf(m, x);
    const float alpha = exp2f(m - m_new);  // exp2f(-inf) = 0 on the first key
    const float w = exp2f(x - m_new);
    l = l * alpha + w;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = fmaf(w, vx[e], acc[e] * alpha);
    m = m_new;
  }

  // rows x wavefronts -> LDS, then one merge
  const int nrows = nwaves * 4;
  float* sm_m = smem;                 // [nrows]
  float* sm_l = smem + nrows;         // [nrows]
  float* sm_acc = smem + 2 * nrows;   // [nrows][D]
  const int r = wave * 4 + row;
  if (col == 0) { sm_m[r] = m; sm_l[r] = l; }
#pragma unroll
  for (int e = 0; e < E; ++e) sm_acc[r * D + col * E + e] = acc[e];
  __syncthreads();

  for (int d = threadIdx.x; d < D; d += blockDim.x) {
    float M = -INFINITY;
    for (int i = 0; i < nrows; ++i) M = fmaxf(M, sm_m[i]);
    float nums[4] = {0.f, 0.f, 0.f, 0.f}, dens[4] = {0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < nrows; i += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float mi = sm_m[i + u];
        if (mi == -INFINITY) continue;  // a row that saw no key (all rows: the partial is (-inf, 0, 0))
        const float wgt = exp2f(mi - M);
        nums[u] += wgt * sm_acc[(i + u) * D + d];
        dens[u] += wgt * sm_l[i + u];
      }
    }
    const float num = (nums[0] + nums[1]) + (nums[2] + nums[3]), den = (dens[0] + dens[1]) + (dens[2] + dens[3]);
    if (p.direct) {
      static_cast<float*>(p.out)[(((int64_t)b * p.io_steps + cq) * p.Hq + hq) * D + d] = num / den;
    } else {
      const int64_t part = (((int64_t)b * p.queries + cq) * p.Hq + hq) * p.num_splits + split;
      p.ws_acc[part * D + d] = num;
      if (d == 0) {
        p.ws_ml[part * 2] = M;
        p.ws_ml[part * 2 + 1] = den;
      }
    }
  }
}

}  // namespace

// No padding bound; p.k_new (the fused write) with one query step, or from step 0 on.
hipError_t launch_step_f32(const AttnParams& p, int batch, int D, int grid_splits, int waves, hipStream_t stream) {
  const bool rows = p.k_new && p.io_steps > 1;  // (one step a call: [B][Hkv][D] either way)
  if ((rows && (p.rope_cos || p.t_per_seq || p.t != 0)) || p.pad_t != 0 || batch > 65535 || grid_splits > 65535) return hipErrorInvalidConfiguration;
  const dim3 grid(p.Hq * p.queries, batch, grid_splits);
  const dim3 block(64 * waves);
  const size_t lds = (size_t)waves * 4 * (2 + (size_t)D) * sizeof(float);
  if (rows) {
    if (D == 128) return launch((attn_step_f32<128, true>), grid, block, lds, stream, p);
    return launch((attn_step_f32<64, true>), grid, block, lds, stream, p);
  }
  if (D == 128) return launch((attn_step_f32<128, false>), grid, block, lds, stream, p);
  return launch((attn_step_f32<64, false>), grid, block, lds, stream, p);
}

}  // namespace tempo
