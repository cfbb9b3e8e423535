// Prompt processing: attention of many consecutive query steps over the tiled
// keys/values, bf16, MFMA on gfx950.
//
// What is computed (Section 2, Eq. 1 for every step t .. t+count-1 of a sequence,
// with the causal or window pattern; Section 4.3 index masks): exactly what the
// decode kernel computes for each of those steps, one after the other.  With many
// steps per key the products dominate the reads.
//
// Mapping.  One workgroup = one (sequence, kv head, block of (step, head) columns, split of the
// block's key range; normally one split); column = c*G + g, 32 per wavefront, as the columns of
// 32x32x16 products:
//   logits tile  = K (32 slots x 16 dims) * Q^T (16 dims x 32 columns)   D/16 steps
//   output tiles = V^T (32 dims x 16 slots) * P^T (16 slots x 32 columns)  D/32 tiles x 2 steps
// A lane then holds logits, weights, sum and output of ONE column: no exchange but one lane
// swap for the maximum, and the weights of a lane are the operand of the second product as
// they stand.  The block store's units, made for 16x16x32 operands, are read as 32x32x16
// ones by taking two units side by side (16-lane runs of 256 bytes: no bank conflict).
// Every wavefront walks ALL 32-slot groups of the block's key range, so each column's
// softmax is finished inside one wavefront.  A group's key/value image (16 KiB at D = 128)
// is the same for all wavefronts: it is copied once per workgroup from the pool into LDS.
// 32 columns per wavefront, because LDS operand reads are per wavefront: 16 columns
// (16x16x32 products) read twice as much for the same products.
//
// What bounds it.  Matrix cores: 16 products of 32 cycles per wavefront and group = 512
// cycles; vector ALU 450 cycles; two wavefronts per SIMD.  A wavefront issues about one
// instruction in five cycles, so what is not a product has to lie between products, and
// products that queue behind a busy matrix core keep the SIMD's other wavefront from
// issuing LDS and memory instructions (measured: two copies 148 cycles alone, 658 beside
// back-to-back products; separate product and softmax phases of the two wavefronts, with a
// barrier between, were slower than this order for that reason).  Measured on 16 prompts of
// 4096 steps, 24 query heads in 8 groups, D = 128 (1.65 Tflop): 16-column kernel 2082 us a
// call, this one 1800 us (back to back, the clock at 1.8 GHz); 1700 cycles per group and pair of
// wavefronts (1020 of them products), 11000 before the first and 4400 after the last group of a
// workgroup.  Every vector instruction of the loop counts: without the eight moves of the next
// group's logits and with one comparison for a reference that stays, 1859 -> 1800 us; 499 steps of
// one sequence, 32/8 heads of 64, 15.2 -> 14.7; 4 x 2048 with window 512 105 -> 102.8.
//
// A prompt from step 0 on sees its own rows only, so they need not pass through the store (kRows): every
// workgroup copies them from the caller's arrays, keys as 16-byte pieces gathered into operand order,
// values row by row and turned by gfx950's transposing LDS read (two of 8 bytes where the pools' order
// takes one of 16), and the workgroup whose columns begin a group's first step writes that group to the
// store while it lies in LDS.  One launch instead of a write and a launch that waits for it: 499 steps of
// one sequence, 32/8 heads of 64, 14.7 -> 11.8 us, 40 steps 8.2 -> 5.8; 4 x 2048 with window 512 on a
// ring, which had staged its rows in the workspace, 102.7 -> 84.5.  The extra reads cost 3 to 4% of a long
// causal prompt's loop (prompt_from_rows() in tempo_api.hip draws the line).
//
// Workgroups of one (sequence, head) are adjacent in the work list and run together on
// one die, so the pool is streamed from HBM about once per (sequence, head) and the
// blocks that follow find it in that die's L2; the longest blocks come first.
#include "attn_bf16_columns32.h"

namespace tempo {
namespace {

typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int kWaveColumns = 32;

// Where the keys/values of a group come from: the store's pools; the pools and, from the call's first step
// on, the staging area; or the caller's rows (a prompt from step 0 on, which sees nothing else).
enum Source { kPools, kStage, kRows };

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4* lds_i16x4_ptr;

template <int D, int NW, int NBUF, bool kRope, Source kFrom>
__global__ __launch_bounds__(64 * NW, 2) void attn_prefill_bf16(PromptParams p) {
  constexpr int KT = D / 16;                  // 16-dim contraction steps of the logits
  constexpr int OT = D / 32;                  // 32-dim tiles of the output
  constexpr int KU = D / 16;                  // 1 KiB units of one group's keys
  constexpr int UNITS = 2 * KU;               // ... and of its keys and values together
  constexpr int PER_WAVE = UNITS / NW;        // units each wavefront copies per group
  constexpr bool kStaged = kFrom == kStage;
  static_assert(KU % NW == 0 && (NBUF == 4 || NBUF == 8), "copy split");
  static_assert(kFrom == kPools || !kRope, "unrotated keys come from the store");
  constexpr bool kEarly = NBUF > 4;           // first operands of an iteration are read at the end of the one before
  constexpr int kPair = kEarly ? 2 : 1;       // groups per barrier
  constexpr int kRead = KT;                   // operands read ahead of the matrix instruction that takes them
  extern __shared__ u32x4 lds[];              // [NBUF][UNITS][64] x 16 bytes: a group's keys, then its values
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const BlockWork work = block_work<true>(p, kWaveColumns * NW);
  if (!work.any) return;                       // uniform over the workgroup, before any barrier
  const int b = work.b, hkv = work.hkv, c0 = work.c0, ncols = work.ncols, split = work.split;
  const int t_last = work.t_last, start = work.start, g_first = work.g_first, g_last = work.g_last;
  // The block-table entries of the range's first 64 tiles, one per lane, are asked for before anything
  // else: the first copies wait for them and for nothing else.
  const int32_t* table = p.block_table + (int64_t)b * p.max_blocks_per_seq;
  const int tile_groups = p.z_log2 - 5;             // log2(groups per tile)
  const int tile_last = g_last >> tile_groups;
  int tile_base = g_first >> tile_groups;           // lane i holds the byte offset, in either pool, of tile tile_base + i
  // kRows: the groups whose first step's first column is this block's are written to the store by it
  const unsigned block_first = (unsigned)c0 * (unsigned)p.G + (unsigned)work.skip, group_columns = 32u * (unsigned)p.G;
  const int write_first = kFrom != kRows ? 0 : (int)((block_first + group_columns - 1) / group_columns);
  const int write_past = kFrom != kRows ? 0 : (int)((block_first + (unsigned)ncols + group_columns - 1) / group_columns);
  // ... the last one, if the call goes on in it behind the block's last step, from a copy of its own
  const bool write_tail = kFrom == kRows && cut_tail(work) && t_last + 1 < work.all_steps && g_last >= write_first && g_last < write_past;
  const int write_loop = write_tail ? g_last : write_past;
  uint32_t tile_lo, tile_hi;
  auto fetch_entry = [&]() {
    if (kFrom == kRows) {                           // of group write_first + lane (at most 9 groups)
      const int g = write_first + lane < write_past ? write_first + lane : g_last;
      return table[(g >> tile_groups) & p.tile_mask];
    }
    const int tile = tile_base + lane < tile_last ? tile_base + lane : tile_last;  // never past the range's last tile
    return table[tile & p.tile_mask];
  };
  auto place_tiles = [&](int found) {
    const uint64_t at = ((uint64_t)((int64_t)clamp_block(found, p.num_blocks) * p.Hkv + hkv) << p.z_log2) * (D * 2);
    tile_lo = (uint32_t)at;
    tile_hi = (uint32_t)(at >> 32);
    // waited for here: the use in the loop must not become a wait for the copies in flight
    asm volatile("" : "+v"(tile_lo), "+v"(tile_hi));
  };
  const int entry = fetch_entry();

  const int first_col = kWaveColumns * wave;
  const WaveBounds own = wave_bounds(p, work, first_col, kWaveColumns);

  // This lane's column, its query operand (lane half h: dims 16 s + 8 h .. +7), its softmax state.
  const int half = lane >> 5;
  const int col = first_col + (lane & 31);
  const LaneColumn mine = lane_column(p, work, col);
  const int cq = mine.cq, gq = mine.gq, step = mine.step, lo_col = mine.lo, hi_col = mine.hi;
  u32x4 qreg[KT];
  {
    const uint16_t* qp = static_cast<const uint16_t*>(p.q) +
                         (((int64_t)b * p.io_steps + c0 + cq) * p.Hq + (int64_t)hkv * p.G + gq) * D + 8 * half;
#pragma unroll
    for (int s = 0; s < KT; ++s) qreg[s] = *reinterpret_cast<const u32x4*>(qp + 16 * s);
  }
  __builtin_amdgcn_sched_barrier(0);           // ... on their way before the first copies are, and used behind them
  float m_run = -INFINITY;                     // softmax reference of this lane's column (log2 units)
  float l_run = 0.f;                           // running sum over this lane's slots
  f32x16 acc[OT];                              // dims 32 ot + 8 (r / 4) + 4 h + (r mod 4) of this lane's column
#pragma unroll
  for (int ot = 0; ot < OT; ++ot) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[ot][r] = 0.f;
  }

  // Copy of a group: wavefront w moves units w, w + NW, ... of the group's 1 KiB units
  // (keys first, then values).  The pool image is already what the consumers read, so
  // the copy goes from global memory straight into LDS (gfx950's 16-byte global -> LDS
  // load: lane i's piece lands at the wavefront's LDS base + 16 i); completion is counted
  // by the vector-memory counter.  Where a group sits in either pool follows from its
  // block-table entry.  The range's entries are fetched 64 at a time, one per lane, and read
  // from there: a scalar load inside the loop would share the LDS reads' counter, and as the
  // two kinds return out of order every wait for an operand would become a wait for all.  Beyond the range's last group the last one is
  // copied again (into a buffer nobody reads any more): every iteration then issues the
  // same number of copies, and "the group before the newest has landed" is one counted wait.
  if (kFrom != kRows) place_tiles(entry);
  // kRows: byte offset, from the row of the group's first step, of each piece this lane copies.  Keys land
  // in operand order, as from the pools.  Values land row by row, 16-byte pieces in the order piece ^ (row
  // part), which spreads the four rows a transposing read takes over all LDS banks.
  constexpr int kRowBytes = 2 * D, kPieces = D / 8, kUnitRows = 64 / kPieces;
  const uint32_t row_stride = (uint32_t)p.Hkv * kRowBytes;
  auto swizzle = [](int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); };
  uint32_t row_piece[PER_WAVE];
#pragma unroll
  for (int i = 0; i < PER_WAVE; ++i) {
    const int u = wave + NW * i;
    const int key_row = 16 * (u / (D / 32)) + (lane & 15), value_row = (u - KU) * kUnitRows + lane / kPieces;
    row_piece[i] = u < KU ? (uint32_t)key_row * row_stride + 64u * (uint32_t)(u % (D / 32)) + 16u * (uint32_t)(lane >> 4)
                          : (uint32_t)value_row * row_stride + 16u * (uint32_t)((lane % kPieces) ^ swizzle(lane / kPieces));
  }
  // A prompt on a ring store: the groups from its first step on lie, as one run per (sequence,
  // head), in the staging area; the ring holds the history.
  const int64_t stage_run = ((int64_t)b * p.Hkv + hkv) * p.stage_groups * (64 * D);
  const char* from_pool[PER_WAVE];                  // this wavefront's units in the pools' first group
  const char* from_stage[PER_WAVE];                 // ... and in the staging area's
#pragma unroll
  for (int i = 0; i < PER_WAVE; ++i) {
    const int u = wave + NW * i;                    // wave-uniform
    from_pool[i] = u < KU ? static_cast<const char*>(p.k_pool) + u * 1024
                          : static_cast<const char*>(p.v_pool) + (u - KU) * 1024;
    if (kStaged)
      from_stage[i] = stage_run + (u < KU ? static_cast<const char*>(p.k_stage) + u * 1024
                                          : static_cast<const char*>(p.v_stage) + (u - KU) * 1024);
  }
  const uint32_t lane_bytes = 16u * (uint32_t)lane;
  // kRows: rows outside the block's range read as zeros, as the pools' way masks them (a value that is not finite would
  // show through its weight of 0): those behind the block's last step lie beyond the buffer, `hidden` ones are
  // asked for there.  The copies beyond the range's last group hold all of that group's rows, to be written.
  auto bytes_of = [&](int count) { return (uint32_t)((count < 32 ? count : 32) - 1) * row_stride + kRowBytes; };
  const uint32_t last_bytes = bytes_of(t_last + 1 - 32 * g_last), tail_bytes = bytes_of(work.all_steps - 32 * g_last);
  // `at`: the buffer's offset in LDS, in 16-byte pieces; `hidden` (kRows): first rows whose values read as zeros
  auto issue = [&](int at, int g, int hidden = 0) {
    const int gc = g < g_last ? g : g_last;
    if (kFrom == kRows) {
      const uint32_t bytes = g < g_last ? bytes_of(32) : g == g_last ? last_bytes : tail_bytes;
      const uint64_t from = (((uint64_t)b * (uint32_t)p.io_steps + 32u * (uint32_t)gc) * (uint32_t)p.Hkv + (uint32_t)hkv) * kRowBytes;
      char* const rows[2] = {const_cast<char*>(static_cast<const char*>(p.k_new)) + from,
                             const_cast<char*>(static_cast<const char*>(p.v_new)) + from};
#pragma unroll
      for (int i = 0; i < PER_WAVE; ++i) {
        const auto group = __builtin_amdgcn_make_buffer_rsrc(rows[i / (PER_WAVE / 2)], 0, (int)bytes, 0x00020000);
        uint32_t piece = row_piece[i];
        if (i >= PER_WAVE / 2 && hidden > 0 && (wave + NW * i - KU) * kUnitRows + lane / kPieces < hidden) piece = 0x7FFFFF00u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(group, (lds_ptr)(lds + at + (wave + NW * i) * 64), 16, (int)piece, 0, 0, 0);
      }
      return;
    }
    if (kStaged && gc >= p.stage_first) {
      const uint64_t from = (uint64_t)(gc - p.stage_first) * (64u * D);
#pragma unroll
      for (int i = 0; i < PER_WAVE; ++i) {
        const auto unit = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(from_stage[i] + from), 0, 1024, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(unit, (lds_ptr)(lds + at + (wave + NW * i) * 64), 16, lane_bytes, 0, 0, 0);
      }
      return;
    }
    const int tile = gc >> tile_groups;
    if (tile - tile_base >= 64) {
      tile_base = tile;
      place_tiles(fetch_entry());
    }
    const uint32_t lo = __builtin_amdgcn_readlane(tile_lo, tile - tile_base);
    const uint32_t hi = __builtin_amdgcn_readlane(tile_hi, tile - tile_base);
    const uint64_t from = (((uint64_t)hi << 32) | lo) + (uint32_t)(gc & ((1 << tile_groups) - 1)) * (64u * D);
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      // (the buffer form: the compiler takes the global form for a flat access that may also be
      // an LDS access, and then waits for ALL outstanding LDS reads wherever it waits for one)
      const auto unit = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(from_pool[i] + from), 0, 1024, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(unit, (lds_ptr)(lds + at + (wave + NW * i) * 64), 16, lane_bytes, 0, 0, 0);
    }
  };
  const bool head = kFrom != kRows && cut_head(work), tail = kFrom != kRows && cut_tail(work);
  auto mask_values = [&](int g, int at) {  // the buffer of group g: the first, and head, or the last, and tail
    uint32_t keep[4];
    value_masks(g, start, t_last, lane, keep);
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const int u = wave + NW * i;
      if (u >= KU) mask_piece(lds + at + u * 64 + lane, keep);
    }
  };
  // Waits and barriers are written out instead of __syncthreads() so that they are the ones
  // this loop needs (builtins, not assembly: the compiler then knows what has been waited for
  // and counts its own waits for LDS operands); the empty statements with a "memory" clobber
  // keep it from moving LDS accesses across.
  // landed(): all but the newest kPair groups' copies of this wavefront are in LDS.
  auto landed = [&]() {
    constexpr int kLeft = PER_WAVE * kPair;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((kLeft & 15) | 0x0F70 | ((kLeft >> 4) << 14));  // vmcnt only
    asm volatile("" ::: "memory");
  };
  auto meet = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  // Raw dot products of this wavefront's columns with the 32 keys of the group in `buf`.
  // Key row l & 31 of the operand is slot l & 31: unit (slot / 16, s / 2), lanes
  // (slot & 15) + 16 (2 (s & 1) + h).
  const int k_lane = ((lane >> 4) & 1) * (D / 32) * 64 + (lane & 15) + 16 * half;
  auto key_operand = [&](int at, int s) { return as_bf16x8(lds[at + k_lane + (s >> 1) * 64 + (s & 1) * 32]); };
  // Value rows: dim l & 31 of tile ot is unit 2 ot + (dim / 16), lanes (dim & 15) + 16 (2 chunk + h).
  const int v_lane = KU * 64 + ((lane >> 4) & 1) * 64 + (lane & 15) + 16 * half;
  // From rows, gfx950's transposing read: 16 lanes that point at 4 rows x 4 pieces of 4 dims get one dim of
  // the 4 rows each.  Lane 16 q + i gets dim 16 (q & 1) + i of tile ot, rows 8 chunk + 4 (q >> 1) + 0 .. 3 and
  // the same + 16: the slots of the pools' unit.
  const int tr_row = 4 * half + ((lane & 15) >> 2);
  int v_row_lane[OT];
#pragma unroll
  for (int ot = 0; ot < OT; ++ot)
    v_row_lane[ot] = KU * 1024 + tr_row * kRowBytes + 8 * (lane & 1) +
                     16 * ((4 * ot + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ swizzle((lane & 15) >> 2));
  auto rows_of_dim = [&](int byte) {                // of rows r .. r+3 and r+16 .. r+19, where `byte` points into row r
    char* const from = reinterpret_cast<char*>(lds) + byte;
    struct Both { i16x4 low, high; } both;
    both.low = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)from);
    both.high = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(from + 16 * kRowBytes));
    return __builtin_bit_cast(u32x4, both);
  };
  auto value_operand = [&](int at, int chunk, int ot) {
    if (kFrom == kRows) return as_bf16x8(rows_of_dim(16 * at + v_row_lane[ot] + chunk * 8 * kRowBytes));
    return as_bf16x8(lds[at + v_lane + ot * 128 + chunk * 32]);
  };
  // kRows: group g, in the buffer at `at`, into the store: its keys' units as they lie in LDS, its values'
  // units (tile_off_v_bf16) by transposing reads.  Slots of a group that the call does not write are left alone.
  auto write_group = [&](int g, int at) {
    const int lo = p.keep_first - 32 * g > 0 ? p.keep_first - 32 * g : 0;
    const int hi = work.all_steps - 32 * g < 32 ? work.all_steps - 32 * g : 32;
    if (lo >= hi) return;
    const int phys = clamp_block(__builtin_amdgcn_readlane(entry, g - write_first), p.num_blocks);
    const int64_t to = (((int64_t)phys * p.Hkv + hkv) << p.z_log2) * D + (int64_t)((g << 5) & ((1 << p.z_log2) - 1)) * D;
    u32x4* const k_to = reinterpret_cast<u32x4*>(static_cast<uint16_t*>(p.k_pool) + to) + lane;
    u32x4* const v_to = reinterpret_cast<u32x4*>(static_cast<uint16_t*>(p.v_pool) + to) + lane;
    const int c = lane >> 4;
#pragma unroll
    for (int i = 0; i < PER_WAVE / 2; ++i) {
      const int u = wave + NW * i, slot = 16 * (u / (D / 32)) + (lane & 15);
      const u32x4 keys = lds[at + u * 64 + lane];
      if (slot >= lo && slot < hi) k_to[u * 64] = keys;
      const int row = 4 * c + ((lane & 15) >> 2);
      const u32x4 values = rows_of_dim(16 * at + KU * 1024 + row * kRowBytes + 8 * (lane & 1) +
                                       16 * ((2 * u + ((lane & 3) >> 1)) ^ swizzle(row)));
      if (lo == 0 && hi == 32) {
        v_to[u * 64] = values;
        continue;
      }
      uint16_t* const each = reinterpret_cast<uint16_t*>(v_to + u * 64);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int s = e < 4 ? 4 * c + e : 12 + 4 * c + e;
        if (s >= lo && s < hi) each[e] = (uint16_t)(values[e >> 1] >> (16 * (e & 1)));
      }
    }
  };

  // The groups this wavefront has work in: own_first .. own_last.  The others it only helps
  // to copy: loops of their own, so that no path around the arithmetic carries the accumulators.
  const int own_first = own.idle ? g_last + 1 : (own.lo_first > (g_first << 5) ? own.lo_first >> 5 : g_first);
  const int own_last = own.idle ? g_last : own.hi >> 5;

  int grp = g_first;
  // LDS offset of the buffer of group grp + ahead (NBUF is a power of two)
  constexpr int kBuf = UNITS * 64;
  int at0 = 0;
  auto next = [&](int ahead) { return (at0 + ahead * kBuf) & (NBUF * kBuf - 1); };
  // Into the buffer of group grp - kPair, which everybody finished before the last barrier.
  auto copies = [&]() { issue(next(NBUF - kPair), grp + NBUF - kPair); };
  // The groups no column's range cuts: first_whole .. last_whole.
  const int first_whole = (own.lo_last + 31) >> 5, last_whole = ((own.hi_min + 1) >> 5) - 1;
  float base = 0.f;                            // m_run, or 0 while the column has seen no key
  float limit = -INFINITY;                     // raw dot product from which on m_run has to move
  // mask and reference of group g, whose logits are in x, their maximum in this lane mx
  auto enter = [&](int g, f32x16& x, float mx) {
    if (g < first_whole || g > last_whole) {
      mask_tile(g, lo_col, hi_col, lane, x);
      mx = tile_max(x);
    }
    softmax_reference<D>(mx, p.scale_log2e, limit, m_run, base, acc, l_run);
  };
  // End of an iteration.  After a barrier the next kPair groups, the group behind them (its
  // logits are computed one group ahead) and, with early operand reads, one more are in LDS.
  constexpr int kAhead = 2 * kPair;            // of grp, which may be the second of a pair
  auto finish = [&]() {
    if (kFrom == kRows && grp >= write_first && grp < write_loop) write_group(grp, at0);
    if (kPair == 1 || ((grp - g_first) & 1)) {
      landed();
      if (tail && g_last <= grp + kAhead && g_last > grp + kAhead - kPair) mask_values(g_last, next(g_last - grp));
      meet();
    }
    at0 = next(1);
    ++grp;
  };

  // (a first group that its range cuts is an earlier block's to write)
#pragma unroll
  for (int i = 0; i < NBUF - kPair; ++i) issue(i * kBuf, g_first + i, kFrom == kRows && i == 0 ? start & 31 : 0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < KT; ++s) {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    qreg[s] = col < ncols ? qreg[s] : zero;
  }
  if (kRope) {  // queries arrive unrotated; a dim's partner D/2 further sits in the same lane
#pragma unroll
    for (int s = 0; s < KT / 2; ++s)
      rotate_pieces(p.rope_cos, p.rope_sin, step, D / 2, 16 * s + 8 * half, qreg[s], qreg[s + KT / 2]);
  }
  landed();                                    // groups g_first .. g_first + kAhead - 1
  if (head) mask_values(g_first, 0);
  if (tail && g_last - g_first < kAhead) mask_values(g_last, (g_last - g_first) * kBuf);
  meet();
  for (; grp < own_first && grp <= g_last; finish()) copies();
  // operand i of an iteration: keys of group grp + 1, then values of group grp
  constexpr int kSlots = KT + 2 * OT;
  bf16x8 op[kSlots];
  auto read_operand = [&](int i) {
    op[i] = i < KT ? key_operand(next(1), i) : value_operand(at0, (i - KT) / OT, (i - KT) % OT);
  };
  f32x16 xa, xb;                               // logits of group grp, masked, its reference already moved: in turn
  if (grp <= own_last) {
#pragma unroll
    for (int r = 0; r < 16; ++r) xa[r] = 0.f;
#pragma unroll
    for (int s = 0; s < KT; ++s)
      xa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(key_operand(at0, s), as_bf16x8(qreg[s]), xa, 0, 0, 0);
    enter(grp, xa, tile_max(xa));
    if (kEarly) {
#pragma unroll
      for (int i = 0; i < kRead; ++i) read_operand(i);
    }
  }
  // Group grp, logits in xc; those of group grp + 1 to xn.
  auto iterate = [&](const f32x16& xc, f32x16& xn) {
    if (!kEarly) {
#pragma unroll
      for (int i = 0; i < kRead; ++i) read_operand(i);
    }
    u32x4 pa[2];
    float even, mx[5];
#pragma unroll
    for (int r = 0; r < 16; ++r) xn[r] = 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
      if (s < KT) {
        xn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[s], as_bf16x8(qreg[s]), xn, 0, 0, 0);
      } else {
        const int ot = (s - KT) % OT;
        acc[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[s], as_bf16x8(pa[(s - KT) / OT]), acc[ot], 0, 0, 0);
      }
      if (s + kRead < kSlots) read_operand(s + kRead);
      else if (kEarly) op[s + kRead - kSlots] = key_operand(next(2), s + kRead - kSlots);
      if (s == KT + OT) copies();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (i * (KT + OT) / 16 == s) softmax_weight(xc, p.scale_log2e, base, i, even, pa, l_run);
      }
      if (s >= KT + OT) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
          if (i * OT / 5 == s - KT - OT) {
            mx[i] = max3(xn[3 * i], xn[3 * i + 1], xn[3 * i + 2]);
            asm volatile("" : "+v"(mx[i]));    // here, not behind the products
          }
        }
      }
      asm volatile("" : "+v"(l_run));
      __builtin_amdgcn_sched_barrier(0);
    }
    enter(grp + 1, xn, max3(max3(mx[0], mx[1], mx[2]), max3(mx[3], mx[4], xn[15]), xn[15]));
    finish();
  };
  // Two groups a turn: with one, the logits move to other registers at its end.
  while (grp <= own_last) {
    iterate(xa, xb);
    if (grp > own_last) break;
    iterate(xb, xa);
  }
  for (; grp <= g_last; finish()) copies();
  // the copies issued last may still be in flight: they must land before the LDS is given up
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // Whole range: every column saw its own key, so its sum is > 0 and the output is
  // acc / sum.  One split of the range: the column's partial (reference, sum,
  // accumulator) goes to the workspace; a column that saw no key in this split leaves
  // (-inf, 0, 0).
  const float l_j = half_sum(l_run);
  if (col < ncols) {
    if (p.direct) {
      __bf16* orow = static_cast<__bf16*>(p.out) +
                     (((int64_t)b * p.io_steps + c0 + cq) * p.Hq + (int64_t)hkv * p.G + gq) * D + 4 * half;
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      const float inv = 1.0f / l_j;
#pragma unroll
      for (int ot = 0; ot < OT; ++ot) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          bf16x4 o;
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r] = (__bf16)(acc[ot][4 * i + r] * inv);
          *reinterpret_cast<bf16x4*>(orow + 32 * ot + 8 * i) = o;
        }
      }
    } else {
      const int64_t row = ((int64_t)b * p.queries + c0 + cq) * p.Hq + (int64_t)hkv * p.G + gq;
      const int64_t part = row * p.num_splits + split;
      float* arow = p.ws_acc + part * D + 4 * half;
#pragma unroll
      for (int ot = 0; ot < OT; ++ot) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<f32x4*>(arow + 32 * ot + 8 * i) =
              f32x4{acc[ot][4 * i], acc[ot][4 * i + 1], acc[ot][4 * i + 2], acc[ot][4 * i + 3]};
      }
      if (half == 0) {
        p.ws_ml[part * 2] = m_run;
        p.ws_ml[part * 2 + 1] = l_j;
      }
    }
  }
  if (write_tail) {                            // uniform over the workgroup
    meet();
    write_group(g_last, at0);                  // (the first copy beyond the last group's)
  }
}

}  // namespace

namespace {
template <int D, int NW, int NBUF>
hipError_t launch_from(const PromptParams& p, dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  if (p.k_new) return launch((attn_prefill_bf16<D, NW, NBUF, false, kRows>), grid, block, lds, stream, p);
  if (p.k_stage) return launch((attn_prefill_bf16<D, NW, NBUF, false, kStage>), grid, block, lds, stream, p);
  if (p.rope_cos) return launch((attn_prefill_bf16<D, NW, NBUF, true, kPools>), grid, block, lds, stream, p);
  return launch((attn_prefill_bf16<D, NW, NBUF, false, kPools>), grid, block, lds, stream, p);
}

template <int NW>
hipError_t launch_prefill_nw(const PromptParams& p, int batch, int D, int grid_splits, hipStream_t stream) {
  // Eight wavefronts (one workgroup per compute unit): eight buffers, two groups per
  // barrier, an iteration's first operands read in the one before.  Fewer: four buffers, so that
  // at least two workgroups share a compute unit.
  constexpr int NBUF = NW == 8 ? 8 : 4;
  if (p.G > kWaveColumns * NW || p.block_columns != kWaveColumns * NW) return hipErrorInvalidConfiguration;
  const int64_t nblocks = prompt_blocks(p.queries, p.G, kWaveColumns * NW);
  // the kernel renumbers its workgroups with 32-bit arithmetic on the linear index
  if (nblocks * grid_splits * p.Hkv * batch > INT32_MAX) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)(nblocks * grid_splits), p.Hkv, batch);
  const dim3 block(64 * NW);
  const size_t lds = NBUF * (size_t)(D / 8) * 1024;
  if ((p.k_stage || p.k_new) && p.rope_cos) return hipErrorInvalidConfiguration;  // unrotated keys go to the store first
  if constexpr (NW == 8) {
    if (D != 128) return hipErrorInvalidConfiguration;  // four wavefronts are always the better shape at D = 64
  }
  if constexpr (NW < 8) {
    if (D == 64) return launch_from<64, NW, NBUF>(p, grid, block, lds, stream);
  }
  return launch_from<128, NW, NBUF>(p, grid, block, lds, stream);
}
}  // namespace

// waves: 2, 4 or (D = 128) 8 wavefronts of 32 columns per workgroup; p.block_columns is set to match.
// grid_splits: splits of a block's key range (1 = every workgroup walks its block's whole
// range and writes `out`; p.tps_log2 must then be kWholeRange).
hipError_t launch_prefill_bf16(const PromptParams& p, int batch, int D, int waves, int grid_splits, hipStream_t stream) {
  switch (waves) {
    case 2: return launch_prefill_nw<2>(p, batch, D, grid_splits, stream);
    case 4: return launch_prefill_nw<4>(p, batch, D, grid_splits, stream);
    case 8: return launch_prefill_nw<8>(p, batch, D, grid_splits, stream);
    default: return hipErrorInvalidConfiguration;
  }
}

}  // namespace tempo
