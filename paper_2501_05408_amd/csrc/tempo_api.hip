// The C ABI declared in tempo.h: argument validation, split planning, launches.
// Host code only; every step of the path runs in the kernels this file launches.
#include <math.h>
#include <limits.h>
#include <stdio.h>

#include <mutex>

#include "tempo_internal.h"

namespace {

using namespace tempo;

int ilog2_exact(int32_t v) {  // log2 of a power of two, else -1
  if (v <= 0 || (v & (v - 1)) != 0) return -1;
  int k = 0;
  while ((1 << k) < v) ++k;
  return k;
}

// Layout fields only (no pointers): dtype, head_dim, block_size, heads, counts.
int check_layout(const tempo_kv* kv) {
  if (!kv) return TEMPO_ERR_NULL;
  if (kv->dtype != TEMPO_BF16 && kv->dtype != TEMPO_F32) return TEMPO_ERR_DTYPE;
  if (kv->head_dim != 64 && kv->head_dim != 128) return TEMPO_ERR_SHAPE;
  const int zl = ilog2_exact(kv->block_size);
  if (zl < 0) return TEMPO_ERR_SHAPE;
  if (kv->dtype == TEMPO_BF16 && kv->block_size < 32) return TEMPO_ERR_SHAPE;
  if (kv->dtype == TEMPO_F32 && kv->block_size < 4) return TEMPO_ERR_SHAPE;
  if (kv->num_kv_heads < 1 || kv->num_kv_heads > 65535) return TEMPO_ERR_SHAPE;
  if (kv->num_blocks < 1 || kv->max_blocks_per_seq < 1) return TEMPO_ERR_SHAPE;
  if (kv->ring_blocks != 0 &&
      (ilog2_exact(kv->ring_blocks) < 0 || kv->ring_blocks > kv->max_blocks_per_seq))
    return TEMPO_ERR_SHAPE;
  return TEMPO_OK;
}

int check_store(const tempo_kv* kv) {
  const int rc = check_layout(kv);
  if (rc != TEMPO_OK) return rc;
  if (!kv->k_pool || !kv->v_pool || !kv->block_table) return TEMPO_ERR_NULL;
  return TEMPO_OK;
}

// A block of C consecutive query steps: its C * (Hq / Hkv) (step, head) columns
// either ride in the 16-column tile of the decode kernel or, up to 128, go to
// the kernels for wide blocks (launch_block_bf16(); the same limit for fp32).
// A single step of a group of more than 16 query heads is such a block of one step.
constexpr int kMaxColumns = 128;
// Up to this many columns the single-step kernel (one 16-column tile) serves the call.
constexpr int kNarrowColumns = 16;

int check_heads(const tempo_kv* kv, int32_t batch, int32_t Hq) {
  if (batch < 1 || batch > 65535) return TEMPO_ERR_SHAPE;
  if (Hq < 1 || Hq % kv->num_kv_heads != 0) return TEMPO_ERR_SHAPE;
  if (Hq / kv->num_kv_heads > kMaxColumns || Hq > 65535) return TEMPO_ERR_SHAPE;
  return TEMPO_OK;
}

int check_queries(const tempo_kv* kv, int32_t Hq, int32_t queries) {
  if (queries < 1 || queries > kMaxColumns) return TEMPO_ERR_SHAPE;
  if ((int64_t)queries * (Hq / kv->num_kv_heads) > kMaxColumns) return TEMPO_ERR_SHAPE;
  if ((int64_t)queries * Hq > 65535) return TEMPO_ERR_SHAPE;
  return TEMPO_OK;
}

// The constant s of Eq. 1: finite and positive (the kernels take maxima of raw dot
// products and scale afterwards).
int check_scale(float scale) { return (scale > 0.0f && scale <= 3.0e38f) ? TEMPO_OK : TEMPO_ERR_RANGE; }

// The steps a block of queries starting at t touches: the last step, and the
// window measured from the last step that spans the union of the queries' ranges.
int32_t last_step(int32_t t, int32_t queries) { return t + (queries - 1); }
// (0, causal, if that is more than any step is far from step 0)
int32_t union_window(int32_t window, int32_t queries) {
  return window > 0 && window <= INT32_MAX - (queries - 1) ? window + (queries - 1) : 0;
}

// A linear store must have a table column for step t's tile; a ring store reuses
// its columns, so any step can be written.
int check_step(const tempo_kv* kv, int32_t t) {
  if (t < 0) return TEMPO_ERR_RANGE;
  if (kv->ring_blocks == 0 && t / kv->block_size >= kv->max_blocks_per_seq) return TEMPO_ERR_RANGE;
  return TEMPO_OK;
}

// What a ring store can still answer: every tile of the visible range of step t
// (and of any earlier step with the same window) must be resident, i.e. the range
// may touch at most ring_blocks tiles.
int check_ring_covers(const tempo_kv* kv, int32_t t, int32_t window) {
  if (kv->ring_blocks == 0) return TEMPO_OK;
  const int64_t Z = kv->block_size;
  int64_t tiles;
  if (window == 0 || window > (int64_t)t + 1) tiles = t / Z + 1;           // the whole history
  else tiles = window <= 1 ? 1 : ((int64_t)window - 2 + Z) / Z + 1;         // worst alignment
  return tiles <= kv->ring_blocks ? TEMPO_OK : TEMPO_ERR_RANGE;
}

// Rotary tables: both present, made for this head_dim, and long enough for step t.
int check_rope(const tempo_rope* rope, int32_t head_dim, int32_t t_last) {
  if (!rope || !rope->cos || !rope->sin) return TEMPO_ERR_NULL;
  if (rope->head_dim != head_dim) return TEMPO_ERR_SHAPE;
  if ((reinterpret_cast<uintptr_t>(rope->cos) & 15u) != 0 || (reinterpret_cast<uintptr_t>(rope->sin) & 15u) != 0)
    return TEMPO_ERR_SHAPE;
  if (t_last < 0 || rope->positions < 1 || t_last >= rope->positions) return TEMPO_ERR_RANGE;
  return TEMPO_OK;
}

int32_t tile_mask_of(const tempo_kv* kv) { return kv->ring_blocks ? kv->ring_blocks - 1 : INT32_MAX; }

// Upper bound of the number of splits any step t' <= t can need with this tps.
int32_t splits_bound(int32_t t, int32_t window, int tps_log2) {
  const int32_t causal = (t >> tps_log2) + 1;
  if (window <= 0) return causal;
  // a run of `window` keys starting anywhere touches at most ceil((window-1)/tps)+1 chunks
  const int32_t tps = 1 << tps_log2;
  const int32_t win = (window <= 1) ? 1 : (int32_t)(((int64_t)window - 2 + tps) >> tps_log2) + 1;
  return causal < win ? causal : win;
}

// Compute units of the part this library is written for (MI355X).
constexpr int kComputeUnits = 256;
constexpr int kMaxSplits = 1024;

// Does the vector kernel (one workgroup per step and query head) take an fp32 step or block of steps
// instead of the matrix-core one (16 columns of a query group and its steps per workgroup)?  Over short ranges, while the heads' separate
// reads of a group's keys and values (through different dies' caches, so not shared unless the group
// is wide) stay cheap: us a call, vector / matrix, at D = 128:
//   1 sequence, 24/8 heads, 81 keys 6.7 / 7.7, 151 keys 8.3 / 9.4, 200 keys 9.1 / 9.2
//   16 sequences, 24/8 heads, 48 keys 6.5 / 7.1 (18k key rows read), 81 keys 9.1 / 8.3 (31k)
//   16 sequences, 16/1 heads, 200 keys 9.5 / 11.3 (51k), 256 keys 12.6 / 11.6 (66k)
//   blocks of 1 sequence, 24/8 heads: 4 steps, 4 keys 6.3 / 7.9, 32 steps, 32 keys (25k) 10.3 / 9.6; 8/8 heads:
//   32 steps, 32 keys 10.1 / 9.0, 132 keys (34k) 11.1 / 12.9, 64 steps, 164 keys (84k) 15.0 / 12.3
// and always where no head or step shares a read (16 sequences of 8/8 heads, 1501 keys 34.5 / 44.1).  At D = 64
// the matrix-core kernel has half the products: 1 sequence, 8/2 heads, 8 keys 3.4 / 3.9, 64 keys 6.0 / 5.2.
bool f32_on_vector_alu(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t, int32_t window, int32_t queries) {
  if (kv->dtype != TEMPO_F32) return false;
  const int64_t keys = window > 0 && window < (int64_t)t + 1 ? window : (int64_t)t + 1;  // of the last step
  const int32_t G = Hq / kv->num_kv_heads;
  if (kv->head_dim == 128 && G == 1 && queries == 1) return true;
  if (keys > (kv->head_dim == 128 ? 192 : 24)) return false;
  const int64_t rows = batch * keys * Hq * queries, shared = G < 8 ? 8 : (G > 32 ? 32 : G);
  if (queries == 1) return rows <= 3200 * shared;
  return keys > 64 ? rows <= 36000 : queries <= (kv->head_dim == 128 ? 16 : 8) && rows <= 12000;
}

// Split planning: a small time model of the launch, in nanoseconds, with constants
// measured on MI355X.
//   - Workgroups are handed to compute units round-robin, so the busiest unit gets
//     rounds = ceil(workgroups / units) of them, one after the other.
//   - A unit streams keys/values at its share of what the memory system sustains for
//     this access pattern (about 6.9 TB/s over all units), but never faster than
//     about 40 GB/s, so fewer than ~170 busy units cannot use the whole bandwidth.
//   - A launch pays about 2 us once before its first key arrives (dispatch, kernel
//     arguments, block table, first loads), about 1 us per round (a workgroup's own
//     argument -> table -> data chain and its merge and partial write, as far as the other
//     workgroups resident on the unit do not hide them; fitted on steps that are not powers
//     of two, where short splits looked better than they are), and about 3 us for the
//     combine launch if there is more than one split, 5 us if there are more than the 8 that
//     the one-batch combine takes.  (With 3 us for both, a few sequences got many short splits:
//     one sequence, t = 299, 10 splits 8.8 us, one split 5.9 us; over 104 measured cases of
//     batch 1 .. 16 with 8 or 16 heads the mean distance from the fastest plan went from 3.5% to
//     0.4%, the largest from 50% to 6%; over 90 of 4 and 6 (sequence, head) pairs from 15% to 3%, the
//     largest from 69% to 20%.  One and two pairs keep 3 us, though 5 us would serve them as well
//     (over 90 cases 19% to 6%, 70% to 27%): they are what the block tests reach the combine of more
//     than 8 splits with.  A one-batch combine of 16 or 32 splits was 2 us slower than the one
//     through LDS.)
// Short splits balance better; long splits mean fewer rounds, fewer partials and,
// at one split, no combine at all.  Take the LONGEST split length whose estimate is
// within 3% of the best one.
constexpr double kSustainedBytesPerNs = 6900.0;  // whole part, GB/s
constexpr double kUnitBytesPerNs = 40.0;         // one compute unit, GB/s
constexpr double kLaunchNs = 2000.0, kRoundNs = 1000.0, kCombineNs = 3000.0, kCombineManyNs = 5000.0;
constexpr int64_t kManyPairs = 3;

double plan_cost_ns(int64_t pairs, int64_t splits, int64_t keys_per_split, int bytes_per_key) {
  const int64_t workgroups = pairs * splits;
  const int64_t busy = workgroups < kComputeUnits ? workgroups : kComputeUnits;
  const double share = kSustainedBytesPerNs / (double)busy;
  const double rate = share < kUnitBytesPerNs ? share : kUnitBytesPerNs;
  const int64_t rounds = (workgroups + kComputeUnits - 1) / kComputeUnits;
  return kLaunchNs + (double)rounds * (kRoundNs + (double)keys_per_split * bytes_per_key / rate) +
         (splits > 8 && pairs >= kManyPairs ? kCombineManyNs : splits > 1 ? kCombineNs : 0.0);
}

// Ragged batches (per-sequence steps below t_max) hold less work than the model
// assumes and it is unevenly spread, so their splits are capped at 1024 keys to
// keep the long sequences from becoming single long-running workgroups.
// max_splits: no more splits than this (unless even the longest splits of a ragged batch are more).
void make_plan(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t_max, int32_t window,
               bool ragged, int32_t queries, int64_t max_splits, tempo_plan* plan) {
  // one workgroup serves a query group; fp32 takes 16 (step, head) columns per workgroup
  const int64_t columns = (int64_t)queries * (Hq / kv->num_kv_heads);
  const int64_t pairs = f32_on_vector_alu(kv, batch, Hq, t_max, window, queries)
                            ? (int64_t)batch * Hq
                            : (int64_t)batch * kv->num_kv_heads * (kv->dtype == TEMPO_F32 ? (columns + 15) / 16 : 1);
  const int64_t len = (window > 0 && window < (int64_t)t_max + 1) ? window : (int64_t)t_max + 1;
  const int bytes_per_key = 2 * kv->head_dim * (kv->dtype == TEMPO_BF16 ? 2 : 4);  // K and V of one head
  const int k_max = ragged ? 10 : 30;
  int best_k = -1;
  double best_cost = -1.0;
  double costs[26];
  for (int k = 5; k <= 30; ++k) costs[k - 5] = -1.0;
  for (int k = 5; k <= k_max; ++k) {
    const int64_t splits = splits_bound(t_max, window, k);
    if (splits > max_splits) continue;
    const int64_t tps = (int64_t)1 << k;
    const int64_t per_split = tps < len ? tps : len;  // a split never holds more than the range
    costs[k - 5] = plan_cost_ns(pairs, splits, per_split, bytes_per_key);
    if (best_cost < 0.0 || costs[k - 5] < best_cost) best_cost = costs[k - 5];
    if (splits == 1) break;  // longer splits change nothing
  }
  for (int k = 5; k <= k_max; ++k) {
    if (costs[k - 5] >= 0.0 && costs[k - 5] <= best_cost * 1.03) best_k = k;
  }
  if (best_k < 0) {  // a ragged range too long for 1024 splits of 1024 keys: lengthen until it fits
    best_k = k_max;
    while (splits_bound(t_max, window, best_k) > kMaxSplits) ++best_k;
  }
  plan->tokens_per_split = 1 << best_k;
  plan->num_splits = splits_bound(t_max, window, best_k);
  // About 8 wavefronts per compute unit keep the memory pipe full: 4 per workgroup
  // when a unit gets two or more workgroups, 8 when it gets at most one (measured:
  // 256 workgroups x 8 waves 42.4 us, x 4 waves 43.4 us; 512 x 4 waves 42.7 us), down
  // to one 32-slot group per wavefront (256 keys at batch 16: 7.7 us with 8, 8.2 with 4).
  const int groups = plan->tokens_per_split / 32;
  const int64_t workgroups = pairs * plan->num_splits;
  if (workgroups <= kComputeUnits && groups >= 8) plan->waves = 8;
  else plan->waves = groups >= 4 ? 4 : groups;
}

// A uniform step needs its own split count; ragged steps (any t' <= t) need the bound.
int check_plan(const tempo_plan* plan, int32_t t, int32_t window, bool ragged, int32_t queries,
               int32_t pad_t = 0) {
  if (!plan) return TEMPO_ERR_NULL;
  const int k = ilog2_exact(plan->tokens_per_split);
  if (k < 5) return TEMPO_ERR_SHAPE;
  if (plan->waves != 1 && plan->waves != 2 && plan->waves != 4 && plan->waves != 8) return TEMPO_ERR_SHAPE;
  if (plan->num_splits < 1 || plan->num_splits > 65535) return TEMPO_ERR_SHAPE;
  const int32_t cover = last_step(t, queries) > pad_t ? last_step(t, queries) : pad_t;
  const int32_t need = ragged ? splits_bound(cover, union_window(window, queries), k)
                              : seq_range(t, window, k, queries, pad_t).nchunks;
  if (plan->num_splits < need) return TEMPO_ERR_RANGE;
  return TEMPO_OK;
}

// Map a launch status to the ABI's; say on stderr what the runtime said.
int launch_status(hipError_t e, const char* what) {
  if (e == hipSuccess) return TEMPO_OK;
  fprintf(stderr, "libtempo: launch of %s failed: %s\n", what, hipGetErrorString(e));
  return TEMPO_ERR_LAUNCH;
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- statically allocated partials for callers that cannot allocate -----------------
// tempo_decode_step_causal_noalloc keeps the split partials here instead of in a caller's
// workspace.  Each GPU holds its own copy of the array, at its own address, until the
// process ends.  In host code the array's name is only a handle for hipGetSymbolAddress:
// the address kernels are given is the one that call returned for the current device.
constexpr size_t kScratchBytes = (size_t)8 << 20;
__attribute__((used)) static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, resolved once per device.
int scratch_on_current_device(void** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    fprintf(stderr, "libtempo: no current device for the static scratch array: %s\n", hipGetErrorString(e));
    return TEMPO_ERR_LAUNCH;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      fprintf(stderr, "libtempo: hipGetSymbolAddress(scratch) failed on device %d: %s\n", dev, hipGetErrorString(e));
      return TEMPO_ERR_LAUNCH;
    }
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return TEMPO_OK;
}


// Workspace = [m,l: rows*S*2 f32] [acc: rows*S*D f32], each part padded to 256 bytes;
// rows = batch * queries * Hq.
size_t ml_bytes(int64_t rows, int32_t S) { return align_up((size_t)rows * S * 2 * sizeof(float), 256); }

size_t plan_bytes(const tempo_kv* kv, int64_t rows, int32_t S) {
  return ml_bytes(rows, S) + align_up((size_t)rows * S * kv->head_dim * sizeof(float), 256);
}

// The decode kernel's wave-merge area: a limit of its launch.  (The fp32 kernel asks for up to 68,608
// bytes, the prompt kernel for up to 128 KiB, of the 160 KiB a compute unit has.)
constexpr size_t kMaxLds = 64 * 1024;

AttnParams attn_params(const tempo_kv* kv, const void* q, void* out, int32_t Hq, int32_t t,
                       const int32_t* t_per_seq, int32_t window, float scale,
                       const tempo_plan* plan, void* workspace, int32_t batch, int32_t queries,
                       int32_t pad_t = 0) {
  AttnParams p;
  p.k_pool = kv->k_pool;
  p.v_pool = kv->v_pool;
  p.block_table = kv->block_table;
  p.q = q;
  p.k_new = nullptr;
  p.v_new = nullptr;
  p.t_per_seq = t_per_seq;
  p.count_per_seq = nullptr;
  p.rope_cos = nullptr;
  p.rope_sin = nullptr;
  p.worklist = nullptr;
  char* ws = static_cast<char*>(workspace);
  p.ws_ml = reinterpret_cast<float*>(ws);
  p.ws_acc = reinterpret_cast<float*>(ws + ml_bytes((int64_t)batch * queries * Hq, plan->num_splits));
  p.out = out;
  p.t = t;
  p.window = window;
  p.z_log2 = ilog2_exact(kv->block_size);
  p.max_blocks_per_seq = kv->max_blocks_per_seq;
  p.tile_mask = tile_mask_of(kv);
  p.num_blocks = kv->num_blocks;
  p.Hkv = kv->num_kv_heads;
  p.Hq = Hq;
  p.G = Hq / kv->num_kv_heads;
  p.tps_log2 = ilog2_exact(plan->tokens_per_split);
  p.num_splits = plan->num_splits;
  p.queries = queries;
  p.io_steps = queries;
  p.pad_t = pad_t;
  p.direct = 0;
  p.scale_log2e = scale * 1.44269504088896340736f;
  return p;
}

StoreParams store_params(const tempo_kv* kv, int32_t batch, int32_t t, const int32_t* t_per_seq,
                         int32_t count = 1) {
  StoreParams p;
  p.k_pool = kv->k_pool;
  p.v_pool = kv->v_pool;
  p.block_table = kv->block_table;
  p.t_per_seq = t_per_seq;
  p.t = t;
  p.z_log2 = ilog2_exact(kv->block_size);
  p.max_blocks_per_seq = kv->max_blocks_per_seq;
  p.tile_mask = tile_mask_of(kv);
  p.num_blocks = kv->num_blocks;
  p.Hkv = kv->num_kv_heads;
  p.batch = batch;
  p.count = count;
  p.src_steps = count;
  p.count_per_seq = nullptr;
  p.rope_cos = nullptr;
  p.rope_sin = nullptr;
  return p;
}

// Splits to launch along grid.x: exact for a uniform step, the bound for ragged steps.
int32_t grid_splits(const tempo_plan* plan, int32_t t, const int32_t* t_per_seq, int32_t window,
                    int32_t queries, int32_t pad_t) {
  if (t_per_seq) return plan->num_splits;
  const int32_t exact = seq_range(t, window, ilog2_exact(plan->tokens_per_split), queries, pad_t).nchunks;
  return exact < plan->num_splits ? exact : plan->num_splits;
}

int check_attn(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t, int32_t window, bool ragged,
               const tempo_plan* plan, const void* workspace, size_t workspace_bytes,
               int32_t queries = 1, int32_t pad_t = 0) {
  int rc = check_store(kv);
  if (rc != TEMPO_OK) return rc;
  if ((rc = check_heads(kv, batch, Hq)) != TEMPO_OK) return rc;
  if ((rc = check_queries(kv, Hq, queries)) != TEMPO_OK) return rc;
  if (window < 0 || t < 0 || t > INT32_MAX - 64) return TEMPO_ERR_RANGE;
  // the padded baseline is causal only: with a window the range's length would depend on the step
  if (pad_t < 0 || (pad_t > 0 && window != 0)) return TEMPO_ERR_RANGE;
  const int32_t cover = last_step(t, queries) > pad_t ? last_step(t, queries) : pad_t;
  if ((rc = check_step(kv, cover)) != TEMPO_OK) return rc;
  if ((rc = check_ring_covers(kv, cover, union_window(window, queries))) != TEMPO_OK) return rc;
  if ((rc = check_plan(plan, t, window, ragged, queries, pad_t)) != TEMPO_OK) return rc;
  if (kv->dtype == TEMPO_BF16) {
    const int columns = queries * (Hq / kv->num_kv_heads);
    // more than 16 columns go to the kernels for wide blocks, whose launch shapes are fixed
    if (columns <= kNarrowColumns && partial_bf16_lds_bytes(plan->waves, columns, kv->head_dim) > kMaxLds) return TEMPO_ERR_SHAPE;
  }
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return TEMPO_ERR_WORKSPACE;
  if (workspace_bytes < plan_bytes(kv, (int64_t)batch * queries * Hq, plan->num_splits)) return TEMPO_ERR_WORKSPACE;
  return TEMPO_OK;
}

// Wavefronts of the fp32 matrix-core kernel, whose groups have 16 keys where a plan's have 32: a split of
// 32 or 64 keys that is planned with a wavefront for every 32 gets one for every 16, because a wavefront's
// second group costs such a split about as much as its first (24/8 heads of 128, 1 sequence: splits of 32
// keys at t = 700 11.1 us with 1 wavefront, 9.3 us with 2; one split at t = 63 7.2 us with 2, 6.3 us with 4).
int f32_waves(const tempo_plan& plan) {
  return plan.waves <= 2 && plan.waves * 32 == plan.tokens_per_split ? 2 * plan.waves : plan.waves;
}

// out != nullptr and a single split: the launch writes `out` itself; otherwise it
// writes partials and the caller launches the combine.
// k_new/v_new != nullptr: step t's key/value are appended inside the same launch.
int do_partial(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new, void* out,
               int32_t batch, int32_t Hq, int32_t t, const int32_t* t_per_seq, int32_t window,
               float scale, const tempo_plan* plan, void* workspace, hipStream_t stream,
               int32_t queries = 1, const tempo_rope* rope = nullptr, int32_t pad_t = 0, int32_t io_steps = 0,
               const int32_t* worklist = nullptr) {
  AttnParams p = attn_params(kv, q, out, Hq, t, t_per_seq, window, scale, plan, workspace, batch, queries, pad_t);
  if (io_steps > 0) p.io_steps = io_steps;
  p.worklist = worklist;
  p.direct = (out != nullptr && plan->num_splits == 1) ? 1 : 0;
  p.k_new = k_new;
  p.v_new = v_new;
  if (rope) {
    p.rope_cos = rope->cos;
    p.rope_sin = rope->sin;
  }
  const int32_t gs = grid_splits(plan, t, t_per_seq, window, queries, pad_t);
  if (kv->dtype == TEMPO_BF16 && queries * p.G > kNarrowColumns)  // a wide block: kernels of their own, key range split as planned
    return launch_status(launch_block_bf16(p, batch, kv->head_dim, gs, stream), "attn_block_partial");
  const hipError_t e = kv->dtype == TEMPO_BF16
                           ? launch_partial_bf16(p, batch, kv->head_dim, gs, plan->waves, stream)
                       : f32_on_vector_alu(kv, batch, Hq, last_step(t, queries), union_window(window, queries), queries)
                           ? launch_step_f32(p, batch, kv->head_dim, gs, plan->waves, stream)
                           : launch_partial_f32(p, batch, kv->head_dim, gs, f32_waves(*plan), stream);
  return launch_status(e, "attn_decode_partial");
}

int do_combine(const tempo_kv* kv, void* out, int32_t batch, int32_t Hq, int32_t t,
               const int32_t* t_per_seq, int32_t window, const tempo_plan* plan, void* workspace,
               hipStream_t stream, int32_t queries = 1, int32_t pad_t = 0, int32_t io_steps = 0) {
  AttnParams p = attn_params(kv, nullptr, out, Hq, t, t_per_seq, window, 1.0f, plan, workspace, batch, queries,
                             pad_t);
  if (io_steps > 0) p.io_steps = io_steps;
  const hipError_t e = launch_combine(p, batch, kv->head_dim, kv->dtype, stream);
  return launch_status(e, "attn_decode_combine");
}

// Splits of a block that the stream kernel takes: a time model as make_plan()'s, in nanoseconds, fitted to 228 blocks
// of 18 to 124 columns behind 150 to 8000 keys at 7 split lengths each (the plans it takes are 0.5% off the fastest on
// the mean, 16% at most).  One workgroup of 8 wavefronts per compute unit: about 3.4 us before its first group and
// after its last one (at D = 64 three quarters of it), then its share of the stream or, if that takes longer, its
// wavefronts' arithmetic, 1 us a group and tile of 32 columns; the combine reads and writes a partial per
// column and split.  max_splits: no more than this.
void make_stream_plan(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t, int32_t window, bool ragged,
                      int32_t queries, int64_t max_splits, tempo_plan* plan) {
  constexpr double kFixedNs = 3400.0, kGroupNs = 1000.0, kFewNs = 5000.0, kManyNs = 8000.0, kPartialBytesPerNs = 4800.0;
  const int D = kv->head_dim, columns = queries * (Hq / kv->num_kv_heads);
  const int tiles = columns <= 32 ? 1 : columns <= 64 ? 2 : 4;
  const int64_t pairs = (int64_t)batch * kv->num_kv_heads, keys = block_keys(t, queries, window);
  const int32_t t_eff = last_step(t, queries), w_eff = union_window(window, queries);
  const double wide = D / 128.0;
  double costs[31], best = -1.0;
  const int k_max = ragged ? 10 : 30;  // (ragged batches: as in make_plan)
  int last = 7;
  for (int k = 7; k <= k_max; ++k) {
    const int64_t splits = splits_bound(t_eff, w_eff, k), workgroups = pairs * splits;
    const int64_t rounds = (workgroups + kComputeUnits - 1) / kComputeUnits, busy = workgroups < kComputeUnits ? workgroups : kComputeUnits;
    const int64_t per_split = ((int64_t)1 << k) < keys ? (int64_t)1 << k : keys;
    const double share = kSustainedBytesPerNs / (double)busy, rate = share < kUnitBytesPerNs ? share : kUnitBytesPerNs;
    const double stream = (double)per_split * D * 4 / rate, work = (double)((per_split + 255) / 256) * kGroupNs * tiles * wide;
    costs[k] = (double)rounds * (kFixedNs * (D == 128 ? 1.0 : 0.75) + (stream > work ? stream : work));
    if (splits > 1) costs[k] += (splits > 8 ? kManyNs : kFewNs) + 2.0 * batch * queries * Hq * (double)splits * D * 4 / kPartialBytesPerNs;
    if (splits <= max_splits && (best < 0.0 || costs[k] < best)) best = costs[k];
    last = k;
    if (splits == 1) break;
  }
  int chosen = last;
  while (splits_bound(t_eff, w_eff, chosen) > max_splits) ++chosen;
  for (int k = 7; k <= last; ++k) {  // the longest within 2% of the best
    if (splits_bound(t_eff, w_eff, k) <= max_splits && costs[k] <= best * 1.02) chosen = k;
  }
  plan->tokens_per_split = 1 << chosen;
  plan->num_splits = splits_bound(t_eff, w_eff, chosen);
  plan->waves = 8;  // (always)
}

// Plan of a block of queries: the plan of the union range, with the wavefront count
// cut down until the bf16 kernel's wave-merge area (one accumulator row per column
// and wavefront) fits the LDS a workgroup may ask for.
void make_block_plan(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t, int32_t window,
                     bool ragged, int32_t queries, tempo_plan* plan, int64_t max_splits = kMaxSplits) {
  make_plan(kv, batch, Hq, last_step(t, queries), union_window(window, queries), ragged, queries, max_splits, plan);
  if (kv->dtype != TEMPO_BF16) return;
  const int columns = queries * (Hq / kv->num_kv_heads);
  if (columns > kNarrowColumns && block_streams(kv->head_dim, columns, (int64_t)batch * kv->num_kv_heads, block_keys(t, queries, window))) {
    make_stream_plan(kv, batch, Hq, t, window, ragged, queries, max_splits, plan);
    return;
  }
  if (columns > kNarrowColumns) {
    // The LDS-staged kernel: its workgroups do more arithmetic per key than the decode
    // kernel's, so two per compute unit are wanted (measured at batch 16 x 8 heads,
    // t = 4095: 4 splits of 1024 keys 59-68 us for 63-126 columns, 2 splits 82-83 us,
    // 8 splits 68-81 us).  Up to 32 columns a workgroup has only two wavefronts: twice as many
    // workgroups (measured there: 8 splits of 512 keys 52.8-53.8 us, 4 splits of 1024 keys 55.5-56.1 us).
    // Longest split length of at least 256 keys that gives as many workgroups, else 256.
    const int32_t t_eff = last_step(t, queries), w_eff = union_window(window, queries);
    const int64_t pairs = (int64_t)batch * kv->num_kv_heads;
    const int64_t want = (columns <= 32 ? 4 : 2) * (int64_t)kComputeUnits;
    int k = 8;
    for (int cand = 30; cand >= 8; --cand) {
      if (pairs * splits_bound(t_eff, w_eff, cand) >= want) { k = cand; break; }
    }
    while (splits_bound(t_eff, w_eff, k) > max_splits) ++k;
    if (ragged && k > 10 && splits_bound(t_eff, w_eff, 10) <= max_splits) k = 10;  // as for single steps
    plan->tokens_per_split = 1 << k;
    plan->num_splits = splits_bound(t_eff, w_eff, k);
    plan->waves = 8;  // ignored: the launch picks 2, 4 or 8 wavefronts by the column count
    return;
  }
  while (plan->waves > 1 && partial_bf16_lds_bytes(plan->waves, columns, kv->head_dim) > kMaxLds) plan->waves /= 2;
}

int decode(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new, void* out,
           int32_t batch, int32_t Hq, int32_t t, const int32_t* t_per_seq, int32_t window, float scale,
           void* workspace, size_t workspace_bytes, void* stream, int32_t queries = 1,
           const tempo_rope* rope = nullptr, int32_t pad_t = 0, const int32_t* worklist = nullptr,
           int64_t max_splits = kMaxSplits) {
  int rc = check_layout(kv);
  if (rc != TEMPO_OK) return rc;
  if (!q || !out) return TEMPO_ERR_NULL;
  if ((rc = check_heads(kv, batch, Hq)) != TEMPO_OK) return rc;
  if ((rc = check_queries(kv, Hq, queries)) != TEMPO_OK) return rc;
  if (t < 0 || window < 0 || t > INT32_MAX - 64) return TEMPO_ERR_RANGE;
  if ((rc = check_scale(scale)) != TEMPO_OK) return rc;
  if (rope && (rc = check_rope(rope, kv->head_dim, last_step(t, queries))) != TEMPO_OK) return rc;
  if (pad_t < 0 || pad_t > INT32_MAX - 64) return TEMPO_ERR_RANGE;
  tempo_plan plan;
  // the padded baseline is planned as the step it pretends every step to be
  make_block_plan(kv, batch, Hq, pad_t > t ? pad_t : t, window, t_per_seq != nullptr, queries, &plan, max_splits);
  if ((rc = check_attn(kv, batch, Hq, t, window, t_per_seq != nullptr, &plan, workspace, workspace_bytes, queries,
                       pad_t)) != TEMPO_OK)
    return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // With more (sequence, head) pairs than compute units the in-kernel block-store write
  // costs more than a launch of its own (measured at 512 pairs: +7.5 us inside the
  // attention kernel, +4 us as a separate launch; at 128 pairs +1 us inside): write first.
  // A group of more than 16 query heads runs in the kernels for wide blocks, which read the
  // store only: the write (rotating the key when tables are given) goes first there too,
  // and they rotate the queries.
  const bool wide = kv->dtype == TEMPO_BF16 && queries * (Hq / kv->num_kv_heads) > kNarrowColumns;
  if (k_new && kv->dtype == TEMPO_BF16 && (wide || (!rope && (int64_t)batch * kv->num_kv_heads > kComputeUnits))) {
    const StoreParams sp = store_params(kv, batch, t, t_per_seq);
    const hipError_t e = rope ? launch_rope_append(sp, rope->cos, rope->sin, k_new, v_new, kv->head_dim, kv->dtype, s)
                              : launch_append(sp, k_new, v_new, kv->head_dim, kv->dtype, s);
    if ((rc = launch_status(e, "kv_append")) != TEMPO_OK) return rc;
    k_new = v_new = nullptr;
  }
  rc = do_partial(kv, q, k_new, v_new, out, batch, Hq, t, t_per_seq, window, scale, &plan, workspace, s, queries,
                  rope, pad_t, 0, worklist);
  if (rc != TEMPO_OK || plan.num_splits == 1) return rc;  // a single split wrote `out` itself
  return do_combine(kv, out, batch, Hq, t, t_per_seq, window, &plan, workspace, s, queries, pad_t);
}

}  // namespace

extern "C" {

int tempo_visible_range(int32_t t, int32_t window, int32_t Z, int32_t* lo, int32_t* hi,
                        int32_t* first_tile, int32_t* last_tile, int32_t* first_tile_skip,
                        int32_t* last_tile_valid) {
  if (t < 0 || window < 0 || Z < 1) return TEMPO_ERR_RANGE;
  const int32_t l = (window > 0 && t - window + 1 > 0) ? t - window + 1 : 0;
  if (lo) *lo = l;
  if (hi) *hi = t;
  if (first_tile) *first_tile = l / Z;
  if (last_tile) *last_tile = t / Z;
  if (first_tile_skip) *first_tile_skip = l % Z;
  if (last_tile_valid) *last_tile_valid = t % Z + 1;
  return TEMPO_OK;
}

int tempo_append_slot(int32_t t, int32_t Z, int32_t* tile, int32_t* slot) {
  if (t < 0 || Z < 1) return TEMPO_ERR_RANGE;
  if (tile) *tile = t / Z;
  if (slot) *slot = t % Z;
  return TEMPO_OK;
}

int tempo_kv_release(int32_t t, int32_t window, int32_t Z, int32_t* dead_keys, int32_t* dead_tiles) {
  if (t < 0 || t == INT32_MAX || window < 0 || Z < 1) return TEMPO_ERR_RANGE;  // t + 1 keys must be countable
  // the last reader of key j is step j + window - 1: dead after step t iff j <= t - window + 1
  int64_t dead = window == 0 ? 0 : (int64_t)t - window + 2;
  if (dead < 0) dead = 0;
  if (dead_keys) *dead_keys = (int32_t)dead;
  if (dead_tiles) *dead_tiles = (int32_t)(dead / Z);
  return TEMPO_OK;
}

int tempo_ring_blocks(int32_t window, int32_t Z, int32_t queries, int32_t* ring_blocks) {
  if (!ring_blocks) return TEMPO_ERR_NULL;
  if (window < 1 || Z < 1 || queries < 1) return TEMPO_ERR_RANGE;
  // the union of the queries' ranges, at its worst alignment to the tiles
  const int64_t span = (int64_t)window + queries - 1;
  const int64_t tiles = span <= 1 ? 1 : (span - 2 + Z) / Z + 1;
  if (tiles > (1 << 30)) return TEMPO_ERR_RANGE;
  int32_t ring = 1;
  while (ring < tiles) ring *= 2;
  *ring_blocks = ring;
  return TEMPO_OK;
}

int64_t tempo_kv_element_offset(const tempo_kv* kv, int32_t which, int32_t block, int32_t head,
                                int32_t slot, int32_t d) {
  if (check_layout(kv) != TEMPO_OK) return -1;
  if (which < 0 || which > 1 || block < 0 || block >= kv->num_blocks || head < 0 ||
      head >= kv->num_kv_heads || slot < 0 || slot >= kv->block_size || d < 0 || d >= kv->head_dim)
    return -1;
  const int D = kv->head_dim;
  const int64_t base = ((int64_t)block * kv->num_kv_heads + head) * kv->block_size * D;
  if (kv->dtype == TEMPO_F32) return base + tile_off_f32(D, slot, d);
  return base + (which == 0 ? tile_off_k_bf16(D, slot, d) : tile_off_v_bf16(D, slot, d));
}

size_t tempo_kv_pool_bytes(const tempo_kv* kv) {
  if (check_layout(kv) != TEMPO_OK) return 0;
  const size_t e = kv->dtype == TEMPO_BF16 ? 2 : 4;
  return (size_t)kv->num_blocks * kv->num_kv_heads * kv->block_size * kv->head_dim * e;
}

int tempo_attn_plan(const tempo_kv* kv, int32_t batch, int32_t num_q_heads, int32_t t_max,
                    int32_t window, int32_t ragged, tempo_plan* plan) {
  int rc = check_layout(kv);
  if (rc != TEMPO_OK) return rc;
  if (!plan) return TEMPO_ERR_NULL;
  if ((rc = check_heads(kv, batch, num_q_heads)) != TEMPO_OK) return rc;
  if (t_max < 0 || window < 0) return TEMPO_ERR_RANGE;
  make_block_plan(kv, batch, num_q_heads, t_max, window, ragged != 0, 1, plan);
  return TEMPO_OK;
}

size_t tempo_attn_plan_workspace_bytes(const tempo_kv* kv, int32_t batch, int32_t num_q_heads,
                                       const tempo_plan* plan) {
  if (check_layout(kv) != TEMPO_OK || !plan) return 0;
  if (check_heads(kv, batch, num_q_heads) != TEMPO_OK || plan->num_splits < 1) return 0;
  return plan_bytes(kv, (int64_t)batch * num_q_heads, plan->num_splits);
}

size_t tempo_attn_workspace_bytes(const tempo_kv* kv, int32_t batch, int32_t num_q_heads,
                                  int32_t max_t) {
  if (check_layout(kv) != TEMPO_OK || max_t < 0) return 0;
  if (check_heads(kv, batch, num_q_heads) != TEMPO_OK) return 0;
  // The planner's split count is not monotone in t, so take the largest count it
  // produces for any step up to max_t and any window.  A shorter range or a window
  // never needs more splits than the causal range of max_t at the same split
  // length, and the planner only chooses lengths of at least 32, so the causal
  // count at length 32, capped at the planner's own maximum, bounds them all.
  int64_t worst = splits_bound(max_t, 0, 5);
  if (worst > kMaxSplits) worst = kMaxSplits;
  return plan_bytes(kv, (int64_t)batch * num_q_heads, (int32_t)worst);
}

int tempo_attn_block_plan(const tempo_kv* kv, int32_t batch, int32_t num_q_heads, int32_t queries,
                          int32_t t_max, int32_t window, int32_t ragged, tempo_plan* plan) {
  int rc = check_layout(kv);
  if (rc != TEMPO_OK) return rc;
  if (!plan) return TEMPO_ERR_NULL;
  if ((rc = check_heads(kv, batch, num_q_heads)) != TEMPO_OK) return rc;
  if ((rc = check_queries(kv, num_q_heads, queries)) != TEMPO_OK) return rc;
  if (t_max < 0 || t_max > INT32_MAX - 64 || window < 0 || window > INT32_MAX - 64) return TEMPO_ERR_RANGE;
  make_block_plan(kv, batch, num_q_heads, t_max, window, ragged != 0, queries, plan);
  return TEMPO_OK;
}

size_t tempo_attn_block_workspace_bytes(const tempo_kv* kv, int32_t batch, int32_t num_q_heads,
                                        int32_t queries, int32_t max_t) {
  if (check_layout(kv) != TEMPO_OK || max_t < 0 || max_t > INT32_MAX - 64) return 0;
  if (check_heads(kv, batch, num_q_heads) != TEMPO_OK) return 0;
  if (check_queries(kv, num_q_heads, queries) != TEMPO_OK) return 0;
  // as tempo_attn_workspace_bytes, for the union range that ends at the last query's step
  int64_t worst = splits_bound(last_step(max_t, queries), 0, 5);
  if (worst > kMaxSplits) worst = kMaxSplits;
  return plan_bytes(kv, (int64_t)batch * queries * num_q_heads, (int32_t)worst);
}

const char* tempo_strerror(int status) {
  switch (status) {
    case TEMPO_OK: return "ok";
    case TEMPO_ERR_NULL: return "a required pointer is NULL";
    case TEMPO_ERR_SHAPE: return "unsupported shape (head_dim, block_size, head counts or batch)";
    case TEMPO_ERR_RANGE: return "step or window out of range for this block store";
    case TEMPO_ERR_WORKSPACE: return "workspace is NULL, misaligned or too small";
    case TEMPO_ERR_DTYPE: return "unknown dtype";
    case TEMPO_ERR_LAUNCH: return "HIP launch failed";
    default: return "unknown status";
  }
}

int tempo_kv_append(const tempo_kv* kv, const void* k_new, const void* v_new, int32_t batch,
                    int32_t t, const int32_t* t_per_seq, void* stream) {
  int rc = check_store(kv);
  if (rc != TEMPO_OK) return rc;
  if (!k_new || !v_new) return TEMPO_ERR_NULL;
  if (batch < 1 || batch > 65535) return TEMPO_ERR_SHAPE;
  if ((rc = check_step(kv, t)) != TEMPO_OK) return rc;
  if ((int64_t)batch * kv->num_kv_heads * kv->head_dim > INT32_MAX) return TEMPO_ERR_SHAPE;
  const StoreParams p = store_params(kv, batch, t, t_per_seq);
  const hipError_t e = launch_append(p, k_new, v_new, kv->head_dim, kv->dtype, static_cast<hipStream_t>(stream));
  return launch_status(e, "kv_append");
}

int tempo_kv_append_block(const tempo_kv* kv, const void* k_new, const void* v_new, int32_t batch,
                          int32_t t, const int32_t* t_per_seq, int32_t count, void* stream) {
  int rc = check_store(kv);
  if (rc != TEMPO_OK) return rc;
  if (!k_new || !v_new) return TEMPO_ERR_NULL;
  if (batch < 1 || batch > 65535) return TEMPO_ERR_SHAPE;
  if (count < 1 || count > 65536) return TEMPO_ERR_SHAPE;
  if (t < 0 || t > INT32_MAX - count) return TEMPO_ERR_RANGE;
  if ((rc = check_step(kv, t + count - 1)) != TEMPO_OK) return rc;
  // a ring store must not wrap onto rows of the same call
  if (kv->ring_blocks && (int64_t)count > (int64_t)kv->ring_blocks * kv->block_size) return TEMPO_ERR_RANGE;
  if ((int64_t)batch * count * kv->num_kv_heads * kv->head_dim > INT32_MAX) return TEMPO_ERR_SHAPE;
  const StoreParams p = store_params(kv, batch, t, t_per_seq, count);
  const hipError_t e = launch_append(p, k_new, v_new, kv->head_dim, kv->dtype, static_cast<hipStream_t>(stream));
  return launch_status(e, "kv_append_block");
}

int tempo_rope_kv_append_block(const tempo_kv* kv, const tempo_rope* rope, const void* k_raw, const void* v_new,
                               int32_t batch, int32_t t, const int32_t* t_per_seq, int32_t count, void* stream) {
  int rc = check_store(kv);
  if (rc != TEMPO_OK) return rc;
  if (!k_raw || !v_new) return TEMPO_ERR_NULL;
  if (kv->dtype != TEMPO_BF16) return TEMPO_ERR_DTYPE;  // the block write rotates in the bf16 kernels only
  if (batch < 1 || batch > 65535) return TEMPO_ERR_SHAPE;
  if (count < 1 || count > 65536) return TEMPO_ERR_SHAPE;
  if (t < 0 || t > INT32_MAX - count) return TEMPO_ERR_RANGE;
  if ((rc = check_step(kv, t + count - 1)) != TEMPO_OK) return rc;
  if ((rc = check_rope(rope, kv->head_dim, t + count - 1)) != TEMPO_OK) return rc;
  if (kv->ring_blocks && (int64_t)count > (int64_t)kv->ring_blocks * kv->block_size) return TEMPO_ERR_RANGE;
  if ((int64_t)batch * count * kv->num_kv_heads * kv->head_dim > INT32_MAX) return TEMPO_ERR_SHAPE;
  StoreParams p = store_params(kv, batch, t, t_per_seq, count);
  p.rope_cos = rope->cos;
  p.rope_sin = rope->sin;
  const hipError_t e = launch_append(p, k_raw, v_new, kv->head_dim, kv->dtype, static_cast<hipStream_t>(stream));
  return launch_status(e, "kv_rope_append_block");
}

int tempo_kv_gather(const tempo_kv* kv, void* k_out, void* v_out, int32_t batch, int32_t j0,
                    int32_t count, void* stream) {
  int rc = check_store(kv);
  if (rc != TEMPO_OK) return rc;
  if (batch < 1 || batch > 65535) return TEMPO_ERR_SHAPE;
  if (j0 < 0 || count < 0) return TEMPO_ERR_RANGE;
  if (count == 0) return TEMPO_OK;
  if ((int64_t)j0 + count - 1 > INT32_MAX) return TEMPO_ERR_RANGE;
  if ((rc = check_step(kv, j0 + count - 1)) != TEMPO_OK) return rc;
  if (kv->ring_blocks && (int64_t)count > (int64_t)kv->ring_blocks * kv->block_size) return TEMPO_ERR_RANGE;
  const StoreParams p = store_params(kv, batch, 0, nullptr);
  const hipError_t e = launch_gather(p, k_out, v_out, kv->head_dim, kv->dtype, j0, count,
                                     static_cast<hipStream_t>(stream));
  return launch_status(e, "kv_gather");
}

int tempo_attn_decode_causal(const tempo_kv* kv, const void* q, void* out, int32_t batch,
                             int32_t num_q_heads, int32_t t, const int32_t* t_per_seq,
                             float scale, void* workspace, size_t workspace_bytes, void* stream) {
  return decode(kv, q, nullptr, nullptr, out, batch, num_q_heads, t, t_per_seq, 0, scale, workspace,
                workspace_bytes, stream);
}

int tempo_attn_decode_window(const tempo_kv* kv, const void* q, void* out, int32_t batch,
                             int32_t num_q_heads, int32_t t, const int32_t* t_per_seq,
                             int32_t window, float scale, void* workspace,
                             size_t workspace_bytes, void* stream) {
  if (window < 1) return TEMPO_ERR_RANGE;
  return decode(kv, q, nullptr, nullptr, out, batch, num_q_heads, t, t_per_seq, window, scale, workspace,
                workspace_bytes, stream);
}

int tempo_decode_step_causal(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new,
                             void* out, int32_t batch, int32_t num_q_heads, int32_t t,
                             const int32_t* t_per_seq, float scale, void* workspace,
                             size_t workspace_bytes, void* stream) {
  if (!k_new || !v_new) return TEMPO_ERR_NULL;
  return decode(kv, q, k_new, v_new, out, batch, num_q_heads, t, t_per_seq, 0, scale, workspace,
                workspace_bytes, stream);
}

int tempo_decode_step_window(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new,
                             void* out, int32_t batch, int32_t num_q_heads, int32_t t,
                             const int32_t* t_per_seq, int32_t window, float scale, void* workspace,
                             size_t workspace_bytes, void* stream) {
  if (!k_new || !v_new) return TEMPO_ERR_NULL;
  if (window < 1) return TEMPO_ERR_RANGE;
  return decode(kv, q, k_new, v_new, out, batch, num_q_heads, t, t_per_seq, window, scale, workspace,
                workspace_bytes, stream);
}

int tempo_decode_step_causal_noalloc(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new,
                                     void* out, int32_t batch, int32_t num_q_heads, int32_t t,
                                     const int32_t* t_per_seq, float scale, void* stream) {
  if (!k_new || !v_new) return TEMPO_ERR_NULL;
  int rc = check_layout(kv);
  if (rc != TEMPO_OK) return rc;
  if (!q || !out) return TEMPO_ERR_NULL;
  if ((rc = check_heads(kv, batch, num_q_heads)) != TEMPO_OK) return rc;
  if (t < 0 || t > INT32_MAX - 64) return TEMPO_ERR_RANGE;
  // the partials of this call's own plan must fit the static array
  const int64_t rows = (int64_t)batch * num_q_heads;
  int64_t max_splits = kMaxSplits;
  tempo_plan plan;
  make_block_plan(kv, batch, num_q_heads, t, 0, t_per_seq != nullptr, 1, &plan, max_splits);
  // (fp32, and the kernels for bf16 groups of more than 16 heads, want more splits than fit there
  // for many heads and long ranges: then the best plan that fits)
  if (plan_bytes(kv, rows, plan.num_splits) > kScratchBytes && (kv->dtype == TEMPO_F32 || num_q_heads / kv->num_kv_heads > kNarrowColumns)) {
    while (max_splits > 1 && plan_bytes(kv, rows, (int32_t)max_splits) > kScratchBytes) --max_splits;
    make_block_plan(kv, batch, num_q_heads, t, 0, t_per_seq != nullptr, 1, &plan, max_splits);
  }
  const size_t need = plan_bytes(kv, rows, plan.num_splits);
  if (need > kScratchBytes) {
    fprintf(stderr, "libtempo: tempo_decode_step_causal_noalloc: this step needs %zu bytes of split partials, "
                    "the static array holds %zu; use tempo_decode_step_causal with a workspace\n", need, kScratchBytes);
    return TEMPO_ERR_WORKSPACE;
  }
  void* ws = nullptr;
  if ((rc = scratch_on_current_device(&ws)) != TEMPO_OK) return rc;
  return decode(kv, q, k_new, v_new, out, batch, num_q_heads, t, t_per_seq, 0, scale, ws, kScratchBytes, stream, 1,
                nullptr, 0, nullptr, max_splits);
}

// The work list of a ragged step is tied to the plan the step will use: both come from
// make_block_plan with the same arguments.
static int worklist_plan(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t_max, int32_t window, tempo_plan* plan) {
  int rc = check_layout(kv);
  if (rc != TEMPO_OK) return rc;
  if ((rc = check_heads(kv, batch, Hq)) != TEMPO_OK) return rc;
  if (t_max < 0 || t_max > INT32_MAX - 64 || window < 0) return TEMPO_ERR_RANGE;
  // the list is read by the single-step bf16 kernel only
  if (kv->dtype != TEMPO_BF16) return TEMPO_ERR_DTYPE;
  if (Hq / kv->num_kv_heads > kNarrowColumns) return TEMPO_ERR_SHAPE;
  make_block_plan(kv, batch, Hq, t_max, window, true, 1, plan);
  if ((int64_t)batch * plan->num_splits > 65535) return TEMPO_ERR_SHAPE;  // one grid row per possible item
  return TEMPO_OK;
}

size_t tempo_attn_worklist_bytes(const tempo_kv* kv, int32_t batch, int32_t num_q_heads, int32_t t_max,
                                 int32_t window) {
  tempo_plan plan;
  if (worklist_plan(kv, batch, num_q_heads, t_max, window, &plan) != TEMPO_OK) return 0;
  return align_up(sizeof(int32_t) * (1 + (size_t)batch * plan.num_splits), 256);
}

int tempo_attn_worklist_build(const tempo_kv* kv, int32_t batch, int32_t num_q_heads, int32_t t_max,
                              const int32_t* t_per_seq, int32_t window, void* worklist, size_t worklist_bytes,
                              void* stream) {
  tempo_plan plan;
  const int rc = worklist_plan(kv, batch, num_q_heads, t_max, window, &plan);
  if (rc != TEMPO_OK) return rc;
  if (!t_per_seq || !worklist) return TEMPO_ERR_NULL;
  if ((reinterpret_cast<uintptr_t>(worklist) & 3u) != 0) return TEMPO_ERR_WORKSPACE;
  if (worklist_bytes < sizeof(int32_t) * (1 + (size_t)batch * plan.num_splits)) return TEMPO_ERR_WORKSPACE;
  const hipError_t e = launch_worklist_build(t_per_seq, batch, t_max, window, ilog2_exact(plan.tokens_per_split),
                                             plan.num_splits, static_cast<int32_t*>(worklist),
                                             static_cast<hipStream_t>(stream));
  return launch_status(e, "worklist_build");
}

int tempo_decode_step_ragged(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new, void* out,
                             int32_t batch, int32_t num_q_heads, int32_t t_max, const int32_t* t_per_seq,
                             int32_t window, float scale, const void* worklist, void* workspace,
                             size_t workspace_bytes, void* stream) {
  if (!t_per_seq || !worklist) return TEMPO_ERR_NULL;
  if ((k_new == nullptr) != (v_new == nullptr)) return TEMPO_ERR_NULL;
  tempo_plan plan;
  const int rc = worklist_plan(kv, batch, num_q_heads, t_max, window, &plan);
  if (rc != TEMPO_OK) return rc;
  return decode(kv, q, k_new, v_new, out, batch, num_q_heads, t_max, t_per_seq, window, scale, workspace,
                workspace_bytes, stream, 1, nullptr, 0, static_cast<const int32_t*>(worklist));
}

int tempo_attn_decode_padded_causal(const tempo_kv* kv, const void* q, void* out, int32_t batch,
                                    int32_t num_q_heads, int32_t t, const int32_t* t_per_seq,
                                    int32_t t_pad, float scale, void* workspace, size_t workspace_bytes,
                                    void* stream) {
  if (kv && kv->dtype == TEMPO_F32) return TEMPO_ERR_DTYPE;  // the baseline exists for the bf16 kernel only
  // ... and in the single-step kernel only: the kernels that serve larger query
  // groups walk the step's own range and know no padding bound
  if (kv && kv->num_kv_heads > 0 && num_q_heads / kv->num_kv_heads > kNarrowColumns) return TEMPO_ERR_SHAPE;
  if (t_pad < t) return TEMPO_ERR_RANGE;
  return decode(kv, q, nullptr, nullptr, out, batch, num_q_heads, t, t_per_seq, 0, scale, workspace,
                workspace_bytes, stream, 1, nullptr, t_pad);
}

int tempo_rope_rotate(const tempo_rope* rope, const void* x, void* y, int32_t dtype, int32_t batch,
                      int32_t heads, int32_t t, const int32_t* t_per_seq, void* stream) {
  if (!rope || !x || !y) return TEMPO_ERR_NULL;
  if (dtype != TEMPO_BF16 && dtype != TEMPO_F32) return TEMPO_ERR_DTYPE;
  if (rope->head_dim < 2 || rope->head_dim % 2 != 0 || rope->head_dim > 65536) return TEMPO_ERR_SHAPE;
  if (batch < 1 || heads < 1 || (int64_t)batch * heads * rope->head_dim > INT32_MAX) return TEMPO_ERR_SHAPE;
  const int rc = check_rope(rope, rope->head_dim, t);
  if (rc != TEMPO_OK) return rc;
  const hipError_t e = launch_rope_rotate(rope->cos, rope->sin, x, y, dtype, batch, heads, rope->head_dim, t,
                                          t_per_seq, static_cast<hipStream_t>(stream));
  return launch_status(e, "rope_rotate");
}

int tempo_rope_kv_append(const tempo_kv* kv, const tempo_rope* rope, const void* k_raw, const void* v_new,
                         int32_t batch, int32_t t, const int32_t* t_per_seq, void* stream) {
  int rc = check_store(kv);
  if (rc != TEMPO_OK) return rc;
  if (!k_raw || !v_new) return TEMPO_ERR_NULL;
  if (batch < 1 || batch > 65535) return TEMPO_ERR_SHAPE;
  if ((rc = check_step(kv, t)) != TEMPO_OK) return rc;
  if ((rc = check_rope(rope, kv->head_dim, t)) != TEMPO_OK) return rc;
  if ((int64_t)batch * kv->num_kv_heads * kv->head_dim > INT32_MAX) return TEMPO_ERR_SHAPE;
  const StoreParams p = store_params(kv, batch, t, t_per_seq);
  const hipError_t e = launch_rope_append(p, rope->cos, rope->sin, k_raw, v_new, kv->head_dim, kv->dtype,
                                          static_cast<hipStream_t>(stream));
  return launch_status(e, "kv_rope_append");
}

int tempo_rope_decode_step_causal(const tempo_kv* kv, const tempo_rope* rope, const void* q_raw,
                                  const void* k_raw, const void* v_new, void* out, int32_t batch,
                                  int32_t num_q_heads, int32_t t, const int32_t* t_per_seq, float scale,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  if (!rope || !k_raw || !v_new) return TEMPO_ERR_NULL;
  return decode(kv, q_raw, k_raw, v_new, out, batch, num_q_heads, t, t_per_seq, 0, scale, workspace,
                workspace_bytes, stream, 1, rope);
}

int tempo_rope_decode_step_window(const tempo_kv* kv, const tempo_rope* rope, const void* q_raw,
                                  const void* k_raw, const void* v_new, void* out, int32_t batch,
                                  int32_t num_q_heads, int32_t t, const int32_t* t_per_seq,
                                  int32_t window, float scale, void* workspace, size_t workspace_bytes,
                                  void* stream) {
  if (!rope || !k_raw || !v_new) return TEMPO_ERR_NULL;
  if (window < 1) return TEMPO_ERR_RANGE;
  return decode(kv, q_raw, k_raw, v_new, out, batch, num_q_heads, t, t_per_seq, window, scale, workspace,
                workspace_bytes, stream, 1, rope);
}

// Do a prompt's blocks of 128 columns alone give every compute unit one?
bool prompt_fills_part(const tempo_kv* kv, int32_t batch, int32_t G, int32_t count) {
  return (int64_t)prompt_blocks(count, G, kMaxColumns) * kv->num_kv_heads * batch >= kComputeUnits;
}

// Does a bf16 prompt go to the block kernel's form for prompts over short ranges?  At D = 128, more columns
// than 64, and at most 128 keys for the longest block of 128 columns (us, block kernel / prompt kernel, 24/8
// heads: 16 sequences of 64 steps 12.2 / 13.5, 128 steps 22.8 / 24.0, 200 steps 35.3 / 35.9, 300 steps behind
// a history with window 64 41.3 / 45.1, 1 sequence of 42 steps 11.5 / 12.2; windows only if the blocks fill the
// part: 1 sequence of 42 steps behind a history 14.3 / 13.3).  At D = 64 the prompt kernel is
// the faster one throughout (8 sequences, 32/8 heads, 128 steps 12.7 / 11.9).
bool short_prompt(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t, int32_t count, int32_t window) {
  const int32_t G = Hq / kv->num_kv_heads, QB = kMaxColumns / G;
  const int64_t all = (int64_t)t + count, most = (int64_t)window + QB - 1;
  if (kv->head_dim != 128 || (int64_t)count * G <= 64) return false;
  return all <= 128 || (window > 0 && most <= 128 && prompt_fills_part(kv, batch, G, count));
}

// Is a prompt answered block by block (blocks of 128 columns, each written, attended with split key ranges and
// combined) rather than in one launch?  The one launch cuts key ranges into at most 8 splits and its kernels
// are made for many columns; a block's attention spreads a long range over the whole part.
//   fp32: one block does, always (1 sequence, 24/8 heads, 1 step behind 2000 keys 12.6 us, in one launch 37;
//   behind 30000 49, 128).  More do not (2 blocks behind 2000 keys 62, 51).
//   bf16, a range of few groups, which no kernel splits: one launch where the merge of a block's wavefronts, by column
//   or tile of 32 columns, takes longer than the prompt kernel's beginning (us, by blocks / in one launch, D = 64, 60 columns,
//   16 keys 9.3 / 6.9, 143 keys 9.2 / 8.1; D = 128, 15 columns, 8 keys 9.9 / 7.0, 10 columns 8.0 / 7.1, 6 columns 7.0 / 7.2;
//   30 columns, 22 keys 8.1 / 7.2; queries to be turned to their position hide it below 25 columns, 7.9 / 8.4).
//   bf16, at most 16 columns, which the single-step kernel takes: by blocks else (24/8 heads, 1 step, 1 sequence behind
//   8000 keys 14, 27; 16 sequences behind 300 keys 10, 12), but for one or two (sequence, head) pairs with a
//   few columns behind a short range, whose many splits cost more to combine (1 sequence, 8/1 heads, 2 steps
//   behind 1000 keys 14.0, 11.1).
//   bf16, more columns: by two estimates in us, fitted to 4754 measured prompts of 1 to 255 blocks of all pairs (on the mean
//   0.3% from the better of the two, 21% at most), unless their blocks fill the part.  A block takes a time of its own and a
//   share of its keys' stream from HBM, both by the kernel its columns go to; one launch 7.7 and the longer of a
//   workgroup's walk through an eighth of the keys and 1.63 times the stream (us, by blocks / in one launch: 2 sequences,
//   32/8 heads of 64, 5 steps behind 8000 keys 13.3 / 22.3, 24/8 heads of 128, 6 sequences, 15 steps behind 3600 29.4 / 34.7,
//   1 sequence, 16 steps behind 1650 16.5 / 15.4).
bool prompt_by_blocks(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t, int32_t count, int32_t window, bool rope) {
  const int32_t G = Hq / kv->num_kv_heads, block = kMaxColumns / G;
  if (kv->dtype != TEMPO_BF16) return count <= block;
  if (prompt_fills_part(kv, batch, G, count)) return false;
  const bool narrow = kv->head_dim == 64;
  const int64_t pairs = (int64_t)batch * kv->num_kv_heads, columns = (int64_t)count * G;
  const int64_t keys = window > 0 && window <= t ? (int64_t)window + count - 1 : (int64_t)t + count;
  if (columns <= kNarrowColumns) {
    if (narrow ? columns >= 12 && keys <= 32 : (columns > 8 && keys <= 32) || (columns > 13 && keys <= 64)) return false;
    tempo_plan plan;
    make_block_plan(kv, batch, Hq, t, window, false, count, &plan);
    return !(pairs < kManyPairs && plan.num_splits > 8 && columns >= 8 && count > 1 && keys <= 2200);
  }
  if (short_prompt(kv, batch, Hq, t, count, window)) return false;
  if (columns <= 32 && (narrow ? keys <= 32 : columns > 24 ? keys <= 64 : keys <= 32 && !rope)) return false;
  if (narrow && columns > 32 && columns <= 64 && keys <= 256) return false;
  const double stream = (double)pairs * keys * kv->head_dim * 4 / (kSustainedBytesPerNs * 1000.0);
  const int64_t blocks = (count + block - 1) / block, widest = columns < kMaxColumns ? columns : kMaxColumns;
  const int size = widest <= 32 ? 0 : widest <= 64 ? 1 : 2;
  constexpr double kOwn[2][3] = {{5.0, 13.0, 14.1}, {7.0, 9.6, 12.5}}, kShare[2][3] = {{0.73, 0.51, 2.23}, {1.12, 0.68, 0.72}};
  const double by_blocks = (double)blocks * (kOwn[narrow][size] + kShare[narrow][size] * stream);
  const int64_t workgroups = 8 * pairs * blocks, rounds = (workgroups + 2 * kComputeUnits - 1) / (2 * kComputeUnits);
  const double walk = (workgroups <= kComputeUnits ? 0.74 : 0.85) * (narrow ? 0.35 : 1.0) * (columns > 64 ? 1.36 : 1.0) * rounds * (double)keys / 256.0;
  const double one_launch = 7.7 + (walk > 1.63 * stream ? walk : 1.63 * stream) + (narrow && size == 1 ? 0.06 * count : 0.0);
  return by_blocks < one_launch;
}

constexpr int kWaveColumns = 32;  // of the prompt kernel

// How the prompt kernel takes a prompt: wavefronts of 32 columns per workgroup, and splits of
// a block's key range (tps_log2 = kWholeRange, splits = 1: none).
struct PromptPlan {
  int waves, tps_log2, splits;
};

// A time model of the launch, in nanoseconds, with constants measured on MI355X at D = 128 (at D = 64
// an iteration takes 0.68 of it: 128 groups per workgroup 48 us against 68 us).  Two workgroups of 2 or
// 4 wavefronts share a compute unit (at D = 128 by their 64 KiB of LDS each); a workgroup spends about
// 5 us before its first and after its last group, and an iteration over a 32-slot group takes 0.55 us
// with one wavefront on a SIMD, 0.78 us with two, and 0.64 us with one where two workgroups of 2 copy
// each their own keys/values.  So 4 wavefronts win once they fill the part; 2, and a key range cut into
// splits (a combine launch, and partials of (D + 2) * 4 bytes per column and split), when the query
// columns alone do not (100 steps behind 1900 keys, one sequence: no splits 52 us, 8 splits 25 us).
// The combine is priced at 1.5 us beside the rest of the model: over 1496 measured prompts that fits
// best (0.4% off the fastest of 1.5, 2.5, 3.5 and 5 us on the mean, 9% at most; 5 us 3.1% and 51%: 4
// sequences of 21 steps, 24/8 heads, window 512: 19.6 us unsplit, 14.8; 1 and 2 us like 1.5).
// 8 wavefronts in one workgroup read each key/value half as often, but nothing covers the
// workgroup's beginning and end: the better shape only for long ranges at D = 128 (us with 4 / 8:
// 16 x 200 steps 32.7 / 35.7, 16 x 1000 185 / 200, 4 x 4000 449 / 437; D = 64, 8 x 1500 125 / 147).
PromptPlan plan_prompt(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t, int32_t count, int32_t window,
                       size_t workspace_bytes, bool rows) {
  const int G = Hq / kv->num_kv_heads;
  const double scale = kv->head_dim == 128 ? 1.0 : 0.68;
  PromptPlan best = {4, kWholeRange, 1};
  double best_ns = -1.0;
  const bool may_split = !prompt_fills_part(kv, batch, G, count);
  const int64_t pairs = (int64_t)batch * kv->num_kv_heads;
  const int64_t mean_keys = window > 0 && window < t + count / 2 ? window : t + count / 2;
  if (kv->head_dim == 128 && mean_keys >= 1800 && prompt_blocks(count, G, 8 * kWaveColumns) * pairs >= 4 * kComputeUnits) return {8, kWholeRange, 1};
  for (int waves = 4; waves >= 2; waves /= 2) {
    if (G > waves * kWaveColumns) break;
    const int32_t QB = prompt_block_span(G, waves * kWaveColumns);
    const int64_t blocks = prompt_blocks(count, G, waves * kWaveColumns);
    // keys of the longest block; from the store in whole steps, as the constants were fitted (with a step more of 3 heads a
    // window of 107 crossed into a fifth group for 2 wavefronts and got 4: 125 steps, 2 sequences, 15.3 -> 17.5 us; from
    // rows that step decides the other way: 122 steps, 3 sequences, window 21 8.6 by 2 wavefronts, 10.9 by 4)
    const int64_t seen = (int64_t)window + (rows ? QB : waves * kWaveColumns / G);
    const int64_t keys = window > 0 && seen < (int64_t)t + count ? seen : (int64_t)t + count;
    const int resident = 2;  // (at D = 64 more would fit; the constants were fitted with 2 there too)
    for (int k = kWholeRange; k >= 7; k = k == kWholeRange ? 13 : k - 1) {
      const int splits = k == kWholeRange ? 1 : splits_bound(t + count - 1, union_window(window, QB), k);
      if (k != kWholeRange && !may_split) break;
      if (k != kWholeRange && splits == 1) continue;
      if (splits > 8) break;  // the combine reads up to 8 splits in one batch
      const int64_t answers = (int64_t)batch * count * Hq;
      if (k != kWholeRange && (answers * splits * kv->head_dim > INT32_MAX || plan_bytes(kv, answers, splits) > workspace_bytes)) break;
      const int64_t workgroups = blocks * pairs * splits;
      const int64_t rounds = (workgroups + resident * kComputeUnits - 1) / (resident * kComputeUnits);
      const bool shared = workgroups > kComputeUnits;  // two workgroups on some compute unit
      const int64_t span = k == kWholeRange || keys < ((int64_t)1 << k) ? keys : (int64_t)1 << k;
      // a causal prompt's blocks are half the longest on average: beyond the first round that counts
      const double mean = window == 0 && rounds > 1 ? (double)(t + count / 2) / (t + count) : 1.0;
      double ns = (double)rounds * (5000.0 + mean * (double)((span + 31) / 32) * (!shared ? 550.0 : waves == 4 ? 780.0 : 640.0) * scale);
      if (splits > 1) ns += 1500.0 + 2.0 * (double)answers * splits * kv->head_dim * 4 / 4000.0;
      if (best_ns < 0.0 || ns < 0.97 * best_ns) {  // the wider workgroup and the fewer splits unless clearly slower
        best_ns = ns;
        best = {waves, k, splits};
      }
    }
  }
  return best;
}

// Does one launch answer all steps of a prompt (of a ring store's chunk)?  It does unless the call
// is too large for the index range of its launches.
bool prompt_in_one_launch(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t count) {
  const int32_t heads = kv->dtype == TEMPO_BF16 ? kv->num_kv_heads : Hq;
  return (int64_t)batch * count * heads * kv->head_dim <= INT32_MAX;
}

// fp32: tiles of 16 (step, head) columns, the keys of a tile spread over 8 wavefronts.  A tile's
// group of 16 keys costs about 2 us at D = 128; the key range is split (and combined, 5 us) only
// if the tiles leave most of the part idle and a wavefront would walk more than 6 groups (1 sequence,
// 16/1 heads, 16 steps behind 1000 keys: one split 33.6 us, 4 splits 22; 64 steps of 24/8 heads behind
// 500: 25.0, 3 splits 26.4).
PromptPlan plan_prompt_f32(const tempo_kv* kv, int32_t batch, int32_t Hq, int32_t t, int32_t count, int32_t window,
                           size_t workspace_bytes) {
  const int64_t columns = (int64_t)count * (Hq / kv->num_kv_heads);
  const int64_t tiles = (columns + 15) / 16 * kv->num_kv_heads * batch, rows = (int64_t)batch * count * Hq;
  PromptPlan plan = {8, kWholeRange, 1};
  const int64_t steps = 16 / (columns / count) + 1;  // of a tile
  const int64_t keys = window > 0 && window + steps < (int64_t)t + count ? window + steps : (int64_t)t + count;
  if (keys <= 256) plan.waves = 4;
  for (int k = 8; k <= 20 && keys >= 768 && tiles < kComputeUnits / 2; ++k) {
    const int splits = splits_bound(t + count - 1, union_window(window, count), k);
    if (splits == 1) break;
    if (splits > 8 || tiles * splits > 2 * kComputeUnits || plan_bytes(kv, rows, splits) > workspace_bytes) continue;
    plan = {8, k, splits};
    break;
  }
  return plan;
}

// A ring store holds a limited range: the most steps from t on that one chunk may write and
// answer (every tile of the chunk's ranges resident), ending on a 32-slot group if that leaves
// at least `block` steps, which are known to fit.
int32_t ring_chunk(const tempo_kv* kv, int32_t t, int32_t left, int32_t window, int32_t block) {
  int32_t C = left;
  if (kv->ring_blocks) {
    const int64_t slots = (int64_t)kv->ring_blocks * kv->block_size;
    // check_ring_covers: ceil((window + C - 2) / Z) + 1 <= ring_blocks, or the whole history fits
    const int64_t most = t + (int64_t)left <= slots ? left : slots - kv->block_size - window + 2;
    C = most < left ? (int32_t)(most < 1 ? 1 : most) : left;
    if (C < block) C = left < block ? left : block;
    const int32_t aligned = ((t + C) & ~31) - t;
    if (C < left && aligned >= block) C = aligned;
  }
  return C;
}

// A prompt from step 0 on whose keys/values the attention kernel reads from the caller's rows; it writes the
// steps from keep_first on to the store itself.
struct PromptRows {
  const void *k, *v;
  int32_t keep_first;
};

// Is `out` clear of the rows?
bool rows_apart(const tempo_kv* kv, const void* k_new, const void* v_new, const void* out, int32_t batch, int32_t Hq,
                int32_t count) {
  const uintptr_t k = reinterpret_cast<uintptr_t>(k_new), v = reinterpret_cast<uintptr_t>(v_new);
  const uintptr_t o = reinterpret_cast<uintptr_t>(out);
  const uintptr_t step_bytes = (uintptr_t)batch * count * kv->head_dim * (kv->dtype == TEMPO_BF16 ? 2 : 4);
  const uintptr_t out_bytes = step_bytes * Hq, row_bytes = step_bytes * kv->num_kv_heads;
  return (o + out_bytes <= k || k + row_bytes <= o) && (o + out_bytes <= v || v + row_bytes <= o);
}

// Do answers of steps before the call's step c lie over rows (its k_new or v_new) of steps from c on?
bool answers_over_later_rows(const tempo_kv* kv, const void* rows, const void* out, int32_t batch, int32_t Hq,
                             int32_t count, int32_t c) {
  const int64_t step_bytes = (int64_t)kv->head_dim * (kv->dtype == TEMPO_BF16 ? 2 : 4);
  const int64_t row = step_bytes * kv->num_kv_heads, answer = step_bytes * Hq;
  const int64_t apart = (int64_t)(reinterpret_cast<uintptr_t>(out) - reinterpret_cast<uintptr_t>(rows));
  for (int32_t b = 0; b < batch; ++b) {
    const int64_t from = apart + (int64_t)b * count * answer, to = from + c * answer;  // sequence b's answers, from the first row
    const int64_t other = from > 0 ? from / (count * row) : 0;                // the first sequence whose rows end behind `from`
    if (other < batch && (other * count + c) * row < to) return true;
  }
  return false;
}

// May it?  Not where `out` lies over the rows (which a write launch of its own has read before), nor where
// 16-byte pieces of them are not aligned.
bool rows_readable(const tempo_kv* kv, const void* k_new, const void* v_new, const void* out, int32_t batch, int32_t Hq,
                   int32_t count) {
  return ((reinterpret_cast<uintptr_t>(k_new) | reinterpret_cast<uintptr_t>(v_new)) & 15u) == 0 &&
         rows_apart(kv, k_new, v_new, out, batch, Hq, count);
}

// And is it the faster way?  It saves a launch and a pass over memory, and costs a little per group and workgroup, which
// shows where the longest walk or the last round decides.  (us, write and attend / from rows)
//   bf16, causal: up to about 1.15e11 flops (24/8 heads of 128: 16 x 160 steps 23.6 / 16.8, 16 x 1300 (1.7e11) 243 / 247;
//   16/16 heads of 64: 16 x 320 25.0 / 17.1, 16 x 1900 (1.2e11) 207 / 214).  Less at D = 128: groups of 1 head, with more
//   blocks than units, up to 1320 steps, or 1700 with blocks for two rounds (8 heads: 3 sequences of 1591 steps 54.3 / 59.3,
//   2 of 2339 71.7 / 81.4; but 2 of 1568, 208 blocks, 43.2 / 39.4, 6 of 1459 71.0 / 65.0); of 2 or 3 heads up to 2800 steps (1
//   sequence of 2888 steps 83.0 / 90.0, 2175 65.6 / 61.8), or 1700 with more than 1024 blocks (5% on the mean).
//   Windows: all, but for stores that hold the prompt and windows so short that the block kernel takes the written prompt, with
//   blocks for many rounds (8 heads a group, 52 keys, 2400 blocks 64.6 / 69.1, 780 28.4 / 27.9; 3 heads, 36 keys, 3072 blocks
//   98.5 / 101.2, 1800 64.8 / 63.6).
//   fp32: at D = 128 up to about 4.5e9 flops (8/8 heads: 4 x 128 17.5 / 10.4, 1 x 1534 (4.8e9) 124.5 / 124.4); at D = 64 but
//   for long walks with tiles for a little more than one round of the units, of few pairs (2 pairs, 4 heads
//   a group: 948 steps, 474 tiles 25.0 / 30.7, 414 steps 14.2 / 10.1, 1254 steps, 628 tiles 40.7 / 36.2; 8 pairs, 1 head: 674
//   steps, 344 tiles 24.4 / 28.5, 854 steps, 432 tiles 32.2 / 31.1).
constexpr double kRowsMostFlops = 1.15e11, kRowsMostFlopsF32 = 4.5e9;

bool prompt_from_rows(const tempo_kv* kv, const void* k_new, const void* v_new, const void* out, int32_t batch, int32_t Hq,
                      int32_t t, int32_t count, int32_t window) {
  if (t != 0 || !prompt_in_one_launch(kv, batch, Hq, count)) return false;
  const int32_t G = Hq / kv->num_kv_heads;
  const int64_t pairs = (int64_t)batch * kv->num_kv_heads;
  const double mean_keys = window > 0 && window < count / 2 ? window : 0.5 * count;
  const double flops = 4.0 * batch * Hq * kv->head_dim * count * mean_keys;
  if (kv->dtype == TEMPO_BF16) {
    const int64_t blocks = (int64_t)prompt_blocks(count, G, kMaxColumns) * pairs;
    if (window == 0) {
      if (flops > kRowsMostFlops) return false;
      if (kv->head_dim == 128 && (G == 1 ? blocks > 240 && count > (blocks <= 2 * kComputeUnits ? 1320 : 1700)
                                         : G < 4 && (count > 2800 || (count > 1700 && blocks > 1024))))
        return false;
    } else if ((kv->ring_blocks == 0 || count <= (int64_t)kv->ring_blocks * kv->block_size) && window < count &&
               short_prompt(kv, batch, Hq, t, count, window) && blocks >= (G < 8 ? 2048 : 1400)) {
      return false;
    }
  } else if (kv->head_dim == 128) {
    if (flops > kRowsMostFlopsF32) return false;
  } else {
    const int64_t tiles = ((int64_t)count * G + 15) / 16 * pairs;
    if (count >= 530 && tiles > kComputeUnits && tiles <= (pairs < 8 ? 2 * kComputeUnits : pairs == 8 ? 352 : 0)) return false;
  }
  return rows_readable(kv, k_new, v_new, out, batch, Hq, count);
}

// One launch (and the combine, if it splits key ranges) for `count` steps from t on, already in
// the store.  q, out: the caller's, `io_steps` steps per sequence.
int attend_prompt(const tempo_kv* kv, const void* q, void* out, int32_t batch, int32_t Hq, int32_t t, int32_t count,
                  int32_t io_steps, const int32_t* count_per_seq, int32_t window, float scale, void* workspace,
                  size_t workspace_bytes, hipStream_t s, const tempo_rope* rope, const StageParams* staged = nullptr,
                  const PromptRows* rows = nullptr) {
  const bool bf16 = kv->dtype == TEMPO_BF16;
  // (a sequence with fewer steps than the others has blocks, and splits, the combine does not know)
  // (and staged keys/values lie where the partials of split ranges would)
  const bool is_short = bf16 && !staged && !rows && short_prompt(kv, batch, Hq, t, count, window);
  const PromptPlan plan = is_short ? PromptPlan{8, kWholeRange, 1}
                          : bf16   ? plan_prompt(kv, batch, Hq, t, count, window, count_per_seq || staged ? 0 : workspace_bytes, rows != nullptr)
                                   : plan_prompt_f32(kv, batch, Hq, t, count, window, workspace_bytes);
  const tempo_plan cut = {32, plan.splits, plan.waves};  // (its split length is set below)
  PromptParams p;
  static_cast<AttnParams&>(p) = attn_params(kv, q, out, Hq, t, nullptr, window, scale, &cut, workspace, batch, count);
  p.io_steps = io_steps;
  p.tps_log2 = plan.tps_log2;
  p.direct = plan.splits == 1;
  p.block_columns = plan.waves * kWaveColumns;
  p.k_stage = p.v_stage = nullptr;
  p.stage_first = p.stage_groups = p.keep_first = 0;
  if (rows) {
    p.k_new = rows->k;
    p.v_new = rows->v;
    p.keep_first = rows->keep_first;
  }
  p.count_per_seq = count_per_seq;
  if (rope) {
    p.rope_cos = rope->cos;
    p.rope_sin = rope->sin;
  }
  if (staged) {
    p.k_stage = staged->k_stage;
    p.v_stage = staged->v_stage;
    p.stage_first = t >> 5;
    p.stage_groups = staged->stage_groups;
  }
  const hipError_t e = is_short ? launch_short_prompt_bf16(p, batch, kv->head_dim, s)
                       : bf16   ? launch_prefill_bf16(p, batch, kv->head_dim, plan.waves, plan.splits, s)
                                : launch_partial_f32(p, batch, kv->head_dim, plan.splits, plan.waves, s);
  const int rc = launch_status(e, "attn_prefill");
  if (rc != TEMPO_OK || plan.splits == 1) return rc;
  return launch_status(bf16 ? launch_prompt_combine(p, batch, kv->head_dim, s)
                            : launch_combine(p, batch, kv->head_dim, kv->dtype, s), "attn_prefill_combine");
}

// A ring store holds little more than the window, so a prompt written into it has to be answered
// in chunks, each too small to fill the part (2048 steps of 4 sequences, window 512, 4 blocks of
// 256: 8 chunks, 253 us).  Instead the prompt's key/value groups are laid out in the workspace
// first, one launch answers all steps from there (and from the ring, for the history), and the
// steps the ring holds in the end are written last.  How many steps from t on the workspace has
// room for, if any; less than `left` ends on a group.
int32_t staged_steps(const tempo_kv* kv, int32_t batch, int32_t t, int32_t left, size_t workspace_bytes) {
  if (kv->dtype != TEMPO_BF16 || kv->ring_blocks == 0) return 0;
  const int64_t group_bytes = (int64_t)batch * kv->num_kv_heads * 2 * 32 * kv->head_dim * 2;  // keys and values of all sequences
  const int64_t room = (int64_t)workspace_bytes / group_bytes, first = t >> 5;
  const int64_t end = (first + room) << 5;                       // first step without room
  return end >= (int64_t)t + left ? left : (end > t ? (int32_t)(end - t) : 0);
}

// Steps c0 .. c0+C-1 of the call, staged.
int prefill_staged(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new, void* out, int32_t batch,
                   int32_t Hq, int32_t t, int32_t count, int32_t c0, int32_t C, int32_t window, float scale,
                   void* workspace, hipStream_t s) {
  const char* k = static_cast<const char*>(k_new);
  const char* v = static_cast<const char*>(v_new);
  const size_t row = (size_t)kv->num_kv_heads * kv->head_dim * 2, q_at = (size_t)c0 * Hq * kv->head_dim * 2;
  StageParams sp;
  static_cast<StoreParams&>(sp) = store_params(kv, batch, t + c0, nullptr, C);
  sp.src_steps = count;
  sp.stage_groups = ((t + c0 + C - 1) >> 5) - ((t + c0) >> 5) + 1;
  sp.k_stage = workspace;
  sp.v_stage = static_cast<char*>(workspace) + (size_t)batch * kv->num_kv_heads * sp.stage_groups * 64 * kv->head_dim;
  int rc = launch_status(launch_stage(sp, k + c0 * row, v + c0 * row, kv->head_dim, s), "kv_stage");
  if (rc != TEMPO_OK) return rc;
  rc = attend_prompt(kv, static_cast<const char*>(q) + q_at, static_cast<char*>(out) + q_at, batch, Hq, t + c0, C, count,
                     nullptr, window, scale, workspace, 0, s, nullptr, &sp);
  if (rc != TEMPO_OK) return rc;
  const int64_t slots = (int64_t)kv->ring_blocks * kv->block_size;
  const int32_t kept = C < slots ? C : (int32_t)slots, from = c0 + C - kept;
  StoreParams last = store_params(kv, batch, t + from, nullptr, kept);
  last.src_steps = count;
  return launch_status(launch_append(last, k + from * row, v + from * row, kv->head_dim, kv->dtype, s), "kv_append_block");
}

// `count` steps from t on, in blocks of 128 columns: write (fp32, one block from step 0 on: the attention launch
// does), attend, combine.
int prefill_by_blocks(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new, void* out, int32_t batch,
                      int32_t Hq, int32_t t, int32_t count, int32_t window, float scale, void* workspace, hipStream_t s,
                      const tempo_rope* rope = nullptr) {
  const size_t esz = kv->dtype == TEMPO_BF16 ? 2 : 4;
  const int32_t block = kMaxColumns / (Hq / kv->num_kv_heads);
  const bool rows = kv->dtype == TEMPO_F32 && t == 0 && count <= block && rows_readable(kv, k_new, v_new, out, batch, Hq, count);
  // `out` over the rows: a block's answers would stand where the next one's rows are read, so all are written first
  const bool write_first = !kv->ring_blocks && count > block && !rows_apart(kv, k_new, v_new, out, batch, Hq, count);
  const auto write = [&](int32_t c0, int32_t C) {
    const size_t at = (size_t)c0 * kv->num_kv_heads * kv->head_dim * esz;
    StoreParams sp = store_params(kv, batch, t + c0, nullptr, C);
    sp.src_steps = count;
    if (rope) {
      sp.rope_cos = rope->cos;
      sp.rope_sin = rope->sin;
    }
    return launch_status(launch_append(sp, static_cast<const char*>(k_new) + at, static_cast<const char*>(v_new) + at, kv->head_dim, kv->dtype, s),
                         "kv_append_block");
  };
  for (int32_t c0 = 0; write_first && c0 < count; c0 += block) {
    const int rc = write(c0, count - c0 < block ? count - c0 : block);
    if (rc != TEMPO_OK) return rc;
  }
  for (int32_t c0 = 0; c0 < count; c0 += block) {
    const int32_t C = count - c0 < block ? count - c0 : block;
    tempo_plan plan;
    make_block_plan(kv, batch, Hq, t + c0, window, false, C, &plan);
    const char* qc = static_cast<const char*>(q) + (size_t)c0 * Hq * kv->head_dim * esz;
    char* oc = static_cast<char*>(out) + (size_t)c0 * Hq * kv->head_dim * esz;
    int rc = rows || write_first ? TEMPO_OK : write(c0, C);
    if (rc != TEMPO_OK) return rc;
    rc = do_partial(kv, qc, rows ? k_new : nullptr, rows ? v_new : nullptr, oc, batch, Hq, t + c0, nullptr, window, scale, &plan, workspace, s, C, rope,
                    0, count);
    if (rc != TEMPO_OK) return rc;
    if (plan.num_splits > 1) {
      rc = do_combine(kv, oc, batch, Hq, t + c0, nullptr, window, &plan, workspace, s, C, 0, count);
      if (rc != TEMPO_OK) return rc;
    }
  }
  return TEMPO_OK;
}

// Prompt processing: `count` steps per sequence, written and answered in one launch each, or
// in blocks of as many steps as the column tiles hold.
static int prefill(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new, void* out, int32_t batch,
            int32_t Hq, int32_t t, int32_t count, const int32_t* count_per_seq, int32_t window, float scale,
            void* workspace, size_t workspace_bytes, void* stream, const tempo_rope* rope = nullptr) {
  int rc = check_store(kv);
  if (rc != TEMPO_OK) return rc;
  if (!q || !k_new || !v_new || !out) return TEMPO_ERR_NULL;
  if ((rc = check_heads(kv, batch, Hq)) != TEMPO_OK) return rc;
  if (count < 1 || count > (1 << 24)) return TEMPO_ERR_SHAPE;
  if (t < 0 || window < 0 || t > INT32_MAX - 64 - count) return TEMPO_ERR_RANGE;
  if ((rc = check_scale(scale)) != TEMPO_OK) return rc;
  if ((rc = check_step(kv, t + count - 1)) != TEMPO_OK) return rc;
  const int G = Hq / kv->num_kv_heads;
  const int32_t block = kMaxColumns / G;  // steps per block: all four column tiles
  if ((int64_t)batch * block * Hq * kv->head_dim > INT32_MAX) return TEMPO_ERR_SHAPE;
  const size_t esz = kv->dtype == TEMPO_BF16 ? 2 : 4;
  const bool ragged = false;  // every sequence starts at step t
  hipStream_t s = static_cast<hipStream_t>(stream);
  // validate every block before the first launch, so that an error leaves the store untouched
  size_t need = 0;  // of the workspace, for the partials of any block
  for (int32_t c0 = 0; c0 < count; c0 += block) {
    const int32_t C = count - c0 < block ? count - c0 : block;
    tempo_plan plan;
    make_block_plan(kv, batch, Hq, t + c0, window, ragged, C, &plan);
    if ((rc = check_attn(kv, batch, Hq, t + c0, window, ragged, &plan, workspace, workspace_bytes, C)) != TEMPO_OK)
      return rc;
    if (kv->ring_blocks && (int64_t)C > (int64_t)kv->ring_blocks * kv->block_size) return TEMPO_ERR_RANGE;
    const size_t partials = plan_bytes(kv, (int64_t)batch * C * Hq, plan.num_splits);
    need = partials > need ? partials : need;
  }

  const bool one_launch = prompt_in_one_launch(kv, batch, Hq, count);
  // per-sequence prompt lengths exist in the prompt kernel only; the rotary producer is refused where that could not take the prompt
  if ((count_per_seq || rope) && (kv->dtype != TEMPO_BF16 || kv->ring_blocks != 0 || !one_launch))
    return TEMPO_ERR_SHAPE;
  if (rope && (rc = check_rope(rope, kv->head_dim, t + count - 1)) != TEMPO_OK) return rc;
  // A ring store keeps little more than its window, so it can't be written ahead of the answers.  Where the prompt
  // takes several chunks and answers stand over rows that are still to be read (by a later chunk; if it is staged, by the
  // last write), the call reads a copy of the rows, at the workspace's end.
  bool may_stage = true;
  if (kv->ring_blocks && !rows_apart(kv, k_new, v_new, out, batch, Hq, count)) {
    bool chunks = false, over = false;
    for (int32_t c = 0;;) {
      c += one_launch ? ring_chunk(kv, t + c, count - c, window, block) : (count - c < block ? count - c : block);
      if (c >= count) break;
      chunks = true;
      over = over || answers_over_later_rows(kv, k_new, out, batch, Hq, count, c) ||
             answers_over_later_rows(kv, v_new, out, batch, Hq, count, c);
    }
    if (chunks && (over || kv->dtype == TEMPO_BF16)) {  // (fp32 is not staged)
      const size_t bytes = (size_t)batch * count * kv->num_kv_heads * kv->head_dim * esz;
      if (workspace_bytes >= 2 * bytes && ((workspace_bytes - 2 * bytes) & ~(size_t)255) >= need) {
        workspace_bytes = (workspace_bytes - 2 * bytes) & ~(size_t)255;
        char* const copy = static_cast<char*>(workspace) + workspace_bytes;
        const int workgroups = bytes < ((size_t)64 << 20) ? (int)((bytes + 16383) / 16384) : 4096;
        if ((rc = launch_status(launch_stream_copy(k_new, copy, bytes, workgroups, s), "rows_copy")) != TEMPO_OK) return rc;
        if ((rc = launch_status(launch_stream_copy(v_new, copy + bytes, bytes, workgroups, s), "rows_copy")) != TEMPO_OK) return rc;
        k_new = copy;
        v_new = copy + bytes;
      } else if (over) {
        return TEMPO_ERR_WORKSPACE;
      } else {
        may_stage = false;  // every chunk's answers stand clear of later rows
      }
    }
  }
  const bool one_f32_block = kv->dtype == TEMPO_F32 && count <= block;  // (goes by blocks, which know the way by rows too)
  if (!rope && !one_f32_block && prompt_from_rows(kv, k_new, v_new, out, batch, Hq, t, count, window)) {
    const int64_t slots = kv->ring_blocks ? (int64_t)kv->ring_blocks * kv->block_size : count;
    const PromptRows rows = {k_new, v_new, count > slots ? (int32_t)(count - slots) : 0};  // a ring keeps the last steps
    return attend_prompt(kv, q, out, batch, Hq, t, count, count, count_per_seq, window, scale, workspace, workspace_bytes, s,
                         nullptr, nullptr, &rows);
  }
  // (several blocks on a ring, answers over rows: the chunks looked at above, not the blocks)
  const bool blocks_stand = !kv->ring_blocks || count <= block || rows_apart(kv, k_new, v_new, out, batch, Hq, count);
  if (!count_per_seq && blocks_stand && prompt_by_blocks(kv, batch, Hq, t, count, window, rope != nullptr))
    return prefill_by_blocks(kv, q, k_new, v_new, out, batch, Hq, t, count, window, scale, workspace, s, rope);
  // Write the prompt, then answer it in one launch; on a ring store in chunks that it can hold.
  if (one_launch) {
    for (int32_t c0 = 0; c0 < count;) {
      const int32_t C = ring_chunk(kv, t + c0, count - c0, window, block);
      const int32_t S = may_stage && C < count - c0 ? staged_steps(kv, batch, t + c0, count - c0, workspace_bytes) : 0;
      if (S > C) {
        rc = prefill_staged(kv, q, k_new, v_new, out, batch, Hq, t, count, c0, S, window, scale, workspace, s);
        if (rc != TEMPO_OK) return rc;
        c0 += S;
        continue;
      }
      const size_t kv_at = (size_t)c0 * kv->num_kv_heads * kv->head_dim * esz, q_at = (size_t)c0 * Hq * kv->head_dim * esz;
      StoreParams sp = store_params(kv, batch, t + c0, nullptr, C);
      sp.src_steps = count;
      sp.count_per_seq = count_per_seq;
      if (rope) {
        sp.rope_cos = rope->cos;
        sp.rope_sin = rope->sin;
      }
      if ((rc = launch_status(launch_append(sp, static_cast<const char*>(k_new) + kv_at, static_cast<const char*>(v_new) + kv_at,
                                            kv->head_dim, kv->dtype, s), "kv_append_block")) != TEMPO_OK)
        return rc;
      if ((rc = attend_prompt(kv, static_cast<const char*>(q) + q_at, static_cast<char*>(out) + q_at, batch, Hq, t + c0, C,
                              count, count_per_seq, window, scale, workspace, workspace_bytes, s, rope)) != TEMPO_OK)
        return rc;
      c0 += C;
    }
    return TEMPO_OK;
  }

  // A call beyond the index range of one launch goes block by block too.
  return prefill_by_blocks(kv, q, k_new, v_new, out, batch, Hq, t, count, window, scale, workspace, s);
}

int tempo_prefill_causal(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new, void* out,
                         int32_t batch, int32_t num_q_heads, int32_t t, int32_t count,
                         const int32_t* count_per_seq, float scale, void* workspace, size_t workspace_bytes,
                         void* stream) {
  return prefill(kv, q, k_new, v_new, out, batch, num_q_heads, t, count, count_per_seq, 0, scale, workspace,
                 workspace_bytes, stream);
}

int tempo_prefill_window(const tempo_kv* kv, const void* q, const void* k_new, const void* v_new, void* out,
                         int32_t batch, int32_t num_q_heads, int32_t t, int32_t count,
                         const int32_t* count_per_seq, int32_t window, float scale, void* workspace,
                         size_t workspace_bytes, void* stream) {
  if (window < 1 || window > INT32_MAX - 128) return TEMPO_ERR_RANGE;
  return prefill(kv, q, k_new, v_new, out, batch, num_q_heads, t, count, count_per_seq, window, scale, workspace,
                 workspace_bytes, stream);
}

int tempo_rope_prefill_causal(const tempo_kv* kv, const tempo_rope* rope, const void* q_raw, const void* k_raw,
                              const void* v_new, void* out, int32_t batch, int32_t num_q_heads, int32_t t,
                              int32_t count, const int32_t* count_per_seq, float scale, void* workspace,
                              size_t workspace_bytes, void* stream) {
  if (!rope) return TEMPO_ERR_NULL;
  return prefill(kv, q_raw, k_raw, v_new, out, batch, num_q_heads, t, count, count_per_seq, 0, scale, workspace,
                 workspace_bytes, stream, rope);
}

int tempo_rope_prefill_window(const tempo_kv* kv, const tempo_rope* rope, const void* q_raw, const void* k_raw,
                              const void* v_new, void* out, int32_t batch, int32_t num_q_heads, int32_t t,
                              int32_t count, const int32_t* count_per_seq, int32_t window, float scale,
                              void* workspace, size_t workspace_bytes, void* stream) {
  if (!rope) return TEMPO_ERR_NULL;
  if (window < 1 || window > INT32_MAX - 128) return TEMPO_ERR_RANGE;
  return prefill(kv, q_raw, k_raw, v_new, out, batch, num_q_heads, t, count, count_per_seq, window, scale,
                 workspace, workspace_bytes, stream, rope);
}

int tempo_prefill_launches(const tempo_kv* kv, int32_t batch, int32_t num_q_heads, int32_t count) {
  if (check_layout(kv) != TEMPO_OK || check_heads(kv, batch, num_q_heads) != TEMPO_OK || count < 1) return 0;
  const int32_t G = num_q_heads / kv->num_kv_heads, block = kMaxColumns / G;
  if (kv->ring_blocks == 0 && prompt_in_one_launch(kv, batch, num_q_heads, count)) {
    if (kv->dtype != TEMPO_BF16) return 3;
    if (prompt_fills_part(kv, batch, G, count)) return 2;  // one launch, and no key range is split
  }
  return 3 * ((count + block - 1) / block);
}

size_t tempo_prefill_workspace_bytes(const tempo_kv* kv, int32_t batch, int32_t num_q_heads, int32_t max_t) {
  if (check_layout(kv) != TEMPO_OK || check_heads(kv, batch, num_q_heads) != TEMPO_OK) return 0;
  const int32_t block = kMaxColumns / (num_q_heads / kv->num_kv_heads);
  return tempo_attn_block_workspace_bytes(kv, batch, num_q_heads, block, max_t);
}

int tempo_attn_block_with_plan(const tempo_kv* kv, const void* q, void* out, int32_t batch,
                               int32_t num_q_heads, int32_t queries, int32_t t, const int32_t* t_per_seq,
                               int32_t window, float scale, const tempo_plan* plan, void* workspace,
                               size_t workspace_bytes, void* stream) {
  int rc = check_layout(kv);
  if (rc != TEMPO_OK) return rc;
  if (!q || !out || !plan) return TEMPO_ERR_NULL;
  if ((rc = check_scale(scale)) != TEMPO_OK) return rc;
  if ((rc = check_attn(kv, batch, num_q_heads, t, window, t_per_seq != nullptr, plan, workspace, workspace_bytes,
                       queries)) != TEMPO_OK)
    return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  rc = do_partial(kv, q, nullptr, nullptr, out, batch, num_q_heads, t, t_per_seq, window, scale, plan, workspace, s,
                  queries);
  if (rc != TEMPO_OK || plan->num_splits == 1) return rc;
  return do_combine(kv, out, batch, num_q_heads, t, t_per_seq, window, plan, workspace, s, queries);
}

int tempo_attn_block_causal(const tempo_kv* kv, const void* q, void* out, int32_t batch,
                            int32_t num_q_heads, int32_t queries, int32_t t, const int32_t* t_per_seq,
                            float scale, void* workspace, size_t workspace_bytes, void* stream) {
  return decode(kv, q, nullptr, nullptr, out, batch, num_q_heads, t, t_per_seq, 0, scale, workspace,
                workspace_bytes, stream, queries);
}

int tempo_attn_block_window(const tempo_kv* kv, const void* q, void* out, int32_t batch,
                            int32_t num_q_heads, int32_t queries, int32_t t, const int32_t* t_per_seq,
                            int32_t window, float scale, void* workspace, size_t workspace_bytes,
                            void* stream) {
  if (window < 1 || window > INT32_MAX - 64) return TEMPO_ERR_RANGE;
  return decode(kv, q, nullptr, nullptr, out, batch, num_q_heads, t, t_per_seq, window, scale, workspace,
                workspace_bytes, stream, queries);
}

int tempo_rope_attn_block_causal(const tempo_kv* kv, const tempo_rope* rope, const void* q_raw, void* out,
                                 int32_t batch, int32_t num_q_heads, int32_t queries, int32_t t,
                                 const int32_t* t_per_seq, float scale, void* workspace, size_t workspace_bytes,
                                 void* stream) {
  if (!rope) return TEMPO_ERR_NULL;
  return decode(kv, q_raw, nullptr, nullptr, out, batch, num_q_heads, t, t_per_seq, 0, scale, workspace,
                workspace_bytes, stream, queries, rope);
}

int tempo_rope_attn_block_window(const tempo_kv* kv, const tempo_rope* rope, const void* q_raw, void* out,
                                 int32_t batch, int32_t num_q_heads, int32_t queries, int32_t t,
                                 const int32_t* t_per_seq, int32_t window, float scale, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  if (!rope) return TEMPO_ERR_NULL;
  if (window < 1 || window > INT32_MAX - 64) return TEMPO_ERR_RANGE;
  return decode(kv, q_raw, nullptr, nullptr, out, batch, num_q_heads, t, t_per_seq, window, scale, workspace,
                workspace_bytes, stream, queries, rope);
}

int tempo_attn_decode_partial(const tempo_kv* kv, const void* q, const void* k_new,
                              const void* v_new, int32_t batch, int32_t num_q_heads, int32_t t,
                              const int32_t* t_per_seq, int32_t window, float scale,
                              const tempo_plan* plan, void* workspace, size_t workspace_bytes,
                              void* stream) {
  int rc = check_layout(kv);
  if (rc != TEMPO_OK) return rc;
  if (!q || ((k_new == nullptr) != (v_new == nullptr))) return TEMPO_ERR_NULL;
  if ((rc = check_scale(scale)) != TEMPO_OK) return rc;
  if ((rc = check_attn(kv, batch, num_q_heads, t, window, t_per_seq != nullptr, plan, workspace, workspace_bytes)) != TEMPO_OK) return rc;
  // the kernel that serves a group of more than 16 heads does not write the store
  if (k_new && kv->dtype == TEMPO_BF16 && num_q_heads / kv->num_kv_heads > kNarrowColumns) return TEMPO_ERR_SHAPE;
  return do_partial(kv, q, k_new, v_new, nullptr, batch, num_q_heads, t, t_per_seq, window, scale, plan,
                    workspace, static_cast<hipStream_t>(stream));
}

int tempo_attn_decode_combine(const tempo_kv* kv, void* out, int32_t batch, int32_t num_q_heads,
                              int32_t t, const int32_t* t_per_seq, int32_t window,
                              const tempo_plan* plan, const void* workspace,
                              size_t workspace_bytes, void* stream) {
  int rc = check_layout(kv);
  if (rc != TEMPO_OK) return rc;
  if (!out) return TEMPO_ERR_NULL;
  if ((rc = check_attn(kv, batch, num_q_heads, t, window, t_per_seq != nullptr, plan, workspace, workspace_bytes)) != TEMPO_OK) return rc;
  return do_combine(kv, out, batch, num_q_heads, t, t_per_seq, window, plan,
                    const_cast<void*>(workspace), static_cast<hipStream_t>(stream));
}

int tempo_discounted_sum(const float* r, float* g, int32_t batch, int32_t T, int32_t n, float gamma, void* stream) {
  if (!r || !g) return TEMPO_ERR_NULL;
  if (batch < 1 || batch > 65535 || T < 1) return TEMPO_ERR_SHAPE;
  if (n < 0 || !(gamma >= -3.0e38f && gamma <= 3.0e38f)) return TEMPO_ERR_RANGE;       // a finite discount
  if (n > discounted_sum_max_window() && n < T) return TEMPO_ERR_RANGE;                 // neither a short window nor the whole future
  if (r == g) return TEMPO_ERR_SHAPE;                                                   // a step reads rewards of later steps
  if ((int64_t)T > INT32_MAX - 4096) return TEMPO_ERR_SHAPE;
  const hipError_t e = launch_discounted_sum(r, g, batch, T, n, gamma, static_cast<hipStream_t>(stream));
  return launch_status(e, "discounted_sum");
}

int tempo_stream_read(const void* src, size_t bytes, void* sink, int32_t workgroups, void* stream) {
  if (!src || !sink) return TEMPO_ERR_NULL;
  if (bytes < 16 || bytes % 16 != 0 || (reinterpret_cast<uintptr_t>(src) & 15u) != 0) return TEMPO_ERR_SHAPE;
  if (workgroups < 1 || workgroups > (1 << 24)) return TEMPO_ERR_SHAPE;
  const hipError_t e = launch_stream_read(src, bytes, sink, workgroups, static_cast<hipStream_t>(stream));
  return launch_status(e, "stream_read");
}

int tempo_stream_copy(const void* src, void* dst, size_t bytes, int32_t workgroups, void* stream) {
  if (!src || !dst) return TEMPO_ERR_NULL;
  if (bytes < 16 || bytes % 16 != 0 || (reinterpret_cast<uintptr_t>(src) & 15u) != 0 ||
      (reinterpret_cast<uintptr_t>(dst) & 15u) != 0)
    return TEMPO_ERR_SHAPE;
  if (workgroups < 1 || workgroups > (1 << 24)) return TEMPO_ERR_SHAPE;
  const hipError_t e = launch_stream_copy(src, dst, bytes, workgroups, static_cast<hipStream_t>(stream));
  return launch_status(e, "stream_copy");
}

}  // extern "C"
