// The host side of the library (tempo_api.hip) with its launches recorded instead of made: every
// launcher appends one line that says what it was asked for.  Built by test_host_launches.py with
// the host compiler, signed overflow checked; no GPU and no HIP runtime is involved.
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) x
#include "tempo_api.hip"

#include <stdarg.h>

#include <string>

static std::string g_log;

static hipError_t say(const char* format, ...) {
  char line[512];
  va_list args;
  va_start(args, format);
  vsnprintf(line, sizeof line, format, args);
  va_end(args);
  g_log += line;
  g_log += '\n';
  return hipSuccess;
}

// The runtime calls tempo_api.hip makes itself.
extern "C" {
hipError_t hipGetDevice(int* device) { *device = 0; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "recorded"; }
hipError_t hipGetSymbolAddress(void** ptr, const void* symbol) { *ptr = const_cast<void*>(symbol); return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipErrorUnknown; }

// The lines since the last call; valid until the next one.
const char* host_launches_take() {
  static std::string taken;
  taken.swap(g_log);
  g_log.clear();
  return taken.c_str();
}
}

namespace tempo {
// stream: does a wide block go to the kernel that streams its keys?  k, v: of a prompt that is read from its rows.
static hipError_t attend(const char* what, const AttnParams& p, int grid_splits, int waves, bool stream = false) {
  return say("%s t=%d queries=%d window=%d tps_log2=%d num_splits=%d grid_splits=%d direct=%d waves=%d stream=%d out=%zu steps=%d "
             "k=%zu v=%zu",
             what, p.t, p.queries, p.window, p.tps_log2, p.num_splits, grid_splits, p.direct, waves, stream, (size_t)p.out, p.io_steps,
             (size_t)p.k_new, (size_t)p.v_new);
}
hipError_t launch_append(const StoreParams& p, const void* k, const void* v, int, int, hipStream_t) {
  return say("append t=%d count=%d steps=%d k=%zu v=%zu", p.t, p.count, p.src_steps, (size_t)k, (size_t)v);
}
hipError_t launch_stage(const StageParams& p, const void* k, const void* v, int, hipStream_t) {
  return say("stage t=%d count=%d groups=%d steps=%d k=%zu v=%zu", p.t, p.count, p.stage_groups, p.src_steps, (size_t)k, (size_t)v);
}
hipError_t launch_gather(const StoreParams&, void*, void*, int, int, int j0, int count, hipStream_t) {
  return say("gather t=%d count=%d", j0, count);
}
hipError_t launch_partial_bf16(const AttnParams& p, int, int, int grid_splits, int waves, hipStream_t) {
  return attend("partial_bf16", p, grid_splits, waves);
}
size_t partial_bf16_lds_bytes(int waves, int columns, int D) {  // as next to the kernel
  return (size_t)waves * (32 + (size_t)columns * D) * sizeof(float) + (size_t)4 * D;
}
hipError_t launch_prefill_bf16(const PromptParams& p, int, int, int waves, int grid_splits, hipStream_t) {
  return attend(p.k_stage ? "prompt_staged" : "prompt", p, grid_splits, waves);
}
hipError_t launch_prompt_combine(const PromptParams& p, int, int, hipStream_t) { return attend("prompt_combine", p, 0, 0); }
hipError_t launch_short_prompt_bf16(const AttnParams& p, int, int, hipStream_t) { return attend("short_prompt", p, 1, 0); }
hipError_t launch_block_bf16(const AttnParams& p, int batch, int D, int grid_splits, hipStream_t) {
  const bool stream = block_streams(D, p.queries * p.G, (int64_t)batch * p.Hkv, block_keys(p.t, p.queries, p.window));
  return attend("block_bf16", p, grid_splits, 0, stream);
}
hipError_t launch_partial_f32(const AttnParams& p, int, int, int grid_splits, int waves, hipStream_t) {
  return attend("partial_f32", p, grid_splits, waves);
}
hipError_t launch_step_f32(const AttnParams& p, int, int, int grid_splits, int waves, hipStream_t) {
  return attend("step_f32", p, grid_splits, waves);
}
hipError_t launch_rope_rotate(const float*, const float*, const void*, void*, int, int, int, int, int t, const int32_t*,
                              hipStream_t) {
  return say("rope_rotate t=%d", t);
}
hipError_t launch_rope_append(const StoreParams& p, const float*, const float*, const void*, const void*, int, int,
                              hipStream_t) {
  return say("rope_append t=%d count=%d", p.t, p.count);
}
hipError_t launch_combine(const AttnParams& p, int, int, int, hipStream_t) { return attend("combine", p, 0, 0); }
hipError_t launch_worklist_build(const int32_t*, int, int t_max, int, int, int, int32_t*, hipStream_t) {
  return say("worklist t=%d", t_max);
}
hipError_t launch_discounted_sum(const float*, float*, int, int T, int, float, hipStream_t) { return say("discounted T=%d", T); }
int discounted_sum_max_window() { return 1024; }
hipError_t launch_stream_read(const void*, size_t, void*, int, hipStream_t) { return say("stream_read"); }
hipError_t launch_stream_copy(const void* from, void* to, size_t bytes, int, hipStream_t) {
  return say("stream_copy from=%zu to=%zu bytes=%zu", (size_t)from, (size_t)to, bytes);
}
}  // namespace tempo
