// A decode step whose launches or copies fail, on the CPU: the program defines the HIP calls of
// the library's step itself ("device" memory is host memory, kernels do nothing,
// copies stay pending until their stream is waited for), makes one call of a step fail in turn,
// and requires that asr_step returns an error with no copy pending whose host memory (the
// step's own rows, the caller's argmax and logits) may be gone by then.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "asr.h"

namespace {
struct Copy {
  void* dst;
  const void* src;
  size_t n;
};
std::vector<Copy> pending;
int calls = 0, fail_at = -1;   // of the copies and error queries since armed
constexpr int kFailed = 719;
int step_call() { return fail_at >= 0 && calls++ == fail_at ? kFailed : 0; }
}  // namespace

extern "C" {
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipLaunchKernel(const void*, unsigned long long, unsigned long long, void**, size_t, void*) { return 0; }
int hipGetLastError() { return step_call(); }
const char* hipGetErrorString(int) { return "made to fail"; }
int hipMemcpyAsync(void* dst, const void* src, size_t n, int, void*) {
  if (int e = step_call()) return e;
  pending.push_back({dst, src, n});
  return 0;
}
int hipStreamSynchronize(void*) {
  for (const Copy& c : pending) memcpy(c.dst, c.src, c.n);
  pending.clear();
  return 0;
}
int hipDeviceSynchronize() { return hipStreamSynchronize(nullptr); }
}

#define OK(x)                                                                       \
  do {                                                                              \
    if ((x) != ASR_OK) return printf("%s: %s\n", #x, asr_last_error()), 1;          \
  } while (0)

int main() {
  asr_model_cfg cfg{8, 64, 0, 1, 1, 64, 40, ASR_F32, 1, 1, 1, 4};
  asr_ctx* c = nullptr;
  OK(asr_create(&cfg, 0, &c));
  size_t bytes = 0;
  OK(asr_workspace_size(c, &bytes));
  void* block = aligned_alloc(256, bytes);
  memset(block, 0, bytes);
  OK(asr_bind(c, block, bytes, nullptr));
  int32_t n = 0;
  OK(asr_n_params(c, &n));
  std::vector<std::vector<float>> data(n);
  std::vector<const float*> tensors(n);
  for (int i = 0; i < n; ++i) {
    int64_t numel = 0;
    OK(asr_param_numel(c, i, &numel));
    data[i].resize(numel);
    tensors[i] = data[i].data();
  }
  OK(asr_load_weights(c, tensors.data(), n, 0));
  OK(asr_set_decode_graphs(c, 0));
  std::vector<float> E(1500 * 64), logits(40);
  int32_t slot = 0, left = 40, token = 0, argmax = 0, done = 0;
  int64_t id = -1;
  OK(asr_debug_set_encoder_out(c, &slot, &id, &left, 1, E.data(), 0));
  asr_step_in in{0, nullptr, 1, &slot, &token, logits.data()};
  asr_step_out out{nullptr, &argmax, &done};
  int bad = 0, failing = 0;
  for (int at = 0;; ++at) {
    calls = 0;
    fail_at = at;
    const asr_status st = asr_step(c, &in, &out);
    const bool reached = calls > at;
    fail_at = -1;
    if (!reached) {                       // every call of the step has failed once
      OK(st);
      break;
    }
    ++failing;
    if (st != ASR_EDEVICE || !pending.empty()) {
      printf("call %d of the step: status %d, %zu copies pending\n", at, (int)st, pending.size());
      ++bad;
    }
    hipStreamSynchronize(nullptr);
  }
  OK(asr_destroy(c));
  free(block);
  if (failing < 4) return printf("only %d calls failed\n", failing), 1;
  if (!bad) printf("failed steps leave nothing pending: ok (%d)\n", failing);
  return bad != 0;
}
