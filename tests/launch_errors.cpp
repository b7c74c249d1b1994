// Calls the library's peak searches on a HIP runtime of its own, without a GPU: every
// runtime function the library uses is defined here (the program's symbols come
// before the HIP library's), launches do nothing and, once told to, fail.
// Prints "name status error-left" per call.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "ttm.h"

static int last_error = 0;
static bool launches_fail = false;

extern "C" {
struct dim3_t { unsigned x, y, z; };
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { static char scratch; *p = &scratch; return 0; }
int hipMalloc(void** p, size_t n) { *p = malloc(n); return 0; }
int hipFree(void* p) { free(p); return 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipMemcpyAsync(void* d, const void*, size_t n, int, void*) { memset(d, 0, n); return 0; }
const char* hipGetErrorString(int) { return "launch failure"; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
int __hipPushCallConfiguration(dim3_t, dim3_t, size_t, void*) { return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* m, void** s) { *g = *b = {1, 1, 1}; *m = 0; *s = nullptr; return 0; }
int hipLaunchKernel(const void*, dim3_t, dim3_t, void**, size_t, void*) {
  if (launches_fail) last_error = 719;   // hipErrorLaunchFailure
  return last_error;
}
}

int main() {
  ttm_ctx* ctx = nullptr;
  if (ttm_create(&ctx, 0) != TTM_OK) return 2;
  const int32_t lo[3] = {0, 0, 0}, hi[3] = {63, 63, 63}, ext[3] = {64, 64, 64};
  ttm_desc d = {2, 3, 16, 7.0f, 0.1f, 1e-6f, {0, 0, 1}};
  const size_t bytes = ttm_workspace_size(&d, TTM_OP_PEAKS, 0, 64, 64, 64);
  std::vector<char> ws(bytes);
  std::vector<float> score(64 * 64 * 64), vals(10);
  std::vector<int32_t> peaks(30);
  int32_t n = 0;
  ttm_peak_item item = {};
  for (launches_fail = false;; launches_fail = true) {
    const char* name = launches_fail ? "fail" : "ok";
    int rc = ttm_find_peaks(ctx, score.data(), 64, 64, 64, lo, hi, 10, 6.0f, peaks.data(), vals.data(), &n, ws.data(), bytes, nullptr);
    printf("find_peaks/%s %d %d\n", name, rc, hipGetLastError());
    rc = ttm_find_peaks_async(ctx, score.data(), 64, 64, 64, lo, hi, 10, 6.0f, peaks.data(), vals.data(), &n, ws.data(), bytes, nullptr);
    printf("find_peaks_async/%s %d %d\n", name, rc, hipGetLastError());
    rc = ttm_find_peaks_batch(ctx, &item, 1, ext, nullptr);
    printf("find_peaks_batch/%s %d %d\n", name, rc, hipGetLastError());
    if (launches_fail) break;
  }
  ttm_destroy(ctx);
  return 0;
}
