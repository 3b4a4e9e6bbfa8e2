// sdpdem_mlp_read on the host: the copies of the runtime are plain ones here,
// and operator new fails on demand.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

static bool no_memory = false;
void* operator new(size_t n) {
  void* p = no_memory ? nullptr : std::malloc(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept {
  return no_memory ? nullptr : std::malloc(n);
}
void* operator new[](size_t n) { return operator new(n); }
void* operator new[](size_t n, const std::nothrow_t& t) noexcept { return operator new(n, t); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
void operator delete[](void* p) noexcept { std::free(p); }
void operator delete[](void* p, size_t) noexcept { std::free(p); }

static hipError_t copy(void* to, const void* from, size_t n) {
  std::memcpy(to, from, n);
  return hipSuccess;
}
#define hipMemcpyAsync(to, from, n, kind, stream) copy(to, from, n)
#define hipStreamSynchronize(stream) hipSuccess
#include "sdpdem_mlp.hip"

int main() {
  static char store[1 << 20];
  sdpdem_mlp m;
  mlp_layout(reinterpret_cast<char*>(((uintptr_t)store + 255) & ~(uintptr_t)255), &m.T);
  for (int p = 0; p < NP; ++p) {
    m.T.master[p] = 0.5f + p;
    m.T.grad[p] = -1.0f - p;
    m.T.wq[p] = (uint16_t)(7 * p);
  }
  m.T.loss[0] = 3.5f;
  m.steps = 11;
  static float params[NP], used[NP], grad[NP];
  for (int want = 0; want < 16; ++want)
    for (int fail = 0; fail < 2; ++fail) {
      float loss = 0.0f;
      int64_t steps = 0;
      for (int p = 0; p < NP; ++p) params[p] = used[p] = grad[p] = 0.0f;
      no_memory = fail != 0;
      const int rc = sdpdem_mlp_read(&m, want & 1 ? params : nullptr, want & 2 ? used : nullptr,
                                     want & 4 ? grad : nullptr, want & 8 ? &loss : nullptr, &steps,
                                     nullptr);
      no_memory = false;
      bool ok = rc == SDPDEM_OK && steps == 11 && loss == (want & 8 ? 3.5f : 0.0f);
      for (int p = 0; p < NP; ++p) {
        const uint32_t u = (uint32_t)(uint16_t)(7 * p) << 16;
        ok = ok && params[p] == (want & 1 ? 0.5f + p : 0.0f) &&
             grad[p] == (want & 4 ? -1.0f - p : 0.0f) &&
             (want & 2 ? std::memcmp(&used[p], &u, 4) == 0 : used[p] == 0.0f);
      }
      std::printf("%d %d %s\n", want, fail, ok ? "ok" : "wrong");
      if (!ok) return 1;
    }
  return 0;
}
