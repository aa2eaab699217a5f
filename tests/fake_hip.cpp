// A HIP runtime without a device, for host tests of libozaki and its BLAS
// interposer: loaded with global symbols before them, it answers their calls.
// Device memory is a budget of address ranges that nothing may touch, kernels
// and device copies are recorded instead of run, and a launch whose grid the
// runtime may refuse is refused (more than 2^32 - 1 work items in x, more than
// 65535 blocks in y or z). test_host_runtime_cpu.py builds it and reads the log.
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>

namespace {
std::mutex mu;
std::map<char *, size_t> dev, host;           // device and pinned ranges
std::map<const void *, std::string> kernels;  // host stub -> kernel name
size_t used = 0, budget = (size_t)1 << 38;
bool capturing = false;
std::string text;

void note(const char *fmt, unsigned long long a, unsigned long long b = 0, unsigned long long c = 0,
          const char *s = "") {
  char line[512];
  std::snprintf(line, sizeof line, fmt, s, a, b, c);
  text += line;
}
bool within(const std::map<char *, size_t> &m, const void *p) {
  auto it = m.upper_bound((char *)p);
  if (it == m.begin()) return false;
  --it;
  return (char *)p < it->first + it->second;
}
thread_local struct {
  dim3 g, b;
  size_t shmem;
  hipStream_t st;
} call;
}  // namespace

extern "C" {
// ------------------------------------------------------------ for the tests
void fake_budget(size_t bytes) { budget = bytes; }
void fake_capture(int on) { capturing = on != 0; }
size_t fake_used() { return used; }
void *fake_pinned(size_t bytes) {
  void *p = std::malloc(bytes);
  host[(char *)p] = bytes;
  return p;
}
// The log since the last call: one line per allocation, free, launch and copy.
const char *fake_log() {
  static std::string out;
  const std::lock_guard<std::mutex> l(mu);
  out.swap(text);
  text.clear();
  return out.c_str();
}

// ------------------------------------------------------------------ runtime
hipError_t hipMalloc(void **p, size_t n) {
  const std::lock_guard<std::mutex> l(mu);
  if (used + n > budget) {
    note("%.0snomem %llu\n", n);
    return hipErrorOutOfMemory;
  }
  *p = mmap(nullptr, n, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (*p == MAP_FAILED) return hipErrorOutOfMemory;
  used += n;
  dev[(char *)*p] = n;
  note("%.0smalloc %llu\n", n);
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  const std::lock_guard<std::mutex> l(mu);
  if (p == nullptr) return hipSuccess;
  auto it = dev.find((char *)p);
  if (it == dev.end()) return hipErrorInvalidValue;
  used -= it->second;
  note("%.0sfree %llu\n", it->second);
  munmap(p, it->second);
  dev.erase(it);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  const std::lock_guard<std::mutex> l(mu);
  *p = std::malloc(n);
  host[(char *)*p] = n;
  note("%.0spinned %llu\n", n);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  const std::lock_guard<std::mutex> l(mu);
  host.erase((char *)p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  const std::lock_guard<std::mutex> l(mu);
  std::memset(a, 0, sizeof *a);
  a->type = within(dev, p) ? hipMemoryTypeDevice : within(host, p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
  return hipSuccess;
}
hipError_t hipMemcpy(void *, const void *, size_t n, hipMemcpyKind k) {
  const std::lock_guard<std::mutex> l(mu);
  note("%.0scopy %llu %llu\n", n, k);
  return hipSuccess;
}
hipError_t hipMemcpy2D(void *, size_t, const void *, size_t, size_t w, size_t h, hipMemcpyKind k) {
  const std::lock_guard<std::mutex> l(mu);
  note("%.0scopy2d %llu %llu %llu\n", w, h, k);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *, const void *, size_t n, hipMemcpyKind k, hipStream_t) {
  const std::lock_guard<std::mutex> l(mu);
  note("%.0scopyasync %llu %llu\n", n, k);
  return hipSuccess;
}
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;  // compute units
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t)std::malloc(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  std::free(s);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = (hipEvent_t)std::malloc(1);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }

hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shmem, hipStream_t st) {
  call = {g, b, shmem, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shmem, hipStream_t *st) {
  *g = call.g;
  *b = call.b;
  *shmem = call.shmem;
  *st = call.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t, hipStream_t) {
  const std::lock_guard<std::mutex> l(mu);
  const bool ok = (unsigned long long)g.x * b.x <= 0xffffffffull && g.y <= 65535 && g.z <= 65535 &&
                  g.x > 0 && g.y > 0 && g.z > 0;
  note(ok ? "launch %s %llu %llu %llu\n" : "refused %s %llu %llu %llu\n", g.x, g.y, g.z, kernels[f].c_str());
  return ok ? hipSuccess : hipErrorInvalidConfiguration;
}
void **__hipRegisterFatBinary(const void *) {
  static void *handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *) {
  kernels[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
}
