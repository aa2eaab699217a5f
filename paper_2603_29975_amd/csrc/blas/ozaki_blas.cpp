// Host-BLAS interposer: Fortran DGEMM/ZGEMM served by libozaki on the GPU.
// The paper reaches the emulation through intercepted standard BLAS calls
// (Section 3.1); on a discrete GPU that means staging the host operands in
// HBM around each call. See include/ozaki_blas.h for the contract.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cctype>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <thread>

#include "../../../include/ozaki_blas.h"

namespace {

struct Staging {
  void *buf[3] = {nullptr, nullptr, nullptr};  // A, B, C
  size_t cap[3] = {0, 0, 0};
};
Staging g_stage;
std::mutex g_mutex;  // one call at a time: the buffers, lanes and libozaki's state are shared
int g_slices = 0, g_moduli = 0;

char up(char c) { return (char)std::toupper((unsigned char)c); }

int env_int(const char *name) {
  const char *v = std::getenv(name);
  return (v != nullptr && *v) ? std::atoi(v) : 0;
}

void fail(const char *routine, const char *what, int status) {
  std::fprintf(stderr, "ozaki_blas: %s: %s (status %d: %s)\n", routine, what, status,
               ozaki_status_string(status));
  std::abort();
}

void *stage(int which, size_t bytes, const char *routine) {
  if (bytes == 0) bytes = 16;
  if (g_stage.cap[which] < bytes) {
    if (g_stage.buf[which] != nullptr) (void)hipFree(g_stage.buf[which]);
    g_stage.buf[which] = nullptr;
    g_stage.cap[which] = 0;
    if (hipMalloc(&g_stage.buf[which], bytes) != hipSuccess) fail(routine, "hipMalloc", OZAKI_ERR_ALLOC);
    g_stage.cap[which] = bytes;
  }
  return g_stage.buf[which];
}

// ---------------------------------------------------------------- copies
// A host operand is pageable memory. hipMemcpy moves it through the runtime's own
// pinned buffers on one thread, 23 GB/s on a link that does more than twice that,
// so a large operand goes through pinned buffers here: several threads, each with
// a stream and two buffers, take the next chunk in turn and copy it while their
// last one is on the link. Threads live for one copy only; buffers and streams are
// kept until ozaki_blas_release. Whole ZGEMM calls, 7 slices, here / hipMemcpy:
// 2048^3 4.9 / 9.1 ms, 1000^3 1.40 / 2.02, 730^3 (8.5 MB operands) 0.89 / 1.10,
// but 600^3 (5.8 MB) 0.75 / 0.77 and 512^3 0.60 / 0.57. With 2, 8 and 12 lanes
// 2048^3 took 5.3, 5.2 and 5.4 ms, with chunks of 1 and 4 MiB 5.1 and 5.2. A
// pitched block of any size goes this way too (a small one on one lane): a pitched
// copy of pageable memory goes row by row, 2000^3 with ld = 2001 57 ms, here 4.7.
// Pinned arrays are left to the runtime: 2048^3 4.9 this way / 4.5 there, 1000^3
// 1.36 / 1.05, 2000^3 with ld = 2001 4.8 / 4.3, 200^3 with ld = 210 0.16 / 0.13.
constexpr int kLanes = 4;
constexpr size_t kChunk = (size_t)2 << 20;
constexpr size_t kLaneBytes = (size_t)6 << 20;  // smaller operands: one hipMemcpy

struct Lane {
  hipStream_t st = nullptr;
  char *pin[2] = {nullptr, nullptr};
  hipEvent_t ev[2] = {nullptr, nullptr};
};
Lane g_lane[kLanes];
int g_lane_dev = -1;  // device of the streams, -1: none

int release_lanes() {
  int rc = 0;
  for (Lane &l : g_lane) {
    for (int b = 0; b < 2; ++b) {
      if (l.ev[b] != nullptr && hipEventDestroy(l.ev[b]) != hipSuccess) rc = OZAKI_ERR_HIP;
      if (l.pin[b] != nullptr && hipHostFree(l.pin[b]) != hipSuccess) rc = OZAKI_ERR_HIP;
    }
    if (l.st != nullptr && hipStreamDestroy(l.st) != hipSuccess) rc = OZAKI_ERR_HIP;
    l = Lane{};
  }
  g_lane_dev = -1;
  return rc;
}

// The lanes on the current device; false if they cannot be had.
bool lanes_ready() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  if (g_lane_dev == dev) return true;
  (void)release_lanes();
  for (int i = 0; i < kLanes; ++i) {
    Lane &l = g_lane[i];
    bool ok = hipStreamCreateWithFlags(&l.st, hipStreamNonBlocking) == hipSuccess;
    for (int b = 0; b < 2 && ok; ++b)
      ok = hipHostMalloc(reinterpret_cast<void **>(&l.pin[b]), kChunk, hipHostMallocDefault) == hipSuccess &&
           hipEventCreateWithFlags(&l.ev[b], hipEventDisableTiming) == hipSuccess;
    if (!ok) {
      (void)hipGetLastError();
      (void)release_lanes();
      return false;
    }
  }
  g_lane_dev = dev;
  return true;
}

struct Job {
  char *dev;        // packed column-major block on the device
  char *host;       // its first element in host memory
  size_t col, ldb;  // bytes of a column and from one column to the next
  size_t bytes;
  bool up;
  std::atomic<size_t> next{0};
  std::atomic<int> err{0};
};

// Bytes [off, off + len) of the packed block from host memory to p, or back.
void pack(const Job &j, size_t off, size_t len, char *p) {
  while (len > 0) {
    const size_t in = off % j.col, n = j.ldb == j.col ? len : std::min(len, j.col - in);
    char *h = j.host + off / j.col * j.ldb + in;
    std::memcpy(j.up ? p : h, j.up ? h : p, n);
    off += n;
    p += n;
    len -= n;
  }
}

void run_lane(Job &j, Lane &l) {
  size_t off[2] = {0, 0}, len[2] = {0, 0};  // chunk on the link of either buffer
  auto landed = [&](int b) {
    if (len[b] == 0) return true;
    const hipError_t e = hipEventSynchronize(l.ev[b]);
    if (e == hipSuccess && !j.up) pack(j, off[b], len[b], l.pin[b]);
    len[b] = 0;
    return e == hipSuccess;
  };
  bool ok = true;
  int b = 0;
  for (; ok; b ^= 1) {
    ok = landed(b);
    const size_t o = j.next.fetch_add(kChunk);
    if (!ok || j.err.load() != 0 || o >= j.bytes) break;
    const size_t n = std::min(kChunk, j.bytes - o);
    if (j.up) pack(j, o, n, l.pin[b]);
    ok = hipMemcpyAsync(j.up ? j.dev + o : l.pin[b], j.up ? l.pin[b] : j.dev + o, n,
                        j.up ? hipMemcpyHostToDevice : hipMemcpyDeviceToHost, l.st) == hipSuccess &&
         hipEventRecord(l.ev[b], l.st) == hipSuccess;
    off[b] = o;
    len[b] = n;
  }
  // the other buffer's last chunk; nothing may stay on the link
  ok = landed(b ^ 1) && ok;
  if (hipStreamSynchronize(l.st) != hipSuccess) ok = false;
  if (!ok) j.err.store(1);
}

bool lane_copy(Job &j) {
  const int dev = g_lane_dev;
  std::thread th[kLanes];
  const int lanes = (int)std::min<size_t>(kLanes, (j.bytes + kChunk - 1) / kChunk);
  for (int i = 1; i < lanes; ++i) {
    try {
      th[i] = std::thread([&j, dev, i] {
        if (hipSetDevice(dev) == hipSuccess) run_lane(j, g_lane[i]);
        else j.err.store(1);
      });
    } catch (...) {  // no more threads: the others take the chunks
      break;
    }
  }
  run_lane(j, g_lane[0]);
  for (std::thread &t : th)
    if (t.joinable()) t.join();
  return j.err.load() == 0;
}

// Memory the runtime knows (pinned, managed or on a device): a copy of it goes
// straight over the link, and the host need not be able to touch it.
bool known_memory(const void *p) {
  hipPointerAttribute_t at{};
  if (hipPointerGetAttributes(&at, p) == hipSuccess) return at.type != hipMemoryTypeUnregistered;
  (void)hipGetLastError();
  return false;
}

// Copy the rows x cols column-major block at host (leading dimension ld) into
// a packed device buffer, or back. Exactly the block: the rows between `rows`
// and `ld` are neither read nor written.
bool copy_block(void *dev, void *host, int64_t rows, int64_t cols, int64_t ld, size_t esz, bool up) {
  const size_t col = (size_t)rows * esz, ldb = (size_t)ld * esz, bytes = col * (size_t)cols;
  const bool pitched = ld != rows && cols > 1;
  if ((bytes >= kLaneBytes || pitched) && !known_memory(host) && lanes_ready()) {
    Job j;
    j.dev = static_cast<char *>(dev);
    j.host = static_cast<char *>(host);
    j.col = col;
    j.ldb = pitched ? ldb : col;
    j.bytes = bytes;
    j.up = up;
    return lane_copy(j);
  }
  const hipMemcpyKind kind = up ? hipMemcpyHostToDevice : hipMemcpyDeviceToHost;
  void *dst = up ? dev : host, *src = up ? host : dev;
  return (!pitched ? hipMemcpy(dst, src, bytes, kind)
                   : hipMemcpy2D(dst, up ? col : ldb, src, up ? ldb : col, col, cols, kind)) == hipSuccess;
}
void to_device(void *dst, const void *src, int64_t rows, int64_t cols, int64_t ld, size_t esz,
               const char *routine) {
  if (rows == 0 || cols == 0) return;
  if (!copy_block(dst, const_cast<void *>(src), rows, cols, ld, esz, true))
    fail(routine, "copy to device", OZAKI_ERR_HIP);
}
void to_host(void *dst, const void *src, int64_t rows, int64_t cols, int64_t ld, size_t esz,
             const char *routine) {
  if (rows == 0 || cols == 0) return;
  if (!copy_block(const_cast<void *>(src), dst, rows, cols, ld, esz, false))
    fail(routine, "copy to host", OZAKI_ERR_HIP);
}

// Reference-BLAS argument checks; returns the number of the first illegal
// argument or 0.
int check(char ta, char tb, int m, int n, int k, int lda, int ldb, int ldc) {
  ta = up(ta);
  tb = up(tb);
  const bool oka = ta == 'N' || ta == 'T' || ta == 'C';
  const bool okb = tb == 'N' || tb == 'T' || tb == 'C';
  const int nrowa = ta == 'N' ? m : k;
  const int nrowb = tb == 'N' ? k : n;
  if (!oka) return 1;
  if (!okb) return 2;
  if (m < 0) return 3;
  if (n < 0) return 4;
  if (k < 0) return 5;
  if (lda < (nrowa > 1 ? nrowa : 1)) return 8;
  if (ldb < (nrowb > 1 ? nrowb : 1)) return 10;
  if (ldc < (m > 1 ? m : 1)) return 13;
  return 0;
}

template <typename T>
void gemm(bool cplx, const char *routine, char ta, char tb, int m, int n, int k, T alpha,
          const T *A, int lda, const T *B, int ldb, T beta, T *C, int ldc, bool alpha_zero,
          bool beta_zero, bool beta_one) {
  const int info = check(ta, tb, m, n, k, lda, ldb, ldc);
  if (info != 0) {
    std::fprintf(stderr, " ** On entry to %s parameter number %d had an illegal value\n", routine,
                 info);
    return;
  }
  if (m == 0 || n == 0 || ((alpha_zero || k == 0) && beta_one)) return;
  const std::lock_guard<std::mutex> lock(g_mutex);
  const size_t esz = sizeof(T);
  ta = up(ta);
  tb = up(tb);
  const int64_t rowsA = ta == 'N' ? m : k, colsA = ta == 'N' ? k : m;
  const int64_t rowsB = tb == 'N' ? k : n, colsB = tb == 'N' ? n : k;
  const bool need_ab = !alpha_zero && k > 0;
  T *dA = static_cast<T *>(stage(0, need_ab ? rowsA * colsA * esz : 0, routine));
  T *dB = static_cast<T *>(stage(1, need_ab ? rowsB * colsB * esz : 0, routine));
  T *dC = static_cast<T *>(stage(2, (size_t)m * n * esz, routine));
  if (need_ab) {
    to_device(dA, A, rowsA, colsA, lda, esz, routine);
    to_device(dB, B, rowsB, colsB, ldb, esz, routine);
  }
  if (!beta_zero) to_device(dC, C, m, n, ldc, esz, routine);
  const int64_t ldA = rowsA > 1 ? rowsA : 1, ldB = rowsB > 1 ? rowsB : 1;
  int slices = g_slices, moduli = g_moduli;
  if (slices == 0 && moduli == 0) {
    moduli = env_int("OZAKI_BLAS_MODULI");
    slices = moduli > 0 ? 0 : env_int("OZAKI_BLAS_SLICES");
    if (slices == 0 && moduli == 0) slices = 7;
  }
  int rc;
  if constexpr (sizeof(T) == sizeof(ozaki_z)) {
    rc = slices > 0 ? ozaki_zgemm(ta, tb, m, n, k, alpha, dA, ldA, dB, ldB, beta, dC, m, slices)
                    : ozaki2_zgemm(ta, tb, m, n, k, alpha, dA, ldA, dB, ldB, beta, dC, m, moduli);
  } else {
    rc = slices > 0 ? ozaki_dgemm(ta, tb, m, n, k, alpha, dA, ldA, dB, ldB, beta, dC, m, slices)
                    : ozaki2_dgemm(ta, tb, m, n, k, alpha, dA, ldA, dB, ldB, beta, dC, m, moduli);
  }
  (void)cplx;
  if (rc != 0) fail(routine, "emulated GEMM", rc);
  if (hipDeviceSynchronize() != hipSuccess) fail(routine, "synchronize", OZAKI_ERR_HIP);
  to_host(C, dC, m, n, ldc, esz, routine);
}

}  // namespace

extern "C" {

void dgemm_(const char *transa, const char *transb, const int *m, const int *n, const int *k,
            const double *alpha, const double *A, const int *lda, const double *B,
            const int *ldb, const double *beta, double *C, const int *ldc) {
  gemm<double>(false, "DGEMM ", *transa, *transb, *m, *n, *k, *alpha, A, *lda, B, *ldb, *beta, C,
               *ldc, *alpha == 0.0, *beta == 0.0, *beta == 1.0);
}

void zgemm_(const char *transa, const char *transb, const int *m, const int *n, const int *k,
            const ozaki_z *alpha, const ozaki_z *A, const int *lda, const ozaki_z *B,
            const int *ldb, const ozaki_z *beta, ozaki_z *C, const int *ldc) {
  gemm<ozaki_z>(true, "ZGEMM ", *transa, *transb, *m, *n, *k, *alpha, A, *lda, B, *ldb, *beta, C,
                *ldc, alpha->re == 0.0 && alpha->im == 0.0, beta->re == 0.0 && beta->im == 0.0,
                beta->re == 1.0 && beta->im == 0.0);
}

int ozaki_blas_config(int slices, int moduli) {
  if (slices < 0 || slices > OZAKI_S_MAX) return -1;
  if (moduli != 0 && (moduli < OZAKI2_MODULI_MIN || moduli > OZAKI2_MODULI_MAX)) return -2;
  g_slices = slices;
  g_moduli = slices > 0 ? 0 : moduli;
  return 0;
}

int ozaki_blas_release(void) {
  const std::lock_guard<std::mutex> lock(g_mutex);
  int rc = release_lanes();
  for (int w = 0; w < 3; ++w) {
    if (g_stage.buf[w] != nullptr && hipFree(g_stage.buf[w]) != hipSuccess) rc = OZAKI_ERR_HIP;
    g_stage.buf[w] = nullptr;
    g_stage.cap[w] = 0;
  }
  return rc;
}

}  // extern "C"
