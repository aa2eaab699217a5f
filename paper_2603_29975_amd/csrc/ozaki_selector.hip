// Learned slice-count selector of libozaki (gfx950): exponent-statistics
// features and a 64 -> 128 -> 128 -> 1 ReLU MLP with BF16 weights and FP32
// accumulation, trained on the GPU by these kernels (forward, backward, Adam).
//
// The paper observes that emulation accuracy depends on both the arithmetic
// precision and properties of the operator (abstract; Section 4), and tunes the
// precision per run by hand. The selector predicts the number of slices a
// product needs from the one property the slicing is sensitive to: how far
// the entries sit below their row (column) maximum in binary exponent, since
// an entry delta binades below the maximum keeps only 7s - delta bits.
//
// Features of a product (64 floats):
//   [0..31]  fraction of entries of op(A) with delta = e_i - E(a_il) in bin
//            min(delta, 30), bin 31 = zero entries (E = frexp exponent, the
//            larger of the real and imaginary parts for complex data)
//   [32..62] the same for the columns of op(B): bins min(delta, 29), bin 30 =
//            zero entries
//   [63]     log2(k) / 16
//
// MLP parameters (P = 24961 floats, FP32 master copy), in this order:
//   W1 [128 x 64], b1 [128], W2 [128 x 128], b2 [128], w3 [128], b3 [1];
//   y = w3 . relu(W2 relu(W1 x + b1) + b2) + b3. W1, W2 and w3 are used as
//   BF16 (round to nearest even), so are the layer inputs fed to the matrix
//   cores; every product is accumulated in FP32 by v_mfma_f32_32x32x16_bf16.
#include "ozaki_internal.hpp"

namespace oz {

namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------- features
template <bool CPLX>
__device__ __forceinline__ int elem_code2(const void *base, int64_t off) {
  if (CPLX) {
    const double2 z = reinterpret_cast<const double2 *>(base)[off];
    return max(expo_code(z.x), expo_code(z.y));
  }
  return expo_code(reinterpret_cast<const double *>(base)[off]);
}

// Histogram bin of an entry with code c in a row with code rc (nbins bins;
// the last one counts zeros, the one before collects delta >= nbins - 2).
__device__ __forceinline__ int feat_bin(int c, int rc, int nbins) {
  if (c == 0 || code_bad(c) || code_bad(rc)) return nbins - 1;
  const int d = rc - c;
  return min(max(d, 0), nbins - 2);
}

// One block per task and row group: 256 threads walk the rows of the group
// (64 rows with 4 threads each when rows are unit-stride, else 4 rows with a
// wave each) over the whole contraction, into an LDS histogram; the loads of
// four entries are issued together.
template <bool CPLX>
__device__ void feat_block(const FeatTask &t, int64_t rb) {
  __shared__ int hist[32];
  const int tid = threadIdx.x;
  if (tid < 32) hist[tid] = 0;
  __syncthreads();
  const View &v = t.v;
  int64_t r, l, step, off0, stride;
  if (t.rows_fast) {
    r = rb * 64 + (tid & 63);
    l = tid >> 6;
    step = 4;
    off0 = r;
    stride = v.sl;
  } else {
    r = rb * 4 + (tid >> 6);
    l = tid & 63;
    step = 64;
    off0 = r * v.sr;
    stride = 1;
  }
  if (r < v.R) {
    const int rc = t.code[r];
    for (; l + 3 * step < v.L; l += 4 * step) {
      int cq[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) cq[q] = elem_code2<CPLX>(v.base, off0 + (l + q * step) * stride);
#pragma unroll
      for (int q = 0; q < 4; ++q) atomicAdd(&hist[feat_bin(cq[q], rc, t.nbins)], 1);
    }
    for (; l < v.L; l += step)
      atomicAdd(&hist[feat_bin(elem_code2<CPLX>(v.base, off0 + l * stride), rc, t.nbins)], 1);
  }
  __syncthreads();
  if (tid < t.nbins && hist[tid] != 0) atomicAdd(t.hist + tid, hist[tid]);
}

__device__ __forceinline__ int find_task2(const int64_t *start, int ntasks, int64_t b) {
  int lo = 0, hi = ntasks - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (start[mid] <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

__global__ void __launch_bounds__(256) k_feat_hist(const FeatTask *tasks, const int64_t *start,
                                                   int ntasks) {
  const int64_t b = blockIdx.x;
  const int t = find_task2(start, ntasks, b);
  const FeatTask tk = tasks[t];
  if (tk.cplx)
    feat_block<true>(tk, b - start[t]);
  else
    feat_block<false>(tk, b - start[t]);
}

// feat[p][0..63] from the integer histograms hist[p][0..63] (A bins 0..31,
// B bins 32..62) and the problem's m, n, k.
__global__ void __launch_bounds__(64) k_feat_finish(const int *hist, const int64_t *dims, float *feat,
                                                    int64_t np) {
  const int64_t p = blockIdx.x;
  const int j = threadIdx.x;
  if (p >= np) return;
  const int64_t m = dims[3 * p], n = dims[3 * p + 1], k = dims[3 * p + 2];
  float v;
  if (j < 32)
    v = (float)hist[p * 64 + j] / (float)(m * k);
  else if (j < 63)
    v = (float)hist[p * 64 + j] / (float)(k * n);
  else
    v = (float)(log2((double)k) / 16.0);
  feat[p * 64 + j] = v;
}

// ---------------------------------------------------------------- MLP
constexpr int kIn = 64, kH = 128;
constexpr int64_t kP = (int64_t)kH * kIn + kH + (int64_t)kH * kH + kH + kH + 1;  // 24961
// offsets of the parameters in the FP32 vector
constexpr int64_t oW1 = 0, oB1 = oW1 + kH * kIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH,
                  oW3 = oB2 + kH, oB3 = oW3 + kH;

// State layout (bytes): theta, adam m, adam v, grad (FP32, P each), then the
// BF16 copies W1 [128 x 64], W2 [128 x 128], W2^T [128 x 128], w3 [128].
constexpr size_t kStF32 = (size_t)kP * 4;
constexpr size_t sTheta = 0, sM = kStF32, sV = 2 * kStF32, sG = 3 * kStF32;
constexpr size_t sW1h = 4 * kStF32 + 64;  // keep 16-byte alignment (P*4 = 99844)
constexpr size_t sW2h = sW1h + (size_t)kH * kIn * 2;
constexpr size_t sW2th = sW2h + (size_t)kH * kH * 2;
constexpr size_t sW3h = sW2th + (size_t)kH * kH * 2;
constexpr size_t kStateBytes = sW3h + (size_t)kH * 2 + 64;

__device__ __forceinline__ float bf_round(float x) { return (float)(__bf16)x; }

// The network runs as three kernels: forward and the row part of the backward
// pass on 32 batch rows per workgroup (the layers of a row block follow each
// other through LDS), and the sums over the batch (weight and bias gradients,
// loss) with one workgroup per 32 x 32 weight tile or few columns. At batch 256
// they are bound by launch and memory latency: forward, loss and gradients
// 20 us, where one launch per step (12), the head's atomics (296 us) and two
// column sums by one workgroup (41 us each) took 430.
//
// One wave forms one 32 x 32 tile C = A * Bt^T with A, Bt rows of K BF16: lane l
// reads 8 consecutive entries of row l % 32 from contraction offset 8 (l / 32),
// and v_mfma_f32_32x32x16_bf16 leaves C[8 (r/4) + 4 (l/32) + r%4][l % 32] in
// register r.
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
constexpr int kRows = 32;          // batch rows per workgroup
constexpr int kPitch = kH + 8;     // BF16 per LDS row (16-byte aligned, rows 4 banks apart)

__device__ __forceinline__ int mm_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

template <int K>
__device__ __forceinline__ v16f mm_tile(const __bf16 *pa, const __bf16 *pb) {
  v8bf x[K / 16], y[K / 16];
#pragma unroll
  for (int q = 0; q < K / 16; ++q) {
    x[q] = *reinterpret_cast<const v8bf *>(pa + 16 * q);
    y[q] = *reinterpret_cast<const v8bf *>(pb + 16 * q);
  }
  v16f acc = {0};
#pragma unroll
  for (int q = 0; q < K / 16; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[q], y[q], acc, 0, 0, 0);
  return acc;
}

// Stores a wave's tile of BF16 values row-major (cols columns) and transposed
// (bp columns), rows r0.., column col, and into the LDS tile if there is one.
__device__ __forceinline__ void store_tile(const __bf16 (&h)[16], int lane, int64_t r0, int col,
                                           int64_t bp, __bf16 *rm, __bf16 *tr, __bf16 *lds) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int rr = mm_row(4 * g, lane);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      rm[(r0 + rr + b) * kH + col] = h[4 * g + b];
      if (lds) lds[(rr + b) * kPitch + col] = h[4 * g + b];
    }
    const v4bf v = {h[4 * g], h[4 * g + 1], h[4 * g + 2], h[4 * g + 3]};
    *reinterpret_cast<v4bf *>(tr + col * bp + r0 + rr) = v;
  }
}

struct MlpPtrs {
  const float *theta;
  const __bf16 *W1h, *W2h, *W2th, *w3h;
  __bf16 *xh, *xht;
  float *h1, *h2;
  __bf16 *h1h, *h1ht, *h2h, *h2ht, *dh2h, *dh2ht, *dh1h, *dh1ht;
  float *grad;
};

// Rows 32 blockIdx.x .. +31: Xh = bf16(X) (zero rows from b on), H1 = relu(Xh
// W1^T + b1), H2 = relu(bf16(H1) W2^T + b2), y = w3 . H2 + b3. Wave w forms the
// columns 32 w .. +31 of each layer.
__global__ void __launch_bounds__(256) k_mlp_fwd(MlpPtrs p, const float *X, int64_t b, int64_t bp,
                                                 float *y) {
  __shared__ __attribute__((aligned(16))) __bf16 xt[kRows * (kIn + 8)];
  __shared__ __attribute__((aligned(16))) __bf16 ht[kRows * kPitch];
  __shared__ float yp[4][kRows];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kRows;
  for (int c = tid; c < kRows * kIn; c += 256) {
    const int64_t r = r0 + c / kIn;
    const __bf16 v = (__bf16)(r < b ? X[r * kIn + c % kIn] : 0.0f);
    xt[(c / kIn) * (kIn + 8) + c % kIn] = v;
    p.xh[r * kIn + c % kIn] = v;
  }
  __syncthreads();
  for (int c = tid; c < kRows * kIn; c += 256)
    p.xht[(c / kRows) * bp + r0 + c % kRows] = xt[(c % kRows) * (kIn + 8) + c / kRows];

  const int col = 32 * wave + (lane & 31);
  v16f acc = mm_tile<kIn>(xt + (lane & 31) * (kIn + 8) + 8 * (lane >> 5),
                          p.W1h + col * kIn + 8 * (lane >> 5));
  __bf16 h[16];
  const float b1 = p.theta[oB1 + col];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float v = fmaxf(acc[r] + b1, 0.0f);
    p.h1[(r0 + mm_row(r, lane)) * kH + col] = v;
    h[r] = (__bf16)v;
  }
  store_tile(h, lane, r0, col, bp, p.h1h, p.h1ht, ht);
  __syncthreads();
  acc = mm_tile<kH>(ht + (lane & 31) * kPitch + 8 * (lane >> 5), p.W2h + col * kH + 8 * (lane >> 5));
  const float b2 = p.theta[oB2 + col], w3 = (float)p.w3h[col];
  float part[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float v = fmaxf(acc[r] + b2, 0.0f);
    p.h2[(r0 + mm_row(r, lane)) * kH + col] = v;
    h[r] = (__bf16)v;
    part[r] = w3 * v;
  }
  store_tile(h, lane, r0, col, bp, p.h2h, p.h2ht, nullptr);
  // the head: each row's 128 terms over the 32 lanes of the half wave, then the waves
#pragma unroll
  for (int off = 16; off > 0; off >>= 1)
#pragma unroll
    for (int r = 0; r < 16; ++r) part[r] += __shfl_xor(part[r], off);
  if ((lane & 31) == 0)
#pragma unroll
    for (int r = 0; r < 16; ++r) yp[wave][mm_row(r, lane)] = part[r];
  __syncthreads();
  if (tid < kRows && r0 + tid < b)
    y[r0 + tid] = ((yp[0][tid] + yp[1][tid]) + (yp[2][tid] + yp[3][tid])) + p.theta[oB3];
}

// dL/dy of row r for L = (1/b) sum_r w_r (y_r - t_r)^2, w_r = under (y_r < t_r) or 1.
__device__ __forceinline__ float loss_dy(float y, float t, float under, int64_t b) {
  const float e = y - t;
  const float w = y < t ? under : 1.0f;
  return 2.0f * w * e / (float)b;
}

// Rows 32 blockIdx.x .. +31: dH2 = dy w3 [H2 > 0] (BF16, zero rows from b on),
// dH1 = (dH2 W2) [H1 > 0] (BF16).
__global__ void __launch_bounds__(256) k_mlp_bwd_rows(MlpPtrs p, const float *y, const float *t,
                                                      float under, int64_t b, int64_t bp) {
  __shared__ __attribute__((aligned(16))) __bf16 dt[kRows * kPitch];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kRows;
  const int col = 32 * wave + (lane & 31);
  const float w3 = (float)p.w3h[col];
  __bf16 g[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t row = r0 + mm_row(r, lane);
    const float dy = row < b ? loss_dy(y[row], t[row], under, b) : 0.0f;
    g[r] = (__bf16)(row < b && p.h2[row * kH + col] > 0.0f ? dy * w3 : 0.0f);
  }
  store_tile(g, lane, r0, col, bp, p.dh2h, p.dh2ht, dt);
  __syncthreads();
  const v16f acc = mm_tile<kH>(dt + (lane & 31) * kPitch + 8 * (lane >> 5),
                               p.W2th + col * kH + 8 * (lane >> 5));
#pragma unroll
  for (int r = 0; r < 16; ++r)
    g[r] = (__bf16)(p.h1[(r0 + mm_row(r, lane)) * kH + col] > 0.0f ? acc[r] : 0.0f);
  store_tile(g, lane, r0, col, bp, p.dh1h, p.dh1ht, nullptr);
}

// The sums over the batch, 512 threads: blocks 0..15 one 32 x 32 tile of dW2 =
// dH2^T H1, 16..23 of dW1 = dH1^T X (the 8 waves take every eighth 16-row step
// and add up through LDS), 24..55 the bias gradients (one wave per column of
// dH1, dH2), 56..71 dw3 = H2^T dy (8 columns each), 72 db3 and the loss. Every
// sum has a fixed order.
constexpr int kSumTiles2 = (kH / 32) * (kH / 32), kSumTiles1 = (kH / 32) * (kIn / 32);
constexpr int kSumBias = 2 * kH / 8, kSumHead = kH / 8;
constexpr int kSumBlocks = kSumTiles2 + kSumTiles1 + kSumBias + kSumHead + 1;

__global__ void __launch_bounds__(512) k_mlp_bwd_sums(MlpPtrs p, const float *y, const float *t,
                                                      float under, float *loss, int64_t b, int64_t bp) {
  __shared__ float red[8 * 1024];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int blk = blockIdx.x;
  if (blk < kSumTiles2 + kSumTiles1) {
    const bool first = blk >= kSumTiles2;  // dW1
    if (first) blk -= kSumTiles2;
    const int nc = (first ? kIn : kH) / 32;
    const int r0 = (blk / nc) * 32, c0 = (blk % nc) * 32;
    const __bf16 *pa = (first ? p.dh1ht : p.dh2ht) + (r0 + (lane & 31)) * bp + 8 * (lane >> 5);
    const __bf16 *pb = (first ? p.xht : p.h1ht) + (c0 + (lane & 31)) * bp + 8 * (lane >> 5);
    v16f acc = {0};
    const int64_t steps = bp / 16;
    int64_t q = wave;
    for (; q + 24 < steps; q += 32) {  // four steps' loads in flight
      v8bf x[4], z[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        x[u] = *reinterpret_cast<const v8bf *>(pa + 16 * (q + 8 * u));
        z[u] = *reinterpret_cast<const v8bf *>(pb + 16 * (q + 8 * u));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[u], z[u], acc, 0, 0, 0);
    }
    for (; q < steps; q += 8)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const v8bf *>(pa + 16 * q),
                                                    *reinterpret_cast<const v8bf *>(pb + 16 * q), acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave * 1024 + mm_row(r, lane) * 32 + (lane & 31)] = acc[r];
    __syncthreads();
    float *out = p.grad + (first ? oW1 : oW2);
    for (int c = tid; c < 1024; c += 512) {
      float s = red[c];
#pragma unroll
      for (int w = 1; w < 8; ++w) s += red[w * 1024 + c];
      out[(r0 + c / 32) * (first ? kIn : kH) + c0 + c % 32] = s;
    }
    return;
  }
  blk -= kSumTiles2 + kSumTiles1;
  if (blk < kSumBias) {
    const int c = blk * 8 + wave;  // columns of dH1, then of dH2
    const __bf16 *g = (c < kH ? p.dh1ht + c * bp : p.dh2ht + (c - kH) * bp);
    float s = 0.0f;
    for (int64_t r = 8 * lane; r < bp; r += 512) {
      const v8bf x = *reinterpret_cast<const v8bf *>(g + r);
#pragma unroll
      for (int u = 0; u < 8; ++u) s += (float)x[u];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) p.grad[c < kH ? oB1 + c : oB2 + c - kH] = s;
    return;
  }
  blk -= kSumBias;
  if (blk < kSumHead) {
    const int c = blk * 8 + (tid & 7);
    float s = 0.0f;
    int64_t r = tid >> 3;
    for (; r + 192 < b; r += 256) {
      float h[4], d[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        h[u] = p.h2[(r + 64 * u) * kH + c];
        d[u] = loss_dy(y[r + 64 * u], t[r + 64 * u], under, b);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (d[u] != 0.0f) s = fmaf(d[u], h[u], s);  // an infinite H2 of a row without error adds nothing
    }
    for (; r < b; r += 64) {
      const float d = loss_dy(y[r], t[r], under, b);
      if (d != 0.0f) s = fmaf(d, p.h2[r * kH + c], s);
    }
    red[tid] = s;
    __syncthreads();
    if (tid < 8) {
      for (int u = 1; u < 64; ++u) s += red[tid + 8 * u];
      p.grad[oW3 + blk * 8 + tid] = s;
    }
    return;
  }
  float sd = 0.0f, sl = 0.0f;
  for (int64_t r = tid; r < b; r += 512) {
    const float e = y[r] - t[r];
    const float w = y[r] < t[r] ? under : 1.0f;
    sd += loss_dy(y[r], t[r], under, b);
    sl += w * e * e / (float)b;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sd += __shfl_xor(sd, off);
    sl += __shfl_xor(sl, off);
  }
  if (lane == 0) {
    red[wave] = sd;
    red[8 + wave] = sl;
  }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 8; ++w) {
      sd += red[w];
      sl += red[8 + w];
    }
    p.grad[oB3] = sd;
    if (loss) *loss = sl;
  }
}

// BF16 copies of W1, W2, W2^T and w3 from theta.
__global__ void __launch_bounds__(256) k_refresh_bf16(char *state) {
  const float *th = reinterpret_cast<const float *>(state + sTheta);
  __bf16 *W1h = reinterpret_cast<__bf16 *>(state + sW1h);
  __bf16 *W2h = reinterpret_cast<__bf16 *>(state + sW2h);
  __bf16 *W2th = reinterpret_cast<__bf16 *>(state + sW2th);
  __bf16 *w3h = reinterpret_cast<__bf16 *>(state + sW3h);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < kH * kIn) W1h[i] = (__bf16)th[oW1 + i];
  if (i < kH * kH) {
    const int64_t r = i / kH, c = i % kH;
    W2h[i] = (__bf16)th[oW2 + i];
    W2th[c * kH + r] = (__bf16)th[oW2 + i];
  }
  if (i < kH) w3h[i] = (__bf16)th[oW3 + i];
}

__device__ __forceinline__ uint64_t mix64(uint64_t x) {
  uint64_t z = x + 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// He-uniform initialisation: W ~ U(-sqrt(6/fan_in), +sqrt(6/fan_in)) from
// SplitMix64(seed + index), biases 0; Adam moments 0.
__global__ void __launch_bounds__(256) k_init(char *state, uint64_t seed) {
  float *th = reinterpret_cast<float *>(state + sTheta);
  float *m = reinterpret_cast<float *>(state + sM);
  float *v = reinterpret_cast<float *>(state + sV);
  float *g = reinterpret_cast<float *>(state + sG);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= kP) return;
  const double u = (double)(mix64(seed + (uint64_t)i) >> 11) * (1.0 / 9007199254740992.0);  // [0,1)
  float val = 0.0f;
  if (i < oB1)
    val = (float)((2.0 * u - 1.0) * sqrt(6.0 / kIn));
  else if (i >= oW2 && i < oB2)
    val = (float)((2.0 * u - 1.0) * sqrt(6.0 / kH));
  else if (i >= oW3 && i < oB3)
    val = (float)((2.0 * u - 1.0) * sqrt(6.0 / kH));
  th[i] = val;
  m[i] = 0.0f;
  v[i] = 0.0f;
  g[i] = 0.0f;
}

// Adam (Kingma and Ba 2015) with bias correction at step t >= 1.
__global__ void __launch_bounds__(256) k_adam(char *state, float lr, float b1, float b2, float eps,
                                              float c1, float c2) {
  float *th = reinterpret_cast<float *>(state + sTheta);
  float *m = reinterpret_cast<float *>(state + sM);
  float *v = reinterpret_cast<float *>(state + sV);
  const float *g = reinterpret_cast<const float *>(state + sG);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= kP) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

inline unsigned blocks(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// Scratch layout for a batch padded to bp rows (all offsets 256-aligned).
struct Scratch {
  size_t xh, xht, h1, h1h, h1ht, h2, h2h, h2ht, dh2h, dh2ht, dh1h, dh1ht, total;
};
Scratch scratch_layout(int64_t bp) {
  Scratch s{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) / 256 * 256;
    return o;
  };
  s.xh = take(bp * kIn * 2);
  s.xht = take(bp * kIn * 2);
  s.h1 = take(bp * kH * 4);
  s.h1h = take(bp * kH * 2);
  s.h1ht = take(bp * kH * 2);
  s.h2 = take(bp * kH * 4);
  s.h2h = take(bp * kH * 2);
  s.h2ht = take(bp * kH * 2);
  s.dh2h = take(bp * kH * 2);
  s.dh2ht = take(bp * kH * 2);
  s.dh1h = take(bp * kH * 2);
  s.dh1ht = take(bp * kH * 2);
  s.total = off;
  return s;
}

}  // namespace

int64_t mlp_params() { return kP; }
size_t mlp_state_bytes() { return kStateBytes; }
size_t mlp_scratch_bytes(int64_t batch) { return scratch_layout((batch + 31) / 32 * 32).total; }

hipError_t launch_feat_hist(const FeatTask *tasks, const int64_t *start, int ntasks, int64_t nblocks,
                            hipStream_t st) {
  if (ntasks <= 0 || nblocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_feat_hist, dim3((unsigned)nblocks), dim3(256), 0, st, tasks, start, ntasks);
  return hipGetLastError();
}

int64_t feat_task_blocks(const FeatTask &t) {
  return t.rows_fast ? (t.v.R + 63) / 64 : (t.v.R + 3) / 4;
}

hipError_t launch_feat_finish(const int *hist, const int64_t *dims, float *feat, int64_t np,
                              hipStream_t st) {
  if (np <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_feat_finish, dim3((unsigned)np), dim3(64), 0, st, hist, dims, feat, np);
  return hipGetLastError();
}

hipError_t mlp_init(void *state, uint64_t seed, hipStream_t st) {
  char *s = static_cast<char *>(state);
  hipLaunchKernelGGL(k_init, dim3(blocks(kP, 256)), dim3(256), 0, st, s, seed);
  hipLaunchKernelGGL(k_refresh_bf16, dim3(blocks(kH * kH, 256)), dim3(256), 0, st, s);
  return hipGetLastError();
}

hipError_t mlp_refresh(void *state, hipStream_t st) {
  hipLaunchKernelGGL(k_refresh_bf16, dim3(blocks(kH * kH, 256)), dim3(256), 0, st,
                     static_cast<char *>(state));
  return hipGetLastError();
}

namespace {
MlpPtrs mlp_ptrs(const void *state, void *scratch, int64_t bp) {
  // the state is written through `grad` only (backward pass, whose state is not const)
  char *s = static_cast<char *>(const_cast<void *>(state));
  char *w = static_cast<char *>(scratch);
  const Scratch L = scratch_layout(bp);
  auto bf = [](char *q) { return reinterpret_cast<__bf16 *>(q); };
  MlpPtrs p{};
  p.theta = reinterpret_cast<const float *>(s + sTheta);
  p.W1h = bf(s + sW1h);
  p.W2h = bf(s + sW2h);
  p.W2th = bf(s + sW2th);
  p.w3h = bf(s + sW3h);
  p.grad = reinterpret_cast<float *>(s + sG);
  p.xh = bf(w + L.xh);
  p.xht = bf(w + L.xht);
  p.h1 = reinterpret_cast<float *>(w + L.h1);
  p.h2 = reinterpret_cast<float *>(w + L.h2);
  p.h1h = bf(w + L.h1h);
  p.h1ht = bf(w + L.h1ht);
  p.h2h = bf(w + L.h2h);
  p.h2ht = bf(w + L.h2ht);
  p.dh2h = bf(w + L.dh2h);
  p.dh2ht = bf(w + L.dh2ht);
  p.dh1h = bf(w + L.dh1h);
  p.dh1ht = bf(w + L.dh1ht);
  return p;
}
}  // namespace

hipError_t mlp_forward(const void *state, int64_t b, const float *X, float *y, void *scratch,
                       hipStream_t st) {
  if (b <= 0) return hipSuccess;
  const int64_t bp = (b + 31) / 32 * 32;
  hipLaunchKernelGGL(k_mlp_fwd, dim3((unsigned)(bp / kRows)), dim3(256), 0, st,
                     mlp_ptrs(state, scratch, bp), X, b, bp, y);
  return hipGetLastError();
}

hipError_t mlp_backward(void *state, int64_t b, const float *y, const float *target, float under,
                        float *loss, void *scratch, hipStream_t st) {
  if (b <= 0) return hipSuccess;
  const int64_t bp = (b + 31) / 32 * 32;
  const MlpPtrs p = mlp_ptrs(state, scratch, bp);
  hipLaunchKernelGGL(k_mlp_bwd_rows, dim3((unsigned)(bp / kRows)), dim3(256), 0, st, p, y, target,
                     under, b, bp);
  hipLaunchKernelGGL(k_mlp_bwd_sums, dim3(kSumBlocks), dim3(512), 0, st, p, y, target, under, loss, b,
                     bp);
  return hipGetLastError();
}

hipError_t mlp_adam(void *state, float lr, float b1, float b2, float eps, int64_t step,
                    hipStream_t st) {
  const float c1 = 1.0f - powf(b1, (float)step);
  const float c2 = 1.0f - powf(b2, (float)step);
  char *s = static_cast<char *>(state);
  hipLaunchKernelGGL(k_adam, dim3(blocks(kP, 256)), dim3(256), 0, st, s, lr, b1, b2, eps, c1, c2);
  hipLaunchKernelGGL(k_refresh_bf16, dim3(blocks(kH * kH, 256)), dim3(256), 0, st, s);
  return hipGetLastError();
}

}  // namespace oz
