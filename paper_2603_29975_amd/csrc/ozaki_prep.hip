// Exponent scan, slicing and small helper kernels of libozaki (gfx950).
//
// Steps "exponent alignment" and "split into slices by significant bits" of
// the Ozaki-I scheme (Section 2.2 of the paper). Both are HBM-bound: the scan
// reads each operand once, the split reads it again and writes S (real) or
// 2S (complex) bytes per element in the packed fragment layout.
#include "ozaki_split_tile.hpp"

namespace oz {

namespace {

__global__ void __launch_bounds__(256) k_fill_i32(int *p, int64_t n, int value) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = value;
}

// Pseudo-random INT8 digits in [-127, 127] (SplitMix64 finaliser of the byte
// index): stand-in slice data for timing the slice GEMM, whose power draw and
// clock depend on the operand bits.
// Grid-stride: the fills of large workspaces exceed the grid size limit.
__global__ void __launch_bounds__(256) k_fill_digits(int8_t *p, int64_t n, uint64_t seed) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    uint64_t z = seed + 0x9e3779b97f4a7c15ull * (uint64_t)(i + 1);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z ^= z >> 31;
    p[i] = (int8_t)((int)(z % 255u) - 127);
  }
}

template <bool CPLX>
__device__ __forceinline__ int elem_code(const void *base, int64_t off) {
  if (CPLX) {
    const double2 z = reinterpret_cast<const double2 *>(base)[off];
    return max(expo_code(z.x), expo_code(z.y));
  }
  return expo_code(reinterpret_cast<const double *>(base)[off]);
}

// Rows are unit-stride in memory (sr == 1): 64 consecutive rows per block,
// four threads per row walking the contraction index; each warp-wide load is
// one contiguous run of 64 elements.
// `direct`: the block covers the whole contraction range, so the row code is
// stored instead of max-combined with other blocks.
template <bool CPLX>
__device__ __forceinline__ void scan_rowsfast_block(const View &v, int64_t rb, int64_t l0,
                                                    int64_t l1, int *code, bool direct) {
  const int tid = threadIdx.x;
  const int64_t r = rb * 64 + (tid & 63);
  int c = 0;
  if (r < v.R) {
    // eight loads in flight per pass (a block that covers a long contraction
    // alone is latency-bound), then four, then the remainder
    int64_t l = l0 + (tid >> 6);
    for (; l + 28 < l1; l += 32) {
      int a[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) a[q] = elem_code<CPLX>(v.base, r + (l + 4 * q) * v.sl);
      c = max(c, max(max(max(a[0], a[1]), max(a[2], a[3])), max(max(a[4], a[5]), max(a[6], a[7]))));
    }
    for (; l + 12 < l1; l += 16) {
      const int a0 = elem_code<CPLX>(v.base, r + l * v.sl);
      const int a1 = elem_code<CPLX>(v.base, r + (l + 4) * v.sl);
      const int a2 = elem_code<CPLX>(v.base, r + (l + 8) * v.sl);
      const int a3 = elem_code<CPLX>(v.base, r + (l + 12) * v.sl);
      c = max(c, max(max(a0, a1), max(a2, a3)));
    }
    for (; l < l1; l += 4) c = max(c, elem_code<CPLX>(v.base, r + l * v.sl));
  }
  __shared__ int red[256];
  red[tid] = c;
  __syncthreads();
  if (tid < 64) {
    c = max(max(red[tid], red[tid + 64]), max(red[tid + 128], red[tid + 192]));
    if (r < v.R) {
      if (direct)
        code[r] = c;
      else if (c > 0)
        atomicMax(code + r, c);
    }
  }
}

// Each row is unit-stride (sl == 1): one wave per row and contraction chunk,
// lanes read consecutive elements, a wave max-reduction gives the row code.
template <bool CPLX>
__device__ __forceinline__ void scan_rowcontig_block(const View &v, int64_t rb, int64_t l0,
                                                     int64_t l1, int *code, bool direct) {
  const int lane = threadIdx.x & 63;
  const int64_t r = rb * 4 + (threadIdx.x >> 6);
  if (r >= v.R) return;
  int c = 0;
  int64_t l = l0 + lane;
  for (; l + 192 < l1; l += 256) {  // four loads in flight per pass
    const int a0 = elem_code<CPLX>(v.base, r * v.sr + l);
    const int a1 = elem_code<CPLX>(v.base, r * v.sr + l + 64);
    const int a2 = elem_code<CPLX>(v.base, r * v.sr + l + 128);
    const int a3 = elem_code<CPLX>(v.base, r * v.sr + l + 192);
    c = max(c, max(max(a0, a1), max(a2, a3)));
  }
  for (; l < l1; l += 64) c = max(c, elem_code<CPLX>(v.base, r * v.sr + l));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c = max(c, __shfl_xor(c, off));
  if (lane == 0) {
    if (direct)
      code[r] = c;
    else if (c > 0)
      atomicMax(code + r, c);
  }
}

// One thread per (packed row, 16 consecutive packed contraction entries):
// reads the 16 source values (8 complex elements), splits each into S digits
// and writes one 16-byte run per slice into the packed fragment layout.
// Rows and entries beyond the operand are written as zero digits (padding).
// Per-byte negation of four packed digits in [0, 127]: bytes whose mask byte
// is 0xff become (-d) mod 256. (d ^ 0x7f) + 1 = 128 - d never carries out of
// its byte, and xor 0x80 then adds 128.
__device__ __forceinline__ uint32_t neg_bytes(uint32_t w, uint32_t mask) {
  return ((w ^ (mask & 0x7f7f7f7fu)) + (mask & 0x01010101u)) ^ (mask & 0x80808080u);
}

// floor(|x| 2^(7S)) for S <= 9 (at most 63 bits): the top 7S bits of |x|
// below the binary point as one integer, so digit p is bits
// [7(S-p), 7(S-p)+7) of it.
template <int S>
__device__ __forceinline__ uint64_t top_bits(const Sig &x) {
  const int sh = x.sh0 + kDigitBits * S;
  if (sh >= 0) return x.m << sh;  // sh <= 7S - 53 <= 10: no overflow
  return (sh > -64) ? (x.m >> (-sh)) : 0ull;
}

// trunc(|x| 2^NB) for NB <= 62 (|x| < 1 after the exponent shift, so the
// result stays below 2^NB).
template <int NB>
__device__ __forceinline__ uint64_t top_nbits(const Sig &x) {
  const int sh = x.sh0 + NB;
  if (sh >= 0) return x.m << sh;
  return (sh > -64) ? (x.m >> (-sh)) : 0ull;
}

template <bool CPLX, bool SIDEB, int SC, bool TRP, bool B8>
__device__ __forceinline__ void split_block(const View &v, const int *code, int S, int8_t *out,
                                            int64_t nrb, int64_t nkb, int64_t bx, int64_t by,
                                            const double *tile) {
  const int tid = threadIdx.x;
  const int64_t rp = bx * 64 + (tid & 63);
  const int64_t kp0 = (by * 4 + (tid >> 6)) * 16;
  const int64_t Rrows = (CPLX && SIDEB) ? 2 * v.R : v.R;
  const int64_t r = (CPLX && SIDEB) ? (rp >> 1) : rp;
  const int cr = (CPLX && SIDEB) ? (int)(rp & 1) : 0;
  const int c = (rp < Rrows) ? code[r] : 0;
  const bool live = (rp < Rrows) && !code_bad(c);
  const int e = code_exp(c);

  Sig sg[16];
  if (CPLX) {
    const double2 *X = reinterpret_cast<const double2 *>(v.base);
    // every load of the thread is issued before any is used (an entry outside
    // the view reads element (0, 0), or its zero in the staged tile, and
    // counts as zero)
    double2 zs[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int64_t l = (kp0 >> 1) + x;
      if constexpr (TRP) {
        using T = SplitTile<CPLX, SIDEB>;
        zs[x] = *reinterpret_cast<const double2 *>(tile + (r - bx * T::TR) * T::PITCH +
                                                   (l - by * T::TL) * 2);
      } else {
        zs[x] = X[(live && l < v.L) ? r * v.sr + l * v.sl : 0];
      }
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int64_t l = (kp0 >> 1) + x;
      const bool ok = live && l < v.L;
      const double re = ok ? zs[x].x : 0.0;
      const double im = ok ? (v.conj ? -zs[x].y : zs[x].y) : 0.0;
      double v0, v1;
      if (!SIDEB) {
        v0 = re;
        v1 = im;
      } else if (cr == 0) {
        v0 = re;
        v1 = -im;
      } else {
        v0 = im;
        v1 = re;
      }
      sg[2 * x] = decompose(v0, e);
      sg[2 * x + 1] = decompose(v1, e);
    }
  } else {
    const double *X = reinterpret_cast<const double *>(v.base);
    double vs[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const int64_t l = kp0 + x;
      if constexpr (TRP) {
        using T = SplitTile<CPLX, SIDEB>;
        vs[x] = tile[(r - bx * T::TR) * T::PITCH + (l - by * T::TL)];
      } else {
        vs[x] = X[(live && l < v.L) ? r * v.sr + l * v.sl : 0];
      }
    }
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const int64_t l = kp0 + x;
      sg[x] = decompose((live && l < v.L) ? vs[x] : 0.0, e);
    }
  }

  if constexpr (B8) {
    // 8-bit balanced slices: X = trunc(x 2^(8S - 2)) with the sign of x, and
    // its balanced base-256 digits d_p in [-128, 127] (slice p holds the digit
    // of weight 256^(S - p)). With Y = X + 128 (256^S - 1) / 255, which lies in
    // [0, 256^S) because |X| < 2^(8S - 2), the plain base-256 bytes b_p of Y
    // are d_p + 128: the same digits as the recurrence d = ((X + 128) mod 256)
    // - 128, X <- (X - d) / 256, read off as bytes, with d_p = b_p - 128 being
    // b_p XOR 0x80 in two's complement. Every value is split as it stands, so
    // the -Im row of complex B gets the digits of -Im.
    static_assert(SC >= 1 && SC <= 8, "8-bit slices need 8S - 2 <= 62");
    constexpr uint64_t kBias = 0x8080808080808080ull >> (8 * (8 - SC));  // 128 (256^S - 1) / 255
    uint64_t Y[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const uint64_t u = top_nbits<8 * SC - 2>(sg[x]);
      Y[x] = (sg[x].neg ? (0ull - u) : u) + kBias;  // mod 2^64; the true value is in [0, 256^S)
    }
#pragma unroll
    for (int p = SC; p >= 1; --p) {
      const int sh = 8 * (SC - p);
      uint32_t w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) word |= ((uint32_t)(Y[4 * q + b] >> sh) & 0xffu) << (8 * b);
        w[q] = word ^ 0x80808080u;
      }
      int8_t *dst = out + frag_offset(p - 1, rp, kp0, nrb, nkb);
      *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  } else if constexpr (SC > 0) {
    // S known at compile time and 7S <= 63: one integer per value, digits by
    // constant shifts, signs applied four bytes at a time.
    uint64_t T[16];
    uint32_t neg[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t mk = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        T[4 * q + b] = top_bits<SC>(sg[4 * q + b]);
        mk |= (sg[4 * q + b].neg ? 0xffu : 0u) << (8 * b);
      }
      neg[q] = mk;
    }
#pragma unroll
    for (int p = 1; p <= SC; ++p) {
      uint32_t w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b)
          word |= ((uint32_t)(T[4 * q + b] >> (kDigitBits * (SC - p))) & 127u) << (8 * b);
        w[q] = neg_bytes(word, neg[q]);
      }
      int8_t *dst = out + frag_offset(p - 1, rp, kp0, nrb, nkb);
      *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  } else {
    for (int p = 1; p <= S; ++p) {
      uint32_t w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) word |= ((uint32_t)digit(sg[4 * q + b], p) & 0xffu) << (8 * b);
        w[q] = word;
      }
      int8_t *dst = out + frag_offset(p - 1, rp, kp0, nrb, nkb);
      *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

template <bool CPLX, bool SIDEB, bool TRP, bool B8>
__device__ __forceinline__ void split_s(const View &v, const int *code, int S, int8_t *out,
                                        int64_t nrb, int64_t nkb, int64_t bx, int64_t by,
                                        const double *tile) {
  if constexpr (B8) {
    // 1..8 slices (the host rejects more)
    switch (S) {
#define OZ_SPLIT(N) \
  case N: split_block<CPLX, SIDEB, N, TRP, true>(v, code, S, out, nrb, nkb, bx, by, tile); break;
      OZ_SPLIT(1) OZ_SPLIT(2) OZ_SPLIT(3) OZ_SPLIT(4) OZ_SPLIT(5) OZ_SPLIT(6) OZ_SPLIT(7)
      OZ_SPLIT(8)
#undef OZ_SPLIT
      default: break;
    }
  } else {
    switch (S) {
#define OZ_SPLIT(N) \
  case N: split_block<CPLX, SIDEB, N, TRP, false>(v, code, S, out, nrb, nkb, bx, by, tile); break;
      OZ_SPLIT(1) OZ_SPLIT(2) OZ_SPLIT(3) OZ_SPLIT(4) OZ_SPLIT(5) OZ_SPLIT(6) OZ_SPLIT(7)
      OZ_SPLIT(8) OZ_SPLIT(9)
#undef OZ_SPLIT
      default: split_block<CPLX, SIDEB, 0, TRP, false>(v, code, S, out, nrb, nkb, bx, by, tile); break;
    }
  }
}

template <bool CPLX, bool SIDEB, bool B8 = false>
__device__ __forceinline__ void split_dispatch(const View &v, const int *code, int S, int8_t *out,
                                               int64_t nrb, int64_t nkb, int64_t bx, int64_t by,
                                               double *tile) {
  if (tile != nullptr && split_staged(v)) {
    load_split_tile<CPLX, SIDEB>(v, bx, by, tile);
    split_s<CPLX, SIDEB, true, B8>(v, code, S, out, nrb, nkb, bx, by, tile);
  } else {
    split_s<CPLX, SIDEB, false, B8>(v, code, S, out, nrb, nkb, bx, by, nullptr);
  }
}

template <bool CPLX, bool SIDEB, bool STAGED, bool B8>
__global__ void __launch_bounds__(256) k_split(View v, const int *code, int S, int8_t *out,
                                               int64_t nrb, int64_t nkb) {
  if constexpr (STAGED) {
    __shared__ __attribute__((aligned(16))) double tile[kSplitTileDoubles];
    split_dispatch<CPLX, SIDEB, B8>(v, code, S, out, nrb, nkb, blockIdx.x, blockIdx.y, tile);
  } else {
    split_dispatch<CPLX, SIDEB, B8>(v, code, S, out, nrb, nkb, blockIdx.x, blockIdx.y, nullptr);
  }
}

// Both operands of a product in one launch: blocks [0, na) take the first view.
// Each block is one of nr row groups times a contraction chunk.
struct ScanSide {
  View v;
  int *code;
  int64_t nr, lchunk;
  int rows_fast;
};
template <bool CPLX>
__global__ void __launch_bounds__(256) k_scan(ScanSide a, ScanSide b, int64_t na) {
  const bool first = blockIdx.x < na;
  const ScanSide &s = first ? a : b;
  const int64_t blk = first ? blockIdx.x : blockIdx.x - na;
  const int64_t l0 = (blk / s.nr) * s.lchunk, l1 = min(s.v.L, l0 + s.lchunk);
  if (s.rows_fast)
    scan_rowsfast_block<CPLX>(s.v, blk % s.nr, l0, l1, s.code, false);
  else
    scan_rowcontig_block<CPLX>(s.v, blk % s.nr, l0, l1, s.code, false);
}

// Both operands in one launch: blocks [0, na) take the first.
struct SplitSide {
  View v;
  const int *code;
  int8_t *out;
  int64_t nrb, nkb;
};
template <bool CPLX, bool B8>
__global__ void __launch_bounds__(256) k_split_pair(SplitSide a, SplitSide b, int64_t na, int S) {
  __shared__ __attribute__((aligned(16))) double tile[kSplitTileDoubles];
  if (blockIdx.x < na) {
    const int64_t nbx = a.nrb / 2, blk = blockIdx.x;
    split_dispatch<CPLX, false, B8>(a.v, a.code, S, a.out, a.nrb, a.nkb, blk % nbx, blk / nbx, tile);
  } else {
    const int64_t nbx = b.nrb / 2, blk = blockIdx.x - na;
    split_dispatch<CPLX, true, B8>(b.v, b.code, S, b.out, b.nrb, b.nkb, blk % nbx, blk / nbx, tile);
  }
}

// ---------------------------------------------------------------- batched
// Block b of a batched launch belongs to the task t with
// start[t] <= b < start[t + 1] (binary search, uniform per block).
__device__ __forceinline__ int find_task(const int64_t *start, int ntasks, int64_t b) {
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

// One task scans all rows of one operand view over the whole contraction.
__global__ void __launch_bounds__(256) k_scan_batched(const ScanTask *tasks, const int64_t *start,
                                                      int ntasks) {
  const int64_t b = blockIdx.x;
  const int t = find_task(start, ntasks, b);
  const ScanTask tk = tasks[t];
  const int64_t rb = b - start[t];
  if (tk.rows_fast) {
    if (tk.cplx)
      scan_rowsfast_block<true>(tk.v, rb, 0, tk.v.L, tk.code, true);
    else
      scan_rowsfast_block<false>(tk.v, rb, 0, tk.v.L, tk.code, true);
  } else {
    if (tk.cplx)
      scan_rowcontig_block<true>(tk.v, rb, 0, tk.v.L, tk.code, true);
    else
      scan_rowcontig_block<false>(tk.v, rb, 0, tk.v.L, tk.code, true);
  }
}

// One task splits one operand view into its packed buffer; its blocks cover
// nrb * 32 / 64 packed-row groups times nkb * 32 / 64 contraction groups.
__global__ void __launch_bounds__(256) k_split_batched(const SplitTask *tasks, const int64_t *start,
                                                       int ntasks) {
  const int64_t b = blockIdx.x;
  const int t = find_task(start, ntasks, b);
  const SplitTask tk = tasks[t];
  const int64_t local = b - start[t];
  const int64_t nbx = tk.nrb / 2;
  const int64_t bx = local % nbx, by = local / nbx;
  __shared__ __attribute__((aligned(16))) double tile[kSplitTileDoubles];
  if (tk.cplx) {
    if (tk.side_b)
      split_dispatch<true, true>(tk.v, tk.code, tk.S, tk.out, tk.nrb, tk.nkb, bx, by, tile);
    else
      split_dispatch<true, false>(tk.v, tk.code, tk.S, tk.out, tk.nrb, tk.nkb, bx, by, tile);
  } else {
    split_dispatch<false, false>(tk.v, tk.code, tk.S, tk.out, tk.nrb, tk.nkb, bx, by, tile);
  }
}

// ---------------------------------------------------------------- scan + split
// Exponent scan and packing of an operand in one kernel: a block of 256 threads
// scans 16 view rows over the whole contraction and packs one 64-entry fragment
// of them, one thread per row and four packed entries, so that a wave's stores
// are contiguous. Every block of a row scans it again; that costs reads of the
// caches, but one block per row would leave the chip to a few long chains:
// bound by its launch, two loads in a row and the digits' arithmetic. Whole call
// z 32^3 S = 7 12.3 us, d 256^3 14.8 (16 entries per thread and the whole
// contraction per block: 16.1 and 19.5).
constexpr int kPrepRows = 16;

// The slices of four packed entries (complex: re, im, re, im) of view row vr: one
// word per slice, or for complex B two, X' rows 2 vr = (Re, -Im) and 2 vr + 1 =
// (Im, Re), from the same digits: with trunc-7 slices those of -Im are the
// negated ones of Im, with 8-bit slices -Im is split as it stands.
__device__ __forceinline__ uint32_t swap_pairs(uint32_t w) {
  return __builtin_amdgcn_perm(0u, w, 0x02030001u);  // bytes 1, 0, 3, 2
}

template <bool PAIR, bool B8, int SC>
__device__ __forceinline__ void emit_slices(const double (&x)[4], int e, int S, int8_t *dst, int64_t plane) {
  Sig sg[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) sg[q] = decompose(x[q], e);
  auto put = [&](int p, uint32_t a, uint32_t b) {
    int8_t *d = dst + (int64_t)(p - 1) * plane;
    *reinterpret_cast<uint32_t *>(d) = a;
    if constexpr (PAIR) *reinterpret_cast<uint32_t *>(d + 16) = b;
  };
  if constexpr (B8) {
    // the bytes of X + 0x80...80, as in split_block
    constexpr uint64_t kBias = 0x8080808080808080ull >> (8 * (8 - SC));
    uint64_t Y[4], M[2];  // M: -Im
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint64_t u = top_nbits<8 * SC - 2>(sg[q]);
      Y[q] = (sg[q].neg ? 0ull - u : u) + kBias;
      if (PAIR && (q & 1)) M[q >> 1] = (sg[q].neg ? u : 0ull - u) + kBias;
    }
#pragma unroll
    for (int p = SC; p >= 1; --p) {
      const int sh = 8 * (SC - p);
      uint32_t w = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) w |= ((uint32_t)(Y[k] >> sh) & 0xffu) << (8 * k);
      w ^= 0x80808080u;
      if constexpr (PAIR) {
        const uint32_t m = (((uint32_t)(M[0] >> sh) & 0xffu) << 8) | (((uint32_t)(M[1] >> sh) & 0xffu) << 24);
        put(p, (w & 0x00ff00ffu) | (m ^ 0x80008000u), swap_pairs(w));
      } else {
        put(p, w, 0);
      }
    }
  } else {
    uint64_t T[4];
    uint32_t neg = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (SC > 0) T[k] = top_bits<SC>(sg[k]);
      neg |= (sg[k].neg ? 0xffu : 0u) << (8 * k);
    }
    auto slice = [&](int p) {
      uint32_t w = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        uint32_t d;
        if constexpr (SC > 0)
          d = (uint32_t)(T[k] >> (kDigitBits * (SC - p))) & 127u;
        else
          d = (uint32_t)digit(Sig{sg[k].m, sg[k].sh0, false}, p);
        w |= d << (8 * k);
      }
      if constexpr (PAIR)
        put(p, neg_bytes(w, neg ^ 0xff00ff00u), swap_pairs(neg_bytes(w, neg)));
      else
        put(p, neg_bytes(w, neg), 0);
    };
    if constexpr (SC > 0) {
#pragma unroll
      for (int p = 1; p <= SC; ++p) slice(p);
    } else {
      for (int p = 1; p <= S; ++p) slice(p);
    }
  }
}

template <bool CPLX, bool SIDEB, bool B8>
__device__ __forceinline__ void prep_task(const PrepTask &tk, uint32_t block, int *red) {
  using E = typename std::conditional<CPLX, double2, double>::type;
  constexpr int NE = CPLX ? 2 : 4;  // elements per thread
  constexpr int U = 8;              // scan loads in flight per thread
  const View &v = tk.v;
  const E *X = reinterpret_cast<const E *>(v.base);
  const int tid = threadIdx.x;
  const uint32_t nfrag = (uint32_t)(tk.nkb / 2), kb = block % nfrag;
  const int64_t r0 = (int64_t)(block / nfrag) * kPrepRows;
  const int r = (tid >> 2) & 15;
  const int64_t vr = r0 + r;
  const int64_t kk = (int64_t)kb * 64 + (tid >> 6) * 16 + (tid & 3) * 4, l0 = kk / (CPLX ? 2 : 1);
  E val[NE];  // in flight during the scan
#pragma unroll
  for (int x = 0; x < NE; ++x)
    val[x] = X[(vr < v.R && l0 + x < v.L) ? vr * v.sr + (l0 + x) * v.sl : 0];
  // codes: 16 threads per row, along the rows where those are contiguous
  const bool along = v.sl == 1;
  const int sr = along ? tid >> 4 : tid & 15, sl = along ? tid & 15 : tid >> 4;
  int c = 0;
  if (r0 + sr < v.R) {
    const int64_t base = (r0 + sr) * v.sr;
    for (int64_t l = sl; l < v.L; l += 16 * U) {
      int a[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        a[u] = elem_code<CPLX>(v.base, base + (l + 16 * u < v.L ? l + 16 * u : l) * v.sl);
#pragma unroll
      for (int u = 0; u < U; ++u) c = max(c, a[u]);
    }
  }
  red[sr * 17 + sl] = c;
  __syncthreads();
  if (tid < kPrepRows) {
    c = 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) c = max(c, red[tid * 17 + u]);
    red[16 * 17 + tid] = c;
    if (kb == 0 && r0 + tid < v.R) tk.code[r0 + tid] = c;
  }
  __syncthreads();
  c = red[16 * 17 + r];
  const bool live = vr < v.R && !code_bad(c);  // rows with Inf or NaN pack zeros
  double x[4];
#pragma unroll
  for (int q = 0; q < NE; ++q) {
    const bool ok = live && l0 + q < v.L;
    if constexpr (CPLX) {
      x[2 * q] = ok ? val[q].x : 0.0;
      x[2 * q + 1] = ok ? (v.conj ? -val[q].y : val[q].y) : 0.0;
    } else {
      x[q] = ok ? val[q] : 0.0;
    }
  }
  constexpr bool PAIR = CPLX && SIDEB;
  const int e = code_exp(c);
  const int64_t plane = tk.nrb * tk.nkb * kFragBytes;
  int8_t *dst = tk.out + frag_offset(0, PAIR ? 2 * vr : vr, kk, tk.nrb, tk.nkb);
  switch (tk.S) {
#define OZ_EMIT(N) \
  case N: emit_slices<PAIR, B8, N>(x, e, N, dst, plane); break;
    OZ_EMIT(1) OZ_EMIT(2) OZ_EMIT(3) OZ_EMIT(4) OZ_EMIT(5) OZ_EMIT(6) OZ_EMIT(7) OZ_EMIT(8)
    default:
      if constexpr (!B8) {
        if (tk.S == 9)
          emit_slices<PAIR, B8, 9>(x, e, 9, dst, plane);
        else
          emit_slices<PAIR, B8, 0>(x, e, tk.S, dst, plane);
      }
      break;
#undef OZ_EMIT
  }
}

template <bool CPLX, bool B8>
__global__ void __launch_bounds__(256) k_prep(PrepTask a, PrepTask b, int64_t blocks_a) {
  __shared__ int red[kPrepRows * 17 + kPrepRows];
  const uint32_t blk = blockIdx.x, na = (uint32_t)blocks_a;
  if (blk < na)
    prep_task<CPLX, false, B8>(a, blk, red);
  else
    prep_task<CPLX, true, B8>(b, blk - na, red);
}

template <bool CPLX, bool SIDEB>
__global__ void __launch_bounds__(256) k_unpack(const int8_t *packed, int64_t R, int64_t L, int S,
                                                int64_t nrb, int64_t nkb, int8_t *digits) {
  const int cc = CPLX ? 2 : 1;
  const int64_t total = (int64_t)S * R * L * cc;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int part = (int)(idx % cc);
  int64_t rest = idx / cc;
  const int64_t l = rest % L;
  rest /= L;
  const int64_t r = rest % R;
  const int p = (int)(rest / R);
  int val;
  if (!CPLX) {
    val = packed[frag_offset(p, r, l, nrb, nkb)];
  } else if (!SIDEB) {
    val = packed[frag_offset(p, r, 2 * l + part, nrb, nkb)];
  } else {
    // row 2j holds (Re, -Im), row 2j+1 (Im, Re): the Re and Im digits are the
    // even entries of the two rows
    val = packed[frag_offset(p, 2 * r + part, 2 * l, nrb, nkb)];
  }
  digits[idx] = (int8_t)val;
}

__global__ void __launch_bounds__(256) k_codes(const int *code, int64_t R, int32_t *exps,
                                               uint8_t *flags) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= R) return;
  const int c = code[r];
  exps[r] = code_exp(c);
  flags[r] = code_bad(c) ? 1 : 0;
}

template <bool CPLX>
__global__ void __launch_bounds__(256) k_scale(int64_t m, int64_t n, double br, double bi,
                                               int beta_zero, void *C, int64_t ldc) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= m * n) return;
  const int64_t i = idx % m, j = idx / m;
  if (CPLX) {
    double2 *c = reinterpret_cast<double2 *>(C) + i + j * ldc;
    if (beta_zero) {
      *c = make_double2(0.0, 0.0);
    } else {
      const double2 z = *c;
      *c = make_double2(sub_rn(mul_rn(br, z.x), mul_rn(bi, z.y)), add_rn(mul_rn(br, z.y), mul_rn(bi, z.x)));
    }
  } else {
    double *c = reinterpret_cast<double *>(C) + i + j * ldc;
    *c = beta_zero ? 0.0 : mul_rn(br, *c);
  }
}

inline unsigned grid1(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_fill_i32(int *p, int64_t n, int value, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3(grid1(n)), dim3(256), 0, st, p, n, value);
  return hipGetLastError();
}

hipError_t launch_fill_digits(int8_t *p, int64_t n, uint64_t seed, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_digits, dim3((unsigned)std::min<int64_t>(grid1(n), 1 << 20)), dim3(256),
                     0, st, p, n, seed);
  return hipGetLastError();
}

namespace {
// Row groups and contraction chunks of one operand: about 2048 blocks.
ScanSide scan_side(const View &v, int *code, int64_t *blocks) {
  ScanSide s{v, code, 1, v.L, 0};
  *blocks = 0;
  if (v.R <= 0 || v.L <= 0) return s;
  const int64_t target = 2048;
  s.rows_fast = v.sr == 1 && !(v.sl == 1 && v.R < 64);
  // otherwise sl == 1 (each row contiguous): one of the two strides of a BLAS
  // operand is always 1
  const int64_t rows = s.rows_fast ? 64 : 4, depth = s.rows_fast ? 16 : 256;
  s.nr = (v.R + rows - 1) / rows;
  const int64_t ncol = std::max<int64_t>(
      1, std::min<int64_t>((v.L + depth - 1) / depth, std::max<int64_t>(1, target / s.nr)));
  s.lchunk = (v.L + ncol - 1) / ncol;
  *blocks = s.nr * ((v.L + s.lchunk - 1) / s.lchunk);
  return s;
}
}  // namespace

hipError_t launch_scan(const View &va, int *ca, const View &vb, int *cb, bool cplx, hipStream_t st) {
  int64_t na = 0, nb = 0;
  const ScanSide a = scan_side(va, ca, &na), b = scan_side(vb, cb, &nb);
  auto go = [&](const ScanSide &x, const ScanSide &y, int64_t nx, int64_t ny) {
    if (nx + ny == 0) return;
    const dim3 g((unsigned)(nx + ny));
    if (cplx)
      hipLaunchKernelGGL(k_scan<true>, g, dim3(256), 0, st, x, y, nx);
    else
      hipLaunchKernelGGL(k_scan<false>, g, dim3(256), 0, st, x, y, nx);
  };
  if (na + nb <= kMaxBlocks) {
    go(a, b, na, nb);
  } else {
    go(a, a, na, 0);
    go(b, b, nb, 0);
  }
  return hipGetLastError();
}

namespace {
template <bool B8>
void split_launch(const View &v, bool cplx, bool side_b, const int *code, int S, int8_t *out,
                  int64_t nrb, int64_t nkb, dim3 g, hipStream_t st) {
#define OZ_SPLIT_LAUNCH(C, B, T) \
  hipLaunchKernelGGL((k_split<C, B, T, B8>), g, dim3(256), 0, st, v, code, S, out, nrb, nkb)
  const bool staged = split_staged(v);
  if (cplx && side_b) {
    if (staged) OZ_SPLIT_LAUNCH(true, true, true); else OZ_SPLIT_LAUNCH(true, true, false);
  } else if (cplx) {
    if (staged) OZ_SPLIT_LAUNCH(true, false, true); else OZ_SPLIT_LAUNCH(true, false, false);
  } else {
    if (staged) OZ_SPLIT_LAUNCH(false, false, true); else OZ_SPLIT_LAUNCH(false, false, false);
  }
#undef OZ_SPLIT_LAUNCH
}
}  // namespace

hipError_t launch_split(const View &v, bool cplx, bool side_b, const int *code, int S, int8_t *out,
                        int64_t nrb, int64_t nkb, hipStream_t st, bool b8) {
  // nrb * 32 is a multiple of 64 (rows padded to 128) and nkb * 32 a multiple
  // of 64 (contraction padded to 64): the grid covers the buffer exactly.
  if (b8 && (S < 1 || S > kS8Max)) return hipErrorInvalidValue;
  dim3 g((unsigned)(nrb * 32 / 64), (unsigned)(nkb * 32 / 64));
  if (b8)
    split_launch<true>(v, cplx, side_b, code, S, out, nrb, nkb, g, st);
  else
    split_launch<false>(v, cplx, side_b, code, S, out, nrb, nkb, g, st);
  return hipGetLastError();
}

hipError_t launch_split(const View &va, const int *ca, int8_t *oa, int64_t nrba, const View &vb,
                        const int *cb, int8_t *ob, int64_t nrbb, int64_t nkb, bool cplx, int S,
                        hipStream_t st, bool b8) {
  if (b8 && (S < 1 || S > kS8Max)) return hipErrorInvalidValue;
  const int64_t na = (nrba / 2) * (nkb / 2), nb = (nrbb / 2) * (nkb / 2);
  if (na + nb > kMaxBlocks) {
    const hipError_t e = launch_split(va, cplx, false, ca, S, oa, nrba, nkb, st, b8);
    return e != hipSuccess ? e : launch_split(vb, cplx, true, cb, S, ob, nrbb, nkb, st, b8);
  }
  const SplitSide a{va, ca, oa, nrba, nkb}, b{vb, cb, ob, nrbb, nkb};
  const dim3 g((unsigned)(na + nb));
#define OZ_SPLIT_PAIR(C, B) hipLaunchKernelGGL((k_split_pair<C, B>), g, dim3(256), 0, st, a, b, na, S)
  if (cplx) {
    if (b8) OZ_SPLIT_PAIR(true, true); else OZ_SPLIT_PAIR(true, false);
  } else {
    if (b8) OZ_SPLIT_PAIR(false, true); else OZ_SPLIT_PAIR(false, false);
  }
#undef OZ_SPLIT_PAIR
  return hipGetLastError();
}

hipError_t launch_unpack(const int8_t *packed, bool cplx, bool side_b, int64_t R, int64_t L, int S,
                         int64_t nrb, int64_t nkb, int8_t *digits, hipStream_t st) {
  const int64_t total = (int64_t)S * R * L * (cplx ? 2 : 1);
  if (total <= 0) return hipSuccess;
  dim3 g(grid1(total));
  if (cplx) {
    if (side_b)
      hipLaunchKernelGGL((k_unpack<true, true>), g, dim3(256), 0, st, packed, R, L, S, nrb, nkb, digits);
    else
      hipLaunchKernelGGL((k_unpack<true, false>), g, dim3(256), 0, st, packed, R, L, S, nrb, nkb, digits);
  } else {
    hipLaunchKernelGGL((k_unpack<false, false>), g, dim3(256), 0, st, packed, R, L, S, nrb, nkb, digits);
  }
  return hipGetLastError();
}

hipError_t launch_codes_to_exps(const int *code, int64_t R, int32_t *exps, uint8_t *flags,
                                hipStream_t st) {
  if (R <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_codes, dim3(grid1(R)), dim3(256), 0, st, code, R, exps, flags);
  return hipGetLastError();
}

int64_t scan_task_blocks(const ScanTask &t) {
  return t.rows_fast ? (t.v.R + 63) / 64 : (t.v.R + 3) / 4;
}

int64_t split_task_blocks(const SplitTask &t) { return (t.nrb / 2) * (t.nkb / 2); }

hipError_t launch_scan_batched(const ScanTask *tasks, const int64_t *start, int ntasks,
                               int64_t nblocks, hipStream_t st) {
  if (ntasks <= 0 || nblocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scan_batched, dim3((unsigned)nblocks), dim3(256), 0, st, tasks, start, ntasks);
  return hipGetLastError();
}

hipError_t launch_split_batched(const SplitTask *tasks, const int64_t *start, int ntasks,
                                int64_t nblocks, hipStream_t st) {
  if (ntasks <= 0 || nblocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_split_batched, dim3((unsigned)nblocks), dim3(256), 0, st, tasks, start, ntasks);
  return hipGetLastError();
}

namespace {
int64_t prep_task_blocks(const PrepTask &t) {
  return t.nrb * ((t.cplx && t.side_b) ? 16 : 32) / kPrepRows * (t.nkb / 2);
}
}  // namespace

bool prep_fits(const PrepTask &a, const PrepTask &b) {
  const int64_t kpad = a.nkb * 32, blocks = prep_task_blocks(a) + prep_task_blocks(b);
  if (kpad <= 64 || (kpad <= 128 && !a.cplx) || (kpad <= 256 && a.S >= 10)) return blocks <= kMaxBlocks;
  return kpad <= 512 && blocks <= (kpad <= 128 ? 4096 : kpad <= 256 ? 1536 : 1024);
}

hipError_t launch_prep(const PrepTask &a, const PrepTask &b, hipStream_t st, bool b8) {
  if (b8 && (a.S < 1 || a.S > kS8Max)) return hipErrorInvalidValue;
  const int64_t na = prep_task_blocks(a), nb = prep_task_blocks(b);
  const dim3 g((unsigned)(na + nb));
  if (a.cplx) {
    if (b8)
      hipLaunchKernelGGL((k_prep<true, true>), g, dim3(256), 0, st, a, b, na);
    else
      hipLaunchKernelGGL((k_prep<true, false>), g, dim3(256), 0, st, a, b, na);
  } else {
    if (b8)
      hipLaunchKernelGGL((k_prep<false, true>), g, dim3(256), 0, st, a, b, na);
    else
      hipLaunchKernelGGL((k_prep<false, false>), g, dim3(256), 0, st, a, b, na);
  }
  return hipGetLastError();
}

hipError_t launch_scale(bool cplx, int64_t m, int64_t n, double br, double bi, bool beta_zero,
                        void *C, int64_t ldc, hipStream_t st) {
  if (m <= 0 || n <= 0) return hipSuccess;
  dim3 g(grid1(m * n));
  if (cplx)
    hipLaunchKernelGGL(k_scale<true>, g, dim3(256), 0, st, m, n, br, bi, (int)beta_zero, C, ldc);
  else
    hipLaunchKernelGGL(k_scale<false>, g, dim3(256), 0, st, m, n, br, bi, (int)beta_zero, C, ldc);
  return hipGetLastError();
}

}  // namespace oz
