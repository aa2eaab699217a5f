// The operand tile of the kernels that write packed operands (slices in
// ozaki_prep.hip, residues in ozaki2.hip): its size and its copy into LDS.
#pragma once

#include <type_traits>

#include "ozaki_internal.hpp"

namespace oz {

// View rows and contraction entries (elements) covered by one split block.
template <bool CPLX, bool SIDEB>
struct SplitTile {
  static constexpr int TR = (CPLX && SIDEB) ? 32 : 64;  // view rows
  static constexpr int TL = CPLX ? 32 : 64;              // contraction elements
  static constexpr int EW = CPLX ? 2 : 1;                // doubles per element
  static constexpr int PITCH = (TL + 1) * EW;            // doubles per LDS row (padded)
};
constexpr int kSplitTileDoubles = 64 * 33 * 2;  // the largest tile (complex, 64 rows)

// When the contraction is the unit-stride direction (sl == 1) a thread's 16
// packed entries lie along one row in memory, and the lanes of a wave would
// read 64 different rows. The block then first copies its tile into LDS with
// consecutive threads on consecutive elements of a row (coalesced), and the
// threads take their values from there. Rows or elements outside the view
// are stored as zeros.
// Every load is issued before the first store to LDS (an element outside the
// view reads element (0, 0) and is stored as zero), so a thread's loads are in
// flight together.
template <bool CPLX, bool SIDEB>
__device__ __forceinline__ void load_split_tile(const View &v, int64_t bx, int64_t by, double *tile) {
  using T = SplitTile<CPLX, SIDEB>;
  using E = typename std::conditional<CPLX, double2, double>::type;
  constexpr int IT = T::TR * T::TL / 256;
  static_assert(T::TR * T::TL % 256 == 0, "whole passes");
  const int64_t r0 = bx * T::TR, l0 = by * T::TL;
  E val[IT];
  bool in[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int c = threadIdx.x + 256 * it;
    const int64_t r = r0 + c / T::TL, l = l0 + c % T::TL;
    in[it] = r < v.R && l < v.L;
    val[it] = reinterpret_cast<const E *>(v.base)[in[it] ? r * v.sr + l : 0];
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int c = threadIdx.x + 256 * it;
    const int rr = c / T::TL, ll = c % T::TL;
    if constexpr (CPLX)
      *reinterpret_cast<double2 *>(tile + rr * T::PITCH + ll * 2) =
          in[it] ? val[it] : make_double2(0.0, 0.0);
    else
      tile[rr * T::PITCH + ll] = in[it] ? val[it] : 0.0;
  }
  __syncthreads();
}

// The LDS-staged form is taken when the contraction is unit-stride and the
// rows are not (the choice is uniform over the block) and the caller provides
// the LDS tile.
__host__ __device__ __forceinline__ bool split_staged(const View &v) {
  return v.sl == 1 && v.sr != 1;
}

// ---------------------------------------------------------------- whole rows
// Exponent scan and packing of an operand in one kernel: a block of 256 threads
// takes 16 view rows over the whole contraction, first their exponent codes,
// then (the second read comes from the caches) their packed entries, one thread
// per row and 16 packed entries at a time, so a wave writes whole 1 KiB
// fragments. emit(x, e, vr, ch): the thread's 16 values x (complex: re, im
// interleaved; zeros outside the view and in rows that hold Inf or NaN), the row
// exponent e, the view row and the number of the 16-entry chunk.
constexpr int kRowsBlock = 16;
constexpr int kRowsTileElems = 128;  // complex elements per row and pass (256 real ones)
struct RowsLds {
  __attribute__((aligned(16))) double tile[kRowsBlock * (2 * kRowsTileElems + 2)];
  int sc[kRowsBlock], red[64];
};

template <bool CPLX>
__device__ __forceinline__ int entry_code(const void *base, int64_t off) {
  if constexpr (CPLX) {
    const double2 z = reinterpret_cast<const double2 *>(base)[off];
    return max(expo_code(z.x), expo_code(z.y));
  }
  return expo_code(reinterpret_cast<const double *>(base)[off]);
}

// Codes of the view rows r0 .. r0 + 15 into sc (LDS) and code (rows of the view).
template <bool CPLX>
__device__ __forceinline__ void rows_codes(const View &v, int64_t r0, int *code, int *sc, int *red) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int U = 8;  // loads in flight per thread
  if (v.sl == 1) {
    // each row unit-stride: one wave per row
    for (int rr = wave; rr < kRowsBlock; rr += 4) {
      const int64_t r = r0 + rr;
      int c = 0;
      if (r < v.R) {
        int64_t l = lane;
        for (; l + 64 * (U - 1) < v.L; l += 64 * U) {
          int a[U];
#pragma unroll
          for (int u = 0; u < U; ++u) a[u] = entry_code<CPLX>(v.base, r * v.sr + l + 64 * u);
#pragma unroll
          for (int u = 0; u < U; ++u) c = max(c, a[u]);
        }
        for (; l < v.L; l += 64) c = max(c, entry_code<CPLX>(v.base, r * v.sr + l));
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) c = max(c, __shfl_xor(c, off));
      if (lane == 0) sc[rr] = c;
    }
  } else {
    // rows unit-stride: 16 rows side by side, 16 threads along the contraction
    const int64_t r = r0 + (tid & 15);
    int c = 0;
    if (r < v.R) {
      int64_t l = tid >> 4;
      for (; l + 16 * (U - 1) < v.L; l += 16 * U) {
        int a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = entry_code<CPLX>(v.base, r * v.sr + (l + 16 * u) * v.sl);
#pragma unroll
        for (int u = 0; u < U; ++u) c = max(c, a[u]);
      }
      for (; l < v.L; l += 16) c = max(c, entry_code<CPLX>(v.base, r * v.sr + l * v.sl));
    }
    c = max(c, __shfl_xor(c, 16));
    c = max(c, __shfl_xor(c, 32));
    if (lane < 16) red[wave * 16 + lane] = c;
    __syncthreads();
    if (tid < 16) sc[tid] = max(max(red[tid], red[16 + tid]), max(red[32 + tid], red[48 + tid]));
  }
  __syncthreads();
  if (tid < kRowsBlock && r0 + tid < v.R) code[r0 + tid] = sc[tid];
}

template <bool CPLX, typename Emit>
__device__ __forceinline__ void pack_rows(const View &v, int64_t block, int64_t nch, int *code, RowsLds &lds,
                                          Emit emit) {
  using E = typename std::conditional<CPLX, double2, double>::type;
  constexpr int NE = CPLX ? 8 : 16;         // elements per thread and pass
  constexpr int TE = 16 * NE;               // elements per row and pass
  constexpr int PITCH = TE * (CPLX ? 2 : 1) + 2;  // doubles per LDS row
  double *tile = lds.tile;
  int *sc = lds.sc;
  const int tid = threadIdx.x;
  const int64_t r0 = block * kRowsBlock;
  const bool staged = v.sl == 1;
  if (r0 < v.R) {
    rows_codes<CPLX>(v, r0, code, sc, lds.red);
  } else {
    if (tid < kRowsBlock) sc[tid] = 0;
    __syncthreads();
  }
  const int64_t vr = r0 + (tid & 15);
  const int c = sc[tid & 15];
  const bool live = vr < v.R && !code_bad(c);
  const int e = code_exp(c);
  for (int64_t ch0 = 0; ch0 < nch; ch0 += 16) {
    const int64_t ch = ch0 + (tid >> 4);
    E val[NE];
    if (staged) {
      // coalesced along each row through LDS; every load before the first store
      E ld[NE];
      const int64_t l0 = ch0 * NE;
#pragma unroll
      for (int it = 0; it < NE; ++it) {
        const int x = tid + 256 * it;
        const int64_t r = r0 + x / TE, l = l0 + x % TE;
        ld[it] = reinterpret_cast<const E *>(v.base)[(r < v.R && l < v.L) ? r * v.sr + l : 0];
      }
      __syncthreads();  // the previous pass has been read
#pragma unroll
      for (int it = 0; it < NE; ++it) {
        const int x = tid + 256 * it;
        *reinterpret_cast<E *>(tile + (x / TE) * PITCH + (x % TE) * (CPLX ? 2 : 1)) = ld[it];
      }
      __syncthreads();
#pragma unroll
      for (int x = 0; x < NE; ++x)
        val[x] = *reinterpret_cast<const E *>(tile + (tid & 15) * PITCH +
                                              ((tid >> 4) * NE + x) * (CPLX ? 2 : 1));
    } else {
#pragma unroll
      for (int x = 0; x < NE; ++x) {
        const int64_t l = ch * NE + x;
        val[x] = reinterpret_cast<const E *>(v.base)[(vr < v.R && l < v.L) ? vr * v.sr + l * v.sl : 0];
      }
    }
    double x[16];
#pragma unroll
    for (int q = 0; q < NE; ++q) {
      const bool ok = live && ch * NE + q < v.L;
      if constexpr (CPLX) {
        x[2 * q] = ok ? val[q].x : 0.0;
        x[2 * q + 1] = ok ? (v.conj ? -val[q].y : val[q].y) : 0.0;
      } else {
        x[q] = ok ? val[q] : 0.0;
      }
    }
    if (ch < nch) emit(x, e, vr, ch);
  }
}

}  // namespace oz
