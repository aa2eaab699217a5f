// Pieces shared by the INT8 GEMM kernels of libozaki (gfx950): explicit
// wait/barrier primitives, direct-to-LDS copies, the INT32 chunk bound, the
// FP64 epilogue of one block and the tile orders.
//
// Accumulator layout of v_mfma_i32_16x16x64_i8 as used here: the MFMA row index
// is the output column side j', the MFMA column index (lane % 16) is the output
// row i. Register r of a lane holds j' = 16 * block + 4 * (lane / 16) + r.
#pragma once

#include "ozaki_internal.hpp"

namespace oz {
namespace tile {

// Wait until at most N vector-memory operations of this wave are in flight.
// Inline assembly with a memory clobber: the compiler neither moves memory
// accesses across it nor adds a drain of the LDS copies still in flight.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void barrier_only() { asm volatile("s_barrier" ::: "memory"); }

// One 1 KiB fragment from global memory straight into LDS: lane l copies 16
// bytes to LDS address lds_wave + 16 l, from its own address (copy_frag) or from
// base + off_lane (copy_frag_s: the wave-uniform base stays in scalar
// registers). Inline assembly rather than the compiler's builtin for the same
// instruction: with the builtin in a loop the compiler waits for every
// outstanding LDS read (lgkmcnt(0)) before each fragment's first use, which
// serialises the fragment reads with the MFMAs; with the copy hidden from it, it
// waits for exactly the reads each MFMA needs. The copy counts in vmcnt, which
// the kernels wait on explicitly (wait_vmcnt); the LDS base goes through M0, set
// in the same statement.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ uint32_t lds_addr(const int8_t *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) int8_t *)p;
}
__device__ __forceinline__ v4i lds_read(uint32_t addr) {
  return *(const __attribute__((address_space(3))) v4i *)(uintptr_t)addr;
}
__device__ __forceinline__ void copy_frag(const int8_t *src_lane, const int8_t *lds_wave) {
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src_lane),
               "s"(lds_addr(lds_wave))
               : "memory", "m0");
}
__device__ __forceinline__ void copy_frag_s(const int8_t *base, uint32_t off_lane, const int8_t *lds_wave) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off_lane), "s"(base),
               "s"(lds_addr(lds_wave))
               : "memory", "m0");
}
#pragma clang diagnostic pop

// Contraction blocks of 32 a chunk may hold: S * 32 * kb * dmax^2 <= 2^31 - 1
// with dmax = 127 (trunc-7 digits) or 128 (8-bit balanced digits).
__host__ __device__ constexpr int64_t chunk_blocks(int S, int dmax = 127) {
  return (int64_t)(2147483647ll / ((int64_t)S * 32 * dmax * dmax));
}

// Stores of one 16 x 16 block: lane register r is column side j' = j0 + r of row
// i. a: the problem (any address space).

// The exact diagonals, total(t, r) being diagonal t + 2 of register r.
template <int S, typename Problem, typename Total>
__device__ __forceinline__ void store_raw(Problem a, Total total, int64_t i, int64_t j0) {
  if (i >= a->m) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t jp = j0 + r;
    if (jp >= a->nprime) continue;
#pragma unroll
    for (int t = 0; t < S; ++t) {
      const int64_t v = total(t, r);
      if (a->cplx) {
        const int64_t n = a->nprime >> 1;
        a->raw[(((int64_t)t * n + (jp >> 1)) * a->m + i) * 2 + (jp & 1)] = v;
      } else {
        a->raw[((int64_t)t * a->nprime + jp) * a->m + i] = v;
      }
    }
  }
}

// The recombined sums val[r] times 2^(e_i + f_j) and alpha/beta without fused
// multiply-adds; rows or columns flagged non-finite give NaN.
template <typename Problem>
__device__ __forceinline__ void store_block(Problem a, const double (&val)[4], int64_t i, int64_t j0) {
  if (i >= a->m) return;
  const int codeA = a->codeA[i];
  const int ea = code_exp(codeA);
  const bool bad_i = code_bad(codeA);
  const int *codeB = a->codeB;
  const int64_t ldc = a->ldc;
  const double ar = a->ar, ai = a->ai, br = a->br, bi = a->bi;
  const int beta_zero = a->beta_zero;
  // the recombined sums as they are (NaN for non-finite rows/columns): a later
  // diagonal adds to them exactly as the recombination would have
  const int unscaled = a->unscaled;
  if (a->cplx) {
    double2 *C = reinterpret_cast<double2 *>(a->C);
    const int64_t n = a->nprime >> 1;
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
      const int64_t j = (j0 + r) >> 1;
      if (j >= n) continue;
      const int cb = codeB[j];
      double2 *cp = C + i + j * ldc;
      if (bad_i || code_bad(cb)) {
        *cp = make_double2(qnan(), qnan());
        continue;
      }
      if (unscaled) {
        *cp = make_double2(val[r], val[r + 1]);
        continue;
      }
      const int sc = ea + code_exp(cb);
      const double pr = ldexp(val[r], sc);
      const double pi = ldexp(val[r + 1], sc);
      double re = sub_rn(mul_rn(ar, pr), mul_rn(ai, pi));
      double im = add_rn(mul_rn(ar, pi), mul_rn(ai, pr));
      if (!beta_zero) {
        const double2 z = *cp;
        re = add_rn(re, sub_rn(mul_rn(br, z.x), mul_rn(bi, z.y)));
        im = add_rn(im, add_rn(mul_rn(br, z.y), mul_rn(bi, z.x)));
      }
      *cp = make_double2(re, im);
    }
  } else {
    double *C = reinterpret_cast<double *>(a->C);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t j = j0 + r;
      if (j >= a->nprime) continue;
      const int cb = codeB[j];
      double *cp = C + i + j * ldc;
      if (bad_i || code_bad(cb)) {
        *cp = qnan();
        continue;
      }
      if (unscaled) {
        *cp = val[r];
        continue;
      }
      const double p = ldexp(val[r], ea + code_exp(cb));
      double out = mul_rn(ar, p);
      if (!beta_zero) out = add_rn(out, mul_rn(br, *cp));
      *cp = out;
    }
  }
}

// Order 3: workgroup w of a persistent grid runs on XCD w % 8 (workgroups are
// dealt to the 8 XCDs round-robin), and each XCD has its own L2. Within each
// full round of gridDim.x tiles, tile number tn is given to slot w of the
// round as xcd_major(tn): the tiles of one XCD's workgroups are consecutive
// in the grouped order (8 tile rows per group), so they share 8 A' stripes
// and few B' stripes in that XCD's L2 instead of every XCD fetching all the
// stripes of the round. A partial last round keeps the identity.
__device__ __forceinline__ int64_t xcd_major(int64_t tn, int64_t ntiles) {
  const int64_t G = gridDim.x;
  if ((G & 7) != 0) return tn;
  const int64_t r0 = tn - tn % G;
  if (r0 + G > ntiles) return tn;
  const int64_t w = tn - r0;
  return r0 + (w & 7) * (G >> 3) + (w >> 3);
}

// Output tile (tj, ti) of tile number `local` in a grid of tiles BJ x BI:
// order 0 walks down the rows i first, order 1 along the columns j' first,
// order 2 in groups of 16 tile rows, down the rows of a group first (the
// tiles in flight at once then share 16 A' stripes and few B' stripes, which
// keeps long contractions in the caches instead of streaming every B' stripe
// once per round); order 3 in groups of 8 tile rows (after xcd_major).
__device__ __forceinline__ void tile_coords(int64_t local, int order, int64_t m, int64_t nprime,
                                            int BJ, int BI, int64_t &tj, int64_t &ti) {
  const int64_t nti = (m + BI - 1) / BI;
  if (order == 0) {
    tj = local / nti;
    ti = local % nti;
  } else if (order == 1) {
    const int64_t ntj = (nprime + BJ - 1) / BJ;
    ti = local / ntj;
    tj = local % ntj;
  } else {
    const int64_t kGroup = order == 2 ? 16 : 8;
    const int64_t ntj = (nprime + BJ - 1) / BJ;
    const int64_t g = local / (kGroup * ntj), r = local - g * (kGroup * ntj);
    const int64_t gh = nti - g * kGroup < kGroup ? nti - g * kGroup : kGroup;
    ti = g * kGroup + r % gh;
    tj = r / gh;
  }
}

}  // namespace tile
}  // namespace oz
