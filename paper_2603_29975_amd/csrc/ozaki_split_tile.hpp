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

}  // namespace oz
