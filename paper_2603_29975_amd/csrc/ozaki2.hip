// Ozaki-II emulation of FP64 and complex-FP64 GEMM (Section 2.2 of the
// paper): both operands are scaled to integer matrices, each integer product
// is formed modulo N pairwise-coprime moduli as N exact INT8 x INT8 -> INT32
// matrix products, and the Chinese remainder theorem rebuilds the exact
// integer product, which is rounded once to FP64 and scaled back. Section 3
// runs it with 10..18 moduli.
//
// Rules of this library (listed with the C ABI in include/ozaki.h):
//   moduli     the N largest pairwise-coprime integers <= 256, taken greedily
//              from 256 downwards; a residue is the representative of x mod m
//              in [-floor(m/2), ceil(m/2) - 1], which fits INT8.
//   integers   A'_il = trunc(a_il 2^(beta - e_i)), B'_lj = trunc(b_lj 2^(beta -
//              f_j)), with e_i, f_j the frexp exponents of the row/column
//              maxima (the exponent scan of the Ozaki-I path) and beta =
//              min(63, floor((floor(log2 M) - 1 - ceil(log2 K')) / 2)) for
//              M = m_1 ... m_N; |A'B'| < K' 2^(2 beta) <= M/2.
//   products   C_k = (A' mod m_k)(B' mod m_k) in INT32: exact for K' <= 2^17
//              (|r| <= 127 for the odd moduli); for m = 256 the INT32
//              wrap-around keeps the value mod 256.
//   rebuild    the unique c in [-M/2, M/2) with c = C_k mod m_k (mixed-radix
//              digits, balanced), then P = RN(c) 2^(e_i + f_j - 2 beta) and
//              alpha/beta, non-finite rows/columns as NaN, exactly as the
//              Ozaki-I epilogue.
// Complex data is one real product with the contraction interleaved (K' = 2k):
// A' rows (Re, Im), B' rows 2j = (Re, -Im) and 2j+1 = (Im, Re) of column j.
#include "ozaki2_crt.hpp"
#include "ozaki_split_tile.hpp"

namespace oz {
namespace crt {

// ---------------------------------------------------------------- residues
// What the residue of modulus k needs: m_k, 1 / m_k, the residues of 256^b mod
// m_k, b = 0..7, as the bytes of two words (balanced and in [0, m_k)), and
// -2^64 mod m_k.
struct ResConst {
  float rm, fm;
  int w0, w1;
  unsigned u0, u1;
  int c64;
};
struct ResTable {
  ResConst c[kModMax];
};
constexpr ResTable make_res_table() {
  ResTable t{};
  for (int k = 0; k < kModMax; ++k) {
    const int m = kT.m[k];
    t.c[k].rm = 1.0f / (float)m;
    t.c[k].fm = (float)m;
    unsigned w[2] = {0, 0}, u[2] = {0, 0};
    int x = bal_c(1, m);
    for (int b = 0; b < 8; ++b) {
      w[b >> 2] |= (unsigned)(x & 0xff) << (8 * (b & 3));
      u[b >> 2] |= (unsigned)(x < 0 ? x + m : x) << (8 * (b & 3));
      x = bal_c(x * 256, m);
    }
    t.c[k].w0 = (int)w[0];
    t.c[k].w1 = (int)w[1];
    t.c[k].u0 = u[0];
    t.c[k].u1 = u[1];
    t.c[k].c64 = x <= 0 ? -x : m - x;
  }
  return t;
}
__constant__ ResTable kRes = make_res_table();

// X = trunc(x 2^(beta - e)) as eight base-256 digits, byte b the digit of 256^b.
// beta <= 62: signed digits; |X| < 2^62, so X + 0x80...80 lies in (0, 2^64) and
// its bytes less 128 are the digits. BIG (beta = 63, |X| < 2^63, which signed
// digits do not cover): the plain bytes of X modulo 2^64.
template <bool BIG>
__device__ __forceinline__ uint64_t digit_bytes(double x, int e, int beta) {
  const Sig s = decompose(x, e);
  const int sh = s.sh0 + beta;
  uint64_t u;
  if (sh >= 0)
    u = s.m << sh;  // |x| < 2^e: the result stays below 2^beta
  else
    u = sh > -64 ? (s.m >> (-sh)) : 0ull;
  if (s.neg) u = 0ull - u;
  return BIG ? u : (u + 0x8080808080808080ull) ^ 0x8080808080808080ull;
}

// Four residues of modulus k plus 128 as the bytes of a word. Two 4-way INT8
// dot products of digits and weights give |t| <= 8 * 128 * 127 < 2^17 (BIG: 0
// <= t < 2^20) congruent to X, for which one FP32 quotient is exact (see
// bal_mod); t carries + 128, so the remainder is an unsigned byte that one
// conversion packs. m_0 = 256: the residue is the lowest digit.
template <bool BIG>
__device__ __forceinline__ uint32_t residue_word(const ResConst &rc, bool first, const uint64_t *z) {
  uint32_t out = 0;
  if (first) {
#pragma unroll
    for (int b = 0; b < 4; ++b) out |= (uint32_t)(z[b] & 0xff) << (8 * b);
    return out ^ 0x80808080u;
  }
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int lo = (int)z[b], hi = (int)(z[b] >> 32);
    int t;
    if constexpr (BIG)
      t = (int)__builtin_amdgcn_udot4(
          (unsigned)hi, rc.u1,
          __builtin_amdgcn_udot4((unsigned)lo, rc.u0, 128u + (unsigned)((hi >> 31) & rc.c64), false), false);
    else
      t = __builtin_amdgcn_sdot4(hi, rc.w1, __builtin_amdgcn_sdot4(lo, rc.w0, 128, false), false);
    const float tf = (float)t;
    const float q = __builtin_rintf(__builtin_fmaf(tf, rc.rm, -128.0f * rc.rm));
    out = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_fmaf(-q, rc.fm, tf), b, out);
  }
  return out;
}

// The bytes 256 - b of the odd bytes (the residues negated; 256: modulo 256).
__device__ __forceinline__ uint32_t neg_odd(uint32_t w) {
  const uint32_t odd = (0x01000100u - ((w >> 8) & 0x00ff00ffu)) & 0x00ff00ffu;
  return (w & 0x00ff00ffu) | (odd << 8);
}

// One thread per view row and 16 consecutive packed contraction entries (8
// complex elements), as in the split: it reads its values once, keeps their
// digits in registers and writes one 16-byte run per modulus (complex B: one
// per X' row, 2j = (Re, -Im) and 2j + 1 = (Im, Re), from the same residues).
// What bounds it is the arithmetic, about 8 operations per entry and modulus
// (two dot products, conversion, quotient, remainder, packing; 13-bit pieces
// with 24-bit products took 15), and the writes: 2048^3 complex, 14 moduli, A
// 40 us and B 74 us (2.9 and 3.2 TB/s written), before 57 and 77; both operands
// share a launch, which a small product gains most from (z 64^3, whole call, 21.5
// us). Rows and entries beyond the operand give zero residues.
struct ResSide {
  View v;
  int *code;
  int8_t *out;
  int64_t nrb;
};

// Codes of the block's 64 view rows into sc (and, from one block per row group,
// into code): 16 threads per row, along the rows where those are contiguous.
template <bool CPLX>
__device__ __forceinline__ void scan_rows(const ResSide &s, int64_t bx, bool store, int *red, int *sc) {
  const View &v = s.v;
  const int tid = threadIdx.x;
  const int sr = v.sl == 1 ? tid >> 4 : tid & 15, sl = v.sl == 1 ? tid & 15 : tid >> 4;
  int c[4] = {0, 0, 0, 0};
  for (int64_t l = sl; l < v.L; l += 32) {
    int a[4][2];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int64_t r = bx * 64 + 16 * g + sr, ll = l + 16 * u < v.L ? l + 16 * u : l;
        const int64_t off = r < v.R ? r * v.sr + ll * v.sl : 0;
        if constexpr (CPLX) {
          const double2 z = reinterpret_cast<const double2 *>(v.base)[off];
          a[g][u] = max(expo_code(z.x), expo_code(z.y));
        } else {
          a[g][u] = expo_code(reinterpret_cast<const double *>(v.base)[off]);
        }
      }
#pragma unroll
    for (int g = 0; g < 4; ++g) c[g] = max(c[g], max(a[g][0], a[g][1]));
  }
#pragma unroll
  for (int g = 0; g < 4; ++g) red[(16 * g + sr) * 17 + sl] = c[g];
  __syncthreads();
  if (tid < 64) {
    int m = 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) m = max(m, red[tid * 17 + u]);
    sc[tid] = m;
    if (store && bx * 64 + tid < v.R) s.code[bx * 64 + tid] = m;
  }
  __syncthreads();
}

template <bool CPLX, bool SIDEB, bool STAGED, bool BIG, bool SCAN>
__device__ __forceinline__ void residues_block(const ResSide &s, int n, int beta, int64_t nkb,
                                               int64_t bx, int64_t by, double *tile, int *red) {
  using T = SplitTile<CPLX, false>;
  using E = typename std::conditional<CPLX, double2, double>::type;
  const View &v = s.v;
  int8_t *out = s.out;
  const int64_t nrb = s.nrb, plane = nrb * nkb * kFragBytes;
  if constexpr (STAGED) load_split_tile<CPLX, false>(v, bx, by, tile);
  const int tid = threadIdx.x;
  const int64_t vr = bx * 64 + (tid & 63);
  const int64_t kk = (by * 4 + (tid >> 6)) * 16;
  int c;
  if constexpr (SCAN) {
    scan_rows<CPLX>(s, bx, by == 0, red, red + 64 * 17);
    c = vr < v.R ? red[64 * 17 + (tid & 63)] : 0;
  } else {
    c = vr < v.R ? s.code[vr] : 0;
  }
  const bool live = vr < v.R && !code_bad(c);
  const int e = code_exp(c);

  uint64_t z[16];
  constexpr int NE = CPLX ? 8 : 16;  // elements per thread
  const int64_t l0 = CPLX ? kk >> 1 : kk;
  E val[NE];
#pragma unroll
  for (int x = 0; x < NE; ++x) {
    const int64_t l = l0 + x;
    if constexpr (STAGED)
      val[x] = *reinterpret_cast<const E *>(tile + (tid & 63) * T::PITCH + (l - by * T::TL) * T::EW);
    else
      val[x] = reinterpret_cast<const E *>(v.base)[(live && l < v.L) ? vr * v.sr + l * v.sl : 0];
  }
#pragma unroll
  for (int x = 0; x < NE; ++x) {
    const bool ok = live && l0 + x < v.L;
    if constexpr (CPLX) {
      z[2 * x] = digit_bytes<BIG>(ok ? val[x].x : 0.0, e, beta);
      z[2 * x + 1] = digit_bytes<BIG>(ok ? (v.conj ? -val[x].y : val[x].y) : 0.0, e, beta);
    } else {
      z[x] = digit_bytes<BIG>(ok ? val[x] : 0.0, e, beta);
    }
  }

  int8_t *dst = out + frag_offset(0, (CPLX && SIDEB) ? 2 * vr : vr, kk, nrb, nkb);
  for (int k = 0; k < n; ++k) {
    const ResConst rc = kRes.c[k];
    uint32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = residue_word<BIG>(rc, k == 0, z + 4 * q);
    int8_t *d = dst + k * plane;
    if constexpr (CPLX && SIDEB) {
      uint32_t a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[q] = neg_odd(w[q]) ^ 0x80808080u;
        b[q] = __builtin_amdgcn_perm(0u, w[q], 0x02030001u) ^ 0x80808080u;  // bytes 1, 0, 3, 2
      }
      *reinterpret_cast<uint4 *>(d) = make_uint4(a[0], a[1], a[2], a[3]);
      *reinterpret_cast<uint4 *>(d + 16) = make_uint4(b[0], b[1], b[2], b[3]);
    } else {
      *reinterpret_cast<uint4 *>(d) = make_uint4(w[0] ^ 0x80808080u, w[1] ^ 0x80808080u,
                                                 w[2] ^ 0x80808080u, w[3] ^ 0x80808080u);
    }
  }
}

// Both operands in one launch: blocks [0, na) take the first, `groups` row groups
// each. SCAN: the blocks find their rows' exponents themselves (each row group's
// blocks scan it again, out of the caches) instead of a launch before.
template <bool CPLX, bool BIG, bool SCAN>
__global__ void __launch_bounds__(256) k_residues(ResSide a, ResSide b, int64_t na, int n, int beta,
                                                  int64_t nkb) {
  using T = SplitTile<CPLX, false>;
  __shared__ __attribute__((aligned(16))) double tile[T::TR * T::PITCH];
  __shared__ int red[SCAN ? 64 * 18 : 1];
  const uint32_t first = (uint32_t)na;
  if (blockIdx.x < first) {
    const uint32_t groups = (uint32_t)(a.nrb / 2), blk = blockIdx.x;
    if (split_staged(a.v))
      residues_block<CPLX, false, true, BIG, SCAN>(a, n, beta, nkb, blk % groups, blk / groups, tile, red);
    else
      residues_block<CPLX, false, false, BIG, SCAN>(a, n, beta, nkb, blk % groups, blk / groups, tile, red);
  } else {
    const uint32_t groups = (uint32_t)(CPLX ? b.nrb / 4 : b.nrb / 2), blk = blockIdx.x - first;
    if (split_staged(b.v))
      residues_block<CPLX, true, true, BIG, SCAN>(b, n, beta, nkb, blk % groups, blk / groups, tile, red);
    else
      residues_block<CPLX, true, false, BIG, SCAN>(b, n, beta, nkb, blk % groups, blk / groups, tile, red);
  }
}

}  // namespace crt

// ---------------------------------------------------------------- host side
int crt_modulus(int k) { return (k >= 0 && k < kModMax) ? crt::kT.m[k] : 0; }

int crt_log2_floor(int n) {
  if (n < 1 || n > kModMax) return -1;
  uint32_t w[6] = {1, 0, 0, 0, 0, 0};  // little-endian 32-bit limbs of the product
  for (int k = 0; k < n; ++k) {
    uint64_t carry = 0;
    for (int t = 0; t < 6; ++t) {
      const uint64_t v = (uint64_t)w[t] * (uint64_t)crt::kT.m[k] + carry;
      w[t] = (uint32_t)v;
      carry = v >> 32;
    }
  }
  for (int t = 5; t >= 0; --t)
    if (w[t] != 0) return 32 * t + 31 - __builtin_clz(w[t]);
  return -1;
}

int crt_beta(int n, int64_t kprime) {
  const int lm = crt_log2_floor(n);
  if (lm < 0) return 0;
  int lk = 0;
  while (lk < 62 && ((int64_t)1 << lk) < kprime) ++lk;
  const int num = lm - 1 - lk;
  const int b = num >= 0 ? num / 2 : -((-num + 1) / 2);  // floor division
  return b > 63 ? 63 : b;
}

hipError_t launch_residues(const View &va, int *ca, int8_t *oa, int64_t nrba, const View &vb, int *cb,
                           int8_t *ob, int64_t nrbb, bool cplx, int n, int beta, int64_t nkb, bool scan,
                           hipStream_t st) {
  // 64 contraction entries (two blocks) per workgroup; view rows up to the
  // padded X' rows (complex B: two X' rows per view row)
  const int64_t rowsb = cplx ? nrbb * 16 : nrbb * 32;
  if (va.R <= 0 || vb.R <= 0 || nrba <= 0 || nrbb <= 0 || nrba % 4 != 0 || nrbb % 4 != 0 || nkb <= 0 ||
      nkb % 4 != 0 || nrba * 32 < va.R || rowsb < vb.R)
    return hipErrorInvalidValue;
  const int64_t na = nrba / 2 * (nkb / 2), nb = rowsb / 64 * (nkb / 2);
  const crt::ResSide a{va, ca, oa, nrba}, b{vb, cb, ob, nrbb};
  // one launch, or one per operand where both together are too many blocks
  auto go = [&](int64_t n0, int64_t blocks, const crt::ResSide &x) {
    const dim3 grid((unsigned)blocks);
#define OZ_RES(C, G, S) \
  hipLaunchKernelGGL((crt::k_residues<C, G, S>), grid, dim3(256), 0, st, x, b, n0, n, beta, nkb)
#define OZ_RES2(C, G) \
  do {                \
    if (scan)         \
      OZ_RES(C, G, true);  \
    else                   \
      OZ_RES(C, G, false); \
  } while (0)
    if (cplx) {
      if (beta > 62) OZ_RES2(true, true); else OZ_RES2(true, false);
    } else {
      if (beta > 62) OZ_RES2(false, true); else OZ_RES2(false, false);
    }
#undef OZ_RES2
#undef OZ_RES
  };
  if (na + nb <= kMaxBlocks) {
    go(na, na + nb, a);
  } else {
    go(na, na, a);
    go(0, nb, a);
  }
  return hipGetLastError();
}

}  // namespace oz
