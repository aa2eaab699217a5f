// Ozaki-II product of libozaki (gfx950) in two kernels: one plain INT8 product
// per modulus whose results leave the chip as one residue byte per output
// entry, then one rebuild pass over those bytes.
//
// Section 2.2 of the paper: the integer operands are multiplied modulo several
// pairwise-coprime moduli on the integer matrix cores, and the Chinese
// remainder theorem gives back the exact integer product.
//
// Why two kernels: with the digits of all moduli in registers (ozaki2_gemm.hip)
// a wave holds one or two 32 x 32 blocks, so every residue fragment read from
// LDS feeds one or two MFMAs and the LDS bounds the kernel. Here a wave holds
// only the INT32 sums of one modulus, 32 blocks of 16 x 16 (128 x 64), and the
// moduli are further independent work items, so small products fill the chip
// too. The price is one byte written and read per output entry and modulus. At
// 2048^3 complex, 14 moduli, the whole call takes 570 us (626 with 32 x 32 x 32
// MFMAs, whose products alone took 486), with the one kernel 1048.
#include "ozaki2_crt.hpp"
#include "ozaki_gemm_tile.hpp"

namespace oz {

namespace {

// ------------------------------------------------------------ modular products
// What the reduction of modulus k needs: m_k, 1 / m_k, and the balanced
// residues of 256^b (P_k)^-1 mod m_k as byte b of a word.
struct ModConst {
  float rm, fm;
  int w;
};
struct ModTable {
  ModConst c[kModMax];
};
constexpr ModTable make_mod_table() {
  ModTable t{};
  for (int k = 0; k < kModMax; ++k) {
    const int m = crt::kT.m[k];
    t.c[k].rm = 1.0f / (float)m;
    t.c[k].fm = (float)m;
    unsigned w = 0;
    int x = crt::kT.inv[k];
    for (int b = 0; b < 4; ++b) {
      w |= (unsigned)(crt::bal_c(x, m) & 0xff) << (8 * b);
      x = crt::bal_c(crt::bal_c(x, m) * 256, m);
    }
    t.c[k].w = (int)w;
  }
  return t;
}
__constant__ ModTable kMod = make_mod_table();

// Four INT32 sums c of modulus k to the bytes of c (P_k)^-1 mod m_k (balanced).
// The signed base-256 digits of c (c + 0x80808080, each byte less 128; exact
// because |c| <= K' 127^2 <= 2^17 127^2 < 0x7f7f7f7f) times the balanced
// weights give |t| <= 4 * 128 * 127 < 2^17, congruent to the wanted residue, so
// one FP32 quotient is exact (see crt::bal_mod). t carries + 128, which makes
// the remainder an unsigned byte that one conversion packs. m_0 = 256 keeps the
// low byte of the (wrapping) sum.
__device__ __forceinline__ uint32_t residue4(const ModConst &mc, bool first, int c0, int c1, int c2,
                                             int c3) {
  if (first)
    return (uint32_t)(c0 & 0xff) | ((uint32_t)(c1 & 0xff) << 8) | ((uint32_t)(c2 & 0xff) << 16) |
           ((uint32_t)c3 << 24);
  const int c[4] = {c0, c1, c2, c3};
  uint32_t out = 0;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int z = (int)(((uint32_t)c[b] + 0x80808080u) ^ 0x80808080u);
    const float t = (float)__builtin_amdgcn_sdot4(z, mc.w, 128, false);
    const float q = __builtin_rintf(__builtin_fmaf(t, mc.rm, -128.0f * mc.rm));
    out = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_fmaf(-q, mc.fm, t), b, out);
  }
  return out ^ 0x80808080u;
}

// One work item is one output tile of one modulus. WJ x WI waves, JB x IB
// blocks of 16 x 16 per wave (MFMA rows: j', columns: i), v_mfma_i32_16x16x64_i8.
// The contraction runs in 64-entry blocks through an LDS ring of four stages
// filled by direct-to-LDS copies. A wave holds the A' fragments of a block in
// registers and streams the B' ones past them, LA ahead; the next block's A'
// fragments, its first B' ones and the copies of the block after the next but
// one follow a barrier in the middle of a block, so no LDS latency is waited
// out.
template <int WJ, int WI, int JB, int IB, int WPS>
__global__ void __launch_bounds__(64 * WJ * WI, WPS) k_oz2mod(Oz2ModArgs G) {
  constexpr int NW = WJ * WI;
  constexpr int NBUF = 4, D = NBUF - 1;
  constexpr int FJ = WJ * JB, FI = WI * IB, NF = FJ + FI;  // 16-row blocks per tile
  constexpr int CPW = NF / NW;                             // copies per wave and block
  constexpr int STAGE = NF * kFragBytes;
  constexpr int LA = JB > 2 ? 2 : 1, R = 2 * LA;           // B' look-ahead and slots
  constexpr int MID = JB / 2;
  static_assert(NF % NW == 0 && JB % R == 0 && JB - LA >= MID, "schedule");
  static_assert(CPW < 64, "vmcnt immediate (6 bits)");
  static_assert(NBUF * STAGE * (4 * WPS / NW) <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(16))) int8_t lds[NBUF * STAGE];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wj = wave % WJ, wi = wave / WJ;
  const uint32_t lane16 = lane * 16;
  const int nkb = (int)(G.nkb >> 1);  // even: the contraction is padded to 128
  const int64_t rowst = (int64_t)nkb * kFragBytes;
  const int64_t ntj = (G.jn + 16 * FJ - 1) / (16 * FJ), nti = (G.m + 16 * FI - 1) / (16 * FI);
  const int64_t ntiles = ntj * nti, nitems = ntiles * G.n;

  for (int64_t item0 = blockIdx.x; item0 < nitems; item0 += gridDim.x) {
    const int64_t item = tile::xcd_major(item0, nitems);
    const int k = (int)(item / ntiles);
    int64_t tj, ti;
    tile::tile_coords(item - k * ntiles, 3, G.m, G.jn, 16 * FJ, 16 * FI, tj, ti);

    // sources of this wave's copies: fragment rows wave * CPW + y. Row blocks
    // past the padded operand repeat its last one (their products are not
    // stored).
    const int8_t *src[CPW];
#pragma unroll
    for (int y = 0; y < CPW; ++y) {
      const int f = wave * CPW + y;
      int64_t rb;
      const int8_t *base;
      if (f < FJ) {
        rb = G.jrb * 2 + tj * FJ + f;
        rb = rb < G.nrbP * 2 ? rb : G.nrbP * 2 - 1;
        base = G.RB + (k * G.nrbP * 2 + rb) * rowst;
      } else {
        rb = ti * FI + (f - FJ);
        rb = rb < G.nrbQ * 2 ? rb : G.nrbQ * 2 - 1;
        base = G.RA + (k * G.nrbQ * 2 + rb) * rowst;
      }
      src[y] = base;
    }
    auto copy = [&](int y, uint32_t voff, int buf) {
      tile::copy_frag_s(src[y], voff, lds + buf * STAGE + (wave * CPW + y) * kFragBytes);
    };

    v4i acc[JB][IB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
      for (int ib = 0; ib < IB; ++ib) acc[jb][ib] = v4i{0};

#pragma unroll
    for (int d = 0; d < D; ++d)
      if (d < nkb) {
#pragma unroll
        for (int y = 0; y < CPW; ++y) copy(y, lane16 + d * kFragBytes, d);
      }
    // block 0 has landed once at most the younger blocks' copies are in flight
    if (nkb >= D)
      tile::wait_vmcnt<(D - 1) * CPW>();
    else
      tile::wait_vmcnt<0>();
    tile::barrier_only();

    v4i pf[R], qf[2][IB];
    uint32_t lb = tile::lds_addr(lds) + lane16 + wj * JB * kFragBytes;
    uint32_t lq = tile::lds_addr(lds) + lane16 + (FJ + wi * IB) * kFragBytes;
    asm volatile("" : "+v"(lb), "+v"(lq));
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) qf[0][ib] = tile::lds_read(lq + ib * kFragBytes);
#pragma unroll
    for (int jb = 0; jb < LA; ++jb) pf[jb] = tile::lds_read(lb + jb * kFragBytes);

    int buf = 0;
    for (int kb0 = 0; kb0 < nkb; kb0 += 2) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int kb = kb0 + s;
        const int nbuf = (buf + 1) & (NBUF - 1), fbuf = (buf + D) & (NBUF - 1);
        const uint32_t co = buf * STAGE, no = nbuf * STAGE;
        const bool fill = kb + D < nkb;
        const uint32_t voff = lane16 + (uint32_t)(kb + D) * kFragBytes;
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
          if (jb == MID) {
            // the next block has landed: this wave's copies, then every wave's;
            // all reads of the block before this one have been used
            if (kb + D <= nkb)
              tile::wait_vmcnt<(D - 2) * CPW>();
            else
              tile::wait_vmcnt<0>();
            tile::barrier_only();
          }
          const int n = jb + LA;
          pf[n % R] = tile::lds_read(lb + (n < JB ? co : no) + (n % JB) * kFragBytes);
          if (jb >= MID) {
#pragma unroll
            for (int ib = 0; ib < IB; ++ib)
              if (ib * (JB - MID) / IB == jb - MID) qf[s ^ 1][ib] = tile::lds_read(lq + no + ib * kFragBytes);
            if (fill) {
#pragma unroll
              for (int y = 0; y < CPW; ++y)
                if (y * (JB - MID) / CPW == jb - MID) copy(y, voff, fbuf);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int ib = 0; ib < IB; ++ib)
            acc[jb][ib] = __builtin_amdgcn_mfma_i32_16x16x64_i8(pf[jb % R], qf[s][ib], acc[jb][ib], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        buf = nbuf;
      }
    }
    // every wave is done reading the ring before the next item refills it
    tile::barrier_only();

    // ---------------------------------------------------------- residue bytes
    // Lane register r of a block holds j' = 16 block + 4 (lane / 16) + r, row i =
    // lane % 16: four consecutive j' of one row are one word.
    const ModConst mc = kMod.c[k];
    uint32_t *out = reinterpret_cast<uint32_t *>(G.planes) + k * G.plane_words;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
      const int64_t i = (ti * FI + wi * IB + ib) * 16 + (lane & 15);
#pragma unroll
      for (int jb = 0; jb < JB; ++jb) {
        const int64_t jq = (tj * FJ + wj * JB + jb) * 4 + (lane >> 4);
        const v4i &c = acc[jb][ib];
        const uint32_t w = residue4(mc, k == 0, c[0], c[1], c[2], c[3]);
        if (i < G.m && 4 * jq < G.jn) out[jq * G.ldq + i] = w;
      }
    }
  }
}

// --------------------------------------------------------------------- rebuild
// Constants of the rebuild from N residues r_K = C_K (P_K)^-1 mod m_K.
// Digits: d_K = r_K - sum_{j<K} d_j (P_j P_K^-1) mod m_K. Three digits make one
// group value v_h = d_3h + m_3h d_3h+1 + m_3h m_3h+1 d_3h+2 (|v_h| < 2^23), and
// c = sum_h v_h P_3h with P_3h in limbs of 26 bits.
constexpr int kLimb26 = 26;
constexpr int kGroups = (kModMax + 2) / 3;
constexpr int kLimbs26 = 7;
struct RebuildTable {
  unsigned g[(kModMax + 3) / 4][kModMax];  // -P_j P_K^-1 mod m_K in [0, m_K), byte j % 4 of word j / 4
  int off[kModMax];                        // 128 (1 + the sum of those bytes): what the + 128 of the digits adds
  float coef[kModMax];                     // the digit's factor in its group
  double limb[kGroups][kLimbs26];          // P_3h
  int nl[kGroups];                         // its nonzero limbs
  int nlM[kModMax + 1];                    // limbs of M_n
};
constexpr int limbs_of(const int (&p)[crt::kLimbs], int64_t (&out)[kLimbs26]) {
  int top = 0;
  for (int l = 0; l < kLimbs26; ++l) {
    int64_t v = 0;
    for (int b = 0; b < kLimb26; ++b) {
      const int bit = l * kLimb26 + b;
      if (bit / 16 < crt::kLimbs && ((p[bit / 16] >> (bit % 16)) & 1)) v |= (int64_t)1 << b;
    }
    out[l] = v;
    if (v) top = l + 1;
  }
  return top;
}
constexpr RebuildTable make_rebuild_table() {
  RebuildTable t{};
  for (int k = 0; k < kModMax; ++k) {
    const int m = crt::kT.m[k];
    int sum = 0;
    for (int j = 0; j < k; ++j) {
      const int g = ((-crt::kT.g[j][k]) % m + m) % m;
      t.g[j >> 2][k] |= (unsigned)g << (8 * (j & 3));
      sum += g;
    }
    t.off[k] = 128 * (1 + sum);
    t.coef[k] = k % 3 == 0 ? 1.0f : t.coef[k - 1] * (float)crt::kT.m[k - 1];
    int64_t l26[kLimbs26] = {};
    const int top = limbs_of(crt::kT.P[k], l26);
    t.nlM[k] = top;
    if (k % 3 == 0) {
      t.nl[k / 3] = top;
      for (int l = 0; l < kLimbs26; ++l) t.limb[k / 3][l] = (double)l26[l];
    }
  }
  int m20[crt::kLimbs] = {}, carry = 0;  // M_20 = P_19 m_19
  for (int l = 0; l < crt::kLimbs; ++l) {
    const int v = crt::kT.P[kModMax - 1][l] * crt::kT.m[kModMax - 1] + carry;
    m20[l] = v & 0xffff;
    carry = v >> 16;
  }
  int64_t l26[kLimbs26] = {};
  t.nlM[kModMax] = limbs_of(m20, l26);
  return t;
}
constexpr RebuildTable kRb = make_rebuild_table();

// Digit of modulus K of one entry (byte b of the residue words), added to its
// group. W holds the earlier digits plus 128 as bytes, so their share is one
// unsigned 4-way dot product per word; t = sum + 128 - off is at most 20 * 255 *
// 254 < 2^21 in magnitude, where one FP32 quotient is exact (see crt::bal_mod),
// and the remainder plus 128 is an unsigned byte.
template <int K, int NW, int NG>
__device__ __forceinline__ void garner_digit(uint32_t rw, int b, uint32_t (&W)[NW], float (&v)[NG]) {
  const uint32_t rb = ((rw >> (8 * b)) & 0xff) ^ 0x80u;  // r_K + 128
  float d;                                               // d_K + 128
  if constexpr (K == 0) {
    W[0] = rb;
    d = (float)rb;
  } else {
    constexpr float m = (float)crt::kT.m[K], rm = 1.0f / m;
    uint32_t t = rb;
#pragma unroll
    for (int h = 0; h <= (K - 1) / 4; ++h) t = __builtin_amdgcn_udot4(W[h], kRb.g[h][K], t, false);
    const float tf = (float)((int)t + (128 - kRb.off[K]));
    const float q = __builtin_rintf(__builtin_fmaf(tf, rm, -128.0f * rm));
    d = __builtin_fmaf(-q, m, tf);
    W[K >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(d, K & 3, (K & 3) == 0 ? 0u : W[K >> 2]);
  }
  // integers below 2^24: exact
  v[K / 3] = __builtin_fmaf(d, kRb.coef[K], K % 3 == 0 ? 0.0f : v[K / 3]);
}
template <int N, int K, int NW, int NG>
__device__ __forceinline__ void garner_all(const uint32_t (&w)[N], int b, uint32_t (&W)[NW],
                                           float (&v)[NG]) {
  if constexpr (K < N) {
    garner_digit<K, NW, NG>(w[K], b, W, v);
    garner_all<N, K + 1, NW, NG>(w, b, W, v);
  }
}
// 128 times the factors of the digits of group h that N moduli have.
template <int N>
constexpr float group_off(int h) {
  float s = 0.0f;
  for (int k = 3 * h; k < 3 * h + 3 && k < N; ++k) s += 128.0f * kRb.coef[k];
  return s;
}

// a + b = s + e exactly, for |a| >= |b| or a = 0 (Dekker 1971, Fast2Sum).
__device__ __forceinline__ void fast_two_sum(double a, double b, double &s, double &e) {
  s = add_rn(a, b);
  e = sub_rn(b, sub_rn(s, a));
}
// a + b rounded to odd (an inexact sum takes the neighbour with an odd last
// bit), for |a| >= |b| or a = 0: added to a much larger number, the sum then
// rounds as the exact one would (Boldo and Melquiond 2008).
__device__ __forceinline__ double add_odd(double a, double b) {
  double s, e;
  fast_two_sum(a, b, s, e);
  int64_t u = __double_as_longlong(s);
  const int64_t step = ((e > 0.0) == (s > 0.0)) ? 1 : -1;
  u += (e != 0.0 && (u & 1) == 0) ? step : 0;
  return __longlong_as_double(u);
}

// c = sum_h v_h P_3h rounded once to FP64. The limb sums stay below 2^53, so
// every FP64 operation up to the last is exact: products and sums per 26-bit
// limb, one carry pass to limbs of at most 2^25 in magnitude, pairs of limbs as
// one number E_p 2^(52 p) with |E_p| < 2^52, and then the sum of at most four
// such non-overlapping numbers, whose tail is rounded to odd.
template <int N, int NG>
__device__ __forceinline__ double combine_rn(const float (&v)[NG]) {
  constexpr int NL = kRb.nlM[N];
  constexpr int NE = (NL + 1) / 2;
  static_assert(NL <= kLimbs26 && NE <= 4, "limbs of M");
  double L[2 * NE];
#pragma unroll
  for (int l = 0; l < 2 * NE; ++l) L[l] = 0.0;
#pragma unroll
  for (int h = 0; h < NG; ++h) {
    const double x = (double)(v[h] - group_off<N>(h));
#pragma unroll
    for (int l = 0; l < kRb.nl[h]; ++l) L[l] = __builtin_fma(x, kRb.limb[h][l], L[l]);
  }
#pragma unroll
  for (int l = 0; l + 1 < NL; ++l) {
    const double c = __builtin_rint(L[l] * 0x1p-26);
    L[l] = __builtin_fma(-c, 0x1p26, L[l]);
    L[l + 1] = add_rn(L[l + 1], c);
  }
  double E[4] = {0.0, 0.0, 0.0, 0.0};
  constexpr double sc[4] = {1.0, 0x1p52, 0x1p104, 0x1p156};
#pragma unroll
  for (int p = 0; p < NE; ++p) E[p] = __builtin_fma(L[2 * p + 1], 0x1p26, L[2 * p]) * sc[p];
  if constexpr (NE == 1) return E[0];
  if constexpr (NE == 2) return add_rn(E[1], E[0]);
  double s, e;
  if constexpr (NE == 3) {
    fast_two_sum(E[2], E[1], s, e);
    return add_rn(s, add_odd(e, E[0]));
  }
  double e1, r;
  fast_two_sum(E[3], E[2], s, e);
  fast_two_sum(e, E[1], e1, r);
  fast_two_sum(s, e1, s, e);
  return add_rn(s, add_odd(e, add_odd(r, E[0])));
}

// One thread per row i and group of four j' (two complex columns or four real
// ones): the N residue words are loaded together, then each entry takes its
// digits, is combined and rounded once, scaled and finished with alpha and
// beta. Consecutive threads take consecutive rows, so every access is
// contiguous. The arithmetic bounds it: about 190 operations per entry at 14
// moduli, 57 us at 2048^3 complex; with integer digits and 16-bit limbs it was
// 310 operations and 81 us.
template <int N>
__global__ void __launch_bounds__(256) k_oz2rebuild(Oz2ModArgs G) {
  constexpr int NW = (N + 3) / 4, NG = (N + 2) / 3;
  const uint32_t nti = (uint32_t)((G.m + 255) / 256);
  const int64_t i = (int64_t)(blockIdx.x % nti) * 256 + threadIdx.x;
  const int64_t jq = G.jq0 + blockIdx.x / nti;
  if (i >= G.m) return;
  const uint32_t *in = reinterpret_cast<const uint32_t *>(G.planes) + jq * G.ldq + i;
  uint32_t w[N];
#pragma unroll
  for (int k = 0; k < N; ++k) w[k] = in[k * G.plane_words];
  const int ca = G.codeA[i];
  const bool bad_i = code_bad(ca);
  const int ea = code_exp(ca) - 2 * G.beta;
  double val[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    uint32_t W[NW];
    float v[NG];
    garner_all<N, 0, NW, NG>(w, b, W, v);
    val[b] = combine_rn<N, NG>(v);
  }
  const int64_t j0 = G.jrb * 32 + 4 * jq;  // first j' of the group in the whole product
  if (G.cplx) {
    double2 *C = reinterpret_cast<double2 *>(G.C);
#pragma unroll
    for (int b = 0; b < 4; b += 2) {
      const int64_t j = (j0 + b) >> 1;
      if (4 * jq + b >= G.jn) continue;
      const int cb = G.codeB[j];
      double2 *cp = C + i + j * G.ldc;
      if (bad_i || code_bad(cb)) {
        *cp = make_double2(qnan(), qnan());
        continue;
      }
      const int sc = ea + code_exp(cb);
      const double pr = ldexp(val[b], sc), pi = ldexp(val[b + 1], sc);
      double re = sub_rn(mul_rn(G.ar, pr), mul_rn(G.ai, pi));
      double im = add_rn(mul_rn(G.ar, pi), mul_rn(G.ai, pr));
      if (!G.beta_zero) {
        const double2 z = *cp;
        re = add_rn(re, sub_rn(mul_rn(G.br, z.x), mul_rn(G.bi, z.y)));
        im = add_rn(im, add_rn(mul_rn(G.br, z.y), mul_rn(G.bi, z.x)));
      }
      *cp = make_double2(re, im);
    }
  } else {
    double *C = reinterpret_cast<double *>(G.C);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int64_t j = j0 + b;
      if (4 * jq + b >= G.jn) continue;
      const int cb = G.codeB[j];
      double *cp = C + i + j * G.ldc;
      if (bad_i || code_bad(cb)) {
        *cp = qnan();
        continue;
      }
      const double p = ldexp(val[b], ea + code_exp(cb));
      double out = mul_rn(G.ar, p);
      if (!G.beta_zero) out = add_rn(out, mul_rn(G.br, *cp));
      *cp = out;
    }
  }
}

template <int WJ, int WI, int JB, int IB, int WPS>
hipError_t launch_mod(const Oz2ModArgs &a, int num_cu, hipStream_t st) {
  const int64_t ntj = (a.jn + 16 * WJ * JB - 1) / (16 * WJ * JB);
  const int64_t nti = (a.m + 16 * WI * IB - 1) / (16 * WI * IB);
  const int64_t grid = std::min<int64_t>(ntj * nti * a.n, (int64_t)(4 * WPS / (WJ * WI)) * num_cu);
  hipLaunchKernelGGL((k_oz2mod<WJ, WI, JB, IB, WPS>), dim3((unsigned)grid), dim3(64 * WJ * WI), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_oz2mod(const Oz2ModArgs &a, int num_cu, hipStream_t st) {
  if (a.m <= 0 || a.jn <= 0) return hipSuccess;
  if (a.n < 2 || a.n > kModMax || a.nkb <= 0 || a.nkb % 4 != 0) return hipErrorInvalidValue;
  // The tile by the work items it gives. 256 x 256 moves the least per MFMA and
  // is taken while it nearly fills the CUs once; below that the smaller tiles
  // spread the work further. Measured, whole call, us at tiles 256 / 128 / 64,
  // 14 moduli: z 4096^3 3903 / 4787 / 8487 (7168 items of 256), d 1024^3 63.9 /
  // 69.7 / 80.9 (224), z 4096 x 128 x 4096 357 / 395 / 533 (224), z 512 x 512 x
  // 4096 173 / 145 / 192 (112; 448 of 128), z 256^3 44.7 / 38.6 / 36.9 (28;
  // 112), z 128^3 38.6 / 35.3 / 31.8 (14; 28). No tile is twice as long as the
  // shorter side of C: z 100 x 40000 x 16 232 / 183 / 246, x 700 1074 / 1028 / 1256,
  // z 16 x 40000 x 16 202 / 143 / 138, z 40000 x 8 x 100 145 / 111 / 107.
  auto items = [&](int64_t t) { return ((a.m + t - 1) / t) * ((a.jn + t - 1) / t) * a.n; };
  const int64_t side = std::min(a.m, a.jn);
  hipError_t e;
  if (side > 128 && items(256) * 4 >= 3 * (int64_t)num_cu)
    e = launch_mod<2, 4, 8, 4, 2>(a, num_cu, st);
  else if (side > 64 && items(128) >= num_cu)
    e = launch_mod<2, 2, 4, 4, 2>(a, num_cu, st);
  else
    e = launch_mod<2, 2, 2, 2, 2>(a, num_cu, st);
  if (e != hipSuccess) return e;
  // blocks of 256 rows of one group of four j', the rows first, in one launch
  // unless that is too many blocks
  Oz2ModArgs r = a;
  const int64_t nti = (a.m + 255) / 256, ngroups = (a.jn + 3) / 4, most = std::max<int64_t>(kMaxBlocks / nti, 1);
  for (r.jq0 = 0; r.jq0 < ngroups; r.jq0 += most) {
    const dim3 grid((unsigned)(nti * std::min(most, ngroups - r.jq0)));
    switch (a.n) {
#define OZ_N(N) \
  case N: hipLaunchKernelGGL(k_oz2rebuild<N>, grid, dim3(256), 0, st, r); break;
      OZ_N(2) OZ_N(3) OZ_N(4) OZ_N(5) OZ_N(6) OZ_N(7) OZ_N(8) OZ_N(9) OZ_N(10) OZ_N(11)
      OZ_N(12) OZ_N(13) OZ_N(14) OZ_N(15) OZ_N(16) OZ_N(17) OZ_N(18) OZ_N(19) OZ_N(20)
#undef OZ_N
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

}  // namespace oz
