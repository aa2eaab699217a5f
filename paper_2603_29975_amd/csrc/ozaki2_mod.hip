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
// only the INT32 sums of one modulus, eight blocks (128 x 64): a fragment feeds
// 2.7 MFMAs, and the moduli are further independent work items, so small
// products fill the chip too. The price is one byte written and read per output
// entry and modulus. At 2048^3 complex, 14 moduli: products 486 us (1.98 POP/s)
// and rebuild 57 us, where the one kernel took 897; the MFMAs alone, on operands
// left in LDS, take 343 us at the clock the chip holds under them, the operand
// copies cost 70 of the rest and the LDS reads 50.
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
// blocks of 32 x 32 per wave (MFMA rows: j', columns: i). The contraction runs
// in stages of KS 32-entry blocks through an LDS ring of NBUF stages filled by
// direct-to-LDS copies. The fragments of block b + 1 are read into a second
// register set, one read after each MFMA of block b, so a wave never waits out
// an LDS latency; the stage's copies are issued the same way. Two workgroups
// share a CU: one's reduction to bytes runs under the other's MFMAs.
template <int WJ, int WI, int JB, int IB, int NBUF, int KS, int WPS>
__global__ void __launch_bounds__(64 * WJ * WI, WPS) k_oz2mod(Oz2ModArgs G) {
  constexpr int NW = WJ * WI;
  constexpr int NFP = WJ * JB, NFQ = WI * IB, NF = NFP + NFQ;
  constexpr int NC = NF * KS;   // copies per stage
  constexpr int CPW = NC / NW;  // per wave
  constexpr int STAGE = NC * kFragBytes;
  constexpr int D = NBUF - 1;
  constexpr int NM = JB * IB, NR = JB + IB;
  static_assert(NC % NW == 0 && KS % 2 == 0 && D >= 2, "ring");
  constexpr int RPM = (NR + NM - 1) / NM, CPM = (CPW + NM - 1) / NM;
  static_assert((D - 2) * CPW < 64, "vmcnt immediate (6 bits)");
  __shared__ __attribute__((aligned(16))) int8_t lds[NBUF * STAGE];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wj = wave % WJ, wi = wave / WJ;
  const int64_t nkb = G.nkb;  // a multiple of KS
  const int nst = (int)(nkb / KS);
  const int64_t ntj = (G.jn + 32 * NFP - 1) / (32 * NFP), nti = (G.m + 32 * NFQ - 1) / (32 * NFQ);
  const int64_t ntiles = ntj * nti, nitems = ntiles * G.n;

  for (int64_t item0 = blockIdx.x; item0 < nitems; item0 += gridDim.x) {
    const int64_t item = tile::xcd_major(item0, nitems);
    const int k = (int)(item / ntiles);
    int64_t tj, ti;
    tile::tile_coords(item - k * ntiles, 3, G.m, G.jn, 32 * NFP, 32 * NFQ, tj, ti);

    // sources of this wave's copies: copy c = wave * CPW + y moves block c % KS
    // of fragment row c / KS. Row blocks past the padded operand repeat its
    // last one (their products are not stored).
    const int8_t *src[CPW];
#pragma unroll
    for (int y = 0; y < CPW; ++y) {
      const int c = wave * CPW + y, f = c / KS;
      int64_t rb;
      const int8_t *base;
      if (f < NFP) {
        rb = G.jrb + tj * NFP + f;
        rb = rb < G.nrbP ? rb : G.nrbP - 1;
        base = G.RB + (k * G.nrbP + rb) * nkb * kFragBytes;
      } else {
        rb = ti * NFQ + (f - NFP);
        rb = rb < G.nrbQ ? rb : G.nrbQ - 1;
        base = G.RA + (k * G.nrbQ + rb) * nkb * kFragBytes;
      }
      src[y] = base + (c % KS) * kFragBytes;
    }
    auto copy = [&](int y, int st, int buf) {
      tile::copy_frag(src[y] + (int64_t)st * (KS * kFragBytes) + lane * 16,
                      lds + buf * STAGE + (wave * CPW + y) * kFragBytes);
    };

    v16i acc[JB][IB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
      for (int ib = 0; ib < IB; ++ib) acc[jb][ib] = v16i{0};

#pragma unroll
    for (int d = 0; d < D; ++d)
      if (d < nst) {
#pragma unroll
        for (int y = 0; y < CPW; ++y) copy(y, d, d);
      }
    // stage 0 has landed once at most the younger stages' copies are in flight
    if (nst >= D)
      tile::wait_vmcnt<(D - 1) * CPW>();
    else
      tile::wait_vmcnt<0>();
    tile::barrier_only();

    v4i pf[2][JB], qf[2][IB];
    // fragment read r of block x of the stage at L into register set s
    auto read = [&](int r, int s, const int8_t *L, int x) {
      if (r < IB)
        qf[s][r] = *reinterpret_cast<const v4i *>(L + ((NFP + wi * IB + r) * KS + x) * kFragBytes);
      else
        pf[s][r - IB] = *reinterpret_cast<const v4i *>(L + ((wj * JB + r - IB) * KS + x) * kFragBytes);
    };
    const int8_t *L = lds + lane * 16;
#pragma unroll
    for (int r = 0; r < NR; ++r) read(r, 0, L, 0);

    int buf = 0;
    for (int st = 0; st < nst; ++st) {
      const int nbuf = buf + 1 == NBUF ? 0 : buf + 1;
#pragma unroll
      for (int x = 0; x < KS; ++x) {
        const int s = x & 1;
        const bool last = x == KS - 1;
        const bool more = !last || st + 1 < nst;
        bool refill = false;
        int rbuf = 0;
        if (last && st + 1 < nst) {
          // The next stage's copies of this wave have landed, then every
          // wave's; all reads of the stage before this one have been used, so
          // its buffer can be refilled.
          if (D > 2 && st + D < nst)
            tile::wait_vmcnt<(D - 2) * CPW>();
          else
            tile::wait_vmcnt<0>();
          tile::barrier_only();
          refill = st + D < nst;
          rbuf = buf + D >= NBUF ? buf + D - NBUF : buf + D;
        }
        const int8_t *Ln = lds + (last ? nbuf : buf) * STAGE + lane * 16;
        const int xn = last ? 0 : x + 1;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          const int jb = i / IB, ib = i % IB;
          if (more)
#pragma unroll
            for (int r = i * RPM; r < (i + 1) * RPM && r < NR; ++r) read(r, s ^ 1, Ln, xn);
          acc[jb][ib] = __builtin_amdgcn_mfma_i32_32x32x32_i8(pf[s][jb], qf[s][ib], acc[jb][ib], 0, 0, 0);
          if (last && refill) {
#pragma unroll
            for (int y = i * CPM; y < (i + 1) * CPM && y < CPW; ++y) copy(y, st + D, rbuf);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      buf = nbuf;
    }
    // every wave is done reading the ring before the next item refills it
    tile::barrier_only();

    // ---------------------------------------------------------- residue bytes
    // Lane register 4 g + b of a block holds j' = 32 block + 8 g + 4 (lane / 32)
    // + b, row i = lane % 32: four consecutive j' of one row are one word.
    const ModConst mc = kMod.c[k];
    uint32_t *out = reinterpret_cast<uint32_t *>(G.planes) + k * G.plane_words;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
      const int64_t i = ti * (32 * NFQ) + (wi * IB + ib) * 32 + (lane & 31);
#pragma unroll
      for (int jb = 0; jb < JB; ++jb) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int64_t jq = tj * (8 * NFP) + (wj * JB + jb) * 8 + 2 * g + (lane >> 5);
          const uint32_t w = residue4(mc, k == 0, acc[jb][ib][4 * g], acc[jb][ib][4 * g + 1],
                                      acc[jb][ib][4 * g + 2], acc[jb][ib][4 * g + 3]);
          if (i < G.m && 4 * jq < G.jn) out[jq * G.ldq + i] = w;
        }
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

// a + b = s + e exactly, for |a| >= |b| or a = 0.
__device__ __forceinline__ void fast_two_sum(double a, double b, double &s, double &e) {
  s = add_rn(a, b);
  e = sub_rn(b, sub_rn(s, a));
}
// a + b rounded to odd (an inexact sum takes the neighbour with an odd last
// bit), for |a| >= |b| or a = 0: added to a much larger number, the sum then
// rounds as the exact one would.
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
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t jq = blockIdx.y;
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

template <int WJ, int WI, int JB, int IB, int NBUF, int KS, int WPS>
hipError_t launch_mod(const Oz2ModArgs &a, int num_cu, hipStream_t st) {
  const int64_t ntj = (a.jn + 32 * WJ * JB - 1) / (32 * WJ * JB);
  const int64_t nti = (a.m + 32 * WI * IB - 1) / (32 * WI * IB);
  const int64_t per_cu = 4 * WPS / (WJ * WI);
  const int64_t grid = std::min<int64_t>(ntj * nti * a.n, per_cu * num_cu);
  if (a.nkb % KS != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_oz2mod<WJ, WI, JB, IB, NBUF, KS, WPS>), dim3((unsigned)grid),
                     dim3(64 * WJ * WI), 0, st, a);
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
  // 112), z 128^3 38.6 / 35.3 / 31.8 (14; 28).
  auto items = [&](int64_t t) { return ((a.m + t - 1) / t) * ((a.jn + t - 1) / t) * a.n; };
  hipError_t e;
  if (items(256) * 4 >= 3 * (int64_t)num_cu)
    e = launch_mod<2, 4, 4, 2, 4, 2, 2>(a, num_cu, st);
  else if (items(128) >= num_cu)
    e = launch_mod<2, 2, 2, 2, 4, 2, 2>(a, num_cu, st);
  else
    e = launch_mod<2, 2, 1, 1, 4, 2, 2>(a, num_cu, st);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)((a.m + 255) / 256), (unsigned)((a.jn + 3) / 4));
  switch (a.n) {
#define OZ_N(N) \
  case N: hipLaunchKernelGGL(k_oz2rebuild<N>, grid, dim3(256), 0, st, a); break;
    OZ_N(2) OZ_N(3) OZ_N(4) OZ_N(5) OZ_N(6) OZ_N(7) OZ_N(8) OZ_N(9) OZ_N(10) OZ_N(11)
    OZ_N(12) OZ_N(13) OZ_N(14) OZ_N(15) OZ_N(16) OZ_N(17) OZ_N(18) OZ_N(19) OZ_N(20)
#undef OZ_N
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace oz
