// Fused slice-pair INT8 GEMM and FP64 recombination of libozaki (gfx950).
//
// Steps "low-precision matrix multiplications on the slices" and "accumulate
// in higher precision" of the Ozaki-I scheme (Section 2.2 of the paper).
//
// Output orientation: the MFMA row index is the output column side j' and the
// MFMA column index (lane % 16) is the output row i, so 16 lanes hold 16
// consecutive rows of one column of C and every store of the epilogue is a
// contiguous run in column-major C. For complex data j' = 2j + c (c = 0 real, 1
// imaginary part of column j), so a lane holds Re and Im of one C entry in
// neighbouring accumulator registers and writes 16 bytes.
//
// Work per workgroup tile (BJ = 16 WJ columns j', BI = 16 WI IB rows i), per wave
// IB blocks of 16 x 16 side by side along i with one INT32 accumulator set per
// diagonal t = 2..S+1:
//   for each 64-wide contraction block:
//     for p = 1..S, q = 1..S+1-p:  acc[p+q-2] += SB'_q(16x64) * SA'_p(16x64)^T
// using v_mfma_i32_16x16x64_i8 (exact INT8 x INT8 -> INT32).
//
// What bounds it is the chip's power: with random digits the clock falls to
// 1.7-1.8 GHz while the matrix pipe is busy 70-80% of the time, and removing
// stalls lowers the clock further, so the energy per product decides.
//  - The 16x16x64 form keeps half as many accumulators per product as 32x32x32:
//    bare MFMA loops on random operands run at 4.02 against 3.43 POP/s.
//  - The copies into LDS are the largest other share (13% in a timed loop without
//    them, as the 6% of the LDS reads below), so the tile is as
//    large as the accumulators allow (128 x 128 up to S = 6, else 128 x 64),
//    then the LDS reads (6%): each wave holds the B' fragments of all S slices
//    of its 16 columns in registers and streams the A' fragments past them.
// Measured per launch, here / 32x32x32 blocks with every LDS latency of a block
// exposed behind its barrier: 2048^3 complex, 8-bit S = 6 441 / 542 us (0.65 of
// the nominal INT8 rate), 4096^3 3.55 / 4.29 ms; 4096^3 real, 7-bit S = 7 1.22 /
// 1.53 ms, 2048^3 complex S = 7 611 / 720 us.
//
// Slice fragments move from global memory straight into LDS with
// global_load_lds_dwordx4 (one 1 KiB fragment per wave instruction, no staging
// registers). The packed fragment layout makes every global and LDS access one
// contiguous 16-byte run per lane and the LDS reads conflict free. No LDS
// latency is waited out: A' fragments are read LA ahead, also across the block
// boundary, and B' slice q of the next block is read as soon as the slice is done
// with, which needs the next block in LDS before this one ends. Two LDS plans
// give that, both with explicit waits (vmcnt for this wave's own copies, then
// s_barrier), because the generic workgroup barrier would drain every copy in
// flight:
//  RING  three stages of one contraction block; one barrier per block, after the
//        first A' fragment: the next block has landed, the one after it is copied.
//  else  (three stages do not fit) one buffer for B', two for A': a barrier X,
//        when every wave has read its B' fragments, starts the copies of the
//        next block, a barrier Y before the first read of the next B' ends them.
//
// INT32 range: a diagonal of S pairs over 64 * kb contraction entries is bounded
// by S * 64 * kb * 127^2. Past that bound the contraction is cut into chunks
// whose INT32 sums go to workgroup-private memory (as they are, for two chunks,
// else added up in int64); the epilogue adds them in int64. At 16384^3
// complex, S = 6, that is 52 GB of traffic, about 4% of the time, where splitting
// each diagonal over two INT32 sets needed the smaller tile. The FP64 epilogue
// converts every S_t exactly (|S_t| < 2^53) and adds them largest weight first,
// one rounding per addition, then scales by 2^(e_i + f_j) and applies alpha/beta
// without fused multiply-adds.
#include <type_traits>
#include <utility>

#include "ozaki_gemm_tile.hpp"

namespace oz {

namespace {

using tile::barrier_only;
using tile::chunk_blocks;
using tile::wait_vmcnt;

// The kernel's arguments and problem table in constant address space, so that
// fields are fetched by scalar loads where they are used.
typedef const __attribute__((address_space(4))) GemmArgs *ArgsPtr;
typedef const __attribute__((address_space(4))) GemmProblem *ProblemPtr;
typedef const __attribute__((address_space(4))) int *IntPtr;

constexpr int kInt32Chunks = 2;  // up to so many chunks each keeps its own INT32 sums

// f(0), ..., f(N - 1) with constant arguments.
template <typename F, int... N>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, N...>, F f) {
  (f(std::integral_constant<int, N>{}), ...);
}

template <int S, int WJ, int WI, int IB>
struct Cfg {
  static constexpr int NW = WJ * WI;
  static constexpr int FJ = WJ, FI = WI * IB;  // 16-row blocks of B' and A' per tile
  static constexpr int BJ = 16 * FJ, BI = 16 * FI;
  static constexpr int RingBytes = 3 * S * (FJ + FI) * kFragBytes;
  static constexpr int XyBytes = S * (FJ + 2 * FI) * kFragBytes;
};

// How a tile's contraction runs: in one piece, in chunks carried by the workgroup,
// or (few tiles) in parts by different workgroups, whose sums k_ozparts adds.
enum { kWhole, kChunked, kParts };

// Word w of this wave's chunk sums, lane-interleaved: a wave-uniform base and a
// 32-bit lane offset, so that the addresses cost no vector registers. The
// accesses are device-scope, which keeps the traffic in L2, away from stale
// lines of the non-coherent vector L1.
template <typename T>
__device__ __forceinline__ T *carry_word(char *base, int w, uint32_t lane) {
  return reinterpret_cast<T *>(base + (int64_t)w * (64 * sizeof(T)) + lane * (uint32_t)sizeof(T));
}

template <int S, int WJ, int WI, int IB, int WPS, bool RING, int LA, bool RAW, int MODE>
__global__ void __launch_bounds__(64 * WJ * WI, WPS) k_ozgemm(GemmArgs G) {
  using C_ = Cfg<S, WJ, WI, IB>;
  constexpr int NW = C_::NW, FJ = C_::FJ, FI = C_::FI;
  constexpr int NCB = S * FJ, NCA = S * FI;  // copies per block
  constexpr int XB = (NCB + NW - 1) / NW, XA = (NCA + NW - 1) / NW;
  constexpr int XC = XB + XA;                // copies per wave and block (at most)
  constexpr int MINC = NCB / NW + NCA / NW;  // at least
  constexpr int STAGE = (NCB + NCA) * kFragBytes;
  constexpr int LDS = RING ? C_::RingBytes : C_::XyBytes;
  constexpr bool CHUNKED = MODE == kChunked, PARTS = MODE == kParts;
  constexpr int NA = S * IB;  // A' fragments per block
  constexpr int R = LA + 1;   // their register slots
  // X (RING: the one barrier) comes when the first A' fragment is done with,
  // which has used every B' slice of the block; Y before step S - 2 (0-based),
  // which leaves its three slice pairs' MFMAs to cover the first reads of the
  // next B'. The copies go out with the IB fragments after X. Spreading them
  // further, or X and Y a step later or earlier, was at most 1% faster in one
  // case and up to 12% slower in others.
  constexpr int NX = 1, NY = (S - 2) * IB, PY = RING ? 1 : S - 2;
  constexpr int WORDS = IB * S * 4;  // accumulator words per lane
  static_assert(LDS * (4 * WPS / NW) <= 160 * 1024, "LDS");
  static_assert(RING || S >= 4, "X before Y");
  static_assert(NA - LA >= (RING ? NX : NY), "the look-ahead crosses into a block that has landed");
  static_assert(MINC < 64, "vmcnt immediate (6 bits)");
  __shared__ __attribute__((aligned(16))) int8_t lds[LDS];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // wave-uniform
  const int wj = wave % WJ;
  const int wi = wave / WJ;
  const uint32_t lane16 = lane * 16;
  const ArgsPtr ga = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const bool grouped = ga->probs != nullptr;
  const int64_t ntiles = grouped ? ga->ntiles
                                 : ((ga->one.nprime + C_::BJ - 1) / C_::BJ) *
                                       ((ga->one.m + C_::BI - 1) / C_::BI);
  const int64_t nitems = PARTS ? ntiles * ga->ksplit : ntiles;

  for (int64_t item = blockIdx.x; item < nitems; item += gridDim.x) {
    // part first: the workgroups of one part share its A' and B' rows
    const int64_t tn = PARTS ? item % ntiles : item;
    // The problem this tile belongs to (uniform across the workgroup).
    ProblemPtr pr = grouped ? (ProblemPtr)(uint64_t)(ga->probs + ((IntPtr)(uint64_t)ga->tile_prob)[tn])
                            : &ga->one;
    int64_t tj, ti;
    {
      const int order = PARTS ? 0 : ga->order;
      int64_t local = grouped ? (int64_t)((IntPtr)(uint64_t)ga->tile_local)[tn] : tn;
      if (!grouped && order == 3) local = tile::xcd_major(tn, ntiles);
      tile::tile_coords(local, order, pr->m, pr->nprime, C_::BJ, C_::BI, tj, ti);
    }
    const int64_t nkb_all = pr->nkb >> 1;  // pr->nkb counts 32 entries
    const int64_t rowst = nkb_all * kFragBytes;
    const int64_t chunk = CHUNKED ? ga->kb_chunk >> 1 : nkb_all;

    v4i acc[IB][S];
    auto acc_word = [&](int w) { return acc[w / (4 * S)][w / 4 % S][w % 4]; };
    // chunk sums of this wave: one INT32 slot per chunk carried, or (wide) int64
    constexpr int64_t kSlot = (int64_t)NW * WORDS * 64 * sizeof(int32_t);
    const bool wide = nkb_all > kInt32Chunks * chunk;
    int slots = 0;
    auto carry_base = [&]() {
      return reinterpret_cast<char *>(ga->flush_ws) + blockIdx.x * (2 * kSlot) +
             (int64_t)wave * (WORDS * 64) * (wide ? sizeof(int64_t) : sizeof(int32_t));
    };

    int64_t k0 = PARTS ? (item / ntiles) * ga->kpart : 0;
    do {
      const int nkb = PARTS ? (int)(nkb_all - k0 < ga->kpart ? nkb_all - k0 : ga->kpart) : CHUNKED ? (int)(nkb_all - k0 < chunk ? nkb_all - k0 : chunk) : (int)nkb_all;
      // sources of this wave's copies at block k0: copy x moves fragment wave +
      // x NW of the block's B' (then A') fragments, slice-major
      const int8_t *src[XC];
      {
        const int64_t planeB = pr->nrbP * 2 * rowst, planeA = pr->nrbQ * 2 * rowst;
        const int8_t *sp = pr->SP + (tj * FJ) * rowst + k0 * kFragBytes;
        const int8_t *sq = pr->SQ + k0 * kFragBytes;
#pragma unroll
        for (int x = 0; x < XB; ++x) {
          const int c = wave + x * NW;
          src[x] = sp + (int64_t)(c / FJ) * planeB + (int64_t)(c % FJ) * rowst;
        }
#pragma unroll
        for (int x = 0; x < XA; ++x) {
          const int c = wave + x * NW;
          src[XB + x] = sq + (int64_t)(c / FI) * planeA + (ti * FI + c % FI) * rowst;
        }
      }
      // Copy x of block kb. b_buf, a_buf: LDS offsets of the block's B' and A'.
      auto copy = [&](int x, uint32_t voff, int b_buf, int a_buf) {
        const bool isb = x < XB;
        const int c = wave + (isb ? x : x - XB) * NW;
        if (isb ? (NCB % NW == 0 || c < NCB) : (NCA % NW == 0 || c < NCA))
          tile::copy_frag_s(src[x], voff, lds + (isb ? b_buf : a_buf) + c * kFragBytes);
      };
      auto b_off = [&](int st) { return RING ? st * STAGE : 0; };
      auto a_off = [&](int st) {
        return RING ? st * STAGE + NCB * kFragBytes : (NCB + st * NCA) * kFragBytes;
      };

#pragma unroll
      for (int ib = 0; ib < IB; ++ib)
#pragma unroll
        for (int t = 0; t < S; ++t) acc[ib][t] = v4i{0};

      v4i pf[S], qf[R];
      // LDS addresses of this wave's fragments in the first B' and A' buffer. (The
      // asm keeps their constant parts out of the reads' offsets, which then fit
      // the 16 bits of the instruction.)
      uint32_t lb = tile::lds_addr(lds) + lane16 + wj * kFragBytes;
      uint32_t lq = tile::lds_addr(lds) + lane16 + a_off(0) + wi * IB * kFragBytes;
      asm volatile("" : "+v"(lb), "+v"(lq));
      auto rdB = [&](int q, uint32_t base) { pf[q] = tile::lds_read(base + q * FJ * kFragBytes); };
      auto rdA = [&](int n, int slot, uint32_t base) {  // fragment n = p IB + ib
        qf[slot] = tile::lds_read(base + ((n / IB) * FI + n % IB) * kFragBytes);
      };
      constexpr int NST = RING ? 3 : 2;
      constexpr uint32_t kStepB = RING ? STAGE : 0, kStepA = RING ? STAGE : NCA * kFragBytes;

#pragma unroll
      for (int x = 0; x < XC; ++x) copy(x, lane16, b_off(0), a_off(0));
      if (RING && nkb > 1) {
#pragma unroll
        for (int x = 0; x < XC; ++x) copy(x, lane16 + kFragBytes, b_off(1), a_off(1));
        wait_vmcnt<MINC>();
      } else {
        wait_vmcnt<0>();
      }
      barrier_only();
#pragma unroll
      for (int n = 0; n < LA; ++n) rdA(n, n, lq);
#pragma unroll
      for (int q = S - 1; q > 0; --q) rdB(q, lb);

      int st = 0;
      for (int kb = 0; kb < nkb; ++kb) {
        const int st1 = st + 1 == NST ? 0 : st + 1;
        const uint32_t bo = lb + st * kStepB, ao = lq + st * kStepA;
        const uint32_t bn = lb + st1 * kStepB, an = lq + st1 * kStepA;
        // blocks whose copies start in this one: the second next (RING) or the next
        const int ahead = RING ? 2 : 1;
        const int stc = RING ? (st1 + 1 == 3 ? 0 : st1 + 1) : st1;
        const int bc = b_off(stc), ac = a_off(stc);
        const uint32_t voff = lane16 + (uint32_t)(kb + ahead) * kFragBytes;
        const bool fill = kb + ahead < nkb;
        // The reads of the next block are unconditional: after the last one they
        // fetch what LDS happens to hold, which nothing uses.
        unrolled(std::make_integer_sequence<int, NA>{}, [&](auto nc) {
          constexpr int n = decltype(nc)::value;
          constexpr int p = n / IB, ib = n % IB;
          if constexpr (n == NX) {
            // RING: the next block's copies have landed, here and (after the
            // barrier) in every wave. Otherwise X. Either way every wave has
            // used its reads of the block before this one and of this B'.
            if (RING) wait_vmcnt<0>();
            barrier_only();
          }
          if constexpr (!RING && n == NY) {
            wait_vmcnt<0>();
            barrier_only();
          }
          rdA((n + LA) % NA, (n + LA) % R, n + LA < NA ? ao : an);
          // B' slice 1 of this block (used last in the first step), then the
          // next block's slices over those done with
          if constexpr (n == 0) rdB(0, bo);
          if constexpr (p >= 1 && p == PY) {
#pragma unroll
            for (int x = 0; x < PY; ++x)
              if (x * IB / PY == ib) rdB(S - 1 - x, bn);
          } else if constexpr (p > PY && ib == 0) {
            rdB(S - p, bn);
          }
          if (n >= NX && n < NX + IB && fill) {
#pragma unroll
            for (int x = 0; x < XC; ++x)
              if (x * IB / XC == n - NX) copy(x, voff, bc, ac);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int qq = 0; qq < S - p; ++qq) {
            constexpr bool desc = p == 0;
            const int q = desc ? S - 1 - qq : qq;
            acc[ib][p + q] =
                __builtin_amdgcn_mfma_i32_16x16x64_i8(pf[q], qf[n % R], acc[ib][p + q], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (NA % R != 0) {
          // the look-ahead fragments to the slots the next block expects
          v4i tmp[LA];
#pragma unroll
          for (int n = 0; n < LA; ++n) tmp[n] = qf[(NA + n) % R];
#pragma unroll
          for (int n = 0; n < LA; ++n) qf[n] = tmp[n];
        }
        st = st1;
      }
      // every wave is done reading LDS before the next chunk or tile refills it
      barrier_only();

      if (CHUNKED) {
        char *cb = carry_base();
        if (!wide) {
          cb += slots * kSlot;
#pragma unroll
          for (int w = 0; w < WORDS; ++w) {
            __hip_atomic_store(carry_word<int32_t>(cb, w, lane), acc_word(w), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            if (w % 4 == 3) __builtin_amdgcn_sched_barrier(0);
          }
        } else {
#pragma unroll
          for (int w = 0; w < WORDS; ++w) {
            int64_t *p = carry_word<int64_t>(cb, w, lane);
            // (asm: the compiler extended all words ahead of the branch, which
            // spilled 99 registers at S = 9 and 356 at S = 6: z 4096 x 1024 x
            // 16384 S = 9 11.9 ms, now 9.3; 2048^2 x 20000 S = 9 13.3, 11.4, S = 6
            // 5.42, 5.30)
            int32_t a = acc_word(w);
            asm volatile("" : "+v"(a));
            const int64_t v = a;
            if (slots == 0)
              __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else
              __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (w % 4 == 3) __builtin_amdgcn_sched_barrier(0);
          }
        }
        ++slots;
        wait_vmcnt<0>();  // the copies' vmcnt counts stay to themselves
      }
      k0 += chunk;
    } while (CHUNKED && k0 < nkb_all);

    if constexpr (PARTS) {
      char *cb = reinterpret_cast<char *>(ga->parts) + (tn * ga->ksplit + item / ntiles) * kSlot +
                 (int64_t)wave * (WORDS * 64) * sizeof(int32_t);
#pragma unroll
      for (int w = 0; w < WORDS; ++w) {
        *carry_word<int32_t>(cb, w, lane) = acc_word(w);
        if (w % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
      wait_vmcnt<0>();  // the copies' vmcnt counts stay to themselves
      continue;
    }

    // ------------------------------------------------------------ epilogue
    // (the problem's fields are fetched again here, not kept through the loop)
    asm volatile("" : "+s"(pr));
    const int64_t i0 = ti * C_::BI + wi * IB * 16 + (lane & 15);
    const int64_t j0 = tj * C_::BJ + wj * 16 + 4 * (lane >> 4);
    unrolled(std::make_integer_sequence<int, IB>{}, [&](auto ibc) {
      constexpr int ib = decltype(ibc)::value;
      // The block from the accumulators (K 0), or from its chunk sums: one or two INT32
      // ones (1, 2) or int64 (3). The last chunk's go to memory like the others', which ends
      // the accumulators' life there: kept for the epilogue they took registers from the
      // chunk loop (16384^3 complex, S = 6, 1.8% slower).
      auto finish = [&](auto kind) {
        constexpr int K = decltype(kind)::value;
        auto total = [&](int t, int r) -> int64_t {
          const int w = (ib * S + t) * 4 + r;
          int64_t v = K == 0 ? acc[ib][t][r] : 0;
          if constexpr (K == 3)
            v = __hip_atomic_load(carry_word<int64_t>(carry_base(), w, lane), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
          if constexpr (K == 2 || K == 1)
#pragma unroll
            for (int c = 0; c < K; ++c)
              v += __hip_atomic_load(carry_word<int32_t>(carry_base() + c * kSlot, w, lane),
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          return v;
        };
        if constexpr (RAW) {
          tile::store_raw<S>(pr, total, i0 + ib * 16, j0);
        } else {
          double val[4];
          const int wbits = pr->wbits, woff = pr->woff;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            val[r] = 0.0;
#pragma unroll
            for (int t = 0; t < S; ++t)
              val[r] = add_rn(val[r], ldexp(K == 0 ? (double)acc[ib][t][r] : (double)total(t, r),
                                            woff - wbits * (t + 2)));
            // one entry's loads at a time (all at once need too many registers)
            if constexpr (K != 0) __builtin_amdgcn_sched_barrier(0);
          }
          tile::store_block(pr, val, i0 + ib * 16, j0);
        }
      };
      if constexpr (!CHUNKED)
        finish(std::integral_constant<int, 0>{});
      else if (wide)
        finish(std::integral_constant<int, 3>{});
      else if (slots == 1)
        finish(std::integral_constant<int, 1>{});
      else
        finish(std::integral_constant<int, 2>{});
      // one block at a time
      __builtin_amdgcn_sched_barrier(0);
    });
  }
}

// The parts of every tile added (int64: their total may pass 2^31) and finished
// as in the epilogue above. One workgroup per 16 x 16 block, a wave per row r of
// the MFMA result's four: bound by the latency of its loads, so four parts' sums
// are in flight at a time (one wave per block and one part at a time took 1 to 8
// us per part).
template <int S, int WJ, int WI, int IB>
__global__ void __launch_bounds__(256) k_ozparts(GemmArgs G) {
  using C_ = Cfg<S, WJ, WI, IB>;
  constexpr int WORDS = IB * S * 4, kAhead = 4;
  __shared__ double rows[4][64];
  const ArgsPtr ga = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int lane = threadIdx.x & 63;
  const int r = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t tn = blockIdx.x / (C_::NW * IB);
  const int wave = (int)(blockIdx.x / IB % C_::NW), ib = (int)(blockIdx.x % IB);
  const int ksplit = ga->ksplit;
  int64_t sum[S];
#pragma unroll
  for (int t = 0; t < S; ++t) sum[t] = 0;
  const int32_t *p = ga->parts + (tn * ksplit * C_::NW + wave) * (int64_t)(WORDS * 64) +
                     (ib * S * 4 + r) * 64 + lane;
  constexpr int64_t kPart = (int64_t)C_::NW * WORDS * 64;
  for (int k = 0; k < ksplit; k += kAhead) {
    int32_t v[kAhead][S];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int32_t *q = p + (k + u < ksplit ? k + u : k) * kPart;
#pragma unroll
      for (int t = 0; t < S; ++t) v[u][t] = q[t * 256];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
#pragma unroll
      for (int t = 0; t < S; ++t) sum[t] += k + u < ksplit ? v[u][t] : 0;
  }
  double val = 0.0;
  const int wbits = ga->one.wbits, woff = ga->one.woff;
#pragma unroll
  for (int t = 0; t < S; ++t) val = add_rn(val, ldexp((double)sum[t], woff - wbits * (t + 2)));
  rows[r][lane] = val;
  __syncthreads();
  if (r != 0) return;
  int64_t tj, ti;
  tile::tile_coords(tn, 0, ga->one.m, ga->one.nprime, C_::BJ, C_::BI, tj, ti);
  const double all[4] = {rows[0][lane], rows[1][lane], rows[2][lane], rows[3][lane]};
  tile::store_block(&ga->one, all, ti * C_::BI + ((wave / WJ) * IB + ib) * 16 + (lane & 15),
                    tj * C_::BJ + (wave % WJ) * 16 + 4 * (lane >> 4));
}

template <int S, int WJ, int WI, int IB, int WPS, bool RING, int LA, bool RAW, int MODE>
hipError_t launch_cfg(const GemmArgs &a, int num_cu, hipStream_t st) {
  using C_ = Cfg<S, WJ, WI, IB>;
  const int64_t ntiles = a.probs != nullptr
                             ? a.ntiles
                             : ((a.one.nprime + C_::BJ - 1) / C_::BJ) * ((a.one.m + C_::BI - 1) / C_::BI);
  // persistent grid: WPS waves per SIMD, i.e. one workgroup of 8 waves per CU or
  // two of 4 (whose barriers are independent, so one's MFMAs fill the other's waits)
  int64_t grid = std::min<int64_t>(MODE == kParts ? ntiles * a.ksplit : ntiles,
                                   (int64_t)(4 * WPS / C_::NW) * num_cu);
  if (a.max_groups > 0) grid = std::min<int64_t>(grid, a.max_groups);
  if (grid <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_ozgemm<S, WJ, WI, IB, WPS, RING, LA, RAW, MODE>), dim3((unsigned)grid),
                     dim3(64 * C_::NW), 0, st, a);
  if constexpr (MODE == kParts)
    hipLaunchKernelGGL((k_ozparts<S, WJ, WI, IB>), dim3((unsigned)(ntiles * C_::NW * IB)), dim3(256), 0,
                       st, a);
  return hipGetLastError();
}

// Tile shapes. All use 16 x 16 x 64 INT8 MFMA blocks and one INT32 accumulator
// set per diagonal; a wave has one 16-row block of B' and IB of A'.
//   128 x 128 (j' x i): 8 waves of 16 x 128; S <= 6, whose 8 S sets, S B' and 4
//     A' fragments fit the 256 registers
//   128 x 64: 8 waves of 16 x 64; S <= 10 (LDS)
//   64 x 128: 8 waves, 4 x 2, each 16 x 64; S <= 8 (LDS)
//   64 x 64: 4 waves of 16 x 64, two workgroups per CU, while two fit the LDS (S
//     <= 6); else 8 waves, 4 x 2, each 16 x 32
//   32 x 32: 4 waves, 2 x 2, each 16 x 16; 4 <= S (ring LDS plan), no chunks: four
//     times the workgroups and a quarter of the chain per block of 64 x 64, for
//     products that do not fill the chip
// With 32 x 64 (B' halves in turn, S = 6) or 32 x 32 per wave the LDS reads were
// fewer, but one needed a few registers too many and the other larger copies:
// 4096^3 complex S = 6 5264 and 4207 us against 3627, 4096^3 real S = 7 1260
// against 1230; 128 x 96 tiles 3776 and 1279.
enum Shape { kBig, kTall, kWide, kSmall, kTiny };

// Tile configurations 0 .. 6 (the autotuner's candidates): 6 is 128 x 128, 1 is
// 64 x 128, 4 and 5 are 64 x 64, the others 128 x 64; the shapes a slice count
// is too large for fall back to the next smaller one. A tuning id below 14 is 2
// * configuration + tile order (0: consecutive tiles walk down the rows i, 1:
// along the columns j'); ids 14 .. 20 are configurations 0 .. 6 with the grouped
// tile order 2, ids 21 .. 27 with the XCD-aware order 3 (see tile_coords and
// xcd_major).
constexpr int kNumCfg = 7;
constexpr int kTinyId = 4 * kNumCfg;  // beyond the autotuner's: 32 x 32, chosen by sizes only
constexpr int id_cfg(int id) {
  return id == kTinyId ? kNumCfg : id < 2 * kNumCfg ? id >> 1 : (id - 2 * kNumCfg) % kNumCfg;
}
constexpr int id_order(int id) { return id == kTinyId ? 0 : id < 2 * kNumCfg ? (id & 1) : 2 + (id - 2 * kNumCfg) / kNumCfg; }

constexpr Shape shape_of(int S, int cfg) {
  if (cfg == kNumCfg && S >= 4) return kTiny;
  if (S >= 11 || cfg == 4 || cfg == 5 || cfg == kNumCfg) return kSmall;
  if (cfg == 6 && S <= 6) return kBig;
  return cfg == 1 && S <= 8 ? kWide : kTall;
}
constexpr int shape_bj(Shape s) { return s == kTiny ? 32 : s == kBig || s == kTall ? 128 : 64; }
constexpr int shape_bi(Shape s) { return s == kTiny ? 32 : s == kBig || s == kWide ? 128 : 64; }

constexpr bool ring_fits(int bytes, int groups) { return bytes * groups <= 160 * 1024; }

template <int S, bool RAW, int MODE>
hipError_t launch_shape(Shape shape, const GemmArgs &a, int num_cu, hipStream_t st) {
  constexpr int LA = S == 1 ? 1 : 3;
  // raw sums take 128 x 64 or 64 x 64 tiles, parts 64 x 64 ones
  constexpr bool all = !RAW && MODE != kParts;
  if (shape == kBig) {
    if constexpr (S <= 6 && all)
      return launch_cfg<S, 8, 1, 8, 2, ring_fits(Cfg<S, 8, 1, 8>::RingBytes, 1), LA, RAW, MODE>(a, num_cu, st);
  } else if (shape == kTall) {
    if constexpr (S <= 10 && MODE != kParts)
      return launch_cfg<S, 8, 1, 4, 2, ring_fits(Cfg<S, 8, 1, 4>::RingBytes, 1), LA, RAW, MODE>(a, num_cu, st);
  } else if (shape == kWide) {
    if constexpr (S <= 8 && all)
      return launch_cfg<S, 4, 2, 4, 2, ring_fits(Cfg<S, 4, 2, 4>::RingBytes, 1), LA, RAW, MODE>(a, num_cu, st);
  } else if (shape == kTiny) {
    if constexpr (S >= 4 && !RAW && MODE != kChunked)
      return launch_cfg<S, 2, 2, 1, 1, true, LA, RAW, MODE>(a, num_cu, st);
  } else {
    if constexpr (S <= 6)
      return launch_cfg<S, 4, 1, 4, 2, ring_fits(Cfg<S, 4, 1, 4>::RingBytes, 2), LA, RAW, MODE>(a, num_cu, st);
    else
      return launch_cfg<S, 4, 2, 2, 2, false, LA, RAW, MODE>(a, num_cu, st);
  }
  return hipErrorInvalidValue;
}

template <int S>
hipError_t launch_s(int cfg, const GemmArgs &a, int num_cu, hipStream_t st) {
  const bool raw = a.one.raw != nullptr;
  const Shape shape = shape_of(S, raw ? 0 : cfg);
  if (raw)
    return a.chunked ? launch_shape<S, true, kChunked>(shape, a, num_cu, st)
                     : launch_shape<S, true, kWhole>(shape, a, num_cu, st);
  if (a.ksplit > 1) return launch_shape<S, false, kParts>(shape, a, num_cu, st);
  return a.chunked ? launch_shape<S, false, kChunked>(shape, a, num_cu, st)
                   : launch_shape<S, false, kWhole>(shape, a, num_cu, st);
}

}  // namespace

int64_t kb_chunk_for(int S, bool b8) { return chunk_blocks(S, b8 ? 128 : 127); }

int gemm_num_configs() { return 4 * kNumCfg; }

size_t gemm_flush_bytes(int S, int num_cu) {
  // one int64 per accumulator word of one 128 x 128 tile per CU (the other
  // shapes need no more, so that a plan is valid whichever configuration runs);
  // two INT32 sums per word take the same space
  static_assert(kInt32Chunks <= 2, "INT32 chunk sums fit the int64 space");
  return (size_t)num_cu * 128 * 128 * (size_t)S * sizeof(int64_t);
}

int64_t gemm_tiles(int S, int id, int64_t m, int64_t nprime) {
  const Shape s = shape_of(S, id_cfg(id));
  const int64_t BJ = shape_bj(s), BI = shape_bi(s);
  return ((nprime + BJ - 1) / BJ) * ((m + BI - 1) / BI);
}

namespace {
// Estimated time in us of one tile over `kb` contraction blocks of 64. Per block a
// workgroup takes the larger of its share of the MFMA rate (`rate` times that of
// back-to-back MFMAs, two 64 x 64 workgroups of a CU in turn if `full`) and the
// latency of one alone.
constexpr int shape_groups(Shape s, int S) { return s == kSmall && S <= 6 ? 2 : 1; }  // per CU
double tile_time(Shape s, int S, int64_t kb, bool full) {
  const double mfma = S * (S + 1) / 2 * 16 / 2400.0;  // one 16 x 16 x 64 block, on each SIMD
  const double alone = shape_bj(s) * shape_bi(s) / 1024 * mfma;
  if (s == kTiny) return 2.4 + kb * std::max(2.13 * alone, 1.19 * alone + 0.38);
  const int groups = shape_groups(s, S);
  const double rate = s == kBig ? 1.41 : s == kTall ? 1.44 : groups == 2 ? 1.89 : 1.72;
  return 1.7 + kb * std::max((full ? groups : 1) * rate * alone, 1.19 * alone + 0.26);
}
constexpr bool shape_takes(Shape s, int S) {
  return s == kBig ? S <= 6 : s == kTall ? S <= 10 : s == kTiny ? S >= 4 : true;
}
int64_t shape_tiles(Shape s, int64_t m, int64_t nprime) {
  return ((nprime + shape_bj(s) - 1) / shape_bj(s)) * ((m + shape_bi(s) - 1) / shape_bi(s));
}
}  // namespace

GemmChoice gemm_choose(int S, int64_t m, int64_t nprime, int64_t nkb, int64_t kb_chunk, int num_cu,
                       size_t parts_bytes, size_t *need) {
  // The least estimate over tile shapes and numbers of parts. The parts' sums are
  // written and read once, by 64 x 64 and 32 x 32 tiles only (128 x 64 ones were
  // never faster). Fitted to 260 products of sides 16 .. 8192 at S = 3 .. 12 in up
  // to 70 ways each: about 1.5% slower on average than the fastest way of each.
  // Before, 128 x 64 tiles for all: z 64 x 64 x 4096 S = 7 246 us, now 17; z 256 x
  // 256 x 8192 475, now 70; z 517 x 389 x 1031 72, now 41; z 1500 x 700 x 300 57,
  // now 50. 64 x 64 / 32 x 32 tiles: d 256^3 12.2 / 8.8, z 256^3 15.6 / 10.8, d
  // 512^3 16.7 / 11.3, but z 700 x 700 x 128 14.1 / 20.9.
  // Up to 64 rows 128 x 64 tiles read B' no less often than 64 x 64 ones, of which a
  // CU runs two up to S = 6 (z 64 x 100000 x 128 S = 6 264 / 246, z 16 x 40000 x 700
  // S = 5 435 / 417, z 64 x 12500 x 100 S = 5 38.0 / 36.4).
  const int64_t kb = nkb / 2, chunk = std::max<int64_t>(kb_chunk / 2, 1);
  GemmChoice best{0, 1, kb};
  double best_t = 1e300;
  *need = 0;
  for (const Shape s : {kTall, kBig, kSmall, kTiny}) {
    if (!shape_takes(s, S) || (s == kTall && m <= 64 && S <= 6)) continue;
    const int64_t area = (int64_t)shape_bj(s) * shape_bi(s), tiles = shape_tiles(s, m, nprime);
    for (int64_t ks = 1; ks <= (s == kSmall || s == kTiny ? 64 : 1); ++ks) {
      const int64_t part = (kb + ks - 1) / ks, items = tiles * ks;
      const size_t bytes = ks > 1 ? (size_t)items * area * S * sizeof(int32_t) : 0;
      if (ks > 1 && (part < 2 || items > 4 * num_cu)) break;
      if (ks > 1 && ((ks - 1) * part >= kb || bytes > parts_bytes)) continue;
      if ((ks > 1 || s == kTiny) && part > chunk) continue;  // (32 x 32 tiles carry no chunks)
      const int64_t slots = num_cu * shape_groups(s, S), rounds = (items + slots - 1) / slots;
      double t = rounds * tile_time(s, S, part, items > num_cu);
      if (s != kTiny) t += 1.3;
      if (ks > 1) t += 2.1 + 0.38e-6 * bytes + 0.13 * ks;
      if (t < best_t) {
        best_t = t;
        // 128-row tiles in XCD-aware groups, but down the rows where a tall product is
        // much wider still (z 5000 x 40000 x 16 S = 7 1590 / 1351, x 400 7720 / 7380;
        // z 8000^2 x 64 S = 6 475 / 500, z 700 x 5000 x 100 S = 7 69 / 76); the others
        // down the rows
        const bool wide = m >= 4096 && nprime >= 8 * m;
        best = GemmChoice{s == kBig ? (wide ? 12 : 27) : s == kTall ? (wide ? 4 : 21) : s == kSmall ? 8 : kTinyId,
                          (int)ks, part};
        *need = bytes;
      }
    }
  }
  return best;
}

int gemm_choose_grouped(int S, const std::vector<GemmSize> &probs, int64_t kb_chunk, int num_cu) {
  // The tiles of the first CU, the longest of each round (the table is sorted by the
  // contraction), with the estimate above; two workgroups of a CU take their tiles
  // in turn. Against 128 x 128 (S <= 6) or 128 x 64 tiles for every batch (z, sides
  // 32 .. 1024): 9 problems S = 8 47 / 77 us, 23 S = 7 47 / 74, 12 S = 6 37 / 89.
  int best = 0;
  double best_t = 1e300;
  for (const Shape s : {kBig, kTall, kSmall, kTiny}) {
    // (128 x 64 tiles were never the fastest while 128 x 128 ones are there)
    if (!shape_takes(s, S) || (s == kTall && shape_takes(kBig, S))) continue;
    if (s == kTiny && !probs.empty() && probs[0].nkb > kb_chunk) continue;  // carries no chunks
    double t = s == kTiny ? 0.0 : 1.3;
    int64_t done = 0, next = 0;
    for (const GemmSize &p : probs) {
      done += shape_tiles(s, p.m, p.nprime);
      const int64_t mine = done > next ? (done - next + num_cu - 1) / num_cu : 0;
      t += mine * tile_time(s, S, p.nkb / 2, false);
      next += mine * num_cu;
    }
    if (t < best_t) {
      best_t = t;
      best = s == kBig ? 13 : s == kTall ? 1 : s == kSmall ? 8 : kTinyId;
    }
  }
  return best;
}

hipError_t launch_ozgemm(int S, int tune_id, const GemmArgs &a0, int num_cu, hipStream_t st) {
  GemmArgs a = a0;
  a.order = id_order(tune_id);
  const int cfg = id_cfg(tune_id);
  switch (S) {
#define OZ_CASE(N) \
  case N: return launch_s<N>(cfg, a, num_cu, st);
    OZ_CASE(1) OZ_CASE(2) OZ_CASE(3) OZ_CASE(4) OZ_CASE(5) OZ_CASE(6)
    OZ_CASE(7) OZ_CASE(8) OZ_CASE(9) OZ_CASE(10) OZ_CASE(11) OZ_CASE(12)
#undef OZ_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace oz
