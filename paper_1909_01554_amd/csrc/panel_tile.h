// Device code of one workgroup tile of the matrix-core leaves whose operand rows go to LDS
// by direct loads and become matrix-core operands by masks alone.
//
// Tile and staging.  Four waves (2 x 2) own 64 RA rows by 64 RB columns of C, 32 RA x 32 RB
// each.  A stage is 8 words of k (512 bits) of the tile's rows of A and of B^T: 24 KB, two
// buffers.  A stage is loaded with global_load_lds_dwordx4, which needs no registers, so the 128 counts, two sets of raw
// words and the expanded operands fit in 256 registers (two workgroups per CU) without
// scratch.  A row's four 16-byte chunks are stored rotated by an XOR with bits 1..2 of the
// row, so that the 8 lanes served together by a 16-byte LDS read hit distinct banks; the
// direct loads write LDS linearly, so it is the lane's source address that is permuted.
// A stage is two rounds of 256 bits; round 0 of the next stage is read from LDS while the
// last round of this one is computed, and one barrier per stage, before that read, both
// publishes the next stage and frees this one's buffer for the stage after.
//
// Operands.  The order of k inside a dot product is free as long as both sides use the
// same one.  Lane half h of a round holds 128 consecutive bits (4 dwords) of its row; one
// matrix-core step takes bit plane d of all four dwords, i.e. 128 / planes bits per lane:
//   E2M1: nibble bit d, d = 0..2, is the value 0.5, 1 or 2 where it lies, so one AND makes
//   an operand; bit 3 (the sign) is moved to bit 1 first.  The products 0.25, 1, 4 and 1
//   are brought to 1 by the instruction's block scales, and the fp32 sum is the count,
//   exact below 2^24.  4.5 VALU instructions per 32 bits of a row instead of 7.
//   int8: byte bit d of one side is 2^d; the other side has the bits of each byte reversed
//   (2 instructions per dword, once for all planes), so its mask gives 2^(7-d) and every
//   product is 2^7.  For GF(2) the signs of the planes 0 and 7 do not matter (the parity
//   is bit 7 of the sum); for OR these two planes are moved one bit inward, so that all
//   products are positive.  Exact while 2^7 k < 2^31, i.e. k < 2^24.  8 to 10 VALU
//   instructions per 32 bits of a row instead of 11.5 to 15.
//
// Bound by the matrix cores: 2401 fp4 products of 2048^3 on dense bits take 6.6 ms (6.2e15
// bit ops/s; 5.3e15 before, with register-fed 128 x 64 tiles), one of 16384^3 1.20 ms on
// dense bits (7.2e15) and 1.06 ms on sparse ones (8.2e15), where a kernel of nothing but
// these instructions reaches 9.3e15; dense bits lower the clock.  int8: 4.6e15 of 4.7e15.
#pragma once

#include <type_traits>

#include "bit_transpose.h"
#include "lds_load.h"
#include "mfma_tile.h"

namespace bmm {
namespace panel {

using mfma::FMT_F4;
using mfma::FMT_I8;
using mfma::SEMI_ANY;
using mfma::v16f;
using mfma::v16i;
using mfma::v4i;
using mfma::v8i;

typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int kWords = 8;               // words of k per stage
constexpr int kRowBytes = 8 * kWords;   // LDS row
constexpr int64_t kMaxK = kPanelMaxK;

constexpr int lds_bytes(int RA, int RB) { return 2 * 64 * (RA + RB) * kRowBytes; }

// This wave's LDS reads, LDS writes and direct loads are done, then everyone's.
__device__ __forceinline__ void stage_sync() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ---- operands ----

// Bits of each byte reversed.
__device__ __forceinline__ u4 reverse_bytes(u4 x) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    x[i] = __builtin_amdgcn_perm(0, __builtin_bitreverse32(x[i]), 0x00010203u);
  return x;
}

// (x << -S or x >> S) & mask, two dwords per 64-bit shift: the bits that cross dwords or
// fields are outside the masks used here.
template <int S>
__device__ __forceinline__ v4i shift_mask(u4 x, uint32_t mask) {
  v4i o;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint64_t q = ((uint64_t)x[2 * i + 1] << 32) | x[2 * i];
    const uint64_t y = S > 0 ? q >> (S > 0 ? S : 0) : q << (S > 0 ? 0 : -S);
    o[2 * i] = (int)((uint32_t)y & mask);
    o[2 * i + 1] = (int)((uint32_t)(y >> 32) & mask);
  }
  return o;
}

template <int FMT>
struct Planes;
template <>
struct Planes<FMT_F4> {
  static constexpr int N = 4;
};
template <>
struct Planes<FMT_I8> {
  static constexpr int N = 8;
};

// Plane D of 128 bits of a row.  REV (int8): the side with reversed bytes.
template <int FMT, int D, bool REV, bool SIGNED_OK>
__device__ __forceinline__ v4i plane(u4 x) {
  if constexpr (FMT == FMT_F4) {
    if constexpr (D == 3) return shift_mask<2>(x, 0x22222222u);
    else return __builtin_bit_cast(v4i, x & (0x11111111u << D));
  } else {
    if constexpr (!SIGNED_OK && D == (REV ? 7 : 0)) return shift_mask<-1>(x, 0x02020202u);
    else if constexpr (!SIGNED_OK && D == (REV ? 0 : 7)) return shift_mask<1>(x, 0x40404040u);
    else return __builtin_bit_cast(v4i, x & (0x01010101u << (REV ? 7 - D : D)));
  }
}

__device__ __forceinline__ v8i widen(v4i x) {
  return __builtin_shufflevector(x, x, 0, 1, 2, 3, -1, -1, -1, -1);
}

template <int FMT, int D>
__device__ __forceinline__ typename mfma::Acc<FMT>::type step(
    v4i a, v4i b, typename mfma::Acc<FMT>::type acc) {
  if constexpr (FMT == FMT_F4) {
    // E8M0 scales 2^(s - 127) on both sides: 0.25, 1, 4, 1 become 1
    constexpr int s = D == 0 ? 128 : D == 2 ? 126 : 127;
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(a), widen(b), acc, 4, 4, 0, s, 0,
                                                           s);
  } else {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc, 0, 0, 0);
  }
}

// The counts are computed where this is called.
__device__ __forceinline__ void computed(const v16f& acc) { asm volatile("" ::"v"(acc)); }
__device__ __forceinline__ void computed(const v16i& acc) { asm volatile("" ::"v"(acc)); }

// One round: 128 bits per lane (256 per row) of RA rows of A and RB rows of B^T.
template <int SEMI, int FMT, int RA, int RB, class AccV>
__device__ __forceinline__ void mfma_round(u4 (&xa)[RA], u4 (&xb)[RB], AccV (&acc)[RA][RB]) {
  constexpr bool SIGNED_OK = SEMI == GF2;
  constexpr bool REV_A = RA < RB;  // int8: the side with fewer rows is reversed
  if constexpr (FMT == FMT_I8) {
#pragma unroll
    for (int f = 0; f < RA; ++f)
      if constexpr (REV_A) xa[f] = reverse_bytes(xa[f]);
#pragma unroll
    for (int g = 0; g < RB; ++g)
      if constexpr (!REV_A) xb[g] = reverse_bytes(xb[g]);
  }
  auto one = [&](auto dc) {
    constexpr int D = decltype(dc)::value;
    if constexpr (D < Planes<FMT>::N) {
      v4i eb[RB];
#pragma unroll
      for (int g = 0; g < RB; ++g) eb[g] = plane<FMT, D, !REV_A, SIGNED_OK>(xb[g]);
#pragma unroll
      for (int f = 0; f < RA; ++f) {
        const v4i ea = plane<FMT, D, REV_A, SIGNED_OK>(xa[f]);
#pragma unroll
        for (int g = 0; g < RB; ++g) acc[f][g] = step<FMT, D>(ea, eb[g], acc[f][g]);
      }
    }
  };
  one(std::integral_constant<int, 0>{});
  one(std::integral_constant<int, 1>{});
  one(std::integral_constant<int, 2>{});
  one(std::integral_constant<int, 3>{});
  one(std::integral_constant<int, 4>{});
  one(std::integral_constant<int, 5>{});
  one(std::integral_constant<int, 6>{});
  one(std::integral_constant<int, 7>{});
  // the round ends here: the compiler would otherwise sink it below the next barrier, and
  // the LDS reads issued before it would have nothing to hide behind
#pragma unroll
  for (int f = 0; f < RA; ++f)
#pragma unroll
    for (int g = 0; g < RB; ++g) computed(acc[f][g]);
  __builtin_amdgcn_sched_barrier(0);
}

// ---- results ----

// The 16 result bits of a lane's column of one 32 x 32 block, bit v of the upper half of
// the dword (E2M1 parity) or of the lower half (else): two instructions per count, one
// that brings the bit to an end of a register and one that shifts it in.
template <int FMT>
__device__ __forceinline__ constexpr bool packs_high(bool gf2) {
  return FMT == FMT_F4 && gf2;
}
template <int FMT>
__device__ __forceinline__ uint32_t pack16(const typename mfma::Acc<FMT>::type& acc, bool gf2) {
  uint32_t w = 0;
  if (packs_high<FMT>(gf2)) {
#pragma unroll
    for (int v = 0; v < 16; ++v) w = __builtin_amdgcn_alignbit((uint32_t)acc[v], w, 1);
  } else {
#pragma unroll
    for (int v = 15; v >= 0; --v) {
      uint32_t c;  // the result bit in bit 31
      if constexpr (FMT == FMT_F4) c = __float_as_uint(0.0f - acc[v]);  // a sign iff acc > 0
      else c = gf2 ? (uint32_t)acc[v] << 24 : 0u - (uint32_t)acc[v];
      w = __builtin_amdgcn_alignbit(w, c, 31);
    }
  }
  return w;
}

template <int SEMI, int FMT, int RA, int RB>
__device__ __forceinline__ void store_tile(const typename mfma::Acc<FMT>::type (&acc)[RA][RB],
                                           uint64_t* C, int64_t ldc, int64_t m, int64_t n,
                                           int64_t row0, int64_t word0, int accumulate,
                                           int semiring) {
  static_assert(RA % 2 == 0 && RB % 2 == 0, "blocks are packed in pairs");
  const bool gf2 = SEMI == SEMI_ANY ? semiring == GF2 : SEMI == GF2;
  const int lane = fresh_lane(), half = lane >> 5, li = lane & 31;
  const Transpose tr(lane);
  const int64_t n_words = (n + 63) >> 6;
  // after the transposition lane li of half h holds row r(li) of block f + h
  const int r = ((li >> 2) & 3) * 8 + (li >> 4) * 4 + (li & 3);
  const bool vec16 = RB == 4 && word0 + 1 < n_words &&
                     ((reinterpret_cast<uintptr_t>(C) & 15) | (uintptr_t)(ldc & 1)) == 0;
#pragma unroll
  for (int f = 0; f < RA; f += 2) {
    __builtin_amdgcn_sched_barrier(0);  // one row block at a time, to keep registers
    uint64_t word[RB / 2];
#pragma unroll
    for (int g = 0; g < RB; ++g) {
      const auto s = __builtin_amdgcn_permlane32_swap(
          pack16<FMT>(acc[f][g], gf2), pack16<FMT>(acc[f + 1][g], gf2), false, false);
      const uint32_t x =
          tr(__builtin_amdgcn_perm(s[1], s[0], packs_high<FMT>(gf2) ? 0x07060302u : 0x05040100u));
      if (g & 1) word[g / 2] |= (uint64_t)x << 32;
      else word[g / 2] = x;
    }
    const int64_t row = row0 + 32 * (f + half) + r;
    if (row < m) {
#pragma unroll
      for (int h = 0; h < RB / 2; ++h) {
        const int64_t valid = n - 64 * (word0 + h);
        word[h] &= valid >= 64 ? ~0ull : valid > 0 ? ((uint64_t)1 << valid) - 1 : 0ull;
      }
      const mfma::gw_ptr dst = (mfma::gw_ptr)C + row * ldc + word0;
      if (RB == 4 && vec16) {
        const mfma::gw2_ptr d2 = (mfma::gw2_ptr)dst;
        mfma::cpair_t x = {word[0], word[RB / 2 - 1]};
        if (accumulate) x = gf2 ? (x ^ *d2) : (x | *d2);
        *d2 = x;
      } else {
#pragma unroll
        for (int h = 0; h < RB / 2; ++h) {
          if (word0 + h >= n_words) break;  // uniform
          uint64_t x = word[h];
          if (accumulate) x = gf2 ? (x ^ dst[h]) : (x | dst[h]);
          dst[h] = x;
        }
      }
    }
  }
}

// ---- one workgroup tile ----

// The operands of one workgroup tile and the loads of their stages, made and called by all
// its waves.
template <int RA, int RB, bool FAR>
struct Operands {
  static constexpr int TM = 64 * RA, TN = 64 * RB, NL = (TM + TN) / 64;
  static constexpr int STAGE = (TM + TN) * kRowBytes;
  const uint64_t *Ab, *Bb;
  int64_t lda, ldbt, kw;
  int w;
  unsigned char* smem;
  uint32_t voff[NL];  // byte offset of the lane's chunk, or (FAR) its row

  // Load i of wave w fills LDS rows 16 (4 i + w) .. + 15, 4 lanes per row; rows past the
  // end of an operand repeat its last one (their results are not stored).
  static __device__ __forceinline__ int chunk_of(int ln) {  // of a lane's slot
    return (ln & 3) ^ ((ln >> 3) & 3);
  }
  __device__ __forceinline__ Operands(const uint64_t* __restrict__ A, int64_t lda_,
                                      const uint64_t* __restrict__ BT, int64_t ldbt_, int64_t m,
                                      int64_t k, int64_t n, int64_t im, int64_t in, int w_,
                                      unsigned char* smem_)
      : Ab(A + im * TM * lda_), Bb(BT + in * TN * ldbt_), lda(lda_), ldbt(ldbt_),
        kw((k + 63) >> 6), w(w_), smem(smem_) {
    const int lane = fresh_lane();
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const bool isA = 64 * i < TM;
      const int64_t lim = isA ? m - 1 - im * TM : n - 1 - in * TN;
      int r = 16 * (4 * i + w) + (lane >> 2) - (isA ? 0 : TM);
      r = r < lim ? r : (int)lim;
      voff[i] = FAR ? (uint32_t)r
                    : (uint32_t)r * ((uint32_t)(isA ? lda : ldbt) * 8) + 16 * chunk_of(lane);
    }
  }
  // the lane's chunk of load i in the stage at word w0
  __device__ __forceinline__ const uint64_t* source(int i, int64_t w0) const {
    const bool isA = 64 * i < TM;
    const uint64_t* base = (isA ? Ab : Bb) + w0;
    if (FAR) return base + (int64_t)voff[i] * (isA ? lda : ldbt) + 2 * chunk_of(fresh_lane());
    return (const uint64_t*)((const char*)base + voff[i]);
  }
  // Stage st into LDS buffer buf.
  __device__ __forceinline__ void load(int64_t st, int buf) const {
    typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)smem + w * 1024;
    const int64_t w0 = st * kWords;
    if (w0 + kWords <= kw) {  // uniform
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const uint32_t dst = lds0 + buf * STAGE + i * 4096;
        if (FAR) load_lds16(source(i, w0), dst);
        else load_lds16((64 * i < TM ? Ab : Bb) + w0, voff[i], dst);
      }
      return;
    }
    // the last, shorter stage: words past the end of k read as zero (the loads themselves
    // stay inside the row)
    const int lane = fresh_lane();
    const int left = (int)(kw - w0) - 2 * chunk_of(lane);  // words of the lane's chunk and after
    const int o0 = left > 0 ? 0 : left - 1, o1 = left > 1 ? 1 : left - 1;
    // (two loads at a time: the counts leave no registers for all of them)
#pragma unroll
    for (int i = 0; i < NL; i += 2) {
      __builtin_amdgcn_sched_barrier(0);
      uint64_t x[2][2] = {};
      if (kw > 0) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const mfma::gq_ptr src = (mfma::gq_ptr)source(i + j, w0);
          x[j][0] = src[o0];
          x[j][1] = src[o1];
        }
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        ulonglong2 v;
        v.x = left > 0 ? x[j][0] : 0ull;
        v.y = left > 1 ? x[j][1] : 0ull;
        *reinterpret_cast<ulonglong2*>(smem + w * 1024 + buf * STAGE + (i + j) * 4096 + lane * 16) = v;
      }
    }
  }
};

// The sums of one wave of the tile whose first stage is on its way to LDS buffer buf.
// loaded() runs on every wave once it has arrived (and with it whatever the wave had asked
// of memory before).  At the end other waves may still be reading their last stage.
struct NoHook {
  __device__ void operator()() const {}
};
template <int FMT>
using AccV = typename mfma::Acc<FMT>::type;
template <int SEMI, int FMT, int RA, int RB, bool FAR, class Hook = NoHook>
__device__ __forceinline__ void sums(const Operands<RA, RB, FAR>& op, int buf,
                                     AccV<FMT> (&acc)[RA][RB], Hook&& loaded = Hook()) {
  constexpr int TM = 64 * RA, STAGE = Operands<RA, RB, FAR>::STAGE;
  const int wy = op.w >> 1, wx = op.w & 1;
  const int64_t kw = op.kw;
  const int64_t stages = (kw + kWords - 1) / kWords;
  unsigned char* smem = op.smem;
  // raw words of two rounds: lane half h takes chunk 2 s + h of round s
  const int lane = fresh_lane(), half = lane >> 5, li = lane & 31;
  const int slot = (half ^ ((li >> 1) & 3)) * 16;
  const int abase = (wy * 32 * RA + li) * kRowBytes + slot;
  const int bbase = (TM + wx * 32 * RB + li) * kRowBytes + slot;
  u4 xa[2][RA], xb[2][RB];
  auto read = [&](int buf, int s) {
#pragma unroll
    for (int f = 0; f < RA; ++f)
      xa[s][f] = *reinterpret_cast<const u4*>(smem + buf * STAGE + (abase ^ (32 * s)) + 2048 * f);
#pragma unroll
    for (int g = 0; g < RB; ++g)
      xb[s][g] = *reinterpret_cast<const u4*>(smem + buf * STAGE + (bbase ^ (32 * s)) + 2048 * g);
  };
#pragma unroll
  for (int f = 0; f < RA; ++f)
#pragma unroll
    for (int g = 0; g < RB; ++g) acc[f][g] = AccV<FMT>{};
  stage_sync();
  loaded();
  if (stages > 1) op.load(1, buf ^ 1);
  read(buf, 0);
  // waves in their main loop go before the other workgroup's first loads and epilogue
  __builtin_amdgcn_s_setprio(1);
  int cur = buf;
  for (int64_t st = 0; st < stages; ++st) {
    read(cur, 1);
    mfma_round<SEMI, FMT>(xa[0], xb[0], acc);
    if (st + 1 < stages) {
      stage_sync();
      if (st + 2 < stages) op.load(st + 2, cur);
      read(cur ^ 1, 0);
    }
    if (st * kWords + 4 < kw) mfma_round<SEMI, FMT>(xa[1], xb[1], acc);  // else only zero words are left
    cur ^= 1;
  }
  __builtin_amdgcn_s_setprio(0);
}

// Rows [64 RA im, ...) x columns [64 RB in, ...) of C = A B, by the four waves w = 0..3 of
// a workgroup (all of them call it; every one takes part in loads and barriers).  Needs
// k < 2^24 and lds_bytes(RA, RB) of LDS, which nobody reads any more when it is called.
// FAR: pitches of kNearPitch words and more (64-bit row addresses).
// (Workgroups that took several tiles in turn, the next one's first stage loaded during
// the last stage of this one, were 7 to 10% slower than one workgroup per tile, which the
// hardware hands out as CUs come free: 62.8 against 57.8 ms for the n = 65536 recursion.)
template <int SEMI, int FMT, int RA, int RB, bool FAR>
__device__ __forceinline__ void tile(const uint64_t* __restrict__ A, int64_t lda,
                                     const uint64_t* __restrict__ BT, int64_t ldbt, uint64_t* C,
                                     int64_t ldc, int64_t m, int64_t k, int64_t n, int64_t im,
                                     int64_t in, int accumulate, int semiring, int w,
                                     unsigned char* smem) {
  Operands<RA, RB, FAR> op(A, lda, BT, ldbt, m, k, n, im, in, w, smem);
  AccV<FMT> acc[RA][RB];
  op.load(0, 0);
  sums<SEMI, FMT, RA, RB, FAR>(op, 0, acc);
  store_tile<SEMI, FMT, RA, RB>(acc, C, ldc, m, n, im * op.TM + (w >> 1) * 32 * RA,
                                (in * op.TN >> 6) + (w & 1) * (RB / 2), accumulate, semiring);
}

// ---- few rows: B row-major, turned on its way through LDS ----

// Rows [256 im, ...) x columns [64 WX in, ...) of C = A B, B given row-major, by a workgroup of
// 2 x WX waves of 128 x 64.  A's rows are staged as above, B's as they lie (the 512 rows of a
// stage, WX words each), loaded four stages before the products they are for; two stages
// before, every wave turns four of the 64 x 64 blocks in registers (31 VALU instructions
// each) into the columns' rows.  So B is read once where one row of tiles covers C, and is
// never copied.  Bound by the VALU work of the turns and planes beside the matrix
// instructions, among which the compiler spreads them (one run of code, without branches:
// m = 256, k = 32768, n = 32768, fp4 117 us, with the turns before the products of their own
// 129; n = 65536, dense bits, 225 and 236 us, a transpose of B and the panel leaf 303).
// 0 < k < 2^24, pitches below kNearPitch, n of at least WX words; smem: rows_bytes(WX).
constexpr int rows_bytes(int WX) { return (2 * 256 + 5 * 64 * WX) * kRowBytes; }

__device__ __forceinline__ void rows_sync() {  // all but the wave's last two loads
  asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int SEMI, int FMT, int WX>
__device__ __forceinline__ void rows_tile(const uint64_t* __restrict__ A, int64_t lda,
                                          const uint64_t* __restrict__ B, int64_t ldb, uint64_t* C,
                                          int64_t ldc, int64_t m, int64_t k, int64_t n, int64_t im,
                                          int64_t in, int accumulate, int w, unsigned char* smem) {
  constexpr int NW = 2 * WX, NL = 16 / NW, RA = 4, RB = 2;
  constexpr int kA = 256 * kRowBytes, kB = 64 * WX * kRowBytes;  // bytes of a stage
  constexpr int kRaw = 2 * kA, kTurned = kRaw + 3 * kB;          // where they start
  const int wy = w / WX, wx = w % WX;
  const int kw = (int)((k + 63) >> 6), stages = (kw + kWords - 1) / kWords;
  const int64_t row0 = im * 256, nw = (n + 63) >> 6;
  const int64_t word0 = in * WX < nw - WX ? in * WX : nw - WX;  // of the words read
  const int shift = (int)(in * WX - word0);
  const uint64_t* Ab = A + row0 * lda;
  const uint64_t* Bb = B + word0;
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)smem;

  auto chunk_of = [](int ln) { return (ln & 3) ^ ((ln >> 3) & 3); };
  uint32_t voff[NL];
  {
    const int lane = fresh_lane();
    const int64_t lim = m - 1 - row0;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      int r = 16 * (NW * i + w) + (lane >> 2);
      r = r < lim ? r : (int)lim;
      voff[i] = (uint32_t)r * ((uint32_t)lda * 8) + 16 * chunk_of(lane);
    }
  }
  auto load_a = [&](int st, int buf) {
    const int w0 = st * kWords;
    if (w0 + kWords <= kw) {
#pragma unroll
      for (int i = 0; i < NL; ++i)
        load_lds16(Ab + w0, voff[i], lds0 + buf * kA + (NW * i + w) * 1024);
      return;
    }
    // the last, shorter stage: words past the end of k read as zero
    const int lane = fresh_lane();
    const int left = kw - w0 - 2 * chunk_of(lane);
    const int o0 = left > 0 ? 0 : left - 1, o1 = left > 1 ? 1 : left - 1;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const mfma::gq_ptr src = (mfma::gq_ptr)((const char*)(Ab + w0) + voff[i]);
      const uint64_t x0 = src[o0], x1 = src[o1];
      ulonglong2 v;
      v.x = left > 0 ? x0 : 0ull;
      v.y = left > 1 ? x1 : 0ull;
      *reinterpret_cast<ulonglong2*>(smem + buf * kA + (NW * i + w) * 1024 + lane * 16) = v;
    }
  };
  // the stage's rows of B: 1 KB of them per load, two loads per wave (rows past the end
  // of k repeat the last one)
  auto load_b = [&](int st, int buf) {
    constexpr int kLanes = WX / 2, kRows = 64 / kLanes;  // lanes per row, rows per load
    const int lane = fresh_lane();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int64_t r0 = (int64_t)st * 512 + (2 * w + i) * kRows;
      const int64_t first = r0 < k ? r0 : k - 1;
      const int64_t lim = k - 1 - first;
      int r = lane / kLanes;
      r = r < lim ? r : (int)lim;
      load_lds16(Bb + first * ldb, (uint32_t)r * ((uint32_t)ldb * 8) + 16 * (lane % kLanes),
                 lds0 + kRaw + buf * kB + (2 * w + i) * 1024);
    }
  };
  // four blocks of stage st: word wx, rows 64 (4 wy + j)
  auto turn = [&](int st, int from, int buf) {
    const int c = fresh_lane();
    const Transpose tr(c);
    const int word = wx + shift < WX ? wx + shift : WX - 1;
    const unsigned char* raw = smem + kRaw + from * kB + (256 * wy + c) * (8 * WX) + 8 * word;
    unsigned char* out = smem + kTurned + buf * kB + (64 * wx + c) * kRowBytes;
    const int64_t left = k - ((int64_t)st * 512 + 256 * wy + c);  // rows from lane's first on
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      ulonglong2 v;
      uint64_t x = *reinterpret_cast<const uint64_t*>(raw + (2 * q) * 64 * 8 * WX);
      v.x = transpose64(left > 128 * q ? x : 0ull, tr);
      x = *reinterpret_cast<const uint64_t*>(raw + (2 * q + 1) * 64 * 8 * WX);
      v.y = transpose64(left > 128 * q + 64 ? x : 0ull, tr);
      *reinterpret_cast<ulonglong2*>(out + (((2 * wy + q) ^ ((c >> 1) & 3)) * 16)) = v;
    }
  };

  const int lane = fresh_lane(), half = lane >> 5, li = lane & 31;
  const int slot = (half ^ ((li >> 1) & 3)) * 16;
  const int abase = (wy * 32 * RA + li) * kRowBytes + slot;
  const int bbase = (wx * 32 * RB + li) * kRowBytes + slot;
  u4 xa[2][RA], xb[2][RB];
  auto read = [&](int buf, int s) {
#pragma unroll
    for (int f = 0; f < RA; ++f)
      xa[s][f] = *reinterpret_cast<const u4*>(smem + buf * kA + (abase ^ (32 * s)) + 2048 * f);
#pragma unroll
    for (int g = 0; g < RB; ++g)
      xb[s][g] = *reinterpret_cast<const u4*>(smem + kTurned + buf * kB + (bbase ^ (32 * s)) +
                                              2048 * g);
  };
  AccV<FMT> acc[RA][RB];
#pragma unroll
  for (int f = 0; f < RA; ++f)
#pragma unroll
    for (int g = 0; g < RB; ++g) acc[f][g] = AccV<FMT>{};
  load_b(0, 0);
  load_a(0, 0);
  if (stages > 1) load_b(1, 1);
  stage_sync();
  if (stages > 2) load_b(2, 2);
  turn(0, 0, 0);
  rows_sync();
  if (stages > 1) load_a(1, 1);
  if (stages > 3) load_b(3, 0);
  read(0, 0);
  if (stages > 1) turn(1, 1, 1);
  __builtin_amdgcn_s_setprio(1);
  int cur = 0, third = 2, st = 0;  // the buffers of stage st, and of st + 2's rows of B
  for (; st + 2 < stages; ++st) {
    read(cur, 1);
    mfma_round<SEMI, FMT>(xa[0], xb[0], acc);
    // stage st's operands are in registers, st + 1's and st + 2's rows of B have come
    // (st + 3's, if there are any, are this wave's last two loads and on their way)
    if (st + 3 < stages) rows_sync();
    else stage_sync();
    const int fourth = third == 0 ? 2 : third - 1;  // of stage st + 1 and st + 4
    load_a(st + 2, cur);
    if (st + 4 < stages) load_b(st + 4, fourth);
    read(cur ^ 1, 0);
    turn(st + 2, third, cur);
    mfma_round<SEMI, FMT>(xa[1], xb[1], acc);
    third = third == 2 ? 0 : third + 1;
    cur ^= 1;
  }
  for (; st < stages; ++st) {
    read(cur, 1);
    mfma_round<SEMI, FMT>(xa[0], xb[0], acc);
    if (st + 1 < stages) {
      stage_sync();
      read(cur ^ 1, 0);
    }
    if (st * kWords + 4 < kw) mfma_round<SEMI, FMT>(xa[1], xb[1], acc);  // else only zero words are left
    cur ^= 1;
  }
  __builtin_amdgcn_s_setprio(0);
  store_tile<SEMI, FMT, RA, RB>(acc, C, ldc, m, n, row0 + wy * 32 * RA, in * WX + wx, accumulate,
                                SEMI);
}

// ---- small products: k split over a workgroup's waves ----

// Rows [64 im, ...) x columns [64 in, ...) of C = A B by W waves that share the tile and
// take the 512-bit stages of k in turn (w, w + W, ...), each staging its 128 operand rows in
// 8 KB of LDS of its own (no barrier in the loop: a wave reads a stage into registers and
// loads its next one into the same place; a second buffer per wave gained nothing).  Waves
// without a stage leave at once: up to k = 512 one wave does it all, without a barrier (1000 x
// 64 x 1000, B transposed, 3.83 against 4.05 us).  At the end the waves' result bits, one word per
// lane, are XORed or ORed through LDS.  For products whose larger tiles would leave CUs
// idle: a wave's chain of loads is W times shorter, and there are 8 W waves where the panel
// tile of 128 x 256 has 4.  Bound by the latency of those chains (fp4, 704 x 16704 x 2368:
// 17.6 us, with 128 x 128 tiles 31.6 us; 256 x 8192 x 8192: 10.3 and 16.7 us; before, with
// register-fed 64 x 64 wave tiles, 35.6 and 18.2 us).  0 < k < 2^24; smem: kSplitBytes W bytes.
constexpr int kSplitBytes = 128 * kRowBytes;

//
// BT = false: B is given row-major.  A wave then loads its stage's 512 rows of the tile's
// one column word, a row per lane, and turns the 64 x 64 blocks in registers (31 VALU
// instructions each); lane c holds column c's stage, and a swap of the wave's halves gives
// the operands' layout, so B never goes through LDS.
template <int SEMI, int FMT, int W, bool BT>
__device__ __forceinline__ void split_tile(const uint64_t* __restrict__ A, int64_t lda,
                                           const uint64_t* __restrict__ B, int64_t ldb,
                                           uint64_t* C, int64_t ldc, int64_t m, int64_t k,
                                           int64_t n, int64_t im, int64_t in, int accumulate,
                                           int w, unsigned char* smem) {
  const int64_t kw = (k + 63) >> 6;
  const int stages = (int)((kw + kWords - 1) / kWords);
  const int takers = stages < W ? stages : W;  // waves with stages to take
  if (w >= takers) return;                     // (barriers wait for those that are left)
  const int64_t row0 = im * 64, col0 = in * 64;
  unsigned char* const mine = smem + w * kSplitBytes;
  const int lane = fresh_lane(), half = lane >> 5, li = lane & 31;
  const int chunk = (lane & 3) ^ ((lane >> 3) & 3);
  constexpr int NL = BT ? 8 : 4;
  // load i fills LDS rows 16 i .. + 15 (A's 64 rows, then B^T's)
  const uint64_t* src[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const bool isA = i < 4;
    const int64_t lim = isA ? m - 1 - row0 : n - 1 - col0;
    int64_t r = 16 * (i & 3) + (lane >> 2);
    r = r < lim ? r : lim;
    src[i] = (isA ? A + row0 * lda : B + col0 * ldb) + r * (isA ? lda : ldb) + 2 * chunk;
  }
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)mine;
  uint64_t brow[8];  // BT = false: rows 64 j + lane of the stage, the tile's column word
  auto load = [&](int st) {
    const int64_t w0 = (int64_t)st * kWords;
    const bool whole = (w0 + kWords) * 64 <= k;  // uniform
    if constexpr (!BT) {
      const mfma::gq_ptr p = (mfma::gq_ptr)B + (w0 * 64 + lane) * ldb + in;
      if (whole) {
#pragma unroll
        for (int j = 0; j < 8; ++j) brow[j] = p[64 * j * ldb];
      } else {
        const int64_t rows = k - w0 * 64 - lane;  // row 64 j + lane lies in B if 64 j < rows
#pragma unroll
        for (int j = 0; j < 8; ++j) brow[j] = 64 * j < rows ? p[64 * j * ldb] : 0ull;
      }
    }
    if (whole || w0 + kWords <= kw) {
#pragma unroll
      for (int i = 0; i < NL; ++i) load_lds16(src[i] + w0, lds0 + i * 1024);
      return;
    }
    const int left = (int)(kw - w0) - 2 * chunk;  // words of the lane's chunk and after
    const int o0 = left > 0 ? 0 : left - 1, o1 = left > 1 ? 1 : left - 1;
    uint64_t x[NL][2];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      x[i][0] = ((mfma::gq_ptr)src[i])[w0 + o0];
      x[i][1] = ((mfma::gq_ptr)src[i])[w0 + o1];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      ulonglong2 v;
      v.x = left > 0 ? x[i][0] : 0ull;
      v.y = left > 1 ? x[i][1] : 0ull;
      *reinterpret_cast<ulonglong2*>(mine + i * 1024 + lane * 16) = v;
    }
  };
  using AccV = typename mfma::Acc<FMT>::type;
  AccV acc[2][2];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int g = 0; g < 2; ++g) acc[f][g] = AccV{};
  const int base = li * kRowBytes + (half ^ ((li >> 1) & 3)) * 16;
  const Transpose tr(lane);
  load(w);
  for (int st = w; st < stages; st += W) {
    u4 xa[2][2], xb[2][2];
    if constexpr (!BT) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int v = 0; v < 2; ++v) {  // word v of chunks 2 s and 2 s + 1
          const uint64_t c0 = transpose64(brow[4 * s + v], tr);
          const uint64_t c1 = transpose64(brow[4 * s + 2 + v], tr);
          const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)c0, (uint32_t)c1, false, false);
          const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(c0 >> 32),
                                                           (uint32_t)(c1 >> 32), false, false);
          xb[s][0][2 * v] = lo[0];
          xb[s][1][2 * v] = lo[1];
          xb[s][0][2 * v + 1] = hi[0];
          xb[s][1][2 * v + 1] = hi[1];
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        xa[s][f] = *reinterpret_cast<const u4*>(mine + (base ^ (32 * s)) + 2048 * f);
        if constexpr (BT)
          xb[s][f] = *reinterpret_cast<const u4*>(mine + 4096 + (base ^ (32 * s)) + 2048 * f);
      }
    if (st + W < stages) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read: the next stage may land
      load(st + W);
    }
    mfma_round<SEMI, FMT>(xa[0], xb[0], acc);
    if ((int64_t)st * kWords + 4 < kw) mfma_round<SEMI, FMT>(xa[1], xb[1], acc);
  }
  // lane li of half h holds row r(li) of block h: one word of C per lane and wave
  constexpr bool gf2 = SEMI == GF2;
  uint64_t word = 0;
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const auto s = __builtin_amdgcn_permlane32_swap(pack16<FMT>(acc[0][g], gf2),
                                                    pack16<FMT>(acc[1][g], gf2), false, false);
    const uint32_t x =
        tr(__builtin_amdgcn_perm(s[1], s[0], packs_high<FMT>(gf2) ? 0x07060302u : 0x05040100u));
    word |= (uint64_t)x << (32 * g);
  }
  if (takers > 1) {
    uint64_t* const part = reinterpret_cast<uint64_t*>(smem);
    __syncthreads();  // every wave is done with its stages
    if (w > 0) part[w * 64 + lane] = word;
    __syncthreads();
    if (w > 0) return;
#pragma unroll
    for (int i = 1; i < W; ++i) {
      if (i >= takers) break;
      word = gf2 ? word ^ part[i * 64 + lane] : word | part[i * 64 + lane];
    }
  }
  const int r = ((li >> 2) & 3) * 8 + (li >> 4) * 4 + (li & 3);
  const int64_t row = row0 + 32 * half + r;
  if (row < m) {
    const int64_t valid = n - col0;
    if (valid < 64) word &= ((uint64_t)1 << valid) - 1;
    const mfma::gw_ptr dst = (mfma::gw_ptr)C + row * ldc + in;
    if (accumulate) word = gf2 ? (word ^ *dst) : (word | *dst);
    *dst = word;
  }
}

}  // namespace panel
}  // namespace bmm
