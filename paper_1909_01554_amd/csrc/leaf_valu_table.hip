// VALU leaf by tables (the method of four Russians: Arlazarov, Dinic, Kronrod and Faradzhev,
// 1970), for large cubic products whose B is at hand row-major: for every 8 rows of B the
// workgroup writes the 256 sums (XOR or OR) of subsets of them to LDS, and each byte of a
// row of A then picks one sum, 8 x 1024 bit products per 128-byte row of the table.  Two
// tables (16 rows of B) are folded at once, acc ^= t0 ^ t1 or acc |= t0 | t1, one
// v_bitop3_b32 per dword.
//
// Tile: 8 waves, 1024 x 1024 of C.  Lane l of a wave holds 16 bytes (slice l % 8) of the rows
// 8 g + l / 8, g = 0 .. 15; the 8 lanes of a row read one table row, all slices of it, so no
// two lanes read from one bank whatever the bits of A are.  Tables are double buffered (128 KB
// of LDS): a phase of 16 rows of B reads one pair and builds the next.
//
// Bound by LDS: a phase reads 2 x 1024 and writes 2 x 256 rows of 128 bytes and moves 16 raw
// rows, at least 2800 cycles for 2^25 bit operations; 3300 are measured (lanes of two table
// rows still meet in a bank).  n = 16384: Boolean 1.44 ms and GF(2) 1.49 ms, against 2.75 and
// 3.00 ms for the dot-product form, whose folds are bound by the VALU.  On the way there: A by
// single dwords and B's rows loaded by every builder from memory, both through the vector L1
// at the LDS's own pace, 1.83 ms; A by quads 1.61 ms; 32 reads in flight instead of 16, or 8,
// changed nothing.
#include <type_traits>

#include "bit_transpose.h"
#include "lds_load.h"

namespace bmm {
namespace {

typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int TR = 1024, TW = 16;      // rows and C words per workgroup
constexpr int GR = 16;                 // rows per lane
constexpr int TAB = 256 * 128;         // bytes of one table
constexpr int BUF = 2 * TAB;           // one phase's pair

template <int SEMI>
__device__ __forceinline__ u4 sum(u4 a, u4 b) {
  return SEMI == GF2 ? (a ^ b) : (a | b);
}
template <int SEMI>
__device__ __forceinline__ u4 sum3(u4 a, u4 b, u4 c) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    a[i] = __builtin_amdgcn_bitop3_b32(a[i], b[i], c[i], SEMI == GF2 ? 0x96 : 0xFE);
  return a;
}
// acc + (x & mask)
template <int SEMI>
__device__ __forceinline__ u4 fold(u4 x, uint32_t mask, u4 acc) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    acc[i] = __builtin_amdgcn_bitop3_b32(x[i], mask, acc[i], SEMI == GF2 ? 0x6A : 0xEA);
  return acc;
}

template <int SEMI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void
leaf_valu_table_kernel(const uint64_t* __restrict__ A, int64_t lda, const uint64_t* __restrict__ B,
                       int64_t ldb, uint64_t* __restrict__ C, int64_t ldc, int64_t m, int64_t k,
                       int64_t n, int64_t tiles_m, int64_t tiles_n, int accumulate) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * BUF + 4096];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const TileCoord c = xcd_tile(blockIdx.x, gridDim.x, tiles_m, tiles_n);
  const int64_t nw = (n + 63) >> 6;
  const int slice = lane & 7;

  // A: dwords 4 q + lane % 4 of the lane's 16 rows, so a quad holds four consecutive dwords
  // of its row and a phase broadcasts the one it needs (the lanes of a row loading the same
  // dword each time kept the vector L1 as busy as the LDS).  Rows past m repeat the last
  // one, and are not stored; dwords past the end read the last one, against zero rows of B.
  uint32_t a[GR], an[GR];
  const int64_t k32 = 2 * ((k + 63) >> 6);
  auto load_a = [&](int64_t q) {
    const int ln = fresh_lane();
    const int64_t jd = 4 * q + (ln & 3);
    const uint32_t* base = reinterpret_cast<const uint32_t*>(A) + (jd < k32 ? jd : k32 - 1);
    const int64_t r0 = c.tm * TR + wave * 128 + (ln >> 3);
#pragma unroll
    for (int g = 0; g < GR; ++g) {
      const int64_t r = r0 + 8 * g;
      an[g] = base[(r < m ? r : m - 1) * 2 * lda];
    }
  };
  // B: 16 rows of a phase (2 KB) go to LDS raw, a phase before their tables are built; the
  // waves take turns in halves, one half building while a wave of the other loads.
  const int turn = wave >> 2, table = (wave >> 1) & 1;
  unsigned char* const raw = smem + 2 * BUF;
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  const uint32_t raw0 = (uint32_t)(uintptr_t)(lds_ptr)raw;
  auto stage_b = [&](int64_t k0, int half) {  // rows k0 .. + 15 by one wave
    const int ln = fresh_lane();
    const uint64_t* src = B + k0 * ldb + c.tn * TW;  // uniform
    if (k0 + 16 <= k && (c.tn + 1) * TW <= nw) {  // uniform
      const uint64_t* p = src + (ln >> 3) * ldb + 2 * (ln & 7);
      load_lds16(p, raw0 + half * 2048);
      load_lds16(p + 8 * ldb, raw0 + half * 2048 + 1024);
      return;
    }
    // rows past k and words past n as zeros (clamped addresses)
    const int left = (int)(nw - c.tn * TW) - 2 * (ln & 7);  // words of B's rows from the lane's on
    const int o0 = left > 0 ? 2 * (ln & 7) : 0, o1 = left > 1 ? 2 * (ln & 7) + 1 : 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t r = k0 + 8 * h + (ln >> 3);
      const uint64_t* p = B + (r < k ? r : k - 1) * ldb + c.tn * TW;
      const uint64_t lo = p[o0], hi = p[o1];
      ulonglong2 v;
      v.x = r < k && left > 0 ? lo : 0ull;
      v.y = r < k && left > 1 ? hi : 0ull;
      *reinterpret_cast<ulonglong2*>(raw + half * 2048 + h * 1024 + ln * 16) = v;
    }
  };
  // a builder forms 16 sums of one table, those whose upper four bits are u
  const int u = (tid >> 3) & 15;
  uint32_t mask[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) mask[i] = 0u - ((u >> i) & 1u);
  const uint32_t wbase = table * TAB + (u << 4) * 128 + slice * 16;
  auto build = [&](uint32_t buf, int half) {
    u4 b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      b[i] = *reinterpret_cast<const u4*>(raw + half * 2048 + table * 1024 + i * 128 + slice * 16);
    u4 e = b[4] & mask[0];
#pragma unroll
    for (int i = 1; i < 4; ++i) e = fold<SEMI>(b[4 + i], mask[i], e);
    auto put = [&](int j, u4 x) { *reinterpret_cast<u4*>(smem + buf + wbase + j * 128) = x; };
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      u4 f = e;
      if (h & 1) f = sum<SEMI>(f, b[2]);
      if (h & 2) f = sum<SEMI>(f, b[3]);
      const u4 g = sum<SEMI>(f, b[1]);
      put(4 * h, f);
      put(4 * h + 1, sum<SEMI>(f, b[0]));
      put(4 * h + 2, g);
      put(4 * h + 3, sum<SEMI>(g, b[0]));
    }
  };

  u4 acc[GR];
#pragma unroll
  for (int g = 0; g < GR; ++g) acc[g] = u4{0, 0, 0, 0};
  auto sync = [&]() {  // also for the direct loads, which the compiler does not see
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  load_a(0);
  if (wave == 0) {
    stage_b(0, 0);
    stage_b(16, 1);
  }
  sync();
  if (turn == 1) build(0, 0);
  uint32_t cur = slice * 16;  // the lane's slice in the tables to read
  sync();
  const int64_t quads = (k + 127) >> 7;
  // phase PH of the eight of a quad: dword PH / 2, its bytes 0, 1 or 2, 3
  auto phase = [&](int64_t q, auto phc) {
    constexpr int PH = decltype(phc)::value;
    // (half PH & 1 of the raw rows made the tables of this phase)
    if (wave == 4 * (1 - (PH & 1))) stage_b(q * 128 + 16 * (PH + 2), PH & 1);
#pragma unroll
    for (int g = 0; g < GR; ++g) {
      if (g % 8 == 0) __builtin_amdgcn_sched_barrier(0);  // 16 reads in flight, not 32
      const uint32_t d = (uint32_t)__builtin_amdgcn_update_dpp(
          0, (int)a[g], (PH / 2) * 0x55, 0xf, 0xf, true);  // quad_perm: all four lanes PH / 2
      // byte times 128, and the slice
      const uint32_t x0 = (PH & 1) ? d >> 9 : d << 7, x1 = (PH & 1) ? d >> 17 : d >> 1;
      const u4 t0 = *reinterpret_cast<const u4*>(smem + ((x0 & 0x7F80u) | cur));
      const u4 t1 = *reinterpret_cast<const u4*>(smem + ((x1 & 0x7F80u) | cur) + TAB);
      acc[g] = sum3<SEMI>(acc[g], t0, t1);
      asm volatile("" : "+v"(acc[g]));  // here, not after the barrier with t0, t1 kept
    }
    __builtin_amdgcn_sched_barrier(0);
    cur ^= BUF;
    if (turn == (PH & 1)) build(cur & BUF, 1 - (PH & 1));
    sync();
  };
  for (int64_t q = 0; q < quads; ++q) {
#pragma unroll
    for (int g = 0; g < GR; ++g) a[g] = an[g];
    if (q + 1 < quads) load_a(q + 1);
    phase(q, std::integral_constant<int, 0>{});
    phase(q, std::integral_constant<int, 1>{});
    phase(q, std::integral_constant<int, 2>{});
    phase(q, std::integral_constant<int, 3>{});
    phase(q, std::integral_constant<int, 4>{});
    phase(q, std::integral_constant<int, 5>{});
    phase(q, std::integral_constant<int, 6>{});
    phase(q, std::integral_constant<int, 7>{});
  }
  const int el = fresh_lane();
  const int64_t cw = c.tn * TW + 2 * (el & 7);  // first of the lane's two C words
  const int64_t row0 = c.tm * TR + wave * 128 + (el >> 3);
#pragma unroll
  for (int g = 0; g < GR; ++g) {
    const int64_t row = row0 + 8 * g;
    if (row >= m) continue;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (cw + h >= nw) break;
      uint64_t x = (uint64_t)acc[g][2 * h] | ((uint64_t)acc[g][2 * h + 1] << 32);
      const int64_t valid = n - (cw + h) * 64;
      if (valid < 64) x &= ((uint64_t)1 << valid) - 1;  // padding columns stay zero
      uint64_t* dst = C + row * ldc + cw + h;
      if (accumulate) x = SEMI == GF2 ? (x ^ *dst) : (x | *dst);
      *dst = x;
    }
  }
}

}  // namespace

bool leaf_valu_table_fits(int64_t m, int64_t n) {
  // One workgroup per CU and round, of 88 ns per bit of k, against the dot-product form's 3.2
  // bit operations per fs: the two would meet at 1.43e8 bits of C per round.  The line lies
  // above that (12672 x 4096 x 12672, 1.606e8: 442 against 540 us, k = 64 22 and 96; 16384 x
  // 4096 x 20000, two rounds of 1.64e8, 833 and 1050; n = 8192, where 64 tiles leave three CUs
  // in four idle, takes 0.7 ms with them and 0.38 ms without).
  const double rounds = (double)((((m + TR - 1) / TR) * ((n + 64 * TW - 1) / (64 * TW)) + 255) / 256);
  return (double)m * (double)n >= 1.6e8 * rounds;
}

hipError_t launch_leaf_valu_table(int semiring, const uint64_t* A, int64_t lda, const uint64_t* B,
                                  int64_t ldb, uint64_t* C, int64_t ldc, int64_t m, int64_t k,
                                  int64_t n, int accumulate, hipStream_t s) {
  if (m <= 0 || n <= 0) return hipSuccess;
  if (k <= 0) return accumulate ? hipSuccess : launch_zero(C, ldc, m, (n + 63) / 64, s);
  const int64_t tiles_m = (m + TR - 1) / TR, tiles_n = ((n + 63) / 64 + TW - 1) / TW;
  const int64_t blocks = tiles_m * tiles_n;
  if (!grid_fits(blocks, 512)) return kGridTooLarge;
  const dim3 g((unsigned)blocks), b(512);
  if (semiring == GF2)
    hipLaunchKernelGGL(leaf_valu_table_kernel<GF2>, g, b, 0, s, A, lda, B, ldb, C, ldc, m, k, n,
                       tiles_m, tiles_n, accumulate);
  else
    hipLaunchKernelGGL(leaf_valu_table_kernel<BOOLEAN>, g, b, 0, s, A, lda, B, ldb, C, ldc, m, k, n,
                       tiles_m, tiles_n, accumulate);
  return hipGetLastError();
}

}  // namespace bmm
