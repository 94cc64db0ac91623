// Cubic leaf product on the matrix cores of gfx950: which kernel runs a tile choice, and the
// forms fed from registers: int8's long and unrolled ones, and 64 x 64 wave tiles for short k
// and thin results in int8 and fp4 (every other one is the panel leaf).
//
// The cubic product C[i][k] = SUM_j A[i][j] B[j][k] (GF(2): XOR, Boolean: OR)
// is an integer dot product reduced at the end: the int32 count of j with
// A[i][j] = B[j][k] = 1 gives the GF(2) bit as its parity and the Boolean bit
// as (count > 0).  Counts stay exact because k < 2^31.
//
// In the kernel here each wave owns a TM x TN tile of C (TM = 32*RA, TN = 32*RB) and issues
// v_mfma_i32_32x32x32_i8 (fp4: v_mfma_scale_f32_32x32x64_f8f6f4) on RA x RB accumulator
// blocks held in registers.  Operands never touch HBM as bytes: every lane reads
// 64-bit words of packed bits straight from its row of A (or of B transposed) and
// expands them in registers.  The order of k inside a dot product is free as long as A and B
// use the same one, so a 32-bit half x of a word yields the eight dwords
// (x >> d) & 0x01010101 (d = 0..7): byte e of dword d is bit 8e + d of x, 0 or
// 1 (for one side of the tile both halves at once, from a 64-bit shift).
//
// The result bits go back to packed rows with wave ballots: accumulator
// register v of a 32x32 block holds row 8*(v/4) + (v%4) in lanes 0..31 and
// row 8*(v/4) + 4 + (v%4) in lanes 32..63, one column per lane, so one ballot
// yields two 32-bit row words.
#include <algorithm>

#include "panel_tile.h"

namespace bmm {
namespace {

bool aligned16(const LeafBatch& p) {
  return ((reinterpret_cast<uintptr_t>(p.A) | reinterpret_cast<uintptr_t>(p.BT)) & 15) == 0 &&
         ((p.lda | p.ldbt | p.strideA | p.strideB) & 1) == 0;
}

// Each workgroup owns 2 x 2 wave tiles; workgroups are ordered for L2 reuse per XCD.
template <int SEMI, int RA, int RB, int KV, int FMT, int NB = 2, int STEPS = 0, bool WIDE = true,
          bool UNIFORM = false, bool BOTH = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void leaf_mfma_kernel(
    LeafBatch p, int64_t tiles_m, int64_t tiles_n) {
  const int64_t grid_m = (tiles_m + 1) >> 1, grid_n = (tiles_n + 1) >> 1;
  const TileCoord c = xcd_tile(blockIdx.x, gridDim.x, grid_m, grid_n);
  // UNIFORM: the wave index as a uniform value (the tile coordinates then live in scalar
  // registers, which frees the vector registers the long-k loop spilled); the unrolled tile
  // keeps the per-lane form, measured faster there.
  const int w = UNIFORM ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
  const int64_t tm = 2 * c.tm + (w >> 1);
  const int64_t tn = 2 * c.tn + (w & 1);
  if (c.b >= p.batch || tm >= tiles_m || tn >= tiles_n) return;  // uniform per wave
  const int64_t b = c.b;
  mfma::tile<SEMI, RA, RB, KV, FMT, NB, STEPS, WIDE, BOTH>(
      p.A + b * p.strideA, p.lda, p.BT + b * p.strideB, p.ldbt, p.C + b * p.strideC, p.ldc, p.m,
      p.k, p.n, tm, tn, p.accumulate);
}

// int8 from k = 2^24 on, where the panel leaf's products of 2^7 would overflow int32 sums:
// 64 x 128 wave tiles fed from registers, 0/1 operand bytes.  Aligned operands run the load
// pipeline as a loop over fully unrolled chunks of 12 steps, which leaves the compiler's
// conservative wait for outstanding loads at the loop's back edge once per chunk instead of
// once per step pair.
template <int SEMI>
hipError_t launch_long(const LeafBatch& p, hipStream_t s) {
  const int64_t tiles_m = (p.m + 63) / 64, tiles_n = (p.n + 127) / 128;
  const int64_t blocks = ((tiles_m + 1) / 2) * ((tiles_n + 1) / 2) * p.batch;
  if (blocks == 0) return hipSuccess;
  if (!grid_fits(blocks, 256)) return kGridTooLarge;
  const dim3 g((unsigned)blocks), b(256);
  if (aligned16(p))
    hipLaunchKernelGGL((leaf_mfma_kernel<SEMI, 2, 4, 2, mfma::FMT_I8, 2, -12, true, true>), g, b, 0, s, p,
                       tiles_m, tiles_n);
  else
    hipLaunchKernelGGL((leaf_mfma_kernel<SEMI, 2, 4, 1, mfma::FMT_I8, 2, 0, true, true>), g, b, 0,
                       s, p, tiles_m, tiles_n);
  return hipGetLastError();
}

// int8 tile 6 at the recursion's leaf lengths (k = 2048 or 4096 bits, aligned): a fully
// unrolled load pipeline with two register buffers and both operand sides expanded by
// 64-bit shifts.  The panel leaf, which needs 2/3 of its VALU instructions and a third of
// its loads, is faster (the n = 32768 recursion 11.5 against 12.5 ms) and the tuned choice.
template <int SEMI, int STEPS>
hipError_t launch_deep(const LeafBatch& p, hipStream_t s) {
  const int64_t tiles_m = (p.m + 127) / 128, tiles_n = (p.n + 63) / 64;
  const int64_t blocks = ((tiles_m + 1) / 2) * ((tiles_n + 1) / 2) * p.batch;
  if (blocks == 0) return hipSuccess;
  if (!grid_fits(blocks, 256)) return kGridTooLarge;
  hipLaunchKernelGGL((leaf_mfma_kernel<SEMI, 4, 2, 2, mfma::FMT_I8, 2, STEPS, true, false, true>),
                     dim3((unsigned)blocks), dim3(256), 0, s, p, tiles_m, tiles_n);
  return hipGetLastError();
}

// Short k, and results of one row or column of tiles (leaf_regs_fits): 64 x 64 wave tiles, 2 x
// 2 of them per workgroup.  A step takes 2 KV words of k, where a round of the panel leaf is
// four whatever k has left, and nothing goes through LDS.
template <int SEMI, int FMT>
hipError_t launch_regs(const LeafBatch& p, hipStream_t s) {
  const int64_t tiles_m = (p.m + 63) / 64, tiles_n = (p.n + 63) / 64;
  const int64_t blocks = ((tiles_m + 1) / 2) * ((tiles_n + 1) / 2) * p.batch;
  if (!grid_fits(blocks, 256)) return kGridTooLarge;
  const dim3 g((unsigned)blocks), b(256);
  constexpr bool kWide = FMT == mfma::FMT_I8;  // (E2M1 operands have the 32-bit form only)
  // (words past the last step are taken one by one)
  if (aligned16(p) && (p.k + 63) / 64 % 4 == 0)
    hipLaunchKernelGGL((leaf_mfma_kernel<SEMI, 2, 2, 2, FMT, 2, 0, kWide>), g, b, 0, s, p, tiles_m,
                       tiles_n);
  else
    hipLaunchKernelGGL((leaf_mfma_kernel<SEMI, 2, 2, 1, FMT, 2, 0, kWide>), g, b, 0, s, p, tiles_m,
                       tiles_n);
  return hipGetLastError();
}

template <int SEMI, int FMT>
hipError_t launch_semi(const LeafBatch& p, int tile, hipStream_t s) {
  if constexpr (FMT == mfma::FMT_I8) {
    if (p.k >= panel::kMaxK) return launch_long<SEMI>(p, s);
    if (tile == MFMA_DEEP_128x64 && aligned16(p)) {
      if (p.k == 2048) return launch_deep<SEMI, 8>(p, s);
      if (p.k == 4096) return launch_deep<SEMI, 16>(p, s);
    }
  }
  if (tile == MFMA_64x64 || tile == MFMA_64x32) {
    // Results that 2 x 2 wave tiles of the named size per workgroup would not hold in one
    // launch are refused, whichever form would run.
    const int64_t cols = 2 * leaf_mfma_tile_cols(tile);
    if (!grid_fits((p.m + 127) / 128 * ((p.n + cols - 1) / cols) * p.batch, 256))
      return kGridTooLarge;
    if (tile == MFMA_64x64 && leaf_regs_fits(FMT, p.m, p.k, p.n, p.batch))
      return launch_regs<SEMI, FMT>(p, s);
    return launch_leaf_small(SEMI, FMT, p, tile == MFMA_64x32, s);
  }
  return launch_leaf_panel(SEMI, FMT, p, s);
}

}  // namespace

bool leaf_regs_fits(int fmt, int64_t m, int64_t k, int64_t n, int64_t batch) {
  const int64_t tiles_m = (m + 63) / 64, tiles_n = (n + 63) / 64;
  const int64_t tiles = tiles_m * tiles_n * batch;
  // (one column of 2^31 rows: the tall panel tiles still fit a launch)
  if (!grid_fits(((tiles_m + 1) / 2) * ((tiles_n + 1) / 2) * batch, 256)) return false;
  // One row or column of tiles, more of them than the k-split form likes: a 128 x 128 tile
  // would be half empty (60 x 768 x 200000, int8 13.2 against 16.5 us, fp4 10.9 and 15.0; 40000
  // x 1024 x 30 5.9 and 7.2, 5.3 and 5.5).  From k = 2048 on the k-split form takes them.
  if (std::min(m, n) <= 64 && tiles > 512) return k < 2048;
  // Short k, until the larger tiles fill the CUs (int8, 640 x 320 x 6336, 990 tiles, 4.5 against
  // 5.5 us, k = 384 4.7 and 5.4; 4342 x 256 x 1831, 1972 tiles, 4.9 and 6.0; 4096 x 64 x 4096
  // 6.8 and 6.6); for up to 512 tiles only in int8 (64 x 64 x 64 3.1 and 3.4 us, 1000 x 256 x
  // 1000 3.8 and 3.9; fp4 3.3 and 3.3, 3.8 and 3.7; 640 x 256 x 6336 3.9 and 4.7).
  if (fmt == mfma::FMT_I8) return tiles <= 2304 && k <= (tiles > 512 ? 320 : 256);
  return tiles <= 2304 && k <= 256 && tiles > 512;
}

int leaf_mfma_tile_rows(int tile) {
  switch (tile) {
    case MFMA_64x64: return 64;
    case MFMA_64x128: return 64;
    case MFMA_CHUNK_64x128: return 64;
    case MFMA_64x32: return 64;
    case MFMA_LDS_256x256: return 256;
    case MFMA_LDS4_256x128: return 256;
    default: return 128;
  }
}

int leaf_mfma_tile_cols(int tile) {
  switch (tile) {
    case MFMA_64x64: return 64;
    case MFMA_64x128: return 128;
    case MFMA_CHUNK_64x128: return 128;
    case MFMA_64x32: return 32;
    case MFMA_LDS_256x256: return 256;
    case MFMA_LDS4_256x128: return 128;
    default: return 64;
  }
}

hipError_t launch_leaf_mfma(int semiring, const LeafBatch& p, int tile, hipStream_t s) {
  if (p.m <= 0 || p.n <= 0 || p.batch <= 0) return hipSuccess;
  return semiring == GF2 ? launch_semi<GF2, mfma::FMT_I8>(p, tile, s)
                         : launch_semi<BOOLEAN, mfma::FMT_I8>(p, tile, s);
}

hipError_t launch_leaf_mfma_f4(int semiring, const LeafBatch& p, int tile, hipStream_t s) {
  if (p.m <= 0 || p.n <= 0 || p.batch <= 0) return hipSuccess;
  return semiring == GF2 ? launch_semi<GF2, mfma::FMT_F4>(p, tile, s)
                         : launch_semi<BOOLEAN, mfma::FMT_F4>(p, tile, s);
}

}  // namespace bmm
