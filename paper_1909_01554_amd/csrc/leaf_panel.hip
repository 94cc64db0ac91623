// Cubic leaf on the matrix cores with operand rows staged in LDS by direct loads (see
// panel_tile.h for the tiles and their operands): one workgroup per 128 x 256 or 256 x 128
// tile of C, two workgroups per CU; for smaller products one per 128 x 128 tile, or per 64 x
// 64 tile with k split over its waves.
#include <algorithm>

#include "panel_tile.h"

namespace bmm {
namespace {

template <int SEMI, int FMT, int RA, int RB, bool FAR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void leaf_panel_kernel(
    LeafBatch p, int64_t grid_m, int64_t grid_n) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[panel::lds_bytes(RA, RB)];
  const TileCoord c = xcd_tile(blockIdx.x, gridDim.x, grid_m, grid_n);
  panel::tile<SEMI, FMT, RA, RB, FAR>(
      p.A + c.b * p.strideA, p.lda, p.BT + c.b * p.strideB, p.ldbt, p.C + c.b * p.strideC, p.ldc,
      p.m, p.k, p.n, c.tm, c.tn, p.accumulate, SEMI,
      __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), smem);
}

template <int SEMI, int FMT, int RA, int RB, bool FAR>
hipError_t launch_shape(const LeafBatch& p, hipStream_t s) {
  const int64_t grid_m = (p.m + 64 * RA - 1) / (64 * RA);
  const int64_t grid_n = (p.n + 64 * RB - 1) / (64 * RB);
  const int64_t blocks = grid_m * grid_n * p.batch;
  if (!grid_fits(blocks, 256)) return kGridTooLarge;
  hipLaunchKernelGGL((leaf_panel_kernel<SEMI, FMT, RA, RB, FAR>), dim3((unsigned)blocks),
                     dim3(256), 0, s, p, grid_m, grid_n);
  return hipGetLastError();
}

// Workgroups of r x c bits of C, and the rounds of them over 256 CUs.
int64_t tiles(int64_t m, int64_t n, int64_t batch, int64_t r, int64_t c) {
  return ((m + r - 1) / r) * ((n + c - 1) / c) * batch;
}
int64_t rounds(int64_t count) { return (count + 255) / 256; }

// Rounds of tall workgroups (256 x 128), in wide ones: their rows of C go out 8 bytes at a
// time, which weighs while k is short (15633 x 128 x 8192, 16 rounds of either, fp4, 38.5
// against 35.0 us, k = 2048 93.4 and 91.7; one round, 4000 x 512 x 1500, 6.5 and 5.0 us, k =
// 4096 15.9 and 14.9).
double tall_rounds(int64_t m, int64_t k, int64_t n, int64_t batch) {
  return 0.15 + (k <= 1024 ? 1.1 : 1.02) * (double)rounds(tiles(m, n, batch, 256, 128));
}

template <int SEMI, int FMT>
hipError_t launch_semi(const LeafBatch& p, hipStream_t s) {
  // 64-bit row addresses take registers that only the tall shape has left
  if (p.lda >= kNearPitch || p.ldbt >= kNearPitch) return launch_shape<SEMI, FMT, 4, 2, true>(p, s);
  // Wide wave tiles (64 x 128): C's rows are stored 16 bytes at a time.  Tall ones where they
  // take fewer rounds (4342 x 8192 x 1831, 255 against 272 workgroups: 41.1 against 68.2 us;
  // 1000 x 1024 x 6000, 188 and 192, 9.6 and 8.4 us); in int8 from k = 8192 on, where they are
  // the faster ones otherwise too, where they are fewer (7872 x 8192 x 2944 99.6 and 102.4 us).
  const int64_t wides = tiles(p.m, p.n, p.batch, 128, 256);
  const bool wide = FMT == mfma::FMT_I8 && p.k >= 8192
                        ? wides <= tiles(p.m, p.n, p.batch, 256, 128)
                        : (double)rounds(wides) <= tall_rounds(p.m, p.k, p.n, p.batch);
  return wide ? launch_shape<SEMI, FMT, 2, 4, false>(p, s)
              : launch_shape<SEMI, FMT, 4, 2, false>(p, s);
}

constexpr int kSplit = 4;  // waves that share a 64 x 64 tile
static_assert(64 * kSplit == 256, "every workgroup here has 256 threads (grid_fits)");

template <int SEMI, int FMT, bool BT>
__global__ __launch_bounds__(64 * kSplit) __attribute__((amdgpu_waves_per_eu(2))) void
leaf_split_kernel(LeafBatch p, int64_t grid_m, int64_t grid_n) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kSplit * panel::kSplitBytes];
  const TileCoord c = xcd_tile(blockIdx.x, gridDim.x, grid_m, grid_n);
  panel::split_tile<SEMI, FMT, kSplit, BT>(
      p.A + c.b * p.strideA, p.lda, p.BT + c.b * p.strideB, p.ldbt, p.C + c.b * p.strideC, p.ldc,
      p.m, p.k, p.n, c.tm, c.tn, p.accumulate,
      __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), smem);
}

template <int SEMI, int FMT>
hipError_t launch_small(const LeafBatch& p, bool split, hipStream_t s) {
  const int64_t grid_m = (p.m + 63) / 64, grid_n = (p.n + 63) / 64;
  const int64_t blocks = grid_m * grid_n * p.batch;
  // up to 512 tiles of 64 x 64, two workgroups per CU, the split form is the faster one
  // (512: 10.3 against 16.7 us; 1024, at n = 2048: 9.8 against 8.1 us).  Asked for by name it
  // also takes more tiles while k is long for them (int8, 1500 x 4096 x 1500, 576 tiles, 11.3
  // against 13.6 us, 2000 x 8192 x 2000, 1024 tiles, 22.7 and 23.6; 2000 x 4096 x 2000 14.1
  // and 13.6, 7000 x 1500 x 9000, 15510 tiles, 109 and 55).
  // So does one row or column of them from k = 2048 on, where a 128 x 128 tile would be half
  // empty (40000 x 3000 x 30, 625 tiles, fp4, 8.6 against 11.1 us; 60 x 2048 x 200000, 3125,
  // int8, 26.3 and 32.1).
  const bool thin = std::min(p.m, p.n) <= 64 && p.k >= 2048;
  const bool large = blocks > 512 && !(split && p.k >= 6 * blocks) && !thin &&
                     p.lda < kNearPitch && p.ldbt < kNearPitch;
  if (large) return launch_shape<SEMI, FMT, 2, 2, false>(p, s);
  // (far pitches: past the largest launch of these tiles the panel's)
  if (!grid_fits(blocks, 256)) return launch_semi<SEMI, FMT>(p, s);
  hipLaunchKernelGGL((leaf_split_kernel<SEMI, FMT, true>), dim3((unsigned)blocks),
                     dim3(64 * kSplit), 0, s, p, grid_m, grid_n);
  return hipGetLastError();
}

template <int SEMI, int FMT>
hipError_t launch_rows(const LeafBatch& p, hipStream_t s) {
  const int64_t grid_m = (p.m + 63) / 64, grid_n = (p.n + 63) / 64;
  const int64_t blocks = grid_m * grid_n * p.batch;
  if (!grid_fits(blocks, 64 * kSplit)) return kGridTooLarge;
  hipLaunchKernelGGL((leaf_split_kernel<SEMI, FMT, false>), dim3((unsigned)blocks),
                     dim3(64 * kSplit), 0, s, p, grid_m, grid_n);
  return hipGetLastError();
}

template <int SEMI, int FMT, int WX>
__global__ __launch_bounds__(128 * WX) __attribute__((amdgpu_waves_per_eu(2))) void
leaf_turn_kernel(LeafBatch p, int64_t grid_m, int64_t grid_n) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[panel::rows_bytes(WX)];
  const TileCoord c = xcd_tile(blockIdx.x, gridDim.x, grid_m, grid_n);
  panel::rows_tile<SEMI, FMT, WX>(
      p.A + c.b * p.strideA, p.lda, p.BT + c.b * p.strideB, p.ldbt, p.C + c.b * p.strideC, p.ldc,
      p.m, p.k, p.n, c.tm, c.tn, p.accumulate,
      __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), smem);
}

template <int SEMI, int FMT, int WX>
hipError_t launch_turn(const LeafBatch& p, hipStream_t s) {
  const int64_t grid_m = (p.m + 255) / 256, grid_n = (p.n + 64 * WX - 1) / (64 * WX);
  const int64_t blocks = grid_m * grid_n * p.batch;
  if (!grid_fits(blocks, 128 * WX)) return kGridTooLarge;
  hipLaunchKernelGGL((leaf_turn_kernel<SEMI, FMT, WX>), dim3((unsigned)blocks), dim3(128 * WX), 0,
                     s, p, grid_m, grid_n);
  return hipGetLastError();
}

// E2M1: workgroups of eight waves and 256 columns, one per CU, where there are more than one
// tile of 128 columns per CU (256 x 32768 x 65536 as called: 204 against 212 us); int8 always
// takes 128 columns (318 against 297 us).
template <int SEMI>
hipError_t launch_turn_f4(const LeafBatch& p, hipStream_t s) {
  return ((p.m + 255) / 256) * ((p.n + 127) / 128) > 256
             ? launch_turn<SEMI, mfma::FMT_F4, 4>(p, s)
             : launch_turn<SEMI, mfma::FMT_F4, 2>(p, s);
}

}  // namespace

bool leaf_small_tiles(int fmt, int64_t m, int64_t k, int64_t n, int64_t batch) {
  if (tiles(m, n, batch, 64, 64) <= 512 || leaf_regs_fits(fmt, m, k, n, batch)) return true;
  // whole rounds over 256 CUs; a small tile is half the work of a large one, and costs
  // 4 to 13% more per unit (n = 4096, 4 rounds against 2: 25.5 and 24.0 us; n = 3072, 3
  // against 2: 16.0 and 18.7 us; 5001 x 7003 x 3333, 5 against 3: 50.5 and 58.7 us), 16% in
  // fp4 while k is one stage (12000 x 512 x 2400, 7 against 4: 12.8 and 10.9 us).
  const int64_t small = tiles(m, n, batch, 128, 128);
  const double unit = fmt == mfma::FMT_F4 && k <= 512 ? 0.58 : 0.54;
  const double wide = (double)rounds(tiles(m, n, batch, 128, 256));
  return unit * (double)rounds(small) < std::min(wide, tall_rounds(m, k, n, batch)) &&
         grid_fits(small, 256);
}

hipError_t launch_leaf_small(int semiring, int fmt, const LeafBatch& p, bool split,
                             hipStream_t s) {
  if (p.m <= 0 || p.n <= 0 || p.batch <= 0) return hipSuccess;
  if (p.k >= panel::kMaxK) return hipErrorInvalidValue;  // counts would not be exact
  if (fmt == mfma::FMT_F4)
    return semiring == GF2 ? launch_small<GF2, mfma::FMT_F4>(p, split, s)
                           : launch_small<BOOLEAN, mfma::FMT_F4>(p, split, s);
  return semiring == GF2 ? launch_small<GF2, mfma::FMT_I8>(p, split, s)
                         : launch_small<BOOLEAN, mfma::FMT_I8>(p, split, s);
}

bool leaf_rows_fits(int64_t m, int64_t k, int64_t n) {
  // Every row of tiles turns B again, 8 bytes of a line at a time, which a saved launch (and
  // the scratch copy) repays while the product is small: 1024^3 6.2 us against 7.2 us with a
  // transpose of its own, 3000 x 500 x 500 6.3 and 7.3 us, 256 x 4096 x 256 7.4 and 7.7 us,
  // but 256 x 4096 x 4096 10.5 and 9.1 us, 200 x 20000 x 200 21.8 and 14.3 us.
  return k <= 4096 && ((m + 63) / 64) * ((n + 63) / 64) <= 512 &&
         (double)m * (double)k * (double)n <= (double)(1 << 30);
}

hipError_t launch_leaf_rows(int semiring, int fmt, const LeafBatch& p, hipStream_t s) {
  if (p.m <= 0 || p.n <= 0 || p.batch <= 0) return hipSuccess;
  if (p.k >= panel::kMaxK) return hipErrorInvalidValue;  // counts would not be exact
  if (fmt == mfma::FMT_F4)
    return semiring == GF2 ? launch_rows<GF2, mfma::FMT_F4>(p, s)
                           : launch_rows<BOOLEAN, mfma::FMT_F4>(p, s);
  return semiring == GF2 ? launch_rows<GF2, mfma::FMT_I8>(p, s)
                         : launch_rows<BOOLEAN, mfma::FMT_I8>(p, s);
}

bool leaf_turn_fits(int64_t m, int64_t k, int64_t n, int64_t lda, int64_t ldb) {
  // Every row of tiles turns B again, so one or two of them (m = 512: 409 against 444 us with
  // a transpose and the panel leaf, k = 32768, n = 65536; m = 1024: 734 and 728), the last
  // more than half full (k = 8192, n = 65536: m = 130 52 against 64 us, m = 128 53 against 49).
  // Tiles that fill the CUs, one on each or two, in the last round (k = 8192, m = 256: 192
  // tiles 33.6 against 36.3 us, 448 53 and 63, 640 77 and 83, but 128 32.3 and 31.1, in int8
  // 384 75.6 and 73.1).  Whatever k: what is saved at short k is the transpose's launch (fp4, 256
  // x 64 x 32768 5.7 against 7.1 us, 512 x 64 x 16384 5.5 and 7.0, 400 x 512 x 28672 7.9 and
  // 9.0; at the most, 512 x 64 x 65536, 12.8 and 12.5).
  const int64_t rows = (m + 255) / 256, tiles = rows * ((n + 127) / 128), last = tiles % 512;
  return rows <= 2 && m > 256 * rows - 128 && tiles >= 192 && k < panel::kMaxK &&
         lda < kNearPitch && ldb < kNearPitch &&
         (last == 0 || (last >= 192 && last <= 256) || last >= 448 || tiles > 4096);
}

hipError_t launch_leaf_turn(int semiring, int fmt, const LeafBatch& p, hipStream_t s) {
  if (p.m <= 0 || p.n <= 0 || p.batch <= 0) return hipSuccess;
  if (p.k <= 0 || !leaf_turn_fits(p.m, p.k, p.n, p.lda, p.ldbt)) return hipErrorInvalidValue;
  if (fmt == mfma::FMT_F4)
    return semiring == GF2 ? launch_turn_f4<GF2>(p, s) : launch_turn_f4<BOOLEAN>(p, s);
  return semiring == GF2 ? launch_turn<GF2, mfma::FMT_I8, 2>(p, s)
                         : launch_turn<BOOLEAN, mfma::FMT_I8, 2>(p, s);
}

hipError_t launch_leaf_panel(int semiring, int fmt, const LeafBatch& p, hipStream_t s) {
  if (p.m <= 0 || p.n <= 0 || p.batch <= 0) return hipSuccess;
  if (p.k >= panel::kMaxK) return hipErrorInvalidValue;  // counts would not be exact
  if (fmt == mfma::FMT_F4)
    return semiring == GF2 ? launch_semi<GF2, mfma::FMT_F4>(p, s)
                           : launch_semi<BOOLEAN, mfma::FMT_F4>(p, s);
  return semiring == GF2 ? launch_semi<GF2, mfma::FMT_I8>(p, s)
                         : launch_semi<BOOLEAN, mfma::FMT_I8>(p, s);
}

}  // namespace bmm
