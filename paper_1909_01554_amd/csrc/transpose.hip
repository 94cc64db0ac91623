// Bit-matrix transpose in 64 x 64 bit blocks.
//
// A workgroup of RB waves transposes a tile of 64 RB rows x CW words: wave i loads rows
// 64 i .. + 63, a row per lane (16 bytes at a time), turns
// each word's 64 x 64 block in registers (bit_transpose.h: 31 VALU instructions, no
// cross-lane traffic through LDS), and leaves the 64-bit pieces of the transposed rows in
// LDS, from where they go out RB words (8 RB bytes) at a time.  Bits of rows past the end
// read as zero, so the padding of the transposed rows is zero.
//
// Bound by memory (large) and by latency (small).  8 x 8 blocks move whole 64-byte halves of
// a line both ways, in bands of 8 tiles whose pieces of a row are neighbours (16384 x 16384
// bits: 14.0 us, 4.8 TB/s; in row order 18.7 us; with shuffles through LDS, in row order,
// 26.6 us; 65536 x 65536: 292, 385 and 402 us; with odd pitches 391 us, with 8-byte loads for
// them 558).  Matrices of fewer than 256 such tiles take
// 4 x 2 blocks: 2048 x 2048 bits are 128 workgroups instead of 16, 3.5 us instead of 10.1.
#include "bit_transpose.h"

namespace bmm {
namespace {

// 16 bytes of a row: the device loads them at the 8-byte alignment that rows of odd pitch have
typedef uint64_t pair_t __attribute__((ext_vector_type(2), aligned(8)));

template <int RB, int CW>
__global__ __launch_bounds__(64 * RB) void transpose_kernel(
    const uint64_t* __restrict__ src, int64_t lds, int64_t strideS, uint64_t* __restrict__ dst,
    int64_t ldd, int64_t strideD, int64_t rows, int64_t cols, uint32_t n_rt, uint32_t n_wt) {
  constexpr int STR = RB + 1;  // padded LDS row (in words)
  __shared__ uint64_t tile[64 * CW * STR];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const TileCoord c0 = xcd_tile(blockIdx.x, gridDim.x, n_rt, n_wt);
  const int64_t b = c0.b, r0 = c0.tm * (64 * RB), w0 = c0.tn * CW;
  const int64_t src_words = (cols + 63) >> 6, dst_words = (rows + 63) >> 6;
  const uint64_t* S = src + b * strideS;
  uint64_t* D = dst + b * strideD;
  const int64_t r = r0 + 64 * wave + lane;
  uint64_t x[CW];
  if (w0 + CW <= src_words) {  // uniform
    const pair_t* p = reinterpret_cast<const pair_t*>(S + (r < rows ? r : rows - 1) * lds + w0);
#pragma unroll
    for (int i = 0; i < CW / 2; ++i) {
      const pair_t v = p[i];
      x[2 * i] = r < rows ? v[0] : 0ull;
      x[2 * i + 1] = r < rows ? v[1] : 0ull;
    }
  } else {
#pragma unroll
    for (int i = 0; i < CW; ++i)
      x[i] = (r < rows && w0 + i < src_words) ? S[r * lds + w0 + i] : 0ull;
  }
  const Transpose tr(lane);
  // lane c then holds output row 64 (w0 + i) + c, word r0 / 64 + wave
#pragma unroll
  for (int i = 0; i < CW; ++i) tile[(64 * i + lane) * STR + wave] = transpose64(x[i], tr);
  __syncthreads();
  const int sub_r = tid / RB, sub_w = tid % RB;
  const int64_t wd = r0 / 64 + sub_w;
#pragma unroll
  for (int i = 0; i < CW; ++i) {
    const int orow = 64 * i + sub_r;
    const int64_t c = w0 * 64 + orow;
    if (c < cols && wd < dst_words) D[c * ldd + wd] = tile[orow * STR + sub_w];
  }
}

template <int RB, int CW>
hipError_t launch(const uint64_t* src, int64_t lds, int64_t strideS, uint64_t* dst, int64_t ldd,
                  int64_t strideD, int64_t rows, int64_t cols, int64_t batch, hipStream_t s) {
  const int64_t n_rt = (rows + 64 * RB - 1) / (64 * RB);
  const int64_t n_wt = ((cols + 63) / 64 + CW - 1) / CW;
  const int64_t blocks = n_rt * n_wt * batch;
  if (!grid_fits(blocks, 64 * RB)) return kGridTooLarge;
  hipLaunchKernelGGL((transpose_kernel<RB, CW>), dim3((unsigned)blocks), dim3(64 * RB), 0, s, src,
                     lds, strideS, dst, ldd, strideD, rows, cols, (uint32_t)n_rt, (uint32_t)n_wt);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_transpose(const uint64_t* src, int64_t lds, int64_t strideS, uint64_t* dst,
                            int64_t ldd, int64_t strideD, int64_t rows, int64_t cols,
                            int64_t batch, hipStream_t s) {
  if (rows <= 0 || cols <= 0 || batch <= 0) return hipSuccess;
  const int64_t n_rt = (rows + 511) / 512, n_wt = (cols + 511) / 512;
  if (n_rt * n_wt * batch < 256)
    return launch<4, 2>(src, lds, strideS, dst, ldd, strideD, rows, cols, batch, s);
  // 512 threads per 512 x 512 bits: up to twice the largest launch goes in pieces
  if (batch == 1 && !grid_fits(n_rt * n_wt, 512) && grid_fits(n_rt * n_wt, 256)) {
    const bool by_rows = n_rt > n_wt;
    const int64_t step = (((int64_t)1 << 23) - 1) / (by_rows ? n_wt : n_rt) * 512;
    for (int64_t at = 0; at < (by_rows ? rows : cols); at += step) {
      const int64_t r = by_rows ? (rows - at < step ? rows - at : step) : rows;
      const int64_t c = by_rows ? cols : (cols - at < step ? cols - at : step);
      const hipError_t e =
          by_rows ? launch<8, 8>(src + at * lds, lds, 0, dst + at / 64, ldd, 0, r, c, 1, s)
                  : launch<8, 8>(src + at / 64, lds, 0, dst + at * ldd, ldd, 0, r, c, 1, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  return launch<8, 8>(src, lds, strideS, dst, ldd, strideD, rows, cols, batch, s);
}

}  // namespace bmm
