// Expanding and compressing levels of the recursion (sections 3.8, 3.9, 3.11;
// Algorithms 1 and 2 of the paper) for every 2 x 2 scheme in scheme.h: the
// self-inverse design (eqs. mb-tsrecurrence and mb-qrecurrence, matrix form
// eq. mb-albega), the chaining design (eqs. ab-tsrecurrence and
// ab-qrecurrence) and Strassen-Winograd (eqs. sw-input and sw-output).
//
// The right operand is kept transposed throughout (its quadrant (j, k) lives
// at (k, j)), so the right expansion reads the stored 01 quadrant as B10 and
// the stored 10 quadrant as B01; each S_h is then produced already transposed.
//
// Every thread owns one 64-bit word position of a child (or grandchild) and
// moves it through registers: one level reads 4 words and writes 7 (expand)
// or reads 7 and writes 4 (compress); the merged two-level kernels read 16 and
// write 49, or read 49 and write 16, so the intermediate level never goes to
// HBM (section 3.15, merging levels).  With operands in the standard basis the levels'
// basis changes are applied in the same registers, which saves their own passes over A, B
// and C, and the copy of A they would change.  Children of parent p are matrices
// 7p + h, grandchildren 49p + 7h1 + h2, stored compactly one after another.
#include <type_traits>

#include "bmm_internal.h"
#include "scheme.h"

namespace bmm {
namespace {

using scheme::compress_one;
using scheme::expand_one;

// Index of a word: 32 bits where every index of the launch fits (a 64-bit division is about
// 100 instructions, as many as the rest of a thread's work).
inline bool fits32(int64_t total) { return total < ((int64_t)1 << 31); }

// One operand of an expansion: parents of rows x words at base + p * stride, pitch ld.
struct Operand {
  const uint64_t* src;
  int64_t ld, stride;
  uint64_t* dst;
  int64_t rows;
};

// BASIS: the operand is in the standard basis, and each level's forward change is applied
// to the quadrants before they expand (phi then alpha or beta, level by level, is the same
// map as all levels of phi first: both are Kronecker products over the levels).
template <int SCH, int SIDE, int BASIS>
__device__ __forceinline__ void expand_level(uint64_t q00, uint64_t q01, uint64_t q10,
                                             uint64_t q11, uint64_t (&o)[7]) {
  if constexpr (BASIS) {
    if constexpr (SIDE == 0) scheme::fwd<SCH>(q00, q01, q10, q11);
    else scheme::fwd<SCH>(q00, q10, q01, q11);  // stored transposed
  }
  expand_one<SCH, SIDE>(q00, q01, q10, q11, o);
}

template <int SCH, int SIDE, int BASIS, class I>
__device__ __forceinline__ void expand1(const Operand& a, int64_t words, int64_t parents) {
  const I hr = (I)(a.rows >> 1), hw = (I)(words >> 1);
  const I csize = hr * hw, total = csize * (I)parents;
  const I gstride = (I)gridDim.x * blockDim.x;
  for (I e = (I)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gstride) {
    const I p = e / csize, q = e - p * csize, r = q / hw, w = q - r * hw;
    const uint64_t* P = a.src + (int64_t)p * a.stride + (int64_t)r * a.ld + w;
    const int64_t down = (int64_t)hr * a.ld;
    uint64_t o[7];
    expand_level<SCH, SIDE, BASIS>(P[0], P[hw], P[down], P[down + hw], o);
    uint64_t* D = a.dst + 7 * (int64_t)p * csize + q;
#pragma unroll
    for (int h = 0; h < 7; ++h) D[h * (int64_t)csize] = o[h];
  }
}

template <int SCH, int SIDE, int BASIS, class I>
__device__ __forceinline__ void expand2(const Operand& a, int64_t words, int64_t parents) {
  const I qr = (I)(a.rows >> 2), qw = (I)(words >> 2);
  const I gsize = qr * qw, total = gsize * (I)parents;
  const I gstride = (I)gridDim.x * blockDim.x;
  for (I e = (I)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gstride) {
    const I p = e / gsize, q = e - p * gsize, r = q / qw, w = q - r * qw;
    const uint64_t* P = a.src + (int64_t)p * a.stride + (int64_t)r * a.ld + w;
    // x[i1][j1][i2][j2] at row i1*2qr + i2*qr + r, word j1*2qw + j2*qw + w
    uint64_t x[2][2][2][2];
#pragma unroll
    for (int i1 = 0; i1 < 2; ++i1)
#pragma unroll
      for (int j1 = 0; j1 < 2; ++j1)
#pragma unroll
        for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
          for (int j2 = 0; j2 < 2; ++j2)
            x[i1][j1][i2][j2] = P[(2 * i1 + i2) * (int64_t)qr * a.ld + (2 * j1 + j2) * (int64_t)qw];
    // first level: for each inner quadrant (i2, j2), expand over (i1, j1)
    uint64_t t[7][2][2];
#pragma unroll
    for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
      for (int j2 = 0; j2 < 2; ++j2) {
        uint64_t o[7];
        expand_level<SCH, SIDE, BASIS>(x[0][0][i2][j2], x[0][1][i2][j2], x[1][0][i2][j2],
                                       x[1][1][i2][j2], o);
#pragma unroll
        for (int h = 0; h < 7; ++h) t[h][i2][j2] = o[h];
      }
    uint64_t* D = a.dst + 49 * (int64_t)p * gsize + q;
#pragma unroll
    for (int h1 = 0; h1 < 7; ++h1) {
      uint64_t o[7];
      expand_level<SCH, SIDE, BASIS>(t[h1][0][0], t[h1][0][1], t[h1][1][0], t[h1][1][1], o);
#pragma unroll
      for (int h2 = 0; h2 < 7; ++h2) D[(7 * h1 + h2) * (int64_t)gsize] = o[h2];
    }
  }
}

// Both operands in one launch: the left one in grid row 0, the right one in row 1, or in row 0
// where there is no left one (no rows).
template <int SCH, int LEVELS, int BASIS, class I>
__global__ __launch_bounds__(256) void expand_kernel(Operand left, Operand right, int64_t words,
                                                     int64_t parents) {
  if (blockIdx.y == 0 && left.rows > 0) {
    if constexpr (LEVELS == 2) expand2<SCH, 0, BASIS, I>(left, words, parents);
    else expand1<SCH, 0, BASIS, I>(left, words, parents);
  } else {
    if constexpr (LEVELS == 2) expand2<SCH, 1, BASIS, I>(right, words, parents);
    else expand1<SCH, 1, BASIS, I>(right, words, parents);
  }
}

template <int ACC>
__device__ __forceinline__ void put(uint64_t& d, uint64_t v) {
  if (ACC)
    d ^= v;
  else
    d = v;
}

// Seven products into four quadrants; BASIS: and this level's inverse change after it.
template <int SCH, int BASIS>
__device__ __forceinline__ void compress_level(const uint64_t (&v)[7], uint64_t& c00, uint64_t& c01,
                                               uint64_t& c10, uint64_t& c11) {
  compress_one<SCH>(v, c00, c01, c10, c11);
  if constexpr (BASIS) scheme::inv<SCH>(c00, c01, c10, c11);
}

// ACC = 1: the parent quadrants are XORed into dst instead of overwriting it.
template <int SCH, int ACC, int BASIS, class I>
__global__ __launch_bounds__(256) void compress_kernel(const uint64_t* __restrict__ src,
                                                       uint64_t* __restrict__ dst, int64_t ldp,
                                                       int64_t strideP, int64_t rows,
                                                       int64_t words, int64_t parents) {
  const I hr = (I)(rows >> 1), hw = (I)(words >> 1);
  const I csize = hr * hw, total = csize * (I)parents;
  const I gstride = (I)gridDim.x * blockDim.x;
  for (I e = (I)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gstride) {
    const I p = e / csize, q = e - p * csize, r = q / hw, w = q - r * hw;
    const uint64_t* S = src + 7 * (int64_t)p * csize + q;
    uint64_t v[7];
#pragma unroll
    for (int h = 0; h < 7; ++h) v[h] = S[h * (int64_t)csize];
    uint64_t c00, c01, c10, c11;
    compress_level<SCH, BASIS>(v, c00, c01, c10, c11);
    uint64_t* P = dst + (int64_t)p * strideP + (int64_t)r * ldp + w;
    const int64_t down = (int64_t)hr * ldp;
    put<ACC>(P[0], c00);
    put<ACC>(P[hw], c01);
    put<ACC>(P[down], c10);
    put<ACC>(P[down + hw], c11);
  }
}

template <int SCH, int ACC, int BASIS, class I>
__global__ __launch_bounds__(256) void compress2_kernel(const uint64_t* __restrict__ src,
                                                        uint64_t* __restrict__ dst, int64_t ldp,
                                                        int64_t strideP, int64_t rows,
                                                        int64_t words, int64_t parents) {
  const I qr = (I)(rows >> 2), qw = (I)(words >> 2);
  const I gsize = qr * qw, total = gsize * (I)parents;
  const I gstride = (I)gridDim.x * blockDim.x;
  for (I e = (I)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gstride) {
    const I p = e / gsize, q = e - p * gsize, r = q / qw, w = q - r * qw;
    const uint64_t* S = src + 49 * (int64_t)p * gsize + q;
    // inner level: for each h1, combine the seven h2 products into quadrants (i2, k2)
    uint64_t c[7][2][2];
#pragma unroll
    for (int h1 = 0; h1 < 7; ++h1) {
      uint64_t v[7];
#pragma unroll
      for (int h2 = 0; h2 < 7; ++h2) v[h2] = S[(7 * h1 + h2) * (int64_t)gsize];
      compress_level<SCH, BASIS>(v, c[h1][0][0], c[h1][0][1], c[h1][1][0], c[h1][1][1]);
    }
    uint64_t* P = dst + (int64_t)p * strideP + (int64_t)r * ldp + w;
#pragma unroll
    for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        uint64_t v[7];
#pragma unroll
        for (int h1 = 0; h1 < 7; ++h1) v[h1] = c[h1][i2][k2];
        uint64_t c00, c01, c10, c11;
        compress_level<SCH, BASIS>(v, c00, c01, c10, c11);
        const int64_t off = i2 * (int64_t)qr * ldp + k2 * (int64_t)qw;
        put<ACC>(P[off], c00);
        put<ACC>(P[off + 2 * (int64_t)qw], c01);
        put<ACC>(P[off + 2 * (int64_t)qr * ldp], c10);
        put<ACC>(P[off + 2 * (int64_t)qr * ldp + 2 * (int64_t)qw], c11);
      }
  }
}

// One child of one parent (rows x words, pitch ldp): dst (rows/2 x words/2, pitch ldd)
// = XOR of the parent quadrants in `mask` (bit q: quadrant q in the order 00, 01, 10, 11).
__global__ __launch_bounds__(256) void child_kernel(const uint64_t* __restrict__ src,
                                                    int64_t ldp, uint64_t* __restrict__ dst,
                                                    int64_t ldd, int64_t rows, int64_t words,
                                                    uint32_t mask) {
  const int64_t hr = rows >> 1, hw = words >> 1;
  const int64_t total = hr * hw;
  const int64_t gstride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gstride) {
    const int64_t r = e / hw;
    const int64_t w = e - r * hw;
    uint64_t v = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((mask >> q) & 1u) v ^= src[(r + (q >> 1) * hr) * ldp + (q & 1) * hw + w];
    dst[r * ldd + w] = v;
  }
}

// One product (rows/2 x words/2, pitch lds) into the parent's result quadrants in
// `targets`: overwriting those in `overwrite`, XORed into the others.
__global__ __launch_bounds__(256) void gamma_kernel(const uint64_t* __restrict__ src,
                                                    int64_t lds, uint64_t* __restrict__ dst,
                                                    int64_t ldp, int64_t rows, int64_t words,
                                                    uint32_t targets, uint32_t overwrite) {
  const int64_t hr = rows >> 1, hw = words >> 1;
  const int64_t total = hr * hw;
  const int64_t gstride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gstride) {
    const int64_t r = e / hw;
    const int64_t w = e - r * hw;
    const uint64_t v = src[r * lds + w];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (!((targets >> q) & 1u)) continue;
      uint64_t& d = dst[(r + (q >> 1) * hr) * ldp + (q & 1) * hw + w];
      d = ((overwrite >> q) & 1u) ? v : (d ^ v);
    }
  }
}

__global__ __launch_bounds__(256) void copy_kernel(const uint64_t* __restrict__ src, int64_t lds,
                                                   uint64_t* __restrict__ dst, int64_t ldd,
                                                   int64_t rows, int64_t words) {
  const int64_t total = rows * words;
  const int64_t gstride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gstride) {
    const int64_t r = e / words;
    const int64_t w = e - r * words;
    dst[r * ldd + w] = src[r * lds + w];
  }
}

__global__ __launch_bounds__(256) void xor_kernel(const uint64_t* __restrict__ src, int64_t lds,
                                                  uint64_t* __restrict__ dst, int64_t ldd,
                                                  int64_t rows, int64_t words) {
  const int64_t total = rows * words;
  const int64_t gstride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gstride) {
    const int64_t r = e / words;
    const int64_t w = e - r * words;
    dst[r * ldd + w] ^= src[r * lds + w];
  }
}

// Pseudo-random words for the autotuner's timing buffers (the matrix cores' rate
// depends on how many operand bits switch, so tuning runs on dense random bits):
// the 64-bit finalizer of MurmurHash3 applied to seed + index.
__global__ __launch_bounds__(256) void random_kernel(uint64_t* __restrict__ dst, int64_t words,
                                                     uint64_t seed) {
  const int64_t gstride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < words; e += gstride) {
    uint64_t z = seed + (uint64_t)e;
    z ^= z >> 33;
    z *= 0xFF51AFD7ED558CCDull;
    z ^= z >> 33;
    z *= 0xC4CEB9FE1A85EC53ull;
    z ^= z >> 33;
    dst[e] = z;
  }
}

__global__ __launch_bounds__(256) void zero_kernel(uint64_t* __restrict__ dst, int64_t ld,
                                                   int64_t rows, int64_t words) {
  const int64_t total = rows * words;
  const int64_t gstride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gstride) {
    const int64_t r = e / words;
    const int64_t w = e - r * words;
    dst[r * ld + w] = 0ull;
  }
}

inline unsigned grid_for(int64_t total) {
  int64_t blocks = (total + 255) / 256;
  if (blocks > 32768) blocks = 32768;
  if (blocks < 1) blocks = 1;
  return (unsigned)blocks;
}

template <int SCH, int BASIS, class I>
void launch_expand_t(int levels, const Operand& l, const Operand& r, int64_t words,
                     int64_t parents, dim3 g, hipStream_t s) {
  if (levels == 2)
    hipLaunchKernelGGL((expand_kernel<SCH, 2, BASIS, I>), g, dim3(256), 0, s, l, r, words, parents);
  else
    hipLaunchKernelGGL((expand_kernel<SCH, 1, BASIS, I>), g, dim3(256), 0, s, l, r, words, parents);
}

template <int SCH>
hipError_t expand_sch(int levels, const Operand& l, const Operand& r, int64_t words,
                      int64_t parents, int basis, hipStream_t s) {
  const int sh = levels == 2 ? 2 : 1;
  const int64_t rows = l.rows > r.rows ? l.rows : r.rows;
  const int64_t total = (rows >> sh) * (words >> sh) * parents;
  if (total <= 0) return hipSuccess;
  const dim3 g(grid_for(total), l.rows > 0 && r.rows > 0 ? 2 : 1);
  const bool narrow = fits32(total);
  if (basis) narrow ? launch_expand_t<SCH, 1, uint32_t>(levels, l, r, words, parents, g, s)
                    : launch_expand_t<SCH, 1, int64_t>(levels, l, r, words, parents, g, s);
  else narrow ? launch_expand_t<SCH, 0, uint32_t>(levels, l, r, words, parents, g, s)
              : launch_expand_t<SCH, 0, int64_t>(levels, l, r, words, parents, g, s);
  return hipGetLastError();
}

template <int SCH, int ACC, int BASIS, class I>
void launch_compress_t(int levels, const uint64_t* src, uint64_t* dst, int64_t ldp,
                       int64_t strideP, int64_t rows, int64_t words, int64_t parents, dim3 g,
                       hipStream_t s) {
  if (levels == 2)
    hipLaunchKernelGGL((compress2_kernel<SCH, ACC, BASIS, I>), g, dim3(256), 0, s, src, dst, ldp,
                       strideP, rows, words, parents);
  else
    hipLaunchKernelGGL((compress_kernel<SCH, ACC, BASIS, I>), g, dim3(256), 0, s, src, dst, ldp,
                       strideP, rows, words, parents);
}

template <int SCH, int ACC, int BASIS>
void launch_compress_i(int levels, const uint64_t* src, uint64_t* dst, int64_t ldp,
                       int64_t strideP, int64_t rows, int64_t words, int64_t parents, dim3 g,
                       bool narrow, hipStream_t s) {
  if (narrow)
    launch_compress_t<SCH, ACC, BASIS, uint32_t>(levels, src, dst, ldp, strideP, rows, words,
                                                 parents, g, s);
  else
    launch_compress_t<SCH, ACC, BASIS, int64_t>(levels, src, dst, ldp, strideP, rows, words,
                                                parents, g, s);
}

template <int SCH>
hipError_t compress_sch(int levels, const uint64_t* src, uint64_t* dst, int64_t ldp,
                        int64_t strideP, int64_t rows, int64_t words, int64_t parents,
                        hipStream_t s, int accumulate, int basis) {
  const int sh = levels == 2 ? 2 : 1;
  const int64_t total = (rows >> sh) * (words >> sh) * parents;
  if (total <= 0) return hipSuccess;
  const dim3 g(grid_for(total));
  const bool narrow = fits32(total);
  auto go = [&](auto acc, auto bas) {
    launch_compress_i<SCH, decltype(acc)::value, decltype(bas)::value>(
        levels, src, dst, ldp, strideP, rows, words, parents, g, narrow, s);
  };
  const std::integral_constant<int, 0> no;
  const std::integral_constant<int, 1> yes;
  if (accumulate) basis ? go(yes, yes) : go(yes, no);
  else basis ? go(no, yes) : go(no, no);
  return hipGetLastError();
}

hipError_t expand_any(int scheme, int levels, const Operand& l, const Operand& r, int64_t words,
                      int64_t parents, int basis, hipStream_t s) {
  switch (scheme) {
    case BMM_SCHEME_CHAINING:
      return expand_sch<BMM_SCHEME_CHAINING>(levels, l, r, words, parents, basis, s);
    case BMM_SCHEME_WINOGRAD:  // no basis change
      return expand_sch<BMM_SCHEME_WINOGRAD>(levels, l, r, words, parents, 0, s);
    default:
      return expand_sch<BMM_SCHEME_SELF_INVERSE>(levels, l, r, words, parents, basis, s);
  }
}

hipError_t compress_any(int scheme, int levels, const uint64_t* src, uint64_t* dst, int64_t ldp,
                        int64_t strideP, int64_t rows, int64_t words, int64_t parents,
                        hipStream_t s, int accumulate, int basis) {
  switch (scheme) {
    case BMM_SCHEME_CHAINING:
      return compress_sch<BMM_SCHEME_CHAINING>(levels, src, dst, ldp, strideP, rows, words,
                                               parents, s, accumulate, basis);
    case BMM_SCHEME_WINOGRAD:
      return compress_sch<BMM_SCHEME_WINOGRAD>(levels, src, dst, ldp, strideP, rows, words,
                                               parents, s, accumulate, 0);
    default:
      return compress_sch<BMM_SCHEME_SELF_INVERSE>(levels, src, dst, ldp, strideP, rows, words,
                                                   parents, s, accumulate, basis);
  }
}

// Coefficient masks of a scheme, from its own programs run on bit masks: the stored
// quadrants child h of side `side` sums, and the products result quadrant q sums.
template <int SCH>
uint32_t child_mask_of(int side, int h) {
  uint64_t o[7];
  if (side == 0)
    scheme::expand_one<SCH, 0>(1, 2, 4, 8, o);
  else
    scheme::expand_one<SCH, 1>(1, 2, 4, 8, o);
  return (uint32_t)o[h];
}
template <int SCH>
void gamma_masks_of(uint32_t (&g)[4]) {
  const uint64_t in[7] = {1, 2, 4, 8, 16, 32, 64};
  uint64_t c[4];
  scheme::compress_one<SCH>(in, c[0], c[1], c[2], c[3]);
  for (int q = 0; q < 4; ++q) g[q] = (uint32_t)c[q];
}

}  // namespace

uint32_t child_mask(int scheme, int side, int h) {
  if (scheme == BMM_SCHEME_CHAINING) return child_mask_of<BMM_SCHEME_CHAINING>(side, h);
  if (scheme == BMM_SCHEME_WINOGRAD) return child_mask_of<BMM_SCHEME_WINOGRAD>(side, h);
  return child_mask_of<BMM_SCHEME_SELF_INVERSE>(side, h);
}

hipError_t launch_child(int scheme, int side, int h, const uint64_t* src, int64_t ldp,
                        uint64_t* dst, int64_t ldd, int64_t rows, int64_t words, hipStream_t s) {
  const int64_t total = (rows >> 1) * (words >> 1);
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(child_kernel, dim3(grid_for(total)), dim3(256), 0, s, src, ldp, dst, ldd,
                     rows, words, child_mask(scheme, side, h));
  return hipGetLastError();
}

hipError_t launch_gamma(int scheme, int h, const uint64_t* src, int64_t lds, uint64_t* dst,
                        int64_t ldp, int64_t rows, int64_t words, int accumulate,
                        hipStream_t s) {
  const int64_t total = (rows >> 1) * (words >> 1);
  if (total <= 0) return hipSuccess;
  uint32_t g[4];
  if (scheme == BMM_SCHEME_CHAINING)
    gamma_masks_of<BMM_SCHEME_CHAINING>(g);
  else if (scheme == BMM_SCHEME_WINOGRAD)
    gamma_masks_of<BMM_SCHEME_WINOGRAD>(g);
  else
    gamma_masks_of<BMM_SCHEME_SELF_INVERSE>(g);
  uint32_t targets = 0, overwrite = 0;
  for (int q = 0; q < 4; ++q) {
    if (!((g[q] >> h) & 1u)) continue;
    targets |= 1u << q;
    // the first product of a quadrant overwrites it, unless the result accumulates
    if (!accumulate && (g[q] & ((1u << h) - 1u)) == 0) overwrite |= 1u << q;
  }
  hipLaunchKernelGGL(gamma_kernel, dim3(grid_for(total)), dim3(256), 0, s, src, lds, dst, ldp,
                     rows, words, targets, overwrite);
  return hipGetLastError();
}

hipError_t launch_expand(int side, int levels, const uint64_t* src, int64_t ldp, int64_t strideP,
                         uint64_t* dst, int64_t rows, int64_t words, int64_t parents,
                         hipStream_t s, int scheme) {
  const Operand x{src, ldp, strideP, dst, rows}, none{nullptr, 0, 0, nullptr, 0};
  return side == 0 ? expand_any(scheme, levels, x, none, words, parents, 0, s)
                   : expand_any(scheme, levels, none, x, words, parents, 0, s);
}

hipError_t launch_expand_pair(int levels, const uint64_t* T, int64_t ldT, int64_t strideT,
                              uint64_t* dstT, int64_t rowsT, const uint64_t* S, int64_t ldS,
                              int64_t strideS, uint64_t* dstS, int64_t rowsS, int64_t words,
                              int64_t parents, int basis, hipStream_t s, int scheme) {
  return expand_any(scheme, levels, Operand{T, ldT, strideT, dstT, rowsT},
                    Operand{S, ldS, strideS, dstS, rowsS}, words, parents, basis, s);
}

hipError_t launch_compress(int levels, const uint64_t* src, uint64_t* dst, int64_t ldp,
                           int64_t strideP, int64_t rows, int64_t words, int64_t parents,
                           hipStream_t s, int accumulate, int basis, int scheme) {
  return compress_any(scheme, levels, src, dst, ldp, strideP, rows, words, parents, s, accumulate,
                      basis);
}

hipError_t launch_copy(const uint64_t* src, int64_t lds, uint64_t* dst, int64_t ldd,
                       int64_t rows, int64_t words, hipStream_t s) {
  const int64_t total = rows * words;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(copy_kernel, dim3(grid_for(total)), dim3(256), 0, s, src, lds, dst, ldd,
                     rows, words);
  return hipGetLastError();
}

hipError_t launch_xor(const uint64_t* src, int64_t lds, uint64_t* dst, int64_t ldd, int64_t rows,
                      int64_t words, hipStream_t s) {
  const int64_t total = rows * words;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(xor_kernel, dim3(grid_for(total)), dim3(256), 0, s, src, lds, dst, ldd, rows,
                     words);
  return hipGetLastError();
}

hipError_t launch_random(uint64_t* dst, int64_t words, uint64_t seed, hipStream_t s) {
  if (words <= 0) return hipSuccess;
  hipLaunchKernelGGL(random_kernel, dim3(grid_for(words)), dim3(256), 0, s, dst, words, seed);
  return hipGetLastError();
}

hipError_t launch_zero(uint64_t* dst, int64_t ld, int64_t rows, int64_t words, hipStream_t s) {
  const int64_t total = rows * words;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_kernel, dim3(grid_for(total)), dim3(256), 0, s, dst, ld, rows, words);
  return hipGetLastError();
}

}  // namespace bmm
