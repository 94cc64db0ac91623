// Bit-matrix transposes within a wave, without LDS.
#pragma once

#include "bmm_internal.h"

namespace bmm {

// 32 x 32 bit transposes over the 32 lanes of each wave half, by five exchanges between
// lanes 16, 8, 4, 2 and 1 apart (3 VALU instructions each, where a ballot and two selects
// per count take 7 per count); the selectors depend on the lane only.
struct Transpose {
  uint32_t s16, s8, r4, m4, r2, m2, r1, m1;
  __device__ __forceinline__ explicit Transpose(int lane) {
    s16 = (lane & 16) ? 0x07060302u : 0x05040100u;
    s8 = (lane & 8) ? 0x03070105u : 0x06020400u;
    r4 = (lane & 4) ? 4 : 28;
    m4 = (lane & 4) ? 0x0f0f0f0fu : 0xf0f0f0f0u;
    r2 = (lane & 2) ? 2 : 30;
    m2 = (lane & 2) ? 0x33333333u : 0xccccccccu;
    r1 = (lane & 1) ? 1 : 31;
    m1 = (lane & 1) ? 0x55555555u : 0xaaaaaaaau;
  }
  template <int CTRL>
  static __device__ __forceinline__ uint32_t dpp(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
  }
  static __device__ __forceinline__ uint32_t merge(uint32_t m, uint32_t y, uint32_t r, uint32_t x) {
    return (m & __builtin_amdgcn_alignbit(y, y, r)) | (~m & x);
  }
  __device__ __forceinline__ uint32_t operator()(uint32_t x) const {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = __builtin_amdgcn_perm(r[1], r[0], s16);
    x = __builtin_amdgcn_perm(dpp<0x128>(x), x, s8);        // row_ror:8
    x = merge(m4, dpp<0x1B>(dpp<0x141>(x)), r4, x);         // half mirror, then 3 - i
    x = merge(m2, dpp<0x4E>(x), r2, x);                     // quad_perm [2,3,0,1]
    x = merge(m1, dpp<0xB1>(x), r1, x);                     // quad_perm [1,0,3,2]
    return x;
  }
};

// The lane index as a fresh value: what is derived from it (addresses, selectors) is not
// computed earlier than here and kept in registers across a main loop or a persistent one.
__device__ __forceinline__ int fresh_lane() {
  int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  asm volatile("" : "+v"(lane));
  return lane;
}

// 64 x 64 bits: lane r holds row r; afterwards lane c holds column c, bit r from row r.
__device__ __forceinline__ uint64_t transpose64(uint64_t x, const Transpose& tr) {
  // each half takes its 32 columns of rows 0..31 and 32..63
  const auto s = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)(x >> 32), false, false);
  return (uint64_t)tr(s[0]) | ((uint64_t)tr(s[1]) << 32);
}

}  // namespace bmm
