// Sums over the lanes of a wave.
#pragma once

#include <hip/hip_runtime.h>

namespace nk {

// v from the lane that the DPP pattern CTRL selects (a row shift or a row
// broadcast, in the rows of ROWMASK), 0.0 where the pattern has no source
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_take(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWMASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROWMASK, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// sum over the 64 lanes of a wave in a fixed order (DPP row shifts, then the
// row broadcasts; lane 63 ends with the total), returned in every lane
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_take<0x111, 0xf>(v);  // row_shr:1
  v += dpp_take<0x112, 0xf>(v);  // row_shr:2
  v += dpp_take<0x114, 0xf>(v);  // row_shr:4
  v += dpp_take<0x118, 0xf>(v);  // row_shr:8
  v += dpp_take<0x142, 0xa>(v);  // row_bcast:15
  v += dpp_take<0x143, 0xc>(v);  // row_bcast:31
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, 63);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), 63);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The butterfly sums v += v of lane ^ o, for o = 32 .. 1 (wave_xsum), 4 .. 1
// (oct_xsum, over 8 lanes) and 1, 2 (quad_xsum, over 4 lanes): the same bits
// as with shuffles, on DPP and the row swaps instead of LDS permutes.  After a
// step, lanes l and l ^ o agree, so a rotation within the row of 16 that meets
// either of them does for the next one.
// (a step on a and b at once: the sums of a in the even, of b in the odd half or rows)
__device__ __forceinline__ double pair_sum2(double a, double b, bool rows32) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(a);
  const unsigned long long v = (unsigned long long)__double_as_longlong(b);
  const auto l = rows32 ? __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)v, false, false)
                        : __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)v, false, false);
  const auto h = rows32 ? __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(v >> 32), false, false)
                        : __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(v >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
         __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}
__device__ __forceinline__ double pair_sum(double v, bool rows32) { return pair_sum2(v, v, rows32); }
__device__ __forceinline__ double row_xsum(double v) {
  v += dpp_take<0x128, 0xf>(v);  // row_ror:8
  v += dpp_take<0x124, 0xf>(v);  // row_ror:4
  v += dpp_take<0x122, 0xf>(v);  // row_ror:2
  v += dpp_take<0x121, 0xf>(v);  // row_ror:1
  return v;
}
__device__ __forceinline__ double wave_xsum(double v) { return row_xsum(pair_sum(pair_sum(v, true), false)); }
// the same sums of several values at once, in fewer instructions: the first
// steps leave every value in a part of the wave, the later ones serve all.
// Of two, lanes 0 to 31 get the first; of four, row q of 16 lanes gets vq.
__device__ __forceinline__ double wave_xsum2(double v0, double v1) {
  return row_xsum(pair_sum(pair_sum2(v0, v1, true), false));
}
__device__ __forceinline__ double wave_xsum4(double v0, double v1, double v2, double v3) {
  return row_xsum(pair_sum2(pair_sum2(v0, v2, true), pair_sum2(v1, v3, true), false));
}
__device__ __forceinline__ double quad_xsum(double v) {
  v += dpp_take<0xb1, 0xf>(v);  // quad_perm 1, 0, 3, 2
  v += dpp_take<0x4e, 0xf>(v);  // quad_perm 2, 3, 0, 1
  return v;
}
__device__ __forceinline__ double oct_xsum(double v) {
  const double up = dpp_take<0x104, 0xf>(v), dn = dpp_take<0x114, 0xf>(v);  // row_shl:4: lane + 4, row_shr:4: lane - 4
  v += (threadIdx.x & 4) ? dn : up;
  v += dpp_take<0x4e, 0xf>(v);  // quad_perm 2, 3, 0, 1
  v += dpp_take<0xb1, 0xf>(v);  // quad_perm 1, 0, 3, 2
  return v;
}

}  // namespace nk
