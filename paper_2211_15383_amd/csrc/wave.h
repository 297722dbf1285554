// Reductions over the 64 lanes of a wavefront on cross-lane moves (no LDS traffic).  Every
// sum is the balanced tree over the lane index bits 5, 4, 3, 2, 1, 0 in that order, whatever
// the form, so all of them round alike.
#pragma once

#include <hip/hip_runtime.h>

namespace wave {

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false));
}

// lane l takes lane l ^ 4: a shift by 4 one way on the lanes with bit 2 clear, the other way
// on the rest
__device__ __forceinline__ int xor4(int v) {
  const int a = __builtin_amdgcn_update_dpp(0, v, 0x104, 0xf, 0x5, false);
  return __builtin_amdgcn_update_dpp(a, v, 0x114, 0xf, 0xa, false);
}
__device__ __forceinline__ double xor4(double v) {
  return __hiloint2double(xor4(__double2hiint(v)), xor4(__double2loint(v)));
}

// lanes with bit 5 (bit 4) clear get a(l) + a(l ^ 32), the others b(l) + b(l ^ 32) (16): the
// swap exchanges a's upper halves with b's lower ones
__device__ __forceinline__ double fold32(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double fold16(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// Sum of v over the wavefront, in every lane.
__device__ __forceinline__ double sum(double v) {
  v = fold32(v, v);
  v = fold16(v, v);
  v += dpp<0x128>(v);  // rotate the row of 16 by 8, then (equal values 8 apart) by 4
  v += dpp<0x124>(v);
  v += dpp<0x4e>(v);   // lanes 2 3 0 1 of each quad
  v += dpp<0xb1>(v);   // lanes 1 0 3 2
  return v;
}

// v summed over the lanes that differ in the bits lo, 2 lo, .. < hi of their number (lo, hi
// powers of two, hi <= 64), in every lane.
__device__ __forceinline__ double sum_lanes(double v, int lo, int hi) {
  if (lo <= 1 && 1 < hi) v += dpp<0xb1>(v);
  if (lo <= 2 && 2 < hi) v += dpp<0x4e>(v);
  if (lo <= 4 && 4 < hi) v += xor4(v);
  if (lo <= 8 && 8 < hi) v += dpp<0x128>(v);
  if (lo <= 16 && 16 < hi) v = fold16(v, v);
  if (lo <= 32 && 32 < hi) v = fold32(v, v);
  return v;
}

// The sums of v[0..7], v[l >> 3] in lane l.
__device__ __forceinline__ double sum8(double (&v)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = fold32(v[i], v[4 + i]);
#pragma unroll
  for (int i = 0; i < 2; ++i) v[i] = fold16(v[i], v[2 + i]);
  const bool h8 = (threadIdx.x & 8) != 0;
  double s = (h8 ? v[1] : v[0]) + dpp<0x128>(h8 ? v[0] : v[1]);
  s += xor4(s);
  s += dpp<0x4e>(s);
  s += dpp<0xb1>(s);
  return s;
}

// The sums of v[0..15] by recursive halving: at each exchange a lane keeps half of its values
// and adds the partner's copy of that half.  Returns, in lane l, the sum of v[l >> 2].
__device__ __forceinline__ double sum16(double (&v)[16]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = fold32(v[i], v[8 + i]);
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = fold16(v[i], v[4 + i]);
  const bool h8 = (lane & 8) != 0, h4 = (lane & 4) != 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double a = v[i], b = v[2 + i];
    v[i] = (h8 ? b : a) + dpp<0x128>(h8 ? a : b);
  }
  double s = (h4 ? v[1] : v[0]) + xor4(h4 ? v[0] : v[1]);
  s += dpp<0x4e>(s);
  s += dpp<0xb1>(s);
  return s;
}

}  // namespace wave
