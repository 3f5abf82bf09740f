// hop_h16.h -- 16-bit storage of spinors, links and clover blocks: element layout and
// conversions shared by the 16-bit stencil kernels.
#pragma once

#include "ddq_device.h"

namespace ddq {

typedef unsigned short u16_t;

template <typename S>
__device__ __forceinline__ float h2f(u16_t b) {
  return (float)__builtin_bit_cast(S, b);
}
template <typename S>
__device__ __forceinline__ u16_t f2h(float f) {
  return __builtin_bit_cast(u16_t, (S)f);
}

// element <-> four complex numbers; complex j is word j (re: low half, im: high half)
template <typename S>
__device__ __forceinline__ void unpack4(u4_t q, cpx<float>* c) {
#pragma unroll
  for (int j = 0; j < 4; ++j) c[j] = {h2f<S>((u16_t)(q[j] & 0xffffu)), h2f<S>((u16_t)(q[j] >> 16))};
}
template <typename S>
__device__ __forceinline__ u4_t pack4(const cpx<float>* c) {
  u4_t q;
#pragma unroll
  for (int j = 0; j < 4; ++j) q[j] = (unsigned)f2h<S>(c[j].r) | ((unsigned)f2h<S>(c[j].i) << 16);
  return q;
}

constexpr int SP16_E = 3;   // element rows of a spinor
constexpr int LK16_E = 3;   // element rows of one direction's 12-real link pair
constexpr int CL16_E = 10;  // element rows of a site's clover (2 blocks x 5)

template <typename S>
__device__ __forceinline__ Spinor<float> unpack_spinor(const u4_t (&q)[SP16_E]) {
  cpx<float> c[12];
#pragma unroll
  for (int e = 0; e < SP16_E; ++e) unpack4<S>(q[e], c + 4 * e);
  Spinor<float> s;
#pragma unroll
  for (int k = 0; k < 12; ++k) s.c[k / 3][k % 3] = c[k];
  return s;
}
template <typename S, int AUX = DDQ_SPINOR_AUX>
__device__ __forceinline__ Spinor<float> load_spinor16(const Field& v, uint32_t off) {
  u4_t q[SP16_E];
#pragma unroll
  for (int e = 0; e < SP16_E; ++e) q[e] = ld16<AUX>(v, e, off);
  return unpack_spinor<S>(q);
}
template <typename S, int AUX = DDQ_STORE_AUX>
__device__ __forceinline__ void store_spinor16(const Field& v, uint32_t off, const Spinor<float>& s) {
  cpx<float> c[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) c[k] = s.c[k / 3][k % 3];
#pragma unroll
  for (int e = 0; e < SP16_E; ++e) st16<AUX>(v, e, off, pack4<S>(c + 4 * e));
}

}  // namespace ddq
