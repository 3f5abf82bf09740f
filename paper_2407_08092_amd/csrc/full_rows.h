// full_rows.h -- the rows of 64 consecutive sites of one parity in a full vector [site][NE] of
// 16-byte elements (FP64: NE = 12; FP32: NE = 6).
//
// The parity's sites alternate with the other's along x: NE contiguous elements each, every
// second run.  Consecutive lanes take consecutive elements, so an access of a wavefront covers
// 64 / NE whole runs instead of one element in each of 64, and the rows change places in LDS.
#pragma once

#include "ddq_device.h"

namespace ddq {

// an element of a caller's vector: 8-byte alignment is all that an FP32 vector has to have
typedef unsigned int u4a8_t __attribute__((ext_vector_type(4), aligned(8)));

constexpr int FULL_ROW = 65;  // elements between rows in LDS: 64 sites, one of padding against bank conflicts

// orders a wavefront's LDS writes before its reads
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int NE>
struct FullRows {
  int base, count;           // first site, sites
  unsigned long long odd_x;  // bit l: site base + l has odd x
  // every lane of the wavefront calls it
  __device__ __forceinline__ FullRows(const Geo& g, int base_, int end, int parity, int lane)
      : base(base_), count(end - base_), odd_x(__ballot(decode(g, min(base_ + lane, end - 1), parity).x & 1)) {}
  __device__ __forceinline__ size_t at(int l, int e) const {  // element e of site l
    return (2 * (size_t)(base + l) + ((odd_x >> l) & 1)) * NE + e;
  }
  // by THREADS threads (a multiple of 64), t = 0 .. THREADS - 1; rows of sites past the last hold
  // the last one's
  template <int THREADS>
  __device__ __forceinline__ void load(const u4a8_t* full, u4_t (*lds)[FULL_ROW], int t) const {
    u4_t v[64 * NE / THREADS];
#pragma unroll
    for (int k = 0; k < 64 * NE / THREADS; ++k) {
      const int q = t + k * THREADS, l = q / NE;
      v[k] = full[at(min(l, count - 1), q - NE * l)];
    }
#pragma unroll
    for (int k = 0; k < 64 * NE / THREADS; ++k) {
      const int q = t + k * THREADS, l = q / NE;
      lds[q - NE * l][l] = v[k];
    }
  }
  template <int THREADS>
  __device__ __forceinline__ void store(u4a8_t* full, const u4_t (*lds)[FULL_ROW], int t) const {
    u4_t v[64 * NE / THREADS];
#pragma unroll
    for (int k = 0; k < 64 * NE / THREADS; ++k) {
      const int q = t + k * THREADS, l = q / NE;
      v[k] = lds[q - NE * l][l];
    }
#pragma unroll
    for (int k = 0; k < 64 * NE / THREADS; ++k) {
      const int q = t + k * THREADS, l = q / NE;
      if (l < count) full[at(l, q - NE * l)] = v[k];
    }
    store_fence();
  }
};

}  // namespace ddq
