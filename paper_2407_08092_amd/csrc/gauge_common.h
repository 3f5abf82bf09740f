// gauge_common.h -- 3x3 products and packed-link access shared by the clover build and the
// link force.
//
// Both read the FP64 packed links: per parity and direction rows 0..8 hold U_mu(x), 64 sites of
// a row contiguous, so every load of a wavefront is one run of 16-byte elements (two where
// neighbours wrap or cross a block of 64).  Rows 9..17 hold the same links again, daggered,
// at the other end; they are left alone, because with one copy an XCD's 4 MB of L2 hold twice
// the sites, and each link is read by up to twelve of them.
#pragma once

#include "ddq_internal.h"

namespace ddq {

struct C3 {
  cpx<double> a[3][3];
};

// anti-Hermitian 3x3: i d on the diagonal, u = (0,1), (0,2), (1,2); entry (j, i) = -conj (i, j)
struct AH3 {
  double d[3];
  cpx<double> u[3];
};

__device__ __forceinline__ C3 c3_mul(const C3& A, const C3& B) {
  C3 C;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cpx<double> s = A.a[i][0] * B.a[0][j];
      cfma(s, A.a[i][1], B.a[1][j]);
      cfma(s, A.a[i][2], B.a[2][j]);
      C.a[i][j] = s;
    }
  return C;
}
// X = X B (DAG: X B^H), row by row
template <bool DAG>
__device__ __forceinline__ void c3_rmul(C3& X, const C3& B) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    cpx<double> row[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      row[j] = {0.0, 0.0};
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if constexpr (DAG)
          cfma_conj(row[j], B.a[j][k], X.a[i][k]);
        else
          cfma(row[j], X.a[i][k], B.a[k][j]);
      }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) X.a[i][j] = row[j];
  }
}
__device__ __forceinline__ C3 c3_dag(const C3& A) {
  C3 C;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) C.a[i][j] = conj(A.a[j][i]);
  return C;
}
__device__ __forceinline__ C3 c3_add(const C3& A, const C3& B) {
  C3 C;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) C.a[i][j] = A.a[i][j] + B.a[i][j];
  return C;
}
__device__ __forceinline__ C3 c3_sub(const C3& A, const C3& B) {
  C3 C;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) C.a[i][j] = A.a[i][j] - B.a[i][j];
  return C;
}

// entry (i, j) of W
__device__ __forceinline__ cpx<double> ah_at(const AH3& W, int i, int j) {
  if (i == j) return {0.0, W.d[i]};
  const cpx<double> v = W.u[i + j - 1];
  return i < j ? v : cpx<double>{-v.r, v.i};
}
// Y += A W
__device__ __forceinline__ void ah_right(C3& Y, const C3& A, const AH3& W) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (k == j) {
          Y.a[i][j].r = fma(-A.a[i][k].i, W.d[k], Y.a[i][j].r);
          Y.a[i][j].i = fma(A.a[i][k].r, W.d[k], Y.a[i][j].i);
        } else {
          cfma(Y.a[i][j], A.a[i][k], ah_at(W, k, j));
        }
      }
}
// Y += W A
__device__ __forceinline__ void ah_left(C3& Y, const AH3& W, const C3& A) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (k == i) {
          Y.a[i][j].r = fma(-W.d[k], A.a[k][j].i, Y.a[i][j].r);
          Y.a[i][j].i = fma(W.d[k], A.a[k][j].r, Y.a[i][j].i);
        } else {
          cfma(Y.a[i][j], ah_at(W, i, k), A.a[k][j]);
        }
      }
}
__device__ __forceinline__ C3 c3_zero() {
  C3 m;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) m.a[i][j] = {0.0, 0.0};
  return m;
}

// M formed here and the loads that follow issued after it: keeps the instruction selector from
// lifting every link of a plane to the top and spilling them
__device__ __forceinline__ void c3_fence(C3& M) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) asm volatile("" : "+v"(M.a[i][j].r), "+v"(M.a[i][j].i)::"memory");
}

// site s shifted by one step along mu (uniform over the wavefront), periodic; its parity is
// the other one
__device__ __forceinline__ Site site_shift(const Geo& g, Site s, int mu, int step) {
  auto move = [&](int c, int dir) {
    const int n = c + (mu == dir ? step : 0), L = g.L[dir];
    return n < 0 ? n + L : n >= L ? n - L : n;
  };
  s.x = move(s.x, 0);
  s.y = move(s.y, 1);
  s.z = move(s.z, 2);
  s.t = move(s.t, 3);
  s.i = (s.x + g.L[0] * (s.y + g.L[1] * (s.z + g.L[2] * s.t))) >> 1;
  return s;
}

// links of both parities
struct PackedLinks {
  const d2_t* p[2];
};
// U_mu at the site of parity q and index i
__device__ __forceinline__ C3 packed_link(const PackedLinks& L, const Geo& g, int q, int mu, int i) {
  const Link<double> l = load_link_half<double, 0>(
      bfield(L.p[q] + (size_t)mu * LINK_ROWS * field_vh(g.Vh), LINK_ROWS, g.Vh), 0, boff(i, LINK_ROWS));
  C3 m;
#pragma unroll
  for (int e = 0; e < 9; ++e) m.a[e / 3][e % 3] = l.u[e];
  return m;
}

// directions of plane 0..5: (x,y), (x,z), (x,t), (y,z), (y,t), (z,t)
__device__ __forceinline__ void plane_dirs(int plane, int& mu, int& nu) {
  mu = plane < 3 ? 0 : plane < 5 ? 1 : 2;
  nu = plane < 3 ? plane + 1 : plane < 5 ? plane - 1 : 3;
}

// The 64-site group [base, end) of workgroup blk out of launches with `per` workgroups a group
// (which: the workgroup's number within it), consecutive on one XCD: slab order (slab_group)
// where a slice has at least eight groups, else the groups in a row.
__device__ __forceinline__ bool gauge_group(const Geo& g, int blk, int per, int& which, int& base, int& end) {
  const int ng = (g.sT + 63) >> 6;
  if (ng >= 8) {
    const int local = blk >> 3;
    which = local % per;
    return slab_group(g, blk & 7, local / per, base, end);
  }
  which = blk % per;
  base = (blk / per) * 64;
  end = min(base + 64, g.Vh);
  return base < end;
}
inline long long gauge_groups(const Geo& g, int per) {
  const long long ng = (g.sT + 63) / 64;
  return ng >= 8 ? 8LL * per * slab_groups_per_xcd(g) : (long long)per * ((g.Vh + 63) / 64);
}

}  // namespace ddq
