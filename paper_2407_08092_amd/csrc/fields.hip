// fields.hip -- set-up kernels: gauge packing, clover blocks and their inverses,
// parity packing of vectors.
#include "full_rows.h"
#include "gauge_common.h"

namespace ddq {

// ---------------------------------------------------------------------------
// gauge packing: per parity p, direction mu and site i, complex rows 0..8 = U_mu(x)
// and rows 9..17 = U_mu(x-mu)^H (FP64: one complex per 16-byte element), and in the same
// pass the FP32 copy (18- or 12-real).
//
// A pass over memory: 576 B a site read, 2304 B (FP64) and 1152 or 768 B (FP32) written.  A
// workgroup takes the 128 consecutive sites of one 64-site block of both parities, a wavefront
// one direction of them: it reads their links in runs of 144 B into LDS and writes rows of 64
// sites, each link twice -- forward at its own site, daggered at x + mu, whose index runs with
// the lane.  16^3 x 32 with FP32: 51 us (5.9 TB/s) from 180
// in a copy, a pass that read 16-byte elements 576 B apart, and four conversions.
// ---------------------------------------------------------------------------
constexpr int PACK_SITES = 128;

// rows [r0, r0 + 9) of one site in the FP32 field of direction mu
__device__ __forceinline__ void put_link_f32(f2_t* f, int mu, int r0, int i, int vh, int mode, const cpx<double> (&u)[9]) {
  const size_t fv = (size_t)field_vh(vh);
  auto two = [&](int k) {
    f4_t o;
    o.x = (float)u[k].r;
    o.y = (float)u[k].i;
    o.z = (float)u[k + 1].r;
    o.w = (float)u[k + 1].i;
    return o;
  };
  if (mode == 12) {  // rows 0..5 of each half: elements 0..2 and 3..5
    constexpr int ER = LINK12_ROWS / 2;
    f4_t* d = (f4_t*)f + (size_t)mu * ER * fv;
#pragma unroll
    for (int e = 0; e < 3; ++e) d[fidx((r0 ? 3 : 0) + e, i, ER, vh)] = two(2 * e);
    return;
  }
  constexpr int ER = LINK_ROWS / 2;
  f4_t* d = (f4_t*)f + (size_t)mu * ER * fv;
  f2_t one;  // rows 8 and 9 share element 4
  const int k1 = r0 ? 0 : 8;
  one.x = (float)u[k1].r;
  one.y = (float)u[k1].i;
  ((f2_t*)&d[fidx(4, i, ER, vh)])[r0 ? 1 : 0] = one;
#pragma unroll
  for (int e = 0; e < 4; ++e) d[fidx(r0 ? 5 + e : e, i, ER, vh)] = two(r0 ? 2 * e + 1 : 2 * e);
}

__global__ void __launch_bounds__(256) k_pack_gauge(Geo g, const d2_t* __restrict__ U, d2_t* __restrict__ out_e,
                                                    d2_t* __restrict__ out_o, f2_t* __restrict__ f32_e,
                                                    f2_t* __restrict__ f32_o, int f32_mode) {
  __shared__ d2_t lds[4][PACK_SITES * 9];
  const int mu = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  const int vh = g.Vh;
  const long long n0 = (long long)blockIdx.x * PACK_SITES;
  const int sites = (int)min((long long)PACK_SITES, 2LL * vh - n0);
  d2_t* l = lds[mu];
#pragma unroll
  for (int k = 0; k < PACK_SITES * 9 / 64; ++k) {
    const int q = 64 * k + lane, s = q / 9, e = q - 9 * s;
    if (s < sites) l[q] = U[((n0 + s) * 4 + mu) * 9 + e];
  }
  __syncthreads();
  const int i = (int)(n0 >> 1) + lane;
  if (i >= vh) return;
  const size_t fsz = (size_t)LINK_ROWS * field_vh(vh);  // one direction's link field
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const Site s = decode(g, i, p);
    const d2_t* src = l + (2 * lane + (s.x & 1)) * 9;
    cpx<double> u[9], d[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = {src[e].x, src[e].y};
    d2_t* fwd = (p ? out_o : out_e) + mu * fsz;
#pragma unroll
    for (int e = 0; e < 9; ++e) fwd[fidx(e, i, LINK_ROWS, vh)] = d2_t{u[e].r, u[e].i};
    store_fence();
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) d[3 * a + b] = conj(u[3 * b + a]);
    const int j = site_shift(g, s, mu, 1).i;  // the link is the backward one of x + mu
    d2_t* bwd = (p ? out_e : out_o) + mu * fsz;
#pragma unroll
    for (int e = 0; e < 9; ++e) bwd[fidx(9 + e, j, LINK_ROWS, vh)] = d2_t{d[e].r, d[e].i};
    store_fence();
    if (f32_mode) {  // uniform
      put_link_f32(p ? f32_o : f32_e, mu, 0, i, vh, f32_mode, u);
      store_fence();
      put_link_f32(p ? f32_e : f32_o, mu, 9, j, vh, f32_mode, d);
      store_fence();
    }
  }
}

hipError_t launch_pack_gauge(const Geo& g, const d2_t* U, d2_t* out_e, d2_t* out_o, void* f32_e, void* f32_o, int link12,
                             hipStream_t s) {
  const long long blocks = (2LL * g.Vh + PACK_SITES - 1) / PACK_SITES;
  hipLaunchKernelGGL(k_pack_gauge, dim3((unsigned)blocks), dim3(256), 0, s, g, U, out_e, out_o, (f2_t*)f32_e, (f2_t*)f32_o,
                     f32_e ? (link12 ? 12 : 18) : 0);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// clover blocks
// ---------------------------------------------------------------------------
// F_munu(x) of plane (mu, nu): F = (Q - Q^H) / 8 with Q the sum of the four leaves
//   U_mu(x) U_nu(x+mu) U_mu(x+nu)^H U_nu(x)^H,          U_nu(x) U_mu(x-mu+nu)^H U_nu(x-mu)^H U_mu(x-mu),
//   U_mu(x-mu)^H U_nu(x-mu-nu)^H U_mu(x-mu-nu) U_nu(x-nu),  U_nu(x-nu)^H U_mu(x-nu) U_nu(x+mu-nu) U_mu(x)^H,
// each a chain from the left, 12 products.  10 would do (leaves 1 and 4, 2 and 3 share a factor up
// to conjugates that Q - Q^H cancels; 97 us against 119 for the clover build on 16^3 x 32), but their
// last bits differ, and a block entry whose FP32 rounding turns over moves everything that is solved
// with the FP32 blocks by 1e-9 to 1e-8.
__device__ __forceinline__ AH3 field_strength(const PackedLinks& L, const Geo& g, const Site& s, int p, int mu, int nu) {
  const int o = 1 - p;
  const Site fm = site_shift(g, s, mu, 1), fn = site_shift(g, s, nu, 1);
  const Site bm = site_shift(g, s, mu, -1), bn = site_shift(g, s, nu, -1);
  auto U = [&](int q, int dir, int i) { return packed_link(L, g, q, dir, i); };
  // X = X B, the sums of c3_mul, row by row
  auto times = [](C3& X, const C3& B) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cpx<double> row[3];
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        row[b] = X.a[a][0] * B.a[0][b];
        cfma(row[b], X.a[a][1], B.a[1][b]);
        cfma(row[b], X.a[a][2], B.a[2][b]);
      }
#pragma unroll
      for (int b = 0; b < 3; ++b) X.a[a][b] = row[b];
    }
    c3_fence(X);
  };
  const int i0 = s.i, bb = site_shift(g, bm, nu, -1).i, fb = site_shift(g, fm, nu, -1).i;  // x, x-mu-nu, x+mu-nu
  // one product at a time (c3_fence): the matrices in flight fit the registers of three wavefronts
  C3 T = U(p, mu, i0);
  times(T, U(o, nu, fm.i));
  times(T, c3_dag(U(o, mu, fn.i)));
  times(T, c3_dag(U(p, nu, i0)));
  C3 X = U(p, nu, i0);
  times(X, c3_dag(U(p, mu, site_shift(g, fn, mu, -1).i)));
  times(X, c3_dag(U(o, nu, bm.i)));
  times(X, U(o, mu, bm.i));
  T = c3_add(T, X);
  X = c3_dag(U(o, mu, bm.i));
  times(X, c3_dag(U(p, nu, bb)));
  times(X, U(p, mu, bb));
  times(X, U(o, nu, bn.i));
  T = c3_add(T, X);
  X = c3_dag(U(o, nu, bn.i));
  times(X, U(o, mu, bn.i));
  times(X, U(p, nu, fb));
  times(X, c3_dag(U(p, mu, i0)));
  T = c3_add(T, X);
  AH3 F;
#pragma unroll
  for (int a = 0; a < 3; ++a) F.d[a] = 0.25 * T.a[a][a].i;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a + 1; b < 3; ++b)
      F.u[a + b - 1] = {0.125 * (T.a[a][b].r - T.a[b][a].r), 0.125 * (T.a[a][b].i + T.a[b][a].i)};
  return F;
}

// slots of a Hermitian 6x6 block (upper triangle and diagonal of M) into block blk of site i of
// a clover field of R (FP32: two slots per 16-byte element)
template <typename R>
__device__ __forceinline__ void store_packed(void* C, int blk, int i, int vh, const cpx<double> (&M)[6][6]) {
  constexpr int E = 18 / CPE<R>;  // elements of a block
  const Field f = bfield(C, 2 * E, vh);
  const uint32_t off = boff(i, 2 * E);
  cpx<R> sl[18];
#pragma unroll
  for (int k = 0; k < 3; ++k) sl[k] = {(R)M[2 * k][2 * k].r, (R)M[2 * k + 1][2 * k + 1].r};
#pragma unroll
  for (int j = 0; j < 6; ++j)
#pragma unroll
    for (int k = j + 1; k < 6; ++k) sl[tri_slot(j, k)] = {(R)M[j][k].r, (R)M[j][k].i};
#pragma unroll
  for (int e = 0; e < E; ++e) st16<0>(f, E * blk + e, off, pack<R>(sl + e * CPE<R>));
}

// Inverse of a Hermitian positive-definite 6x6 matrix by Cholesky A = L L^H: reads and writes A's
// diagonal and upper triangle, L, L^-1 and the products in place below it; returns false if a
// pivot is not positive.  Y: A's upper triangle before its factor h; the first term of a sum
// takes h Y unrounded where it can.  The fused operations are written out, so that every
// build gives the same bits.
__device__ __forceinline__ bool hpd_inverse6(cpx<double> (&A)[6][6], const cpx<double> (&Y)[6][6], double h) {
  bool ok = true;
  double dg[6];  // L_jj
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    double d = A[j][j].r;
#pragma unroll
    for (int k = 0; k < j; ++k) {
      const double x = A[j][k].r, y = A[j][k].i;
      d -= fma(y, y, x * x);
    }
    if (!(d > 0.0)) {
      ok = false;
      d = 1.0;
    }
    dg[j] = sqrt(d);
#pragma unroll
    for (int r = j + 1; r < 6; ++r) {
      cpx<double> s = conj(A[j][r]);
#pragma unroll
      for (int k = 0; k < j; ++k) {
        const cpx<double> x = A[r][k], y = A[j][k];
        const double tr = fma(x.i, y.i, x.r * y.r), ti = fma(x.i, y.r, -(x.r * y.i));
        if (k > 0) s = {s.r - tr, s.i - ti};
        else s = {j < 3 && r >= 3 ? fma(h, Y[j][r].r, -tr) : s.r - tr, fma(h, -Y[j][r].i, -ti)};
      }
      A[r][j] = {s.r / dg[j], s.i / dg[j]};
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // L^-1 in its place, column by column: column c needs L's rows from column c on
  double inv[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    inv[c] = 1.0 / dg[c];
#pragma unroll
    for (int r = c + 1; r < 6; ++r) {
      cpx<double> s = {A[r][c].r * inv[c], A[r][c].i * inv[c]};
#pragma unroll
      for (int k = c + 1; k < r; ++k) cfma(s, A[r][k], A[k][c]);
      A[r][c] = {-s.r / dg[r], -s.i / dg[r]};
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // A^-1 = (L^-1)^H L^-1
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    double d = inv[j] * inv[j];
#pragma unroll
    for (int r = j + 1; r < 6; ++r) d = fma(A[r][j].i, A[r][j].i, fma(A[r][j].r, A[r][j].r, d));
    A[j][j] = {d, 0.0};
#pragma unroll
    for (int k = j + 1; k < 6; ++k) {
      cpx<double> s = inv[k] * conj(A[k][j]);
#pragma unroll
      for (int r = k + 1; r < 6; ++r) cfma_conj(s, A[r][j], A[r][k]);
      A[j][k] = s;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  return ok;
}

// Per site: A_+- = (4 + m0) 1_6 + (i c_sw / 2) sum_l s_l (x) E_l^+-,
// E_l^+- = +-F_{l t} - F_{jk}, (l, j, k) cyclic over (x, y, z).  This is the
// chiral-basis form of (4 + m0) + (i c_sw / 4) sum sigma_munu F_munu:
// sigma_{l t} = diag(s_l, -s_l) and sigma_{jk} = -diag(s_l, s_l).
//
// A workgroup is 64 sites of one parity x 6 wavefronts, one per plane; the six F meet in LDS,
// from which two wavefronts (one per block) form, and on odd sites invert, the 6x6 blocks.
// Bound by the latency of the links (one product at a time, three wavefronts a SIMD, 52 B of
// scratch): 16^3 x 32 225 us (one thread a site on canonical links, 464 B of scratch, and 2 x 17 us
// for the FP32 copy) -> 119.  With leaves of 10 products, four wavefronts with three planes each of
// both parities, twice the matrices in flight, read 506 MB past L2 against 165 and took 93 us
// against 96.
constexpr int CLOVER_PLANES = 6;
__global__ void __launch_bounds__(64 * CLOVER_PLANES) __attribute__((amdgpu_waves_per_eu(3)))
k_clover_build(Geo g, PackedLinks L, double c_sw, double m0, ClovOut out, int* notpd) {
  __shared__ double Fs[CLOVER_PLANES][9][64];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  int p, base, end;
  if (!gauge_group(g, (int)blockIdx.x, 2, p, base, end)) return;
  const int vh = g.Vh;
  const bool in = base + lane < end;
  const int i = in ? base + lane : end - 1;
  {
    int mu, nu;
    plane_dirs(w, mu, nu);
    const AH3 F = field_strength(L, g, decode(g, i, p), p, mu, nu);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      Fs[w][k][lane] = F.d[k];
      Fs[w][3 + 2 * k][lane] = F.u[k].r;
      Fs[w][4 + 2 * k][lane] = F.u[k].i;
    }
  }
  __syncthreads();
  if (w >= 2 || !in) return;
  const int blk = w;
  const double sg = blk == 0 ? 1.0 : -1.0, h = 0.5 * c_sw;
  // E_l = sg F_lt - F_jk: planes (x,t), (y,t), (z,t) against (y,z), (z,x) = -(x,z), (x,y)
  auto field = [&](int lt, int jk, double sjk) {
    AH3 E;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      E.d[k] = sg * Fs[lt][k][lane] - sjk * Fs[jk][k][lane];
      E.u[k] = {sg * Fs[lt][3 + 2 * k][lane] - sjk * Fs[jk][3 + 2 * k][lane],
                sg * Fs[lt][4 + 2 * k][lane] - sjk * Fs[jk][4 + 2 * k][lane]};
    }
    return E;
  };
  const AH3 E0 = field(2, 3, 1.0), E1 = field(4, 1, -1.0), E2 = field(5, 0, 1.0);
  // M = (i h) [s1 (x) E0 + s2 (x) E1 + s3 (x) E2] + (4 + m0), spin blocks of the bracket
  // [[e2, e0 - i e1], [e0 + i e1, -e2]]: upper triangle
  cpx<double> M[6][6], Y[6][6];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const cpx<double> e0 = ah_at(E0, a, b), e1 = ah_at(E1, a, b), e2 = ah_at(E2, a, b);
      if (a <= b) {
        Y[a][b] = times_i(e2);
        M[a][b] = h * Y[a][b];
        Y[3 + a][3 + b] = {-Y[a][b].r, -Y[a][b].i};
        M[3 + a][3 + b] = {-M[a][b].r, -M[a][b].i};
      }
      Y[a][3 + b] = times_i(e0 - times_i(e1));
      M[a][3 + b] = h * Y[a][3 + b];
    }
#pragma unroll
  for (int k = 0; k < 6; ++k) M[k][k].r += 4.0 + m0;
  if (p == 0) {
    store_packed<double>(out.e, blk, i, vh, M);
    if (out.e32) store_packed<float>(out.e32, blk, i, vh, M);  // uniform
  } else {
    store_packed<double>(out.o, blk, i, vh, M);  // A_oo itself, for the full operator
    if (!hpd_inverse6(M, Y, h)) {
      *notpd = 1;
#pragma unroll
      for (int j = 0; j < 6; ++j)
#pragma unroll
        for (int k = j; k < 6; ++k) M[j][k] = {0.0, 0.0};
    }
    store_packed<double>(out.o_inv, blk, i, vh, M);
    if (out.o_inv32) store_packed<float>(out.o_inv32, blk, i, vh, M);
  }
}

hipError_t launch_clover_build(const Geo& g, const d2_t* links_e, const d2_t* links_o, double c_sw, double m0,
                               const ClovOut& out, int* notpd, hipStream_t s) {
  const long long blocks = gauge_groups(g, 2);
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_clover_build, dim3((unsigned)blocks), dim3(64 * CLOVER_PLANES), 0, s, g,
                     PackedLinks{{links_e, links_o}}, c_sw, m0, out, notpd);
  return hipGetLastError();
}

// packed [2][18][vh] -> dense [vh][2][6][6]
__global__ void k_clover_export(Geo g, const d2_t* __restrict__ P, d2_t* __restrict__ D) {
  const int vh = g.Vh;
  long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= 2LL * vh) return;
  const int blk = (int)(tid / vh);
  const int i = (int)(tid % vh);
  d2_t* out = D + ((size_t)i * 2 + blk) * 36;
  for (int k = 0; k < 3; ++k) {
    d2_t d = P[fidx(18 * blk + k, i, 36, vh)];
    d2_t a, b;
    a.x = d.x; a.y = 0.0;
    b.x = d.y; b.y = 0.0;
    out[(2 * k) * 6 + 2 * k] = a;
    out[(2 * k + 1) * 6 + 2 * k + 1] = b;
    store_fence();
  }
  for (int j = 0; j < 6; ++j)
    for (int k = j + 1; k < 6; ++k) {
      d2_t v = P[fidx(18 * blk + tri_slot(j, k), i, 36, vh)];
      out[j * 6 + k] = v;
      store_fence();
      v.y = -v.y;
      out[k * 6 + j] = v;
      store_fence();
    }
}

hipError_t launch_clover_export(const Geo& g, const d2_t* packed, d2_t* dense, hipStream_t s) {
  long long n = 2LL * g.Vh;
  hipLaunchKernelGGL(k_clover_export, dim3((int)((n + 255) / 256)), dim3(256), 0, s, g, packed, dense);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// parity packing of vectors: full [n][12] <-> parity layout (FP64: [12][vh]
// complex128; FP32: [6][vh] elements of two complex64, rows 2k and 2k+1)
// ---------------------------------------------------------------------------
// A wavefront moves 64 consecutive sites of one parity through LDS (full_rows.h), so that both
// sides are read and written in runs: 24^3 x 48 FP64
// pack 36 -> 27 us, unpack 73 -> 28 (4.6 TB/s) against lanes that walk a site each.
template <typename R, bool UNPACK>
__global__ void __launch_bounds__(256) k_parity_full(Geo g, int parity, const u4a8_t* __restrict__ src,
                                                     u4a8_t* __restrict__ dst) {
  constexpr int NE = SPINOR_ROWS / CPE<R>;
  __shared__ u4_t lds[4][NE][FULL_ROW];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  const int base = ((int)blockIdx.x * 4 + w) * 64, vh = g.Vh;
  if (base >= vh) return;  // uniform over a wavefront
  const FullRows<NE> f(g, base, min(base + 64, vh), parity, lane);
  const size_t r = (size_t)blockIdx.y * NE * (size_t)vh;
  const int i = min(base + lane, vh - 1);
  if constexpr (UNPACK) {
#pragma unroll
    for (int e = 0; e < NE; ++e) lds[w][e][lane] = src[r + (size_t)e * vh + i];
    wave_lds_order();
    f.template store<64>(dst + 2 * r, lds[w], lane);
  } else {
    f.template load<64>(src + 2 * r, lds[w], lane);
    wave_lds_order();
    if (base + lane < vh)
#pragma unroll
      for (int e = 0; e < NE; ++e) dst[r + (size_t)e * vh + i] = lds[w][e][lane];
  }
}

template <typename R>
hipError_t launch_pack_parity(const Geo& g, int parity, int nrhs, const pair<R>* full, pair<R>* v,
                              hipStream_t s) {
  hipLaunchKernelGGL((k_parity_full<R, false>), dim3((g.Vh + 255) / 256, nrhs), dim3(256), 0, s, g, parity, (const u4a8_t*)full,
                     (u4a8_t*)v);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_unpack_parity(const Geo& g, int parity, int nrhs, const pair<R>* v, pair<R>* full,
                                hipStream_t s) {
  hipLaunchKernelGGL((k_parity_full<R, true>), dim3((g.Vh + 255) / 256, nrhs), dim3(256), 0, s, g, parity, (const u4a8_t*)v,
                     (u4a8_t*)full);
  return hipGetLastError();
}

// FP32 parity vectors into FP64 ones and into the sites of `parity` of full FP64 vectors
__global__ void __launch_bounds__(256) k_f32_to_parity_and_full(Geo g, int parity, const f4_t* __restrict__ src,
                                                                d2_t* __restrict__ v, u4a8_t* __restrict__ full) {
  __shared__ u4_t lds[4][SPINOR_ROWS][FULL_ROW];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  const int base = ((int)blockIdx.x * 4 + w) * 64, vh = g.Vh;
  if (base >= vh) return;  // uniform over a wavefront
  const FullRows<SPINOR_ROWS> f(g, base, min(base + 64, vh), parity, lane);
  const size_t r = (size_t)blockIdx.y * SPINOR_ROWS * (size_t)vh;
  const bool in = base + lane < vh;
  const int i = in ? base + lane : vh - 1;
#pragma unroll
  for (int e = 0; e < SPINOR_ROWS / 2; ++e) {
    const f4_t q = src[r / 2 + (size_t)e * vh + i];
    const d2_t a = {q.x, q.y}, b = {q.z, q.w};
    lds[w][2 * e][lane] = __builtin_bit_cast(u4_t, a);
    lds[w][2 * e + 1][lane] = __builtin_bit_cast(u4_t, b);
    if (in) {
      v[r + (size_t)(2 * e) * vh + i] = a;
      v[r + (size_t)(2 * e + 1) * vh + i] = b;
      store_fence();
    }
  }
  wave_lds_order();
  f.store<64>(full + 2 * r, lds[w], lane);
}

hipError_t launch_f32_to_parity_and_full(const Geo& g, int parity, int nrhs, const void* src, d2_t* v, d2_t* full, hipStream_t s) {
  hipLaunchKernelGGL(k_f32_to_parity_and_full, dim3((g.Vh + 255) / 256, nrhs), dim3(256), 0, s, g, parity, (const f4_t*)src, v,
                     (u4a8_t*)full);
  return hipGetLastError();
}

template hipError_t launch_pack_parity<double>(const Geo&, int, int, const d2_t*, d2_t*, hipStream_t);
template hipError_t launch_pack_parity<float>(const Geo&, int, int, const f2_t*, f2_t*, hipStream_t);
template hipError_t launch_unpack_parity<double>(const Geo&, int, int, const d2_t*, d2_t*, hipStream_t);
template hipError_t launch_unpack_parity<float>(const Geo&, int, int, const f2_t*, f2_t*, hipStream_t);

// FP64 parity vectors [nrhs][12][vh] <-> FP32 parity vectors [nrhs][6][vh][2]
__global__ void k_parity_to_f32(f4_t* __restrict__ y, const d2_t* __restrict__ x, long long n6, int vh) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;  // (rhs, k, i)
  if (t >= n6) return;
  const int i = (int)(t % vh);
  const long long rk = t / vh;  // rhs * 6 + k
  const long long rhs = rk / 6;
  const int k = (int)(rk % 6);
  const d2_t* xr = x + rhs * 12LL * vh;
  d2_t a = xr[(size_t)(2 * k) * vh + i], b = xr[(size_t)(2 * k + 1) * vh + i];
  f4_t o;
  o.x = (float)a.x;
  o.y = (float)a.y;
  o.z = (float)b.x;
  o.w = (float)b.y;
  y[t] = o;
}

__global__ void k_parity_to_f64(d2_t* __restrict__ y, const f4_t* __restrict__ x, long long n6, int vh) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n6) return;
  const int i = (int)(t % vh);
  const long long rk = t / vh;
  const long long rhs = rk / 6;
  const int k = (int)(rk % 6);
  d2_t* yr = y + rhs * 12LL * vh;
  f4_t q = x[t];
  d2_t a, b;
  a.x = q.x;
  a.y = q.y;
  b.x = q.z;
  b.y = q.w;
  yr[(size_t)(2 * k) * vh + i] = a;
  store_fence();
  yr[(size_t)(2 * k + 1) * vh + i] = b;
}

hipError_t launch_parity_to_f32(void* y, const d2_t* x, int nrhs, int vh, hipStream_t s) {
  const long long n6 = 6LL * vh * nrhs;
  hipLaunchKernelGGL(k_parity_to_f32, dim3((unsigned)((n6 + 255) / 256)), dim3(256), 0, s, (f4_t*)y, x, n6, vh);
  return hipGetLastError();
}

hipError_t launch_parity_to_f64(d2_t* y, const void* x, int nrhs, int vh, hipStream_t s) {
  const long long n6 = 6LL * vh * nrhs;
  hipLaunchKernelGGL(k_parity_to_f64, dim3((unsigned)((n6 + 255) / 256)), dim3(256), 0, s, y, (const f4_t*)x, n6, vh);
  return hipGetLastError();
}

}  // namespace ddq
