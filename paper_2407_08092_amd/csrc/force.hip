// force.hip -- derivative of Re(chi^H D_S(U) phi) with respect to the gauge links.
//
// With D_S = A_ee - H_eo A_oo^-1 H_oe and psi_o = A_oo^-1 H_oe phi_e,
// lambda_o = A_oo^-1 (H^H)_oe chi_e (kernel A, plain and dagger), the variation is
//   dL = Re[ chi^H dA_ee phi + lambda^H dA_oo psi - chi^H dH_eo psi - lambda^H dH_oe phi ].
// Every term is Re tr(dU M) for a 3x3 matrix M per link; the gradient in torch's
// convention (dL = Re tr(G^H dU)) is G = M^H, and the su(3) force under
// U -> exp(i e T_a) U is F_a = -Im tr(T_a U M).
//
// Hopping part, link U_mu(y): it enters H once as a forward hop out of y and once
// as a backward hop out of y + mu; for a pair (a on rows, b on columns)
//   a^H (1 - g_mu) dU b(y+mu) = tr(dU sum_s [(1 - g_mu) b(y+mu)]_s a(y)_s^H),
//   a^H (1 + g_mu) dU^H b(y)  = conj-transposed of the same with (1 + g_mu).
// Clover part: per site x and plane (p < q) the insertion
//   W~_pq(x) = (W - W^H) / 8,  W = (i c_sw / 2) sum_s (sigma_pq b)_s a_s^H,
// with (a, b) = (chi, phi) on even and (lambda, psi) on odd sites, gives
//   dL = sum_x sum_pq Re tr(dQ_pq(x) W~_pq(x)),
// and each link sits in 2 plaquettes per plane x 3 planes x 4 corners = 24 leaves.
//
// W~ is anti-Hermitian: nine real numbers, stored per parity and plane as INS_E element rows of
// 64-site blocks like the packed links, which the link kernel reads in place of the canonical
// ones, so that every load of a wavefront is a run of 16-byte elements.
#include "full_rows.h"
#include "gauge_common.h"

namespace ddq {

constexpr int INS_E = 5;       // element rows of an insertion: (d0, d1), (d2, -), u01, u02, u12
constexpr int PLANES = 6;

long long force_insertion_elements(const Geo& g) { return 2LL * PLANES * INS_E * field_vh(g.Vh); }

__device__ __forceinline__ int plane_of(int p, int q) { return p == 0 ? q - 1 : p == 1 ? q + 1 : 5; }  // p < q

// insertions of plane `plane` on the sites of parity q
__device__ __forceinline__ Field ins_field(const d2_t* W, const Geo& g, int q, int plane) {
  return bfield(W + (size_t)(q * PLANES + plane) * INS_E * field_vh(g.Vh), INS_E, g.Vh);
}
__device__ __forceinline__ AH3 load_ins(const Field& f, int i) {
  const uint32_t off = boff(i, INS_E);
  d2_t e[INS_E];
#pragma unroll
  for (int k = 0; k < INS_E; ++k) e[k] = __builtin_bit_cast(d2_t, ld16(f, k, off));
  return {{e[0].x, e[0].y, e[1].x}, {{e[2].x, e[2].y}, {e[3].x, e[3].y}, {e[4].x, e[4].y}}};
}

// one parity vector per parity (chi_e, lambda_o) or (phi_e, psi_o)
struct ParityPair {
  const d2_t* p[2];
};
__device__ __forceinline__ Spinor<double> spinor_at(const ParityPair& v, const Geo& g, int q, int i) {
  return load_spinor<double>(vfield(v.p[q], SPINOR_ROWS, g.Vh), voff(i));
}

// Insertions of the six planes at one site, a thread each.  On each chirality the four outer
// products b_s a_t^H of its two spins give K_l = sum_st (s_l)_st b_t a_s^H for the three Pauli
// matrices; with the upper (u) and lower (l) blocks' K
//   sigma_{l t} = diag(s_l, -s_l):  K = u_l - l_l;   sigma_{jk} = -eps_jkl diag(s_l, s_l):  K = -+(u_l + l_l).
// A pass over memory: 384 B of spinors read and 480 B written a site; 16^3 x 32 50 us -> 17.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_force_insertions(Geo g, ParityPair av, ParityPair bv, double c_sw,
                                                          d2_t* __restrict__ W) {
  const int p = (int)blockIdx.y;
  const int i = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (i >= g.Vh) return;
  const Spinor<double> a = spinor_at(av, g, p, i), b = spinor_at(bv, g, p, i);
  const double h = 0.0625 * c_sw;  // W~ = (W - W^H) / 8 with W = (i c_sw / 2) K
  // entry (r, c) of K_l on block blk
  auto entry = [&](int l, int blk, int r, int c) {
    const cpx<double> *a0 = a.c[2 * blk], *a1 = a.c[2 * blk + 1], *b0 = b.c[2 * blk], *b1 = b.c[2 * blk + 1];
    if (l == 0) return cmul_conj(a0[c], b1[r]) + cmul_conj(a1[c], b0[r]);           // b_1 a_0^H + b_0 a_1^H
    if (l == 1) return times_i(cmul_conj(a1[c], b0[r]) - cmul_conj(a0[c], b1[r]));  // i (b_0 a_1^H - b_1 a_0^H)
    return cmul_conj(a0[c], b0[r]) - cmul_conj(a1[c], b1[r]);                       // b_0 a_0^H - b_1 a_1^H
  };
  const uint32_t off = boff(i, INS_E);
  auto put = [&](const Field& f, int row, d2_t v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, v), f.rsrc, (int)off, (int)(row * f.row_bytes), 0);
    store_fence();
  };
  // anti-Hermitian part W~_ij = (i h) (K_ij + conj K_ji) of the planes (l, t) and (j, k)
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const Field lt = ins_field(W, g, p, l == 0 ? 2 : l == 1 ? 4 : 5), jk = ins_field(W, g, p, l == 0 ? 3 : l == 1 ? 1 : 0);
    const double sjk = l == 1 ? h : -h;  // sigma_xz = -sigma_zx
    double dt[3], dk[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const double u = entry(l, 0, r, r).r, v = entry(l, 1, r, r).r;
      dt[r] = 2.0 * h * (u - v);
      dk[r] = 2.0 * sjk * (u + v);
    }
    put(lt, 0, d2_t{dt[0], dt[1]});
    put(lt, 1, d2_t{dt[2], 0.0});
    put(jk, 0, d2_t{dk[0], dk[1]});
    put(jk, 1, d2_t{dk[2], 0.0});
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = r + 1; c < 3; ++c) {
        const cpx<double> u = entry(l, 0, r, c) + conj(entry(l, 0, c, r)), v = entry(l, 1, r, c) + conj(entry(l, 1, c, r));
        const cpx<double> m = times_i(u - v), q = times_i(u + v);
        put(lt, 1 + r + c, d2_t{h * m.r, h * m.i});
        put(jk, 1 + r + c, d2_t{sjk * q.r, sjk * q.i});
      }
  }
}

// P = U2 U3^H and R = (U2 W) U3^H, a row of U2 at a time
__device__ __forceinline__ void two_products(const C3& U2, const C3& U3, const AH3& W, C3& P, C3& R) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    cpx<double> t[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      t[j] = {0.0, 0.0};
#pragma unroll
      for (int k = 0; k < 3; ++k) cfma(t[j], U2.a[i][k], ah_at(W, k, j));
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      P.a[i][j] = {0.0, 0.0};
      R.a[i][j] = {0.0, 0.0};
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        cfma_conj(P.a[i][j], U3.a[j][k], U2.a[i][k]);
        cfma_conj(R.a[i][j], U3.a[j][k], t[k]);
      }
    }
  }
}

// Lower plaquette of link U_mu(y) in plane (mu, nu), y -> y+mu -> y+mu-nu -> y-nu -> y:
// U2 = U_nu(y+mu-nu)^H, U3 = U_mu(y-nu)^H, U4 = U_nu(y-nu), S = U2 U3 U4 and
// T = (U2 W(y+mu-nu) U3 + U2 U3 W(y-nu)) U4.
__device__ __forceinline__ void lower_plaquette(const PackedLinks& L, const Field& Wp, const Field& Wo, const Geo& g,
                                                const Site& y, int p, const Site& fm, int mu, int nu, C3& S, C3& T) {
  const int o = 1 - p, bn = site_shift(g, y, nu, -1).i, c2 = site_shift(g, fm, nu, -1).i;
  const C3 U4 = packed_link(L, g, o, nu, bn);
  two_products(c3_dag(packed_link(L, g, p, nu, c2)), packed_link(L, g, o, mu, bn), load_ins(Wp, c2), S, T);
  c3_fence(S);
  c3_fence(T);
  ah_right(T, S, load_ins(Wo, bn));
  c3_rmul<false>(S, U4);
  c3_rmul<false>(T, U4);
}

// The clover part of M of link U_mu(y) from plane (mu, nu): each plaquette (U the link, U2 U3 U4
// the rest of the loop, W0 at y, W1 at y+mu, W2, W3) gives
//   S W0 + W1 S + T,  S = U2 U3 U4,  T = (U2 W2 U3 + U2 U3 W3) U4,
// upper minus lower, so the products with W0 and W1 are formed once, on the difference of the S:
// 14 products a plane against 18 plaquette by plaquette.  Wp, Wo: the plane's insertions on y's
// parity and on the other.
__device__ __forceinline__ C3 link_terms(const PackedLinks& L, const Field& Wp, const Field& Wo, const Geo& g, const Site& y,
                                         const Site& fm, int p, int mu, int nu) {
  const int o = 1 - p, fn = site_shift(g, y, nu, 1).i;
  C3 S, T, P, R;
  lower_plaquette(L, Wp, Wo, g, y, p, fm, mu, nu, S, T);
  two_products(packed_link(L, g, o, nu, fm.i), packed_link(L, g, o, mu, fn), load_ins(Wp, site_shift(g, fm, nu, 1).i),
               P, R);
  c3_fence(P);
  c3_fence(R);
  ah_right(R, P, load_ins(Wo, fn));
  const C3 U4 = packed_link(L, g, p, nu, y.i);
  c3_rmul<true>(P, U4);
  c3_rmul<true>(R, U4);
  const C3 D = c3_sub(P, S);
  C3 M = c3_sub(R, T);
  ah_right(M, D, load_ins(Wp, y.i));
  ah_left(M, load_ins(Wo, fm.i), D);
  return M;
}

// K += sum over the two projected spins of h_s (ha_s)^H
__device__ __forceinline__ void add_outer(C3& K, const Half<double>& h, const Half<double>& ha) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) cfma_conj(K.a[i][j], ha.c[s][j], h.c[s][i]);
}
// -1/2 s (M_f + M_b^H) of direction MU: with the projectors P = 1 -+ g, P b a^H summed over spins is
// the product of the two projected half spinors
template <int MU>
__device__ __forceinline__ C3 hop_terms(const ParityPair& av, const ParityPair& bv, const Geo& g, const Site& y, int p,
                                        double f) {
  const int j = site_shift(g, y, MU, 1).i, o = 1 - p;
  C3 Mf = c3_zero(), Mb = c3_zero();
  add_outer(Mf, project<MU, double>(spinor_at(bv, g, o, j), -1.0), project<MU, double>(spinor_at(av, g, p, y.i), -1.0));
  c3_fence(Mf);
  add_outer(Mb, project<MU, double>(spinor_at(bv, g, p, y.i), 1.0), project<MU, double>(spinor_at(av, g, o, j), 1.0));
  C3 M;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) M.a[r][c] = f * (Mf.a[r][c] + conj(Mb.a[c][r]));
  return M;
}

// M of the links of 64 sites of one parity, then G = M^H (torch convention) and/or the su(3)
// projection F_a = -Im tr(T_a U M).  Wavefront mu takes direction mu: the hopping term, then the
// three planes of the direction one after the other, summed in the wavefront's own part of LDS,
// from which the links leave in canonical order (144 contiguous bytes a link).
// Bound by the FP64 units (14 3x3 products a plane: about 80 us of issue at 16^3 x 32) and by L2
// misses, which follow the number of sites in flight: 16^3 x 32 361 us (canonical links, one
// thread a link) -> 164 to 171 (234 registers, two wavefronts a SIMD, 718 MB past L2).  Measured
// beside it: links through both packed copies 186 us (1.09 GB); one plaquette at a time in 164
// registers, three wavefronts a SIMD 196 (1.26 GB); twelve wavefronts a group of 64 sites, one
// plane each 189 (555 MB, but 15 % more instructions and a barrier); both links of a plane in one
// wavefront 267 (spills).
constexpr int FORCE_ROW = 65;  // elements between the rows of a wavefront's LDS: 64 sites, one of padding
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_force_links(Geo g, PackedLinks L, const d2_t* __restrict__ W, ParityPair av, ParityPair bv, d2_t* __restrict__ G,
              double* __restrict__ F, int accum) {
  __shared__ d2_t lds[4][9][FORCE_ROW];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  int p, base, end;
  if (!gauge_group(g, (int)blockIdx.x, 2, p, base, end)) return;
  const int i = min(base + lane, end - 1);
  const Site y = decode(g, i, p), fm = site_shift(g, y, w, 1);
  d2_t (*Ms)[FORCE_ROW] = lds[w];
  auto add = [&](const C3& M, double s) {
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      d2_t q = Ms[e][lane];
      q.x = fma(s, M.a[e / 3][e % 3].r, q.x);
      q.y = fma(s, M.a[e / 3][e % 3].i, q.y);
      Ms[e][lane] = q;
    }
  };
  {
    const double f = (g.antiperiodic && w == 3 && y.t == g.L[3] - 1) ? 0.5 : -0.5;
    C3 M;
    switch (w) {
      case 0: M = hop_terms<0>(av, bv, g, y, p, f); break;
      case 1: M = hop_terms<1>(av, bv, g, y, p, f); break;
      case 2: M = hop_terms<2>(av, bv, g, y, p, f); break;
      default: M = hop_terms<3>(av, bv, g, y, p, f); break;
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) Ms[e][lane] = d2_t{M.a[e / 3][e % 3].r, M.a[e / 3][e % 3].i};
  }
#pragma unroll 1
  for (int k = 1; k < 4; ++k) {
    const int nu = (w + k) & 3;
    const int plane = plane_of(min(w, nu), max(w, nu));
    add(link_terms(L, ins_field(W, g, p, plane), ins_field(W, g, 1 - p, plane), g, y, fm, p, w, nu), w < nu ? 1.0 : -1.0);
  }
  {
    C3 M;
#pragma unroll
    for (int e = 0; e < 9; ++e) M.a[e / 3][e % 3] = {Ms[e][lane].x, Ms[e][lane].y};
    if (F && base + lane < end) {
      // UM = U M;  F_a = -Im tr(T_a UM), T_a = lambda_a / 2
      const C3 UM = c3_mul(packed_link(L, g, p, w, i), M);
      const double r3 = 0.57735026918962576451;  // 1 / sqrt(3)
      double f8[8];
      // -Im tr(T_a X), T_a = lambda_a / 2, X = U M, written out per Gell-Mann matrix;
      // for the antisymmetric ones (a = 2, 5, 7) Im(-i X_ji + i X_ij) = Re X_ij - Re X_ji
      f8[0] = -0.5 * (UM.a[1][0].i + UM.a[0][1].i);
      f8[1] = 0.5 * (UM.a[1][0].r - UM.a[0][1].r);
      f8[2] = -0.5 * (UM.a[0][0].i - UM.a[1][1].i);
      f8[3] = -0.5 * (UM.a[2][0].i + UM.a[0][2].i);
      f8[4] = 0.5 * (UM.a[2][0].r - UM.a[0][2].r);
      f8[5] = -0.5 * (UM.a[2][1].i + UM.a[1][2].i);
      f8[6] = 0.5 * (UM.a[2][1].r - UM.a[1][2].r);
      f8[7] = -0.5 * r3 * (UM.a[0][0].i + UM.a[1][1].i - 2.0 * UM.a[2][2].i);
      double* outf = F + ((2LL * i + (y.x & 1)) * 4 + w) * 8;
      for (int k = 0; k < 8; ++k) {
        outf[k] = accum ? outf[k] + f8[k] : f8[k];
        store_fence();
      }
    }
  }
  if (!G) return;  // uniform
  wave_lds_order();
  // M^H of the wavefront's links, nine lanes a link
  for (int q = lane; q < (end - base) * 9; q += 64) {
    const int sl = q / 9, e = q - 9 * sl;
    const Site s = decode(g, base + sl, p);
    d2_t* out = G + ((2LL * (base + sl) + (s.x & 1)) * 4 + w) * 9 + e;
    d2_t v = Ms[3 * (e % 3) + e / 3][sl];
    v.y = -v.y;
    if (accum) {
      const d2_t old = *out;
      v.x += old.x;
      v.y += old.y;
    }
    *out = v;
    store_fence();
  }
}

hipError_t launch_force(const Geo& g, const d2_t* links_e, const d2_t* links_o, const d2_t* chi_e, const d2_t* lam_o,
                        const d2_t* phi_e, const d2_t* psi_o, double c_sw, d2_t* W, d2_t* G, double* F, int accumulate,
                        hipStream_t s) {
  const ParityPair a{{chi_e, lam_o}}, b{{phi_e, psi_o}};
  hipLaunchKernelGGL(k_force_insertions, dim3((unsigned)((g.Vh + 255) / 256), 2), dim3(256), 0, s, g, a, b, c_sw, W);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const long long blocks = gauge_groups(g, 2);
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_force_links, dim3((unsigned)blocks), dim3(256), 0, s, g, PackedLinks{{links_e, links_o}}, W,
                     a, b, G, F, accumulate);
  return hipGetLastError();
}

}  // namespace ddq
