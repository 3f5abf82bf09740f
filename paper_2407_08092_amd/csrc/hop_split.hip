// hop_split.hip -- the stencil of hop.hip / hop_h16.hip for launches of few sites or of several
// right-hand sides: four threads per output site, one per direction.
//
// The one-thread-per-site kernels walk a site's eight hops one after the other with one
// hop's loads in flight, about eight memory latencies per wavefront.  A large lattice hides
// them behind its other wavefronts; a small one has none (16^3 x 32: one wavefront per
// SIMD; 4^4: four on the whole chip) and the chain is its time.  Here a workgroup is 64
// sites x 4 wavefronts: wavefront w sums up both hops of direction w, so all of a site's
// neighbour and link loads are in flight at once, and there are four times the wavefronts.
// The projected and multiplied half spinors of the eight hops meet in LDS; after the barrier
// wavefront w forms spin w of the hopping term, adding the hops in the order of hop.hip, and
// the three rows of the clover block that spin w belongs to.  Every number is formed by the
// same operations in the same order as in the one-thread kernels, so the results are theirs
// bit for bit and a launch may take either.
// What bounds it: the launch itself (about 4 us from one launch to the next) up to 10^4 sites,
// then the caches' bandwidth; 4^4 FP64 8.4 -> 5.3 us a launch, 16^4 FP32 12.6 -> 8.3, 24^3 x 48
// FP32 71 -> 62 (6.2 TB/s of its algorithmic bytes).
#include "full_rows.h"
#include "hop_common.h"
#include "hop_h16.h"

namespace ddq {

// The third row of a 12-real link with the multiply-adds of the one-thread FP32 kernels written
// out: there a product's imaginary part starts from a.r b.i, and from a.i b.r in the forward
// link's products with entry 0.
template <bool FWD, typename R>
__device__ __forceinline__ void third_row_as_hop(Link<R>& l) {
  auto re = [](cpx<R> a, cpx<R> b) -> R { return fma(a.r, b.r, -(a.i * b.i)); };
  auto im = [](cpx<R> a, cpx<R> b) -> R { return fma(a.i, b.r, a.r * b.i); };
  auto im0 = [&](cpx<R> b) -> R { return FWD ? fma(l.u[0].r, b.i, l.u[0].i * b.r) : im(l.u[0], b); };
  const cpx<R>* u = l.u;
  l.u[6] = {re(u[1], u[5]) - re(u[2], u[4]), -(im(u[1], u[5]) - im(u[2], u[4]))};
  l.u[7] = {re(u[2], u[3]) - re(u[0], u[5]), -(im(u[2], u[3]) - im0(u[5]))};
  l.u[8] = {re(u[0], u[4]) - re(u[1], u[3]), -(im0(u[4]) - im(u[1], u[3]))};
}

// What a launch streams past the Infinity Cache (split_policy); everything else may stay there.
enum SplitStream { ST_NONE = 0, ST_LINKS = 1, ST_LINKS_RESULT = 2 };

// Storage policies: how a precision's fields are read and written.  NT: a SplitStream
template <typename RR, bool L12, int NT>
struct SplitR {
  using R = RR;
  static constexpr int STREAM = NT;
  static constexpr int LINK_AUX = NT >= ST_LINKS ? DDQ_STREAM_AUX : 0, ST_AUX = NT == ST_LINKS_RESULT ? DDQ_STORE_AUX : 0;
  static constexpr int SP_E = SPINOR_ROWS / CPE<R>, CL_E = CLOVER_ROWS / CPE<R>;
  static constexpr int LK_E = (L12 ? LINK12_ROWS : LINK_ROWS) / CPE<R>;
  static __device__ __forceinline__ Spinor<R> spinor(const Field& v, uint32_t off) { return load_spinor<R>(v, off); }
  static __device__ __forceinline__ void links(const Field& U, uint32_t off, Link<R>& f, Link<R>& b) {
    if constexpr (L12) {
      load_link_pair12<R, LINK_AUX>(U, off, f, b);
      third_row_as_hop<true>(f);
      third_row_as_hop<false>(b);
    } else if constexpr (CPE<R> == 1) {
      f = load_link_half<R, LINK_AUX>(U, 0, off);
      b = load_link_half<R, LINK_AUX>(U, 1, off);
    } else {
      load_link_pair<R, LINK_AUX>(U, off, f, b);
    }
  }
  static __device__ __forceinline__ void slots(const Field& C, uint32_t off, int b, cpx<R>* sl) {
    load_rows<R>(C, 18 * b, 18, off, sl);
  }
  // complex row r (uniform) of a parity vector
  static __device__ __forceinline__ cpx<R> row(const Field& v, int r, uint32_t off) {
    if constexpr (CPE<R> == 1) {
      cpx<R> c;
      unpack<R>(ld16(v, r, off), &c);
      return c;
    } else {
      const f2_t q = __builtin_bit_cast(
          f2_t, __builtin_amdgcn_raw_buffer_load_b64(v.rsrc, (int)(off + 8u * (r & 1)), (int)((r >> 1) * v.row_bytes), 0));
      return {q.x, q.y};
    }
  }
  static __device__ __forceinline__ cpx<R> stored(cpx<R> c) { return c; }
  static __device__ __forceinline__ cpx<R> formed_here(cpx<R> c) { return c; }
  static __device__ __forceinline__ void put(const Field& v, int r, uint32_t off, cpx<R> c) {
    if constexpr (CPE<R> == 1) {
      __builtin_amdgcn_raw_buffer_store_b128(pack<R>(&c), v.rsrc, (int)off, (int)(r * v.row_bytes), ST_AUX);
    } else {
      f2_t q;
      q.x = c.r;
      q.y = c.i;
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2_t, q), v.rsrc, (int)(off + 8u * (r & 1)),
                                            (int)((r >> 1) * v.row_bytes), ST_AUX);
    }
  }
};

template <typename S, bool C32, int NT>
struct Split16 {
  using R = float;
  static constexpr int STREAM = NT;
  static constexpr int LINK_AUX = NT >= ST_LINKS ? DDQ_STREAM_AUX : 0;
  static constexpr int SP_E = SP16_E, LK_E = LK16_E, CL_E = C32 ? CLOVER_ROWS / CPE<float> : CL16_E;
  static __device__ __forceinline__ Spinor<R> spinor(const Field& v, uint32_t off) { return load_spinor16<S>(v, off); }
  static __device__ __forceinline__ void links(const Field& U, uint32_t off, Link<R>& f, Link<R>& b) {
    cpx<R> l[12];
#pragma unroll
    for (int e = 0; e < LK16_E; ++e) unpack4<S>(ld16<LINK_AUX>(U, e, off), l + 4 * e);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      f.u[k] = l[k];
      b.u[k] = l[6 + k];
    }
    su3_third_row(f);
    su3_third_row(b);
  }
  static __device__ __forceinline__ void slots(const Field& C, uint32_t off, int b, cpx<R>* sl) {
    if constexpr (C32) {
      load_rows<R>(C, 18 * b, 18, off, sl);
    } else {
      cpx<R> q[20];
#pragma unroll
      for (int e = 0; e < 5; ++e) unpack4<S>(ld16(C, 5 * b + e, off), q + 4 * e);
#pragma unroll
      for (int k = 0; k < 18; ++k) sl[k] = q[k];
    }
  }
  static __device__ __forceinline__ cpx<R> row(const Field& v, int r, uint32_t off) {
    const unsigned q =
        __builtin_amdgcn_raw_buffer_load_b32(v.rsrc, (int)(off + 4u * (r & 3)), (int)((r >> 2) * v.row_bytes), 0);
    return {h2f<S>((u16_t)(q & 0xffffu)), h2f<S>((u16_t)(q >> 16))};
  }
  static __device__ __forceinline__ unsigned stored(cpx<R> c) { return (unsigned)f2h<S>(c.r) | ((unsigned)f2h<S>(c.i) << 16); }
  static __device__ __forceinline__ unsigned formed_here(unsigned q) {
    asm("" : "+v"(q));
    return q;
  }
  static __device__ __forceinline__ void put(const Field& v, int r, uint32_t off, unsigned q) {
    __builtin_amdgcn_raw_buffer_store_b32(q, v.rsrc, (int)(off + 4u * (r & 3)), (int)((r >> 2) * v.row_bytes), 0);
  }
};

template <int MU, typename R>
__device__ __forceinline__ void split_hops(const Spinor<R>& pf, const Spinor<R>& pb, const Link<R>& uf,
                                           const Link<R>& ub, R sf, R sb, const Nbr& nb, Half<R>& hf, Half<R>& hb) {
  hf = link_mul<R>(uf, project<MU, R>(pf, sf));
  hb = link_mul<R>(ub, project<MU, R>(pb, sb));
  if (MU == 3) {
    scale_half(hf, (R)nb.sgn_tf);
    scale_half(hb, (R)nb.sgn_tb);
  }
}

// o += spin SP of the spinor that `accumulate` rebuilds from hop (MU, sg)'s half spinor h
template <int MU, int SP, typename R>
__device__ __forceinline__ void split_add(cpx<R> (&o)[3], const cpx<R> (*h)[64], int lane, R sg) {
  // the half spinor's spin that this spin is made of
  constexpr int S = SP < 2 ? SP : (MU < 2 ? 3 - SP : SP - 2);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const cpx<R> v = h[3 * S + c][lane];
    if constexpr (SP < 2) {
      o[c] = o[c] + v;
    } else {
      cpx<R> d;
      if (MU == 0) d = times_i(v);
      else if (MU == 1) d = SP == 2 ? v : cpx<R>{-v.r, -v.i};
      else if (MU == 2) d = SP == 2 ? times_i(v) : times_minus_i(v);
      else d = v;
      o[c] = o[c] + sg * d;
    }
  }
}
template <int SP, typename R>
__device__ __forceinline__ void split_sum(cpx<R> (&o)[3], const cpx<R> (*h)[6][64], int lane, R sf, R sb) {
  split_add<0, SP, R>(o, h[0], lane, sf);
  split_add<0, SP, R>(o, h[1], lane, sb);
  split_add<1, SP, R>(o, h[2], lane, sf);
  split_add<1, SP, R>(o, h[3], lane, sb);
  split_add<2, SP, R>(o, h[4], lane, sf);
  split_add<2, SP, R>(o, h[5], lane, sb);
  split_add<3, SP, R>(o, h[6], lane, sf);
  split_add<3, SP, R>(o, h[7], lane, sb);
}

// rows 3 HF .. 3 HF + 2 of clover_block_apply, each summed in its order
template <int HF, typename R>
__device__ __forceinline__ void clover_rows(const cpx<R>* sl, const cpx<R> in[6], cpx<R> out[3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int r = 3 * HF + c;
    const R d = (r & 1) ? sl[r >> 1].i : sl[r >> 1].r;
    out[c] = d * in[r];
#pragma unroll
    for (int j = 0; j < r; ++j) cfma_conj(out[c], sl[tri_slot(j, r)], in[j]);
#pragma unroll
    for (int k = r + 1; k < 6; ++k) cfma(out[c], sl[tri_slot(r, k)], in[k]);
  }
}

struct SplitArgs {
  Geo g;
  int p_out;
  const void *in, *links, *clov, *x, *b;
  void* out;
  double omega;
  int nrhs;
  int dagger;
  int reuse;        // FieldReuse
  int slab;         // slab order; else the groups of 64 sites in a row
  int t_lo, t_cnt;  // output sites of slices [t_lo, t_lo + t_cnt)
  // M_PREP, M_RECON: b is a full FP64 vector
  void* full;       // M_RECON: the full vector whose sites of parity p_out are written (and, unless null, out)
  void *out32, *scaled32;  // M_PREP: unless null, the result in FP32 and scale times that, in place of out
  float scale;
};

template <class P, int MODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(typename P::R) == 8 ? 1 : 3)))
hop_split_kernel(SplitArgs a) {
  using R = typename P::R;
  __shared__ cpx<R> hs[8][6][64];
  __shared__ cpx<R> ex[MODE == M_PREP ? 1 : 12][64];  // what the clover block acts on: the hopping term, or x
  constexpr bool FULL = MODE == M_RECON || MODE == M_PREP;
  __shared__ u4_t rows[FULL ? SPINOR_ROWS : 1][FULL_ROW];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  int base, end, rhs;
  if (a.slab) {  // uniform
    const int local = (int)blockIdx.x >> 3, xcd = (int)blockIdx.x & 7;
    rhs = local % a.nrhs;
    const int q = local / a.nrhs, ng = (a.g.sT + 63) >> 6;
    const int n = (((xcd + 1) * ng) >> 3) - ((xcd * ng) >> 3);
    if (q >= a.t_cnt * n || !slab_group(a.g, xcd, a.t_lo * n + q, base, end)) return;
  } else {
    rhs = (int)blockIdx.x % a.nrhs;
    base = a.t_lo * a.g.sT + ((int)blockIdx.x / a.nrhs) * 64;
    end = min(base + 64, (a.t_lo + a.t_cnt) * a.g.sT);
  }
  const int vh = a.g.Vh;
  const bool ok = base + lane < end;
  const int i = ok ? base + lane : end - 1;  // lanes past the end repeat the last site and store nothing
  const size_t rb = (size_t)rhs * P::SP_E * (size_t)vh * 16;
  auto vec = [&](const void* p) { return vfield((const char*)p + rb, P::SP_E, vh); };
  const Nbr nb = neighbours(a.g, decode(a.g, i, a.p_out));
  const R sf = a.dagger ? R(1) : R(-1), sb = -sf;  // D: forward (1 - g), backward (1 + g)
  const uint32_t off = voff(i);
  const size_t fb = (size_t)rhs * 2 * SPINOR_ROWS * (size_t)vh;  // FULL: this right-hand side's full vectors
  const FullRows<SPINOR_ROWS> fr(a.g, base, end, a.p_out, lane);
  if constexpr (FULL) fr.template load<256>((const u4a8_t*)a.b + fb, rows, (int)threadIdx.x);

  const Field in = vec(a.in);
  const int jf = w == 0 ? nb.j[0] : w == 1 ? nb.j[2] : w == 2 ? nb.j[4] : nb.j[6];
  const int jb = w == 0 ? nb.j[1] : w == 1 ? nb.j[3] : w == 2 ? nb.j[5] : nb.j[7];
  const Spinor<R> pf = P::spinor(in, voff(jf)), pb = P::spinor(in, voff(jb));
  Link<R> uf, ub;
  P::links(bfield((const char*)a.links + (size_t)w * P::LK_E * field_vh(vh) * 16, P::LK_E, vh), boff(i, P::LK_E), uf, ub);
  // x of spin w; the other spin of its clover block comes through ex, so no wavefront reads rows
  // that another one stores (out may be x)
  const int blk = w >> 1;
  constexpr bool CX = MODE == M_APPLY || MODE == M_RICH || MODE == M_RESID;
  cpx<R> xs[3], bs[3];
  if constexpr (CX) {
    const Field xv = vec(a.x);
#pragma unroll
    for (int c = 0; c < 3; ++c) xs[c] = P::row(xv, 3 * w + c, off);
  }
  {
    Half<R> hf, hb;
    switch (w) {  // uniform over a wavefront
      case 0: split_hops<0, R>(pf, pb, uf, ub, sf, sb, nb, hf, hb); break;
      case 1: split_hops<1, R>(pf, pb, uf, ub, sf, sb, nb, hf, hb); break;
      case 2: split_hops<2, R>(pf, pb, uf, ub, sf, sb, nb, hf, hb); break;
      default: split_hops<3, R>(pf, pb, uf, ub, sf, sb, nb, hf, hb); break;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      hs[2 * w][k][lane] = hf.c[k / 3][k % 3];
      hs[2 * w + 1][k][lane] = hb.c[k / 3][k % 3];
    }
  }
  if constexpr (CX)
#pragma unroll
    for (int c = 0; c < 3; ++c) ex[3 * w + c][lane] = xs[c];
  if constexpr (MODE == M_RICH || MODE == M_RESID) {
    const Field bv = vec(a.b);
#pragma unroll
    for (int c = 0; c < 3; ++c) bs[c] = P::row(bv, 3 * w + c, off);
  }
  cpx<R> sl[18];
  if constexpr (MODE != M_PREP) P::slots(bfield(a.clov, P::CL_E, vh), boff(i, P::CL_E), blk, sl);
  __syncthreads();
  cpx<R> h[3] = {{R(0), R(0)}, {R(0), R(0)}, {R(0), R(0)}};
  switch (w) {
    case 0: split_sum<0, R>(h, hs, lane, sf, sb); break;
    case 1: split_sum<1, R>(h, hs, lane, sf, sb); break;
    case 2: split_sum<2, R>(h, hs, lane, sf, sb); break;
    default: split_sum<3, R>(h, hs, lane, sf, sb); break;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) h[c] = R(0.5) * h[c];
  if constexpr (FULL)
#pragma unroll
    for (int c = 0; c < 3; ++c) unpack<R>(rows[3 * w + c][lane], bs + c);
  cpx<R> o[3];
  decltype(P::stored(o[0])) y[3];
  if constexpr (MODE == M_PREP) {
#pragma unroll
    for (int c = 0; c < 3; ++c) y[c] = P::stored(o[c] = bs[c] + h[c]);
  } else {
    if constexpr (!CX) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if constexpr (MODE == M_RECON) h[c] = bs[c] + h[c];
        ex[3 * w + c][lane] = h[c];
      }
      __syncthreads();
    }
    cpx<R> v6[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) v6[k] = ex[6 * blk + k][lane];
    // A 16-bit result takes its stored form where it is formed, as in the one-thread kernels: the
    // compiler narrows in the multiply-add itself (one rounding, not two), which it cannot across
    // a merge of branches.  Kernel A's last operation is the clover product's.
    auto rows3 = [&](auto half) {
      clover_rows<half.value, R>(sl, v6, o);
      if constexpr (MODE == M_HOP_CLINV)
#pragma unroll
        for (int c = 0; c < 3; ++c) y[c] = P::formed_here(P::stored(o[c]));
    };
    if (w & 1)
      rows3(std::integral_constant<int, 1>{});
    else
      rows3(std::integral_constant<int, 0>{});
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if constexpr (MODE == M_APPLY) o[c] = o[c] - h[c];
      if constexpr (MODE == M_RESID) o[c] = bs[c] - o[c] + h[c];
      if constexpr (MODE == M_RICH) o[c] = ex[3 * w + c][lane] + (R)a.omega * (bs[c] - o[c] + h[c]);
      if constexpr (MODE != M_HOP_CLINV) y[c] = P::stored(o[c]);
    }
  }
  if constexpr (MODE == M_RECON) {
    // every row of b is read (the barrier above): the results take their place
#pragma unroll
    for (int c = 0; c < 3; ++c) rows[3 * w + c][lane] = pack<R>(o + c);
    __syncthreads();
    fr.template store<256>((u4a8_t*)a.full + fb, rows, (int)threadIdx.x);
    if (!a.out) return;  // uniform
  }
  if (!ok) return;
  if constexpr (MODE == M_PREP) {
    if (a.out32) {  // uniform
      using F = SplitR<float, false, ST_NONE>;
      const size_t r32 = (size_t)rhs * F::SP_E * (size_t)vh * 16;
      const Field v32 = vfield((char*)a.out32 + r32, F::SP_E, vh), z32 = vfield((char*)a.scaled32 + r32, F::SP_E, vh);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const cpx<float> v = {(float)o[c].r, (float)o[c].i};
        F::put(v32, 3 * w + c, off, v);
        F::put(z32, 3 * w + c, off, {v.r * a.scale, v.i * a.scale});
        store_fence();
      }
      return;
    }
  }
  const Field out = vec(a.out);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    P::put(out, 3 * w + c, off, y[c]);
    store_fence();
  }
}

// Slab order, but with fewer than eight groups of 64 sites a slice it leaves XCDs without work, and
// where an XCD's last group is missing on most of them (9 to 11 groups, or 17) one right-hand side
// waits for the others: 12 x 12 x 8 x 64 FP32 26 us an apply against 21 with the groups in a row.
// Several right-hand sides share the links that the order keeps together (5: 63 against 71).
static bool split_slab(const Geo& g, int nrhs) {
  const int ng = (g.sT + 63) / 64, padded = (ng + 7) / 8 * 8;
  return ng >= 8 && (nrhs > 1 || 5 * padded <= 7 * ng);
}
// workgroups of a launch on t_cnt slices
static long long split_grid(const Geo& g, int t_cnt, int nrhs) {
  const int ng = (g.sT + 63) / 64;
  return split_slab(g, nrhs) ? 8LL * t_cnt * ((ng + 7) / 8) * nrhs : ((long long)t_cnt * g.sT + 63) / 64 * nrhs;
}
constexpr long long SPLIT_MAX_GRID = 0xffffffffLL / 256;  // a launch has fewer than 2^32 threads

template <class P>
static hipError_t split_launch(SplitArgs a, int mode, hipStream_t s) {
  if (a.t_cnt <= 0) {
    a.t_lo = 0;
    a.t_cnt = a.g.L[3];
  }
  a.slab = split_slab(a.g, a.nrhs);
  const long long grid = split_grid(a.g, a.t_cnt, a.nrhs);
  if (grid > SPLIT_MAX_GRID) return hipErrorInvalidValue;
  const dim3 g((unsigned)grid), b(256);
#define DDQ_SPLIT_LAUNCH(M, TAKEN)                                            \
  case M:                                                                     \
    if constexpr (!(TAKEN)) return hipErrorInvalidValue;                      \
    else hipLaunchKernelGGL((hop_split_kernel<P, M>), g, b, 0, s, a);         \
    break
  // the modes of eq. 2 and the residual run in FP64 only; applies and sweeps as split_policy has them
  constexpr bool WIDE = sizeof(typename P::R) == 8;
  switch (mode) {
    DDQ_SPLIT_LAUNCH(M_HOP_CLINV, true);
    DDQ_SPLIT_LAUNCH(M_APPLY, P::STREAM != ST_LINKS_RESULT);
    DDQ_SPLIT_LAUNCH(M_RICH, P::STREAM != ST_LINKS);
    DDQ_SPLIT_LAUNCH(M_RECON, WIDE);
    DDQ_SPLIT_LAUNCH(M_RESID, WIDE);
    DDQ_SPLIT_LAUNCH(M_PREP, WIDE);
    default: return hipErrorInvalidValue;
  }
#undef DDQ_SPLIT_LAUNCH
  return hipGetLastError();
}

// Where four threads a site beat one.  Microseconds, one thread a site -> four, with the fields as
// left by the same call before / x written by another kernel just before / 1 GB written just
// before / 1 GB read just before:
//   FP64, one right-hand side: 8^4 20 -> 12 / 20 -> 12 / 34 -> 15 / 34 -> 15, 20 x 16^3 (40,960 sites)
//     44 -> 38 / 46 -> 38 / 48 -> 48 / 45 -> 41.  Repeated sweeps gain up to 200,000 sites, but a lone
//     apply that finds its fields in no cache does not (16^3 x 32 55 -> 53 / 57 -> 53 / 59 -> 67 / 56 -> 57);
//   FP32, one: applies up to 40,960 sites (26 -> 23 / 27 -> 24 / 28 -> 28 / 27 -> 25), again from 65,536
//     sites, where one thread a site begins a second wavefront on a SIMD (65,536: 30 -> 31 / 32 -> 31 /
//     33 -> 38 / 32 -> 33; 82,944: 46 -> 38 / 48 -> 39 / 49 -> 49 / 47 -> 43), to 340,000 (24^3 x 48
//     139 -> 125 / 142 -> 133 / 150 -> 148 / 139 -> 135; 28^3 x 32 143 -> 143 / 149 -> 147 / 158 -> 157 /
//     144 -> 148); between them 1 GB written just before costs up to 8 % (24^2 x 20 x 32 78 -> 69 / 79 ->
//     70 / 84 -> 91 / 78 -> 80).  Sweeps to 400,000 sites: two on 16^3 x 32 63 -> 57, on 24^3 x 48 287 -> 250,
//     on 387,072 sites 308 -> 303.  A solve's applies, whose fields the steps before left: 16^3 x 32
//     with nothing streamed 29 (the mixed solve there 3.99 ms -> 3.89);
//   several: the wavefronts of one 64-site group follow each other and take links and clover
//     from L2, at every size measured.  FP32 (no tile set): 2 on 16^3 x 32 51 -> 36 / 52 -> 36 / 55 -> 60 /
//     51 -> 45, 4 on 32^4 571 -> 575 (the closest: the one-thread kernel takes four together) and on
//     32^3 x 64 1176 -> 1122, 12 on 40^3 x 48 5054 -> 4555; FP64: 2 on 16^3 x 32 108 -> 79 / 107 -> 80 /
//     113 -> 103 / 108 -> 82, 8 on 32^3 x 64 4720 -> 4154;
//   16 bits, one: 65,536 sites (20 -> 20 / 21 -> 21 / 22 -> 23 / 22 -> 21), 73,728 26 -> 28, 128,000 28 -> 29.
//     Several, against a kernel that shares a link among two or three: 2 on 49,152 sites 26 -> 23,
//     3 on 32,768 31 -> 23, 9 on 10,368 30 -> 26, 16 on 4,096 24 -> 17 and on 4,608 24 -> 27; counts that
//     two and three do not divide, where it shares nothing and has the more wavefronts: 5 on 4,608
//     15 -> 14 and on 10,368 16 -> 18, 7 on 4,096 17 -> 13 and on 4,608 15 -> 17.
// And four threads a site reach a launch's limit of threads at a quarter of the sites.
bool hop_split_takes(const Geo& g, int bytes_per_complex, int nrhs, int reuse) {
  const long long n = (long long)g.Vh * nrhs;
  if (split_grid(g, g.L[3], nrhs) > SPLIT_MAX_GRID) return false;
  if (bytes_per_complex == 4)
    return n <= (nrhs == 1 || nrhs > 9 ? 65536 : nrhs % 2 != 0 && nrhs % 3 != 0 ? 24576 : 98304);
  if (nrhs > 1) return true;
  if (bytes_per_complex == 16) return n <= 40960;
  if (reuse == REUSE_NONE) return n <= 40960 || (n > 65536 && n <= 340000);
  return n <= (reuse == REUSE_SOLVE ? 340000 : 400000);
}

// What a launch streams past the Infinity Cache.  A line that is allocated there pushes another one
// out, which has to be written back first where an earlier kernel wrote it.
// * One right-hand side, a lone launch: the links, read once and the largest part.  FP32 applies as
//   above, nothing streamed -> links: 16^4 18 -> 19 / 19 -> 20 / 29 -> 23 / 21 -> 20, 24^3 x 32 95 -> 79 /
//   97 -> 79 / 127 -> 105 / 98 -> 96; FP16 16^3 x 32 19 -> 20 / 20 -> 21 / 26 -> 23 / 21 -> 21.  The results
//   too: 24^3 x 32 84 / 84 / 116 / 99; clover blocks, which two wavefronts read, too: 16^3 x 32 31 -> 35.
// * One right-hand side in a sweep or a solve, whose next launches read the same fields: nothing where
//   the links and clover blocks of both parities fit the cache's 256 MB, else a sweep's links and
//   results (24^3 x 48 six FP32 sweeps 739, links only 778, nothing 852) and an apply's links.
// * Several: nothing; the next wavefronts read the links again (streamed with the results: 2 on 32^4
//   FP32 329 -> 342, 4 575 -> 617, 8 on 32^3 x 64 FP64 4154 -> 4474).
static int split_policy(const SplitArgs& a, long long field_bytes) {
  if (a.nrhs > 1 || (a.reuse != REUSE_NONE && field_bytes <= (256LL << 20))) return ST_NONE;
  return a.reuse == REUSE_SWEEP ? ST_LINKS_RESULT : ST_LINKS;
}

template <typename R, bool L12>
static hipError_t split_launch_r(const SplitArgs& a, int mode, hipStream_t s) {
  switch (split_policy(a, 2LL * a.g.Vh * ((L12 ? 4 * LINK12_ROWS : 4 * LINK_ROWS) + CLOVER_ROWS) * (long long)sizeof(pair<R>))) {
    case ST_NONE: return split_launch<SplitR<R, L12, ST_NONE>>(a, mode, s);
    case ST_LINKS: return split_launch<SplitR<R, L12, ST_LINKS>>(a, mode, s);
  }
  // in FP64 hop_split_takes has no sweep of one right-hand side past the cache
  if constexpr (sizeof(R) == 4) return split_launch<SplitR<R, L12, ST_LINKS_RESULT>>(a, mode, s);
  return split_launch<SplitR<R, L12, ST_NONE>>(a, mode, s);
}

template <typename R>
hipError_t launch_hop_split(const HopArgs<R>& h, int mode, bool dagger, int nrhs, hipStream_t s) {
  SplitArgs a{};
  a.g = h.g;
  a.p_out = h.p_out;
  a.in = h.in;
  a.links = h.links;
  a.clov = h.clov;
  a.x = h.x;
  a.b = h.b;
  a.out = h.out;
  a.omega = (double)h.omega;
  a.nrhs = nrhs;
  a.dagger = dagger ? 1 : 0;
  a.reuse = h.reuse;
  a.t_lo = h.t_lo;
  a.t_cnt = h.t_cnt;
  a.full = h.full;
  a.out32 = h.out32;
  a.scaled32 = h.scaled32;
  a.scale = h.scale;
  if (nrhs < 1 || a.t_lo < 0 || a.t_cnt < 0 || a.t_lo + a.t_cnt > a.g.L[3]) return hipErrorInvalidValue;
  if constexpr (sizeof(R) == 4)
    if (h.link12) return split_launch_r<float, true>(a, mode, s);
  return split_launch_r<R, false>(a, mode, s);
}
template hipError_t launch_hop_split<double>(const HopArgs<double>&, int, bool, int, hipStream_t);
template hipError_t launch_hop_split<float>(const HopArgs<float>&, int, bool, int, hipStream_t);

template <typename S>
static hipError_t split_launch_16(const SplitArgs& a, bool c32, int mode, hipStream_t s) {
  if (split_policy(a, 0) == ST_LINKS)  // a field of the sizes that hop_split_takes fits the cache
    return c32 ? split_launch<Split16<S, true, ST_LINKS>>(a, mode, s) : split_launch<Split16<S, false, ST_LINKS>>(a, mode, s);
  return c32 ? split_launch<Split16<S, true, ST_NONE>>(a, mode, s) : split_launch<Split16<S, false, ST_NONE>>(a, mode, s);
}

hipError_t launch_hop16_split(int kind, const Hop16Args& h, int mode, hipStream_t s) {
  SplitArgs a{};
  a.g = h.g;
  a.p_out = h.p_out;
  a.in = h.in;
  a.links = h.links;
  a.clov = h.clov32 ? (const void*)h.clov32 : h.clov;
  a.x = h.x;
  a.b = h.b;
  a.out = h.out;
  a.omega = (double)h.omega;
  a.nrhs = h.nrhs;
  if (h.nrhs < 1) return hipErrorInvalidValue;
  a.reuse = h.reuse;
  return kind == H16_BF16 ? split_launch_16<__bf16>(a, h.clov32 != nullptr, mode, s) : split_launch_16<_Float16>(a, h.clov32 != nullptr, mode, s);
}

}  // namespace ddq
