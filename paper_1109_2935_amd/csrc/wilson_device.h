// Device code of the Wilson hopping and clover terms shared by the kernels: spin
// projection, the hop of each storage format, spinor and link access, the
// clover product and the kernel arguments.
#pragma once

#include <type_traits>

#include "lqcd_internal.h"

namespace lqcd {

// ---------------------------------------------------------------------------
// spin projection in the chiral basis.
// For P = 1 + g gamma_mu (g = +-1) the result has rows 2,3 proportional to
// rows 0,1, so only h0 = row 0 and h1 = row 1 are formed:
//   x: h0 = s0 - g i s3, h1 = s1 - g i s2;  rows 2,3 = ( g i h1,  g i h0)
//   y: h0 = s0 - g s3,   h1 = s1 + g s2;    rows 2,3 = ( g h1,   -g h0)
//   z: h0 = s0 - g i s2, h1 = s1 + g i s3;  rows 2,3 = ( g i h0, -g i h1)
//   t: h0 = s0 + g s2,   h1 = s1 + g s3;    rows 2,3 = ( g h0,    g h1)

template <int MU, typename R>
__device__ __forceinline__ void project(const cpx<R> (&s)[4][3], R g, cpx<R> (&h)[2][3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if constexpr (MU == 0) {
      h[0][c] = s[0][c] - g * times_i(s[3][c]);
      h[1][c] = s[1][c] - g * times_i(s[2][c]);
    } else if constexpr (MU == 1) {
      h[0][c] = s[0][c] - g * s[3][c];
      h[1][c] = s[1][c] + g * s[2][c];
    } else if constexpr (MU == 2) {
      h[0][c] = s[0][c] - g * times_i(s[2][c]);
      h[1][c] = s[1][c] + g * times_i(s[3][c]);
    } else {
      h[0][c] = s[0][c] + g * s[2][c];
      h[1][c] = s[1][c] + g * s[3][c];
    }
  }
}

template <int MU, typename R>
__device__ __forceinline__ void expand_acc(cpx<R> (&acc)[4][3], const cpx<R> (&u)[2][3], R g) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    acc[0][c] = acc[0][c] + u[0][c];
    acc[1][c] = acc[1][c] + u[1][c];
    if constexpr (MU == 0) {
      acc[2][c] = acc[2][c] + g * times_i(u[1][c]);
      acc[3][c] = acc[3][c] + g * times_i(u[0][c]);
    } else if constexpr (MU == 1) {
      acc[2][c] = acc[2][c] + g * u[1][c];
      acc[3][c] = acc[3][c] - g * u[0][c];
    } else if constexpr (MU == 2) {
      acc[2][c] = acc[2][c] + g * times_i(u[0][c]);
      acc[3][c] = acc[3][c] - g * times_i(u[1][c]);
    } else {
      acc[2][c] = acc[2][c] + g * u[0][c];
      acc[3][c] = acc[3][c] + g * u[1][c];
    }
  }
}

// ---------------------------------------------------------------------------
// FP16 storage: a hop in packed half arithmetic. The spin projection runs on
// packed FP16 pairs (each component of h rounded once to FP16; the sign flips
// and factors i are exact) and the colour products U h on v_dot2_f32_f16
// (products of two FP16 values are exact in FP32, sums in FP32). With 12
// stored link reals the third row is rebuilt in FP32 from the same dot2 sums
// and multiplied in FP32. Against the FP32-arithmetic hop this removes the 36
// half-to-float conversions of a hop and halves its colour-product
// instructions; the one new rounding (of h) is a quarter of the storage
// rounding already in the input.
typedef _Float16 h2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ h2v h2_times_i(h2v a) { return h2v{-a.y, a.x}; }
__device__ __forceinline__ float dot2(h2v a, h2v b, float c) { return __builtin_amdgcn_fdot2(a, b, c, false); }

template <int MU>
__device__ __forceinline__ void project_h2(const h2v (&s)[4][3], h2v g, h2v (&h)[2][3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if constexpr (MU == 0) {
      h[0][c] = s[0][c] - g * h2_times_i(s[3][c]);
      h[1][c] = s[1][c] - g * h2_times_i(s[2][c]);
    } else if constexpr (MU == 1) {
      h[0][c] = s[0][c] - g * s[3][c];
      h[1][c] = s[1][c] + g * s[2][c];
    } else if constexpr (MU == 2) {
      h[0][c] = s[0][c] - g * h2_times_i(s[2][c]);
      h[1][c] = s[1][c] + g * h2_times_i(s[3][c]);
    } else {
      h[0][c] = s[0][c] + g * s[2][c];
      h[1][c] = s[1][c] + g * s[3][c];
    }
  }
}

// u_k = U h_k (FWD) or U^+ h_k for both half-spinor rows k; U as stored: rows
// 0 and 1 (and 2 with 18 reals) as packed (re, im) pairs, row-major.
template <int RECON, bool FWD>
__device__ __forceinline__ void su3_h2(const h2v (&U)[RECON / 2], const h2v (&h)[2][3], cpx<float> (&u)[2][3]) {
  static_assert(RECON == 12 || RECON == 18, "16-bit links hold 12 or 18 reals");
  // conj-swapped forms of h: Re(a b) = dot2(a, hc), Im(a b) = dot2(a, hs);
  // Re(conj(a) b) = dot2(a, b), Im(conj(a) b) = dot2(a, ha)
  h2v hx[2][3], hy[2][3];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      hx[k][c] = FWD ? h2v{h[k][c].x, -h[k][c].y} : h[k][c];
      hy[k][c] = FWD ? h2v{h[k][c].y, h[k][c].x} : h2v{h[k][c].y, -h[k][c].x};
    }
  constexpr int NR = RECON == 18 ? 3 : 2;  // rows taken from storage
  // forward: output rows i < NR over all columns j; adjoint: all outputs i
  // over the stored rows j < NR
  constexpr int NI = FWD ? NR : 3, NJ = FWD ? 3 : NR;
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      float re = 0.f, im = 0.f;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        // forward: row i of U, column j of h; adjoint: column i of U (row j)
        const h2v a = FWD ? U[3 * i + j] : U[3 * j + i];
        re = dot2(a, hx[k][j], re);
        im = dot2(a, hy[k][j], im);
      }
      u[k][i] = mk<float>(re, im);
    }
  if constexpr (RECON == 12) {
    // third row conj(row0 x row1) in FP32: U2j = conj(U0k U1l - U0l U1k)
    cpx<float> r2[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int k = (j + 1) % 3, l = (j + 2) % 3;
      const h2v a = U[k], b = U[3 + l], c = U[l], d = U[3 + k];
      const float re = dot2(a, h2v{b.x, -b.y}, dot2(-c, h2v{d.x, -d.y}, 0.f));
      const float im = dot2(c, h2v{d.y, d.x}, dot2(-a, h2v{b.y, b.x}, 0.f));
      r2[j] = mk<float>(re, im);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      cpx<float> hf[3];
#pragma unroll
      for (int j = 0; j < 3; ++j) hf[j] = mk<float>((float)h[k][j].x, (float)h[k][j].y);
      if constexpr (FWD) {
        cpx<float> a = r2[0] * hf[0];
        cmac(a, r2[1], hf[1]);
        cmac(a, r2[2], hf[2]);
        u[k][2] = a;
      } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) cmac_conj(u[k][i], r2[i], hf[2]);
      }
    }
  }
}

// One FP16 hop from stored values: psi the neighbour's 24 halves, link its
// RECON halves, ps the projection sign (+-1); u as su3_h2.
template <int MU, int DIR, int RECON>
__device__ __forceinline__ void hop_h2(const uint32_t (&psi)[12], const uint32_t (&link)[RECON / 2], float ps,
                                       cpx<float> (&u)[2][3]) {
  h2v s[4][3], hh[2][3], U[RECON / 2];
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int c = 0; c < 3; ++c) s[sp][c] = __builtin_bit_cast(h2v, psi[3 * sp + c]);
#pragma unroll
  for (int k = 0; k < RECON / 2; ++k) U[k] = __builtin_bit_cast(h2v, link[k]);
  const _Float16 g16 = (_Float16)ps;
  project_h2<MU>(s, h2v{g16, g16}, hh);
  su3_h2<RECON, (DIR > 0)>(U, hh, u);
}

template <typename S, typename R>
__device__ __forceinline__ void load_spinor(const S *__restrict__ f, int64_t vh, int s, cpx<R> (&v)[4][3]) {
  R r[24];
  load_spinor_reals<S, 24, R>(f, vh, s, r);
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int c = 0; c < 3; ++c) v[sp][c] = mk<R>(r[6 * sp + 2 * c], r[6 * sp + 2 * c + 1]);
}

template <typename S, typename R, bool NT = false>
__device__ __forceinline__ void store_spinor(S *__restrict__ f, int64_t vh, int s, const cpx<R> (&v)[4][3]) {
  R r[24];
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      r[6 * sp + 2 * c] = v[sp][c].re;
      r[6 * sp + 2 * c + 1] = v[sp][c].im;
    }
  store_spinor_reals<S, 24, R, NT>(f, vh, s, r);
}

// Round to the storage precision and back (what a store followed by a load returns).
template <typename S, typename R> __device__ __forceinline__ R quantize(R v) { return to_real<R>(Store<S>::from(v)); }

// Storage whose Wilson kernels agree bit for bit with those of wilson_split.hip.
template <typename S> constexpr bool fused_products() { return sizeof(S) >= 4; }

// stream: the link is read once per launch (one right-hand side)
template <typename S, typename R, int RECON>
__device__ __forceinline__ Link<R> load_link(const S *__restrict__ gauge, int64_t vh, int mu, int parity, int s,
                                             bool stream) {
  R v[RECON];
  load_site_once<S, RECON, R>(gauge + (int64_t)(2 * mu + parity) * vh * RECON, vh, s, v, stream);
  return unpack_link<RECON, R, fused_products<S>()>(v);
}

// Clover: per site and chirality block a Hermitian 6x6 (index = spin-in-block*3
// + colour): 6 real diagonal entries, then the strictly lower triangle in row
// order as (re, im); block 0 = spins 0,1, block 1 = spins 2,3 (72 reals).
template <typename S, typename R>
__device__ __forceinline__ void clover_mul(const S *__restrict__ clov, int64_t vh, int s, const cpx<R> (&in)[4][3],
                                           cpx<R> (&out)[4][3], bool stream) {
  R a[72];
  load_site_once<S, 72, R>(clov, vh, s, a, stream);
  if constexpr (is_fixed<S>()) {
    const R m = (R)site_norms<S, 72>(clov, vh)[s];
#pragma unroll
    for (int k = 0; k < 72; ++k) a[k] *= m;
  }
  if constexpr (is_float16<S>()) {
    // converted here, as in the hops: kept from folding into mixed-precision FMAs
#pragma unroll
    for (int k = 0; k < 72; ++k) __asm__ volatile("" : "+v"(a[k]));
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const R *A = a + 36 * b;
    cpx<R> x[6], y[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) x[i] = in[2 * b + i / 3][i % 3];
#pragma unroll
    for (int i = 0; i < 6; ++i) y[i] = A[i] * x[i];
    int off = 6;
#pragma unroll
    for (int i = 1; i < 6; ++i)
#pragma unroll
      for (int j = 0; j < i; ++j) {
        const cpx<R> aij = mk<R>(A[off], A[off + 1]);
        off += 2;
        cmac(y[i], aij, x[j]);
        cmac_conj(y[j], aij, x[i]);
      }
#pragma unroll
    for (int i = 0; i < 6; ++i) out[2 * b + i / 3][i % 3] = y[i];
  }
}

template <typename S> struct WArgs {
  Geom g;
  S *out;
  const S *in;
  const S *gauge;
  const S *clov;
  const S *xin;
  double *partials;
  double coef;
  int parity;
  int dagger;
  int nrhs;  // right-hand sides
  int rg;    // sources per block of the multi-source layout (rhs_group(nrhs))
};

// Software-pipelined hops for launches without a cut (FP32 and 16-bit
// storage): the raw inputs of a hop (neighbour spinor, link as stored, wrap
// count) go to one of two buffers, refilled alternately, so each wave keeps
// the loads of the next hop in flight while it multiplies the current one.
// Scheduling barriers hold that order
// (without them the compiler issues the loads of all eight hops first and
// spills).
// The raw values stay in the storage type until they are used, so that no
// conversion forces an early wait for the loads.
template <typename S, int RECON> struct HopIn {
  S psi[24];
  S link[RECON];
  int w;
};

template <int MU, int DIR, bool STREAM, typename S, int RECON>
__device__ __forceinline__ void hop_fetch(const WArgs<S> &a, const Site &x, int s, int rhs, HopIn<S, RECON> &h) {
  const int64_t vh = a.g.Vh, vs = vh * a.nrhs;
  const int n = hop1<MU, DIR>(a.g, x, &h.w);
  load_chunks_raw<S, 24, spinor_chunk<24>()>(a.in, vs, rhs_index(rhs, n, vh, a.rg), h.psi);
  // forward hop: U_mu(x) of x's parity; backward: U_mu(x - mu) of the other
  const int lp = DIR > 0 ? x.p : 1 - x.p, ls = DIR > 0 ? s : n;
  load_chunks_raw<S, RECON, chunk_reals<S, RECON>(), STREAM>(a.gauge + (int64_t)(2 * MU + lp) * vh * RECON, vh, ls,
                                                           h.link);
}

// FP16 storage takes the packed-half hop (hop_h2) with 12 or 18 link reals.
template <typename S, int RECON> constexpr bool half_hop() {
  return std::is_same<S, _Float16>::value && (RECON == 12 || RECON == 18);
}

// The half spinor of a hop: U (or U^+) times the projected neighbour, times the
// boundary sign; ps the projection sign.
template <int MU, int DIR, typename S, typename R, int RECON>
__device__ __forceinline__ void hop_product(const HopIn<S, RECON> &h, R ps, int bc_t, cpx<R> (&u)[2][3]) {
  if constexpr (half_hop<S, RECON>()) {
    uint32_t pw[12], lw[RECON / 2];
#pragma unroll
    for (int j = 0; j < 12; ++j) pw[j] = __builtin_bit_cast(uint32_t, h2v{h.psi[2 * j], h.psi[2 * j + 1]});
#pragma unroll
    for (int j = 0; j < RECON / 2; ++j) lw[j] = __builtin_bit_cast(uint32_t, h2v{h.link[2 * j], h.link[2 * j + 1]});
    hop_h2<MU, DIR, RECON>(pw, lw, ps, u);
  } else {
    cpx<R> psi[4][3], hh[2][3];
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        R re = to_real<R>(h.psi[6 * sp + 2 * c]), im = to_real<R>(h.psi[6 * sp + 2 * c + 1]);
        if constexpr (is_float16<S>()) {
          // convert here: the empty asm keeps the compiler from folding the
          // stored halves into mixed-precision FMAs, which keeps them live
          // across the hop (170-230 VGPRs instead of about 110)
          __asm__ volatile("" : "+v"(re));
          __asm__ volatile("" : "+v"(im));
        }
        psi[sp][c] = mk<R>(re, im);
      }
    project<MU, R>(psi, ps, hh);
    R lv[RECON];
#pragma unroll
    for (int k = 0; k < RECON; ++k) {
      lv[k] = to_real<R>(h.link[k]);
      if constexpr (is_float16<S>()) __asm__ volatile("" : "+v"(lv[k]));
    }
    constexpr bool F = fused_products<S>();
    const Link<R> U = unpack_link<RECON, R, F>(lv);
    if constexpr (DIR > 0) {
      su3_mv<F>(U, hh[0], u[0]);
      su3_mv<F>(U, hh[1], u[1]);
    } else {
      su3_adj_mv<F>(U, hh[0], u[0]);
      su3_adj_mv<F>(U, hh[1], u[1]);
    }
  }
  if constexpr (MU == 3) {
    const R ph = ((h.w & 1) && bc_t < 0) ? R(-1) : R(1);
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) u[k][c] = ph * u[k][c];
  }
}

template <int MU, int DIR, typename S, typename R, int RECON>
__device__ __forceinline__ void hop_apply(const HopIn<S, RECON> &h, R sgn, int bc_t, cpx<R> (&acc)[4][3]) {
  const R ps = DIR > 0 ? -sgn : sgn;
  cpx<R> u[2][3];
  hop_product<MU, DIR, S, R, RECON>(h, ps, bc_t, u);
  expand_acc<MU, R>(acc, u, ps);
}

}  // namespace lqcd
