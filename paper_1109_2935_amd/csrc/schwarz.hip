// Wilson-clover block kernels for gfx950: the MR iterations of the Schwarz
// preconditioner with a Dirichlet block held on chip.
#include <type_traits>

#include "lqcd_internal.h"
#include "wilson_device.h"

namespace lqcd {

// ---------------------------------------------------------------------------
// Additive Schwarz with each block resident in LDS (Section 4's block solver,
// with blocks equal to the tiles and 16-bit storage: FP16, BF16, or fixed
// point with a per-site norm): one workgroup runs every MR step of one block. This
// form serves BF16 and fixed point, sap_half_kernel below FP16. The block's spinor
// of the current half step (r on the even sites, then t on the odd sites) lives in LDS, so neighbours are read
// from there; links and clover stream from memory in each half step; the
// workgroup keeps its sites' r and q (and x, where registers allow) as stored
// 16-bit values. Per step and even site this moves the links twice and both
// clover blocks (672 bytes at 12 link reals, 768 with x in memory) instead of
// the 1152 bytes of two cut Schur launches and an update. The arithmetic is
// the launches' (same operations, same roundings to the storage format, the
// same order of the FP64 sums of <q,r> and <q,q>: per 64-site segment by the
// wave butterfly, then the block's segments in order): with BF16 both forms give the
// same result; in fixed point the compiler folds conversions differently in the two,
// and a few percent of the values differ by rounding steps.
constexpr int kSapMaxSites = 2048;  // sites per parity of one block (96 KiB of 16-bit spinor)

template <typename S> struct SapArgs {
  S *x;           // out: x (even sites)
  const S *r0;    // in: residual (even sites)
  const S *gauge;
  const S *clov_inv_odd;  // A_oo^-1
  const S *clov_even;     // A_ee
  Geom g;                 // for the tile of a colour-restricted launch
  int64_t vh;
  int vt2;
  int b[4];   // block (tile) extents
  int wrap;   // bit mu: the block spans the lattice along mu, its hops wrap inside it
  int bc_t;
  float coef;  // -kappa^2
  double omega;
  int steps;
  int first;  // x starts at zero (not read)
};

// two stored 16-bit values in one register
template <typename S> __device__ __forceinline__ uint32_t pack16(S lo, S hi) {
  return (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
}
template <typename S> __device__ __forceinline__ float lo16(uint32_t u) {
  return to_real<float>(__builtin_bit_cast(S, (uint16_t)(u & 0xffffu)));
}
template <typename S> __device__ __forceinline__ float hi16(uint32_t u) {
  return to_real<float>(__builtin_bit_cast(S, (uint16_t)(u >> 16)));
}

// A site's stored spinor: its 24 16-bit values as 12 registers (register j =
// reals 2j, 2j+1; in LDS and in memory the spinor is chunk-major, chunk c =
// registers 2c, 2c+1) and, with fixed-point storage, the site norm.
template <typename S, bool FIXED = is_fixed<S>()> struct SapSite {
  uint32_t p[12];
};
template <typename S> struct SapSite<S, true> {
  uint32_t p[12];
  float m;
};

// stored -> FP32, as the other kernels load (fixed point: the code's value,
// then times the site norm)
template <typename S> __device__ __forceinline__ void sap_reals(const SapSite<S> &s, float (&v)[24]) {
#pragma unroll
  for (int j = 0; j < 12; ++j) {
    v[2 * j] = lo16<S>(s.p[j]);
    v[2 * j + 1] = hi16<S>(s.p[j]);
  }
  if constexpr (is_fixed<S>()) {
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] *= s.m;
  }
}
// FP32 -> stored, as the other kernels store (fixed point: the norm is the
// largest |v_k|, the codes those of v_k times its reciprocal)
template <typename S> __device__ __forceinline__ void sap_store(const float (&v)[24], SapSite<S> &s) {
  if constexpr (is_fixed<S>()) {
    const float m = fixed_norm<24, float>(v), inv = m > 0 ? 1.0f / m : 0.0f;
    s.m = m;
#pragma unroll
    for (int j = 0; j < 12; ++j)
      s.p[j] = pack16<S>(Store<S>::from((float)v[2 * j] * inv), Store<S>::from((float)v[2 * j + 1] * inv));
  } else {
#pragma unroll
    for (int j = 0; j < 12; ++j) s.p[j] = pack16<S>(Store<S>::from(v[2 * j]), Store<S>::from(v[2 * j + 1]));
  }
}
__device__ __forceinline__ void sap_flat(const cpx<float> (&v)[4][3], float (&f)[24]) {
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      f[6 * sp + 2 * c] = v[sp][c].re;
      f[6 * sp + 2 * c + 1] = v[sp][c].im;
    }
}
__device__ __forceinline__ void sap_cpx(const float (&f)[24], cpx<float> (&v)[4][3]) {
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int c = 0; c < 3; ++c) v[sp][c] = mk<float>(f[6 * sp + 2 * c], f[6 * sp + 2 * c + 1]);
}
// The site's registers become opaque to the compiler here: values derived
// from them (unpacked FP32 copies) are not kept alive across the point.
template <typename S> __device__ __forceinline__ void sap_opaque(SapSite<S> &s) {
#pragma unroll
  for (int j = 0; j < 12; ++j) __asm__ volatile("" : "+v"(s.p[j]));
  if constexpr (is_fixed<S>()) __asm__ volatile("" : "+v"(s.m));
}
// LDS: 6 chunk arrays of vt2 sites (8 bytes each), then (fixed point) the
// vt2 site norms
template <typename S> __device__ __forceinline__ void sap_lds_put(uint2 *lds, int vt2, int k, const SapSite<S> &s) {
#pragma unroll
  for (int c = 0; c < 6; ++c) lds[c * vt2 + k] = make_uint2(s.p[2 * c], s.p[2 * c + 1]);
  if constexpr (is_fixed<S>()) reinterpret_cast<float *>(lds + 6 * vt2)[k] = s.m;
}
template <typename S> __device__ __forceinline__ void sap_lds_get(const uint2 *lds, int vt2, int k, SapSite<S> &s) {
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    const uint2 v = lds[c * vt2 + k];
    s.p[2 * c] = v.x;
    s.p[2 * c + 1] = v.y;
  }
  if constexpr (is_fixed<S>()) s.m = reinterpret_cast<const float *>(lds + 6 * vt2)[k];
}
template <typename S> __device__ __forceinline__ void sap_mem_get(const S *f, int64_t vh, int64_t s, SapSite<S> &o) {
  const uint2 *q = reinterpret_cast<const uint2 *>(f);
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    const uint2 v = q[c * vh + s];
    o.p[2 * c] = v.x;
    o.p[2 * c + 1] = v.y;
  }
  if constexpr (is_fixed<S>()) o.m = site_norms<S, 24>(f, vh)[s];
}
template <typename S> __device__ __forceinline__ void sap_mem_put(S *f, int64_t vh, int64_t s, const SapSite<S> &o) {
  uint2 *q = reinterpret_cast<uint2 *>(f);
#pragma unroll
  for (int c = 0; c < 6; ++c) nt_store(q + c * vh + s, make_uint2(o.p[2 * c], o.p[2 * c + 1]));
  if constexpr (is_fixed<S>()) site_norms<S, 24>(f, vh)[s] = o.m;
}
// bytes of dynamic LDS: the spinor (and norms) of a block, then the segment sums
__host__ __device__ constexpr size_t sap_lds_bytes(int vt2, bool fixed) {
  return (size_t)vt2 * (48 + (fixed ? 4 : 0)) + (size_t)(vt2 / 64) * 3 * sizeof(double);
}

// Hop of STEP along MU from block coordinates l: false if the cut drops it;
// else the neighbour's block-local index and whether the hop wrapped the
// lattice along t with antiperiodic boundary (a sign flip).
template <int MU, int STEP, typename S>
__device__ __forceinline__ bool sap_hop(const SapArgs<S> &a, const int (&l)[4], int *kn, bool *flip) {
  int c[4] = {l[0], l[1], l[2], l[3]};
  c[MU] += STEP;
  const bool out = STEP > 0 ? c[MU] >= a.b[MU] : c[MU] < 0;
  if (out && !((a.wrap >> MU) & 1)) return false;
  c[MU] = out ? (STEP > 0 ? 0 : a.b[MU] - 1) : c[MU];
  *flip = MU == 3 && out && a.bc_t < 0;
  *kn = (c[0] >> 1) + (a.b[0] >> 1) * (c[1] + a.b[1] * (c[2] + a.b[2] * c[3]));
  return true;
}

template <int MU, int STEP, typename S, int RECON>
__device__ __forceinline__ void sap_hop_acc(const SapArgs<S> &a, const uint2 *lds, int base, const int (&l)[4], int k,
                                            int par, cpx<float> (&acc)[4][3]) {
  int kn;
  bool flip;
  if (!sap_hop<MU, STEP>(a, l, &kn, &flip)) return;
  SapSite<S> nb;
  cpx<float> u[2][3];
  sap_lds_get<S>(lds, a.vt2, kn, nb);
  // forward: (1 - gamma_mu) U_mu(x) psi(x+mu); backward: (1 + gamma_mu) U_mu(x-mu)^+ psi(x-mu)
  const float g = STEP > 0 ? -1.f : 1.f;
  float pf[24];
  cpx<float> psi[4][3], h[2][3];
  sap_reals<S>(nb, pf);
  sap_cpx(pf, psi);
  project<MU, float>(psi, g, h);
  // 18-real links (4-byte pieces) through the caches, which hold a block's links for the next half step; streamed,
  // as those of 12 reals are, the K of 4^4 blocks at 32^3 x 64 takes 951 instead of 813 us (BF16, 6 steps)
  const Link<float> U = STEP > 0 ? load_link<S, float, RECON>(a.gauge, a.vh, MU, par, base + k, RECON == 12)
                                 : load_link<S, float, RECON>(a.gauge, a.vh, MU, 1 - par, base + kn, RECON == 12);
  if constexpr (STEP > 0) {
    su3_mv(U, h[0], u[0]);
    su3_mv(U, h[1], u[1]);
  } else {
    su3_adj_mv(U, h[0], u[0]);
    su3_adj_mv(U, h[1], u[1]);
  }
  if constexpr (MU == 3) {
    const float ph = flip ? -1.f : 1.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) u[i][c] = ph * u[i][c];
  }
  expand_acc<MU, float>(acc, u, g);
}

// D restricted to the block at block-local site k of parity par (coordinates
// packed 8 bits each: x/2, y, z, t), neighbours from LDS
template <typename S, int RECON>
__device__ __forceinline__ void sap_hops(const SapArgs<S> &a, const uint2 *lds, int base, int k, uint32_t coords,
                                         int par, cpx<float> (&acc)[4][3]) {
  int l[4];
  l[1] = (coords >> 8) & 255;
  l[2] = (coords >> 16) & 255;
  l[3] = coords >> 24;
  l[0] = 2 * (int)(coords & 255) + ((l[1] + l[2] + l[3] + par) & 1);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[i][c] = mk<float>(0, 0);
  sap_hop_acc<0, +1, S, RECON>(a, lds, base, l, k, par, acc);
  __builtin_amdgcn_sched_barrier(0);
  sap_hop_acc<0, -1, S, RECON>(a, lds, base, l, k, par, acc);
  __builtin_amdgcn_sched_barrier(0);
  sap_hop_acc<1, +1, S, RECON>(a, lds, base, l, k, par, acc);
  __builtin_amdgcn_sched_barrier(0);
  sap_hop_acc<1, -1, S, RECON>(a, lds, base, l, k, par, acc);
  __builtin_amdgcn_sched_barrier(0);
  sap_hop_acc<2, +1, S, RECON>(a, lds, base, l, k, par, acc);
  __builtin_amdgcn_sched_barrier(0);
  sap_hop_acc<2, -1, S, RECON>(a, lds, base, l, k, par, acc);
  __builtin_amdgcn_sched_barrier(0);
  sap_hop_acc<3, +1, S, RECON>(a, lds, base, l, k, par, acc);
  __builtin_amdgcn_sched_barrier(0);
  sap_hop_acc<3, -1, S, RECON>(a, lds, base, l, k, par, acc);
  __builtin_amdgcn_sched_barrier(0);
}

// Clover product for the block kernel: the same operations as clover_mul, one
// chirality block at a time (36 values in registers instead of 72).
template <typename S>
__device__ __forceinline__ void sap_clover(const S *__restrict__ clov, int64_t vh, int s, const cpx<float> (&in)[4][3],
                                           cpx<float> (&out)[4][3]) {
  constexpr int CH = chunk_reals<S, 72>();  // reals per chunk (8 for 16-bit storage)
  static_assert(CH == 8, "16-bit clover chunks of 8 reals");
  float a[72];
  float m = 1.f;  // fixed point: the site norm of the clover term
  if constexpr (is_fixed<S>()) m = site_norms<S, 72>(clov, vh)[s];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    // chunks 0..4 hold block 0 (reals 0..35), chunks 4..8 block 1 (36..71)
#pragma unroll
    for (int c = 5 * b - b; c < 5 * b - b + 5; ++c) {
      if (b == 1 && c == 4) continue;  // loaded with block 0
      const Chunk<S, 8> v = nt_load(reinterpret_cast<const Chunk<S, 8> *>(clov + (c * vh + s) * 8));
#pragma unroll
      for (int j = 0; j < 8; ++j) a[8 * c + j] = to_real<float>(v.v[j]);
    }
#pragma unroll
    for (int k = 36 * b; k < 36 * b + 36; ++k) {
      if constexpr (is_fixed<S>())
        a[k] *= m;
      else
        __asm__ volatile("" : "+v"(a[k]));
    }
    const float *A = a + 36 * b;
    cpx<float> x[6], y[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) x[i] = in[2 * b + i / 3][i % 3];
#pragma unroll
    for (int i = 0; i < 6; ++i) y[i] = A[i] * x[i];
    int off = 6;
#pragma unroll
    for (int i = 1; i < 6; ++i)
#pragma unroll
      for (int j = 0; j < i; ++j) {
        const cpx<float> aij = mk<float>(A[off], A[off + 1]);
        off += 2;
        cmac(y[i], aij, x[j]);
        cmac_conj(y[j], aij, x[i]);
      }
#pragma unroll
    for (int i = 0; i < 6; ++i) out[2 * b + i / 3][i % 3] = y[i];
  }
}

// One workgroup per block (blockIdx.x: the block's tile, or the j-th tile of
// one colour); SPT sites per thread and parity, site k = p * blockDim.x + tid.
// XREG: x stays in registers (else it is read and written in memory each step).
// NT: the most threads per workgroup (512, or 1024 for the wide launches).
template <typename S, int RECON, int SPT, bool XREG, int NT>
__global__ void __launch_bounds__(NT) sap_block_kernel(SapArgs<S> a) {
  extern __shared__ uint2 sap_lds[];  // the block's spinor (and norms), then the segment sums
  const int vt2 = a.vt2, nt = blockDim.x, tid = threadIdx.x;
  double *seg = reinterpret_cast<double *>(reinterpret_cast<char *>(sap_lds) + sap_lds_bytes(vt2, is_fixed<S>()) -
                                           (size_t)(vt2 / 64) * 3 * sizeof(double));  // [Vt2 / 64][3]
  const int tile = a.g.colour >= 0 ? colour_site(a.g, blockIdx.x * vt2) / vt2 : (int)blockIdx.x;
  const int base = tile * vt2;
  SapSite<S> r[SPT], w[SPT];  // w: t (odd sites) or q (even sites)
  SapSite<S> x[XREG ? SPT : 1];
  uint32_t coords[SPT];
#pragma unroll
  for (int p = 0; p < SPT; ++p) {
    const int k = p * nt + tid;
    const int bxh = a.b[0] >> 1;
    const int q1 = k / bxh, q2 = q1 / a.b[1];
    coords[p] = (uint32_t)(k - q1 * bxh) | ((uint32_t)(q1 - q2 * a.b[1]) << 8) |
                ((uint32_t)(q2 % a.b[2]) << 16) | ((uint32_t)(q2 / a.b[2]) << 24);
    sap_mem_get<S>(a.r0, a.vh, base + k, r[p]);
    sap_lds_put<S>(sap_lds, vt2, k, r[p]);
    if constexpr (XREG)
      if (a.first)
        x[p] = SapSite<S>{};
      else
        sap_mem_get<S>(a.x, a.vh, base + k, x[p]);
  }
  __syncthreads();
  // In each phase the thread's site index and coordinates pass through an
  // empty asm, so that the addresses derived from them are recomputed there
  // rather than held in registers across the step loop.
  for (int step = 0; step < a.steps; ++step) {
    // t_o = A_oo^-1 D_oe r on the block's odd sites
#pragma unroll
    for (int p = 0; p < SPT; ++p) {
      int k = p * nt + tid;
      __asm__ volatile("" : "+v"(k));
      cpx<float> acc[4][3], res[4][3];
      float f[24];
      uint32_t cp = coords[p];
      __asm__ volatile("" : "+v"(cp));
      sap_hops<S, RECON>(a, sap_lds, base, k, cp, 1, acc);
      sap_clover<S>(a.clov_inv_odd, a.vh, base + k, acc, res);
      sap_flat(res, f);
      sap_store<S>(f, w[p]);
      sap_opaque<S>(w[p]);
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();  // every read of r is done
#pragma unroll
    for (int p = 0; p < SPT; ++p) {
      int k = p * nt + tid;
      __asm__ volatile("" : "+v"(k));
      sap_lds_put<S>(sap_lds, vt2, k, w[p]);
    }
    __syncthreads();
    // q_e = A_ee r + coef D_eo t, and the segment sums of <q,r>, <q,q> over
    // the values as stored
#pragma unroll
    for (int p = 0; p < SPT; ++p) {
      int k = p * nt + tid;
      __asm__ volatile("" : "+v"(k));
      cpx<float> acc[4][3], res[4][3], xv[4][3];
      float rf[24], qf[24];
      uint32_t cp = coords[p];
      __asm__ volatile("" : "+v"(cp));
      sap_hops<S, RECON>(a, sap_lds, base, k, cp, 0, acc);
      __builtin_amdgcn_sched_barrier(0);
      sap_reals<S>(r[p], rf);
      sap_cpx(rf, xv);
      sap_clover<S>(a.clov_even, a.vh, base + k, xv, res);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) res[i][c] = res[i][c] + a.coef * acc[i][c];
      sap_flat(res, qf);
      sap_store<S>(qf, w[p]);
      if constexpr (is_fixed<S>()) {
        sap_reals<S>(w[p], qf);  // the values as stored
      } else {
#pragma unroll
        for (int j = 0; j < 24; ++j) qf[j] = quantize<S, float>(qf[j]);
      }
      double red[3] = {0, 0, 0};
#pragma unroll
      for (int j = 0; j < 12; ++j) {
        const double qr = qf[2 * j], qi = qf[2 * j + 1], rr = rf[2 * j], ri = rf[2 * j + 1];
        red[0] += qr * rr + qi * ri;
        red[1] += qr * ri - qi * rr;
        red[2] += qr * qr + qi * qi;
      }
      sap_opaque<S>(w[p]);
      sap_opaque<S>(r[p]);
#pragma unroll
      for (int j = 0; j < 3; ++j)
        for (int off = 32; off > 0; off >>= 1) red[j] += __shfl_xor(red[j], off, 64);
      if ((k & 63) == 0)
#pragma unroll
        for (int j = 0; j < 3; ++j) seg[3 * (k >> 6) + j] = red[j];
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();  // every read of t and every segment sum is done
    double qr = 0, qi = 0, qq = 0;
    for (int j = 0; j < (vt2 >> 6); ++j) {
      qr += seg[3 * j];
      qi += seg[3 * j + 1];
      qq += seg[3 * j + 2];
    }
    const float ar = qq > 0 ? (float)(a.omega * qr / qq) : 0.f, ai = qq > 0 ? (float)(a.omega * qi / qq) : 0.f;
    const bool last = step == a.steps - 1, zero_x = a.first && step == 0;
    // x += alpha r, r -= alpha q (the last step needs no new r)
#pragma unroll
    for (int p = 0; p < SPT; ++p) {
      int k = p * nt + tid;
      __asm__ volatile("" : "+v"(k));
      SapSite<S> xo{};
      if constexpr (XREG) {
        xo = x[p];
      } else {
        if (!zero_x) sap_mem_get<S>(a.x, a.vh, base + k, xo);
      }
      float rv[24], qv[24], xv[24];
      sap_reals<S>(r[p], rv);
      sap_reals<S>(w[p], qv);
      sap_reals<S>(xo, xv);
#pragma unroll
      for (int j = 0; j < 24; ++j) xv[j] = zero_x ? 0.f : xv[j];
#pragma unroll
      for (int j = 0; j < 12; ++j) {
        const float re = rv[2 * j], im = rv[2 * j + 1];
        xv[2 * j] += ar * re - ai * im;
        xv[2 * j + 1] += ar * im + ai * re;
        rv[2 * j] = re - (ar * qv[2 * j] - ai * qv[2 * j + 1]);
        rv[2 * j + 1] = im - (ar * qv[2 * j + 1] + ai * qv[2 * j]);
      }
      sap_store<S>(xv, xo);
      if (!last) sap_store<S>(rv, r[p]);
      sap_opaque<S>(r[p]);
      if constexpr (XREG) {
        x[p] = xo;
      } else {
        sap_mem_put<S>(a.x, a.vh, base + k, xo);
      }
      if (!last) sap_lds_put<S>(sap_lds, vt2, k, r[p]);
    }
    __syncthreads();  // the new r is in LDS; the segment sums are read
  }
  if constexpr (XREG) {
#pragma unroll
    for (int p = 0; p < SPT; ++p) sap_mem_put<S>(a.x, a.vh, base + p * nt + tid, x[p]);
  }
}

// ---------------------------------------------------------------------------
// The block kernel for FP16 storage. The form above was bound there not by memory
// but by the vector pipe and the latency of the links (one 8^4 block on each of 64
// CUs took 0.56 ms, on all 256 0.66 ms): a hop spent 130 vector instructions, of
// which the colour products are 36, and waited for its own loads. Here:
// - A hop's projection makes the two forms of h that the dot products take
//   directly, one packed addition each.
// - The two hops of a direction are one chain of dot products, d = u_f - u_b:
//   rows 0, 1 take 2 u_f - d and the other two +-d, instead of both hops apart.
// - A_ee r runs on dot products of stored values, A_oo^-1 on mixed-precision
//   fused multiply-adds (its input is not stored, so it stays FP32).
// - A cut hop reads a zero record from LDS instead of branching, so that loads can
//   run ahead: the links of a hop are loaded before the arithmetic of the hop
//   before it, half the clover words before the last hop.
// - LDS holds 48-byte records (three 16-byte reads; 16 lanes cover all banks
//   once) in SPT + 1 regions of blockDim sites. r is in regions 0 .. SPT - 1; t
//   of the first slab goes to the spare region, t of the second (once every read
//   of r is done) over r of the first, which is also in registers. r of the
//   second slab stays where it is: 12 registers less per lane.
// - The even half takes slabs and directions in reverse, so that it starts with
//   the links that the odd half read last, still in the L2 (1195 -> 1158 us).
// 2170 instead of 3480 vector instructions per pair of sites and MR step. 32^3 x 64,
// 8^4 blocks, 8 steps: 18 link reals 1323 -> 1103 us, 12 reals 1450 -> 908 us; on
// 64 CUs alone 0.56 -> 0.36 ms. Bound now by the links and clover words, which do
// not fit on chip: 7.3 GB read and 0.3 written (x of the second slab among them) at
// 6.7 TB/s, where a plain read of as many bytes per CU in a loop reaches 7.5 (8.0 in
// alternating order). x of both slabs in registers spills (1134 us).
constexpr int kSapHalfThreads = 1024;
constexpr int kNonTemporal = 2;  // of a buffer load
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Sites per thread (1 or 2), or 0 where the kernel does not apply.
static int sap_half_spt(int vt2) {
  if (vt2 % 64 || vt2 > 2 * kSapHalfThreads) return 0;
  if (vt2 <= kSapHalfThreads) return 1;
  return vt2 % 128 == 0 ? 2 : 0;
}
// bytes of dynamic LDS: the regions, the zero record, the segment sums
static size_t sap_half_lds_bytes(int vt2) {
  const int spt = sap_half_spt(vt2);
  return (size_t)(vt2 / spt) * (spt + 1) * 48 + 48 + (size_t)(vt2 / 64) * 3 * sizeof(double);
}

// A packed addition of chosen halves: lo = +-a.{A0} +- b.{B0}, hi = +-a.{A1} +- b.{B1}.
template <int A0, int A1, int B0, int B1, int NA0, int NA1, int NB0, int NB1>
__device__ __forceinline__ h2v pk_add(h2v a, h2v b) {
  h2v r;
  asm("v_pk_add_f16 %0, %1, %2 op_sel:[%3,%4] op_sel_hi:[%5,%6] neg_lo:[%7,%8] neg_hi:[%9,%10]"
      : "=v"(r)
      : "v"(a), "v"(b), "n"(A0), "n"(B0), "n"(A1), "n"(B1), "n"(NA0), "n"(NB0), "n"(NA1), "n"(NB1));
  return r;
}
// h = T (a + G b) or (IMAG) T (a + G i b), T and G +-1, in one of four forms:
// (h.x, h.y), conjugated (h.x, -h.y), swapped (h.y, h.x), turned (h.y, -h.x)
enum { kFormId, kFormConj, kFormSwap, kFormTurn };
template <int FORM, bool IMAG, int G, int T> __device__ __forceinline__ h2v half_row(h2v a, h2v b) {
  constexpr int c0 = FORM >= kFormSwap, c1 = 1 - c0;                 // component in lo, hi
  constexpr int n1 = FORM == kFormConj || FORM == kFormTurn;         // hi negated
  constexpr int nt = T < 0, ng = G < 0;
  constexpr int b0 = IMAG ? 1 - c0 : c0, b1 = IMAG ? 1 - c1 : c1;    // component 0 of i b is -b.y
  constexpr int m0 = nt ^ ng ^ (IMAG && c0 == 0), m1 = nt ^ ng ^ (IMAG && c1 == 0) ^ n1;
  return pk_add<c0, c1, b0, b1, nt, nt ^ n1, m0, m1>(a, b);
}

// u += T U h (FWD) or T U^+ h of the half spinor h of psi for a hop along MU
// (flip: sign bits for an antiperiodic boundary).
template <int MU, bool FWD, int T, int RECON>
__device__ __forceinline__ void half_hop_chain(const h2v (&s)[12], const uint32_t (&lw)[RECON / 2], uint32_t flip,
                                               bool flips, float (&u)[2][3][2]) {
  constexpr int g = FWD ? -1 : 1;
  constexpr bool im = MU == 0 || MU == 2;
  constexpr int r0 = MU < 2 ? 3 : 2, r1 = MU < 2 ? 2 : 3;            // partner rows of rows 0 and 1
  constexpr int g0 = MU == 3 ? g : -g, g1 = MU == 0 ? -g : g;
  constexpr int fx = FWD ? kFormConj : kFormId, fy = FWD ? kFormSwap : kFormTurn;
  h2v hx[2][3], hy[2][3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    hx[0][c] = half_row<fx, im, g0, T>(s[c], s[3 * r0 + c]);
    hy[0][c] = half_row<fy, im, g0, T>(s[c], s[3 * r0 + c]);
    hx[1][c] = half_row<fx, im, g1, T>(s[3 + c], s[3 * r1 + c]);
    hy[1][c] = half_row<fy, im, g1, T>(s[3 + c], s[3 * r1 + c]);
  }
  if (flips)
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        hx[k][c] = __builtin_bit_cast(h2v, __builtin_bit_cast(uint32_t, hx[k][c]) ^ flip);
        hy[k][c] = __builtin_bit_cast(h2v, __builtin_bit_cast(uint32_t, hy[k][c]) ^ flip);
      }
  h2v U[RECON / 2];
#pragma unroll
  for (int j = 0; j < RECON / 2; ++j) U[j] = __builtin_bit_cast(h2v, lw[j]);
  constexpr int NR = RECON == 18 ? 3 : 2, NI = FWD ? NR : 3, NJ = FWD ? 3 : NR;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const h2v a = FWD ? U[3 * i + j] : U[3 * j + i];
        u[k][i][0] = dot2(a, hx[k][j], u[k][i][0]);
        u[k][i][1] = dot2(a, hy[k][j], u[k][i][1]);
      }
  if constexpr (RECON == 12) {
    // third row conj(row 0 x row 1) and its products in FP32
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int k1 = (j + 1) % 3, l1 = (j + 2) % 3;
      const h2v a = U[k1], b = U[3 + l1], c = U[l1], d = U[3 + k1];
      const float re = dot2(a, h2v{b.x, -b.y}, dot2(-c, h2v{d.x, -d.y}, 0.f));
      const float ie = dot2(c, h2v{d.y, d.x}, dot2(-a, h2v{b.y, b.x}, 0.f));
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if constexpr (FWD) {
          const float hr = (float)hx[k][j].x, hn = (float)hx[k][j].y;  // h.x, -h.y
          u[k][2][0] = fmaf(ie, hn, fmaf(re, hr, u[k][2][0]));
          u[k][2][1] = fmaf(ie, hr, fmaf(-re, hn, u[k][2][1]));
        } else {
          const float hr = (float)hx[k][2].x, hi = (float)hx[k][2].y;
          u[k][j][0] = fmaf(ie, hi, fmaf(re, hr, u[k][j][0]));
          u[k][j][1] = fmaf(-ie, hr, fmaf(re, hi, u[k][j][1]));
        }
      }
    }
  }
}

// (x, y) rounded to nearest-even FP16, x in the low half
__device__ __forceinline__ uint32_t pack_half2(float x, float y) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{x, y}, h2v));
}

struct SapHalf {  // a lane's site of one slab in one phase
  uint32_t k;     // its index in the block
  uint32_t edge;  // bits: 0 x position of the row's even sites; per parity (1, 2 and 3, 4) x upper, lower edge;
                  // 5, 6 y upper, lower; 7, 8 z; 9, 10 t
};

// XREG: x of the first slab stays in registers (else it is read and written in memory each step).
// WRAP: the block spans the lattice along some direction.
template <int RECON, int SPT, bool XREG, bool WRAP>
__global__ void __launch_bounds__(kSapHalfThreads) sap_half_kernel(SapArgs<_Float16> a) {
  typedef _Float16 S;
  constexpr int LW = RECON / 2;
  extern __shared__ uint4 sap_rec[];
  char *lds = reinterpret_cast<char *>(sap_rec);
  const uint32_t nt = blockDim.x, tid = threadIdx.x, region = nt * 48, zero = (SPT + 1) * region;
  double *seg = reinterpret_cast<double *>(lds + zero + 48);  // [sites / 64][3]
  const int tile = a.g.colour >= 0 ? colour_site(a.g, blockIdx.x * a.vt2) / a.vt2 : (int)blockIdx.x;
  const int64_t base = (int64_t)tile * a.vt2, vh = a.vh;
  const int bxh = a.b[0] >> 1;
  const int dist[4] = {1, bxh, bxh * a.b[1], bxh * a.b[1] * a.b[2]};
  // the first slab's r (the second's stays in LDS); t is at offset toff, the second slab's wrapped to region 0
  SapSite<S> r0, w[SPT], x0;
  uint32_t edge[SPT];
  const uint32_t toff = SPT * region;

  auto put = [&](uint32_t off, const SapSite<S> &s) __attribute__((always_inline)) {
    uint4 *q = reinterpret_cast<uint4 *>(lds + off);
#pragma unroll
    for (int c = 0; c < 3; ++c) q[c] = make_uint4(s.p[4 * c], s.p[4 * c + 1], s.p[4 * c + 2], s.p[4 * c + 3]);
  };
  auto get = [&](uint32_t off, SapSite<S> &s) __attribute__((always_inline)) {
    const uint4 *q = reinterpret_cast<const uint4 *>(lds + off);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const uint4 v = q[c];
      s.p[4 * c] = v.x, s.p[4 * c + 1] = v.y, s.p[4 * c + 2] = v.z, s.p[4 * c + 3] = v.w;
    }
  };
#pragma unroll
  for (int p = 0; p < SPT; ++p) {
    const uint32_t k = p * nt + tid;
    const uint32_t q1 = k / bxh, xh = k - q1 * bxh, q2 = q1 / a.b[1], y = q1 - q2 * a.b[1], t = q2 / a.b[2],
                   z = q2 - t * a.b[2];
    const uint32_t o = (y + z + t) & 1, hi = xh == (uint32_t)bxh - 1, lo = xh == 0;
    edge[p] = o | ((o & hi) << 1) | (((1 - o) & lo) << 2) | (((1 - o) & hi) << 3) | ((o & lo) << 4) |
              ((uint32_t)(y + 1 == (uint32_t)a.b[1]) << 5) | ((uint32_t)(y == 0) << 6) |
              ((uint32_t)(z + 1 == (uint32_t)a.b[2]) << 7) | ((uint32_t)(z == 0) << 8) |
              ((uint32_t)(t + 1 == (uint32_t)a.b[3]) << 9) | ((uint32_t)(t == 0) << 10);
    SapSite<S> r;
    sap_mem_get<S>(a.r0, vh, base + k, r);
    put(k * 48, r);
    if (p == 0) r0 = r;
    if (XREG && p == 0) {
      x0 = SapSite<S>{};
      if (!a.first) sap_mem_get<S>(a.x, vh, base + k, x0);
    }
  }
  if (tid < 3) sap_rec[zero / 16 + tid] = make_uint4(0, 0, 0, 0);

  // Block index of the neighbour of a site of parity `par` along MU (the site's own where the hop is cut); cut and
  // wrapped are masks of all ones where it is. Masks, not conditions: with branches around the reads the compiler
  // moves arithmetic across them and spills.
  auto neighbour = [&](auto mu_, auto fwd_, int par, SapHalf s, uint32_t *cut, uint32_t *wrapped)
                       __attribute__((always_inline)) {
    if constexpr (WRAP) __asm__ volatile("" : "+v"(s.k), "+v"(s.edge));  // more to compute: not kept from hop to hop
    constexpr int MU = decltype(mu_)::value;
    constexpr bool FWD = decltype(fwd_)::value;
    const int bit = MU == 0 ? (par ? 3 : 1) + (FWD ? 0 : 1) : 3 + 2 * MU + (FWD ? 0 : 1);
    const uint32_t e = (uint32_t)((int)(s.edge << (31 - bit)) >> 31);
    uint32_t d;
    if constexpr (MU == 0) {
      const uint32_t o = (s.edge ^ par) & 1;  // 1: the site is at the odd x of its pair
      d = FWD ? o : o - 1;
    } else {
      d = FWD ? dist[MU] : -dist[MU];
    }
    if constexpr (WRAP) {
      const uint32_t wraps = (a.wrap >> MU) & 1 ? ~0u : 0u;
      const uint32_t span = MU == 0 ? bxh - 1 : (uint32_t)dist[MU] * (a.b[MU] - 1);
      *cut = e & ~wraps;
      *wrapped = e & wraps;
      return s.k + ((e & (FWD ? -span : span) & wraps) | (~e & d));
    } else {
      *cut = e;
      *wrapped = 0;
      return s.k + (~e & d);
    }
  };
  // Addresses in the packed fields: the chunk's base is uniform (scalar), the lane adds its block index. As
  // buffer loads, since the compiler forms per-lane 64-bit sums of global ones (500 instructions a step).
  auto uniform = [&](const S *f) __attribute__((always_inline)) {
    const char *q = reinterpret_cast<const char *>(f);
    __asm__ volatile("" : "+s"(q));  // recomputed at each use, not held in registers
    return q;
  };
  const int block_bytes = a.vt2 * 16;
  auto block_buffer = [&](const char *q) __attribute__((always_inline)) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(q), 0, block_bytes, 0x00027000);
  };
  // links of the hop along MU from s (parity par), as stored
  auto load_link = [&](auto mu_, auto fwd_, int par, const SapHalf &s, uint32_t (&l)[LW]) __attribute__((always_inline)) {
    constexpr int MU = decltype(mu_)::value;
    constexpr bool FWD = decltype(fwd_)::value;
    uint32_t cut, wrapped;
    const uint32_t n = FWD ? s.k : neighbour(mu_, fwd_, par, s, &cut, &wrapped);
    const char *f = uniform(a.gauge + (int64_t)(2 * MU + (FWD ? par : 1 - par)) * vh * RECON);
    if constexpr (RECON == 18) {
#pragma unroll
      for (int c = 0; c < 9; ++c)
        l[c] = __builtin_amdgcn_raw_buffer_load_b32(block_buffer(f + (c * vh + base) * 4), n * 4, 0, 0);
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(block_buffer(f + (c * vh + base) * 8), n * 8, 0, 0);
        l[2 * c] = v.x, l[2 * c + 1] = v.y;
      }
    }
  };
  uint32_t lk[2][LW];
  uint32_t cw[36];
  auto load_clover = [&](const S *f, uint32_t k, auto blk_) __attribute__((always_inline)) {
    constexpr int c0 = decltype(blk_)::value ? 5 : 0, c1 = decltype(blk_)::value ? 9 : 5;
    const char *q = uniform(f);
#pragma unroll
    for (int c = c0; c < c1; ++c) {
      const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(block_buffer(q + (c * vh + base) * 16), k * 16, 0, kNonTemporal);
#pragma unroll
      for (int j = 0; j < 4; ++j) cw[4 * c + j] = v[j];
    }
  };
  // one hop of parity par (source field at LDS offset 0, or t): u += T u_hop
  auto hop_chain = [&](auto mu_, auto fwd_, auto par_, const SapHalf &s, const uint32_t (&l)[LW], float (&u)[2][3][2])
                       __attribute__((always_inline)) {
    constexpr int MU = decltype(mu_)::value, par = decltype(par_)::value;
    constexpr bool FWD = decltype(fwd_)::value;
    uint32_t cut, wrapped;
    const uint32_t n = neighbour(mu_, fwd_, par, s, &cut, &wrapped);
    uint32_t off = n * 48;
    if constexpr (par == 0) {
      off += toff;
      if constexpr (SPT == 2) off = min(off, off - 3 * region);
    }
    off = (cut & zero) | (~cut & off);
    SapSite<S> nb;
    get(off, nb);
    h2v psi[12];
#pragma unroll
    for (int j = 0; j < 12; ++j) psi[j] = __builtin_bit_cast(h2v, nb.p[j]);
    half_hop_chain<MU, FWD, FWD ? 1 : -1, RECON>(psi, l, wrapped & (a.bc_t < 0 ? 0x80008000u : 0u), WRAP && MU == 3, u);
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  typedef std::integral_constant<int, 2> I2;
  typedef std::integral_constant<int, 3> I3;
  typedef std::true_type Fw;
  typedef std::false_type Bw;
  float acc[4][3][2];
  // both hops along MU; `next` issues the loads that follow those of the backward hop
  auto direction = [&](auto mu_, auto par_, auto first_, const SapHalf &s, auto next) __attribute__((always_inline)) {
    constexpr int MU = decltype(mu_)::value, par = decltype(par_)::value;
    constexpr bool first = decltype(first_)::value;
    float u[2][3][2] = {};
    load_link(mu_, Bw{}, par, s, lk[1]);
    __builtin_amdgcn_sched_barrier(0);
    hop_chain(mu_, Fw{}, par_, s, lk[0], u);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[i][c][h] = first ? 2.f * u[i][c][h] : fmaf(2.f, u[i][c][h], acc[i][c][h]);
    __builtin_amdgcn_sched_barrier(0);
    next();
    __builtin_amdgcn_sched_barrier(0);
    hop_chain(mu_, Bw{}, par_, s, lk[1], u);
    // u is u_f - u_b; the lower rows of a hop are g L(u), g = -1 forward, +1 backward: -L(u_f - u_b)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[i][c][h] -= u[i][c][h];
      auto lower = [&](int row, float re, float im) {
        acc[row][c][0] = first ? re : acc[row][c][0] + re;
        acc[row][c][1] = first ? im : acc[row][c][1] + im;
      };
      if constexpr (MU == 0) {  // rows 2, 3: i u1, i u0
        lower(2, u[1][c][1], -u[1][c][0]);
        lower(3, u[0][c][1], -u[0][c][0]);
      } else if constexpr (MU == 1) {  // u1, -u0
        lower(2, -u[1][c][0], -u[1][c][1]);
        lower(3, u[0][c][0], u[0][c][1]);
      } else if constexpr (MU == 2) {  // i u0, -i u1
        lower(2, u[0][c][1], -u[0][c][0]);
        lower(3, -u[1][c][1], u[1][c][0]);
      } else {  // u0, u1
        lower(2, -u[0][c][0], -u[0][c][1]);
        lower(3, -u[1][c][0], -u[1][c][1]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // acc = D restricted to the block at s (its first link is in lk[0]); the clover words' first block follows in cw
  auto hops = [&](auto par_, const SapHalf &s, const S *clov) __attribute__((always_inline)) {
    constexpr int par = decltype(par_)::value;
    if constexpr (par == 1) {
      direction(I0{}, par_, Fw{}, s, [&]() { load_link(I1{}, Fw{}, par, s, lk[0]); });
      direction(I1{}, par_, Bw{}, s, [&]() { load_link(I2{}, Fw{}, par, s, lk[0]); });
      direction(I2{}, par_, Bw{}, s, [&]() { load_link(I3{}, Fw{}, par, s, lk[0]); });
      direction(I3{}, par_, Bw{}, s, [&]() { load_clover(clov, s.k, I0{}); });
    } else {
      direction(I3{}, par_, Fw{}, s, [&]() { load_link(I2{}, Fw{}, par, s, lk[0]); });
      direction(I2{}, par_, Bw{}, s, [&]() { load_link(I1{}, Fw{}, par, s, lk[0]); });
      direction(I1{}, par_, Bw{}, s, [&]() { load_link(I0{}, Fw{}, par, s, lk[0]); });
      direction(I0{}, par_, Bw{}, s, [&]() { load_clover(clov, s.k, I0{}); });
    }
  };
  auto site = [&](int p) __attribute__((always_inline)) {
    SapHalf s{p * nt + tid, edge[p]};
    __asm__ volatile("" : "+v"(s.k), "+v"(s.edge));  // derived values are recomputed, not kept across phases
    return s;
  };
  auto half = [](uint32_t w, int i) { return __builtin_bit_cast(h2v, w)[i]; };
  auto opaque = [](SapSite<S> &s) __attribute__((always_inline)) { sap_opaque<S>(s); };

  load_link(I0{}, Fw{}, 1, site(0), lk[0]);
  __syncthreads();
  for (int step = 0; step < a.steps; ++step) {
    // t_o = A_oo^-1 D_oe r on the block's odd sites
#pragma unroll
    for (int p = 0; p < SPT; ++p) {
      const SapHalf s = site(p);
      hops(I1{}, s, a.clov_inv_odd);
      load_clover(a.clov_inv_odd, s.k, I1{});
      if (p + 1 < SPT)
        load_link(I0{}, Fw{}, 1, site(p + 1), lk[0]);
      else
        load_link(I3{}, Fw{}, 0, site(SPT - 1), lk[0]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float y[6][2];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          const float d = (float)half(cw[18 * b + i / 2], i & 1);
#pragma unroll
          for (int h = 0; h < 2; ++h) y[i][h] = d * acc[2 * b + i / 3][i % 3][h];
        }
        int o = 18 * b + 3;
#pragma unroll
        for (int i = 1; i < 6; ++i)
#pragma unroll
          for (int j = 0; j < i; ++j, ++o) {
            const float re = (float)half(cw[o], 0), im = (float)half(cw[o], 1);
            const float(&xi)[2] = acc[2 * b + i / 3][i % 3], (&xj)[2] = acc[2 * b + j / 3][j % 3];
            y[i][0] = fmaf(-im, xj[1], fmaf(re, xj[0], y[i][0]));
            y[i][1] = fmaf(im, xj[0], fmaf(re, xj[1], y[i][1]));
            y[j][0] = fmaf(im, xi[1], fmaf(re, xi[0], y[j][0]));
            y[j][1] = fmaf(-im, xi[0], fmaf(re, xi[1], y[j][1]));
          }
#pragma unroll
        for (int i = 0; i < 6; ++i) w[p].p[6 * b + i] = pack_half2(y[i][0], y[i][1]);
      }
      opaque(w[p]);
      __builtin_amdgcn_sched_barrier(0);
      if (p == 0) put(toff + s.k * 48, w[0]);
    }
    if constexpr (SPT == 2) {
      __syncthreads();  // every read of r is done
      put(tid * 48, w[1]);
    }
    __syncthreads();
    // q_e = A_ee r + coef D_eo t, and the segment sums of <q,r>, <q,q> over the values as stored
#pragma unroll
    for (int p = SPT - 1; p >= 0; --p) {
      const SapHalf s = site(p);
      hops(I0{}, s, a.clov_even);
      load_clover(a.clov_even, s.k, I1{});
      if (p > 0)
        load_link(I3{}, Fw{}, 0, site(p - 1), lk[0]);
      else
        load_link(I0{}, Fw{}, 1, site(0), lk[0]);
      __builtin_amdgcn_sched_barrier(0);
      SapSite<S> r;
      if (p == 0)
        r = r0;
      else
        get(s.k * 48, r);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float y[6][2];
        h2v xv[6], xs[6];  // as stored, and swapped
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          const uint32_t v = r.p[6 * b + i];
          xv[i] = __builtin_bit_cast(h2v, v);
          xs[i] = __builtin_bit_cast(h2v, (v >> 16) | (v << 16));
          const float d = (float)half(cw[18 * b + i / 2], i & 1);
#pragma unroll
          for (int h = 0; h < 2; ++h)
            y[i][h] = fmaf(d, (float)half(v, h), (float)a.coef * acc[2 * b + i / 3][i % 3][h]);
        }
        int o = 18 * b + 3;
#pragma unroll
        for (int i = 1; i < 6; ++i)
#pragma unroll
          for (int j = 0; j < i; ++j, ++o) {
            const h2v m = __builtin_bit_cast(h2v, cw[o]), mc = __builtin_bit_cast(h2v, cw[o] ^ 0x80000000u);
            y[i][0] = dot2(mc, xv[j], y[i][0]);
            y[i][1] = dot2(m, xs[j], y[i][1]);
            y[j][0] = dot2(m, xv[i], y[j][0]);
            y[j][1] = dot2(mc, xs[i], y[j][1]);
          }
#pragma unroll
        for (int i = 0; i < 6; ++i) w[p].p[6 * b + i] = pack_half2(y[i][0], y[i][1]);
      }
      opaque(w[p]);
      __builtin_amdgcn_sched_barrier(0);
      double red[3] = {0, 0, 0};
#pragma unroll
      for (int j = 0; j < 12; ++j) {
        const double qr = (float)half(w[p].p[j], 0), qi = (float)half(w[p].p[j], 1), rr = (float)half(r.p[j], 0),
                     ri = (float)half(r.p[j], 1);
        red[0] = fma(qi, ri, fma(qr, rr, red[0]));
        red[1] = fma(-qi, rr, fma(qr, ri, red[1]));
        red[2] = fma(qi, qi, fma(qr, qr, red[2]));
      }
#pragma unroll
      for (int j = 0; j < 3; ++j)
        for (int off = 32; off > 0; off >>= 1) red[j] += __shfl_xor(red[j], off, 64);
      if ((tid & 63) == 0)
#pragma unroll
        for (int j = 0; j < 3; ++j) seg[3 * (s.k >> 6) + j] = red[j];
      __builtin_amdgcn_sched_barrier(0);
    }
    const bool last = step == a.steps - 1, zero_x = a.first && step == 0;
    SapSite<S> xm[SPT];
#pragma unroll
    for (int p = XREG; p < SPT; ++p) {
      xm[p] = SapSite<S>{};
      if (!zero_x) sap_mem_get<S>(a.x, vh, base + site(p).k, xm[p]);
    }
    __syncthreads();  // every read of t and every segment sum is done
    double qr = 0, qi = 0, qq = 0;
#pragma unroll 8
    for (int j = 0; j < (a.vt2 >> 6); ++j) {
      qr += seg[3 * j];
      qi += seg[3 * j + 1];
      qq += seg[3 * j + 2];
    }
    const float ar = qq > 0 ? (float)(a.omega * qr / qq) : 0.f, ai = qq > 0 ? (float)(a.omega * qi / qq) : 0.f;
    // x += alpha r, r -= alpha q (the last step needs no new r)
#pragma unroll
    for (int p = 0; p < SPT; ++p) {
      const uint32_t k = site(p).k;
      SapSite<S> &xo = XREG && p == 0 ? x0 : xm[p];
      SapSite<S> r;
      if (p == 0)
        r = r0;
      else
        get(k * 48, r);
      auto cmadd = [&](uint32_t c, float fr, float fi, uint32_t v) __attribute__((always_inline)) {  // c + f v
        const float vr = (float)half(v, 0), vi = (float)half(v, 1);
        const _Float16 re = (_Float16)fmaf(-fi, vi, fmaf(fr, vr, (float)half(c, 0)));
        const _Float16 im = (_Float16)fmaf(fi, vr, fmaf(fr, vi, (float)half(c, 1)));
        return pack16<S>(re, im);
      };
#pragma unroll
      for (int j = 0; j < 12; ++j) xo.p[j] = cmadd(xo.p[j], ar, ai, r.p[j]);
      if (!XREG || p > 0) sap_mem_put<S>(a.x, vh, base + k, xo);
      if (!last) {
#pragma unroll
        for (int j = 0; j < 12; ++j) r.p[j] = cmadd(r.p[j], -ar, -ai, w[p].p[j]);
        opaque(r);
        put(k * 48, r);
        if (p == 0) r0 = r;
      }
    }
    __syncthreads();  // the new r is in LDS; the segment sums are read
  }
  if constexpr (XREG) sap_mem_put<S>(a.x, vh, base + tid, x0);
}

// Sites per thread of the block-resident form for blocks of vt2 sites per
// parity (0: the form does not apply).
int sap_block_spt(int vt2) {
  if (vt2 % 64 || vt2 > kSapMaxSites) return 0;
  for (int spt : {1, 2, 4})
    if (vt2 / spt <= 512 && vt2 % (64 * spt) == 0) return spt;
  return 0;
}

// The wide launch: twice the threads (up to 1024) with half the sites each,
// where a block has at least two sites per thread of the 512-thread launch.
bool sap_block_wide_fits(int vt2) { return sap_block_spt(vt2) >= 2; }

template <typename S> static SapArgs<S> sap_args(const SapLaunch &l) {
  SapArgs<S> a;
  a.x = (S *)l.x;
  a.r0 = (const S *)l.r0;
  a.gauge = (const S *)l.gauge;
  a.clov_inv_odd = (const S *)l.clov_inv_odd;
  a.clov_even = (const S *)l.clov_even;
  a.g = l.g;
  a.vh = l.g.Vh;
  a.vt2 = l.g.Vt2;
  a.wrap = 0;
  for (int m = 0; m < 4; ++m) {
    a.b[m] = l.g.B[m];
    if (l.g.B[m] == l.g.L[m]) a.wrap |= 1 << m;
  }
  a.bc_t = l.g.bc_t;
  a.coef = (float)l.coef;
  a.omega = l.omega;
  a.steps = l.steps;
  a.first = l.first;
  return a;
}

template <typename S, int RECON, int SPT, bool XREG, int NT>
static hipError_t launch_sap4(const SapLaunch &l, hipStream_t st) {
  const SapArgs<S> a = sap_args<S>(l);
  const size_t lds = sap_lds_bytes(l.g.Vt2, is_fixed<S>());
  static bool attr_set = false;  // per instantiation
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&sap_block_kernel<S, RECON, SPT, XREG, NT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)sap_lds_bytes(kSapMaxSites, is_fixed<S>()));
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int nblocks = launch_sites(l.g) / l.g.Vt2;
  hipLaunchKernelGGL((sap_block_kernel<S, RECON, SPT, XREG, NT>), dim3(nblocks), dim3(l.g.Vt2 / SPT), lds, st, a);
  return hipGetLastError();
}

template <typename S, int RECON, int SPT, int NT>
static hipError_t launch_sap3(const SapLaunch &l, hipStream_t st) {
  return l.xreg ? launch_sap4<S, RECON, SPT, true, NT>(l, st) : launch_sap4<S, RECON, SPT, false, NT>(l, st);
}

template <typename S, int RECON>
static hipError_t launch_sap2(const SapLaunch &l, hipStream_t st) {
  const int spt = sap_block_spt(l.g.Vt2);
  if (l.wide) {
    switch (spt) {
      case 2: return launch_sap3<S, RECON, 1, 1024>(l, st);
      case 4: return launch_sap3<S, RECON, 2, 1024>(l, st);
    }
    return hipErrorInvalidValue;
  }
  switch (spt) {
    case 1: return launch_sap3<S, RECON, 1, 512>(l, st);
    case 2: return launch_sap3<S, RECON, 2, 512>(l, st);
    case 4: return launch_sap3<S, RECON, 4, 512>(l, st);
  }
  return hipErrorInvalidValue;
}

template <int RECON, int SPT, bool XREG, bool WRAP>
static hipError_t launch_half3(const SapArgs<_Float16> &a, int nblocks, hipStream_t st) {
  static bool attr_set = false;  // per instantiation
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&sap_half_kernel<RECON, SPT, XREG, WRAP>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)sap_half_lds_bytes(SPT * kSapHalfThreads));
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((sap_half_kernel<RECON, SPT, XREG, WRAP>), dim3(nblocks), dim3(a.vt2 / SPT),
                     sap_half_lds_bytes(a.vt2), st, a);
  return hipGetLastError();
}

template <int RECON, int SPT>
static hipError_t launch_half2(const SapArgs<_Float16> &a, int nblocks, bool xreg, hipStream_t st) {
  if (a.wrap) return xreg ? launch_half3<RECON, SPT, true, true>(a, nblocks, st) : launch_half3<RECON, SPT, false, true>(a, nblocks, st);
  return xreg ? launch_half3<RECON, SPT, true, false>(a, nblocks, st) : launch_half3<RECON, SPT, false, false>(a, nblocks, st);
}

template <int RECON> static hipError_t launch_half1(const SapLaunch &l, hipStream_t st) {
  const SapArgs<_Float16> a = sap_args<_Float16>(l);
  const int nblocks = launch_sites(l.g) / l.g.Vt2;
  switch (sap_half_spt(l.g.Vt2)) {
    case 1: return launch_half2<RECON, 1>(a, nblocks, l.xreg, st);
    case 2: return launch_half2<RECON, 2>(a, nblocks, l.xreg, st);
  }
  return hipErrorInvalidValue;
}

template <typename S>
static hipError_t launch_sap1(const SapLaunch &l, hipStream_t st) {
  switch (l.recon) {
    case 18: return launch_sap2<S, 18>(l, st);
    case 12: return launch_sap2<S, 12>(l, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_sap_block(const SapLaunch &l, hipStream_t st) {
  for (int m = 0; m < 4; ++m)  // blocks are the tiles; coordinates fit 8 bits
    if (l.g.cut[m] != l.g.B[m] || l.g.B[m] > 256) return hipErrorInvalidValue;
  if (l.steps < 1 || !sap_block_spt(l.g.Vt2)) return hipErrorInvalidValue;
  if (l.g.colour >= 0 && (l.g.NT[0] & 1)) return hipErrorInvalidValue;
  if (l.g.Vh == 0) return hipSuccess;
  switch (l.prec) {
    case LQCD_F16: return l.recon == 18 ? launch_half1<18>(l, st) : l.recon == 12 ? launch_half1<12>(l, st) : hipErrorInvalidValue;
    case LQCD_BF16: return launch_sap1<bf16>(l, st);
    case LQCD_HALF: return launch_sap1<fx16>(l, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lqcd
