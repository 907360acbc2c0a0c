// Setup kernels: packing between the natural FP64 exchange format and the
// packed tiled layout, SU(3) link compression, the long links of eq. (3) and
// the clover field of eq. (2) with its per-site inverse.
#include "lqcd_internal.h"

namespace lqcd {

__device__ __forceinline__ int64_t natural_index(const Geom &g, const int X[4]) {
  return X[0] + (int64_t)g.L[0] * (X[1] + (int64_t)g.L[1] * (X[2] + (int64_t)g.L[2] * X[3]));
}

__device__ __forceinline__ void site_global(const Geom &g, const Site &x, int X[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) X[m] = x.t[m] * g.B[m] + x.l[m];
}

// ---------------------------------------------------------------------------
// spinors

// nrhs natural fields (consecutive, V sites each) <-> one packed field in the
// multi-source layout (rhs_index: blocks of rhs_group(nrhs) sources).
template <typename S, int NSP>
__global__ void __launch_bounds__(256) spinor_import_kernel(Geom g, S *packed, const double *nat, int parity,
                                                            int nrhs) {
  const int pidx = blockIdx.x * blockDim.x + threadIdx.x;
  if (pidx >= g.Vh * nrhs) return;
  const int R = rhs_group(nrhs), q = pidx / R, blk = q / g.Vh, s = q - blk * g.Vh, r = blk * R + pidx % R;
  const Site x = decode_site(g, s, parity);
  int X[4];
  site_global(g, x, X);
  const int64_t V = 2 * (int64_t)g.Vh;
  const double *src = nat + NSP * (r * V + natural_index(g, X));
  double v[NSP];
#pragma unroll
  for (int k = 0; k < NSP; ++k) v[k] = src[k];
  store_spinor_reals<S, NSP, double>(packed, (int64_t)g.Vh * nrhs, pidx, v);
}

template <typename S, int NSP>
__global__ void __launch_bounds__(256) spinor_export_kernel(Geom g, double *nat, const S *packed, int parity,
                                                            int nrhs) {
  const int pidx = blockIdx.x * blockDim.x + threadIdx.x;
  if (pidx >= g.Vh * nrhs) return;
  const int R = rhs_group(nrhs), q = pidx / R, blk = q / g.Vh, s = q - blk * g.Vh, r = blk * R + pidx % R;
  const Site x = decode_site(g, s, parity);
  int X[4];
  site_global(g, x, X);
  double v[NSP];
  load_spinor_reals<S, NSP, double>(packed, (int64_t)g.Vh * nrhs, pidx, v);
  const int64_t V = 2 * (int64_t)g.Vh;
  double *dst = nat + NSP * (r * V + natural_index(g, X));
#pragma unroll
  for (int k = 0; k < NSP; ++k) dst[k] = v[k];
}

// out = scale * in between two tiled layouts of the same lattice (one parity
// block each, nrhs sources in the multi-source layout), any precisions: one
// thread per output (site, source), which finds its site in the input layout.
template <typename So, typename Si, int NSP>
__global__ void __launch_bounds__(256) spinor_relayout_kernel(Geom go, So *out, Geom gi, const Si *in, int parity,
                                                              int nrhs, double scale) {
  const int64_t pidx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t vh = go.Vh;
  if (pidx >= vh * nrhs) return;
  const int R = rhs_group(nrhs);
  const int64_t q = pidx / R, blk = q / vh;
  const int s = (int)(q - blk * vh), r = (int)(blk * R + pidx % R);
  int X[4], t[4], l[4];
  site_global(go, decode_site(go, s, parity), X);
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    t[m] = X[m] / gi.B[m];
    l[m] = X[m] - t[m] * gi.B[m];
  }
  const int si = encode_site(gi, t, l);
  double v[NSP];
  load_spinor_reals<Si, NSP, double>(in, vh * nrhs, rhs_index(r, si, vh, R), v);
#pragma unroll
  for (int k = 0; k < NSP; ++k) v[k] *= scale;
  store_spinor_reals<So, NSP, double>(out, vh * nrhs, pidx, v);
}

template <typename So, int NSP>
static hipError_t relayout_in(const Geom &go, So *out, const Geom &gi, int pin, const void *in, int parity, int nrhs,
                              double scale, hipStream_t st) {
  const int bt = 256;
  const int nwg = (int)(((int64_t)go.Vh * nrhs + bt - 1) / bt);
  switch (pin) {
#define CASE(P)                                                                                                     \
  case P:                                                                                                           \
    hipLaunchKernelGGL((spinor_relayout_kernel<So, Prec<P>::S, NSP>), dim3(nwg), dim3(bt), 0, st, go, out, gi,      \
                       (const Prec<P>::S *)in, parity, nrhs, scale);                                                \
    return hipGetLastError();
    CASE(LQCD_F64)
    CASE(LQCD_F32)
    CASE(LQCD_F16)
    CASE(LQCD_BF16)
    CASE(LQCD_HALF)
#undef CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_spinor_relayout(const Geom &go, int pout, void *out, const Geom &gi, int pin, const void *in, int nsp,
                                  int parity, int nrhs, double scale, hipStream_t st) {
  if (go.Vh == 0) return hipSuccess;
  switch (pout) {
#define CASE(P)                                                                                                     \
  case P:                                                                                                           \
    return nsp == 24 ? relayout_in<Prec<P>::S, 24>(go, (Prec<P>::S *)out, gi, pin, in, parity, nrhs, scale, st)    \
                     : relayout_in<Prec<P>::S, 6>(go, (Prec<P>::S *)out, gi, pin, in, parity, nrhs, scale, st);
    CASE(LQCD_F64)
    CASE(LQCD_F32)
    CASE(LQCD_F16)
    CASE(LQCD_BF16)
    CASE(LQCD_HALF)
#undef CASE
  }
  return hipErrorInvalidValue;
}

template <int NSP>
static hipError_t spinor_io(const Geom &g, int prec, void *packed, double *natural, int parity, int nrhs, bool imp,
                            hipStream_t st) {
  const int bt = 256, nwg = (int)(((int64_t)g.Vh * nrhs + bt - 1) / bt);
  switch (prec) {
#define CASE(P)                                                                                               \
  case P:                                                                                                     \
    if (imp)                                                                                                  \
      hipLaunchKernelGGL((spinor_import_kernel<Prec<P>::S, NSP>), dim3(nwg), dim3(bt), 0, st, g,              \
                         (Prec<P>::S *)packed, (const double *)natural, parity, nrhs);                         \
    else                                                                                                      \
      hipLaunchKernelGGL((spinor_export_kernel<Prec<P>::S, NSP>), dim3(nwg), dim3(bt), 0, st, g, natural,     \
                         (const Prec<P>::S *)packed, parity, nrhs);                                           \
    return hipGetLastError();
    CASE(LQCD_F64)
    CASE(LQCD_F32)
    CASE(LQCD_F16)
    CASE(LQCD_BF16)
    CASE(LQCD_HALF)
#undef CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_spinor_import(const Geom &g, int prec, int nsp, void *packed, const double *natural, int parity,
                                int nrhs, hipStream_t st) {
  if (g.Vh == 0) return hipSuccess;
  return nsp == 24 ? spinor_io<24>(g, prec, packed, (double *)natural, parity, nrhs, true, st)
                   : spinor_io<6>(g, prec, packed, (double *)natural, parity, nrhs, true, st);
}

hipError_t launch_spinor_export(const Geom &g, int prec, int nsp, double *natural, const void *packed, int parity,
                                int nrhs, hipStream_t st) {
  if (g.Vh == 0) return hipSuccess;
  return nsp == 24 ? spinor_io<24>(g, prec, (void *)packed, natural, parity, nrhs, false, st)
                   : spinor_io<6>(g, prec, (void *)packed, natural, parity, nrhs, false, st);
}

// ---------------------------------------------------------------------------
// links

struct DLink {
  double re[3][3], im[3][3];
};

__device__ __forceinline__ DLink nat_link(const Geom &g, const double *nat, const int X[4], int mu) {
  const double *p = nat + 18 * (4 * natural_index(g, X) + mu);
  DLink u;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      u.re[i][j] = p[6 * i + 2 * j];
      u.im[i][j] = p[6 * i + 2 * j + 1];
    }
  return u;
}

// c = a * b, each optionally conjugate-transposed
__device__ __forceinline__ DLink dmul(const DLink &a, bool da, const DLink &b, bool db) {
  DLink c;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      double sr = 0, si = 0;
      for (int k = 0; k < 3; ++k) {
        const double ar = da ? a.re[k][i] : a.re[i][k], ai = da ? -a.im[k][i] : a.im[i][k];
        const double br = db ? b.re[j][k] : b.re[k][j], bi = db ? -b.im[j][k] : b.im[k][j];
        sr += ar * br - ai * bi;
        si += ar * bi + ai * br;
      }
      c.re[i][j] = sr;
      c.im[i][j] = si;
    }
  return c;
}

__device__ __forceinline__ void shift(const Geom &g, const int X[4], int mu, int step, int Y[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) Y[m] = X[m];
  Y[mu] = ((X[mu] + step) % g.L[mu] + g.L[mu]) % g.L[mu];
}

template <typename S, int RECON>
__device__ __forceinline__ void pack_link(S *base, int64_t vh, int s, const DLink &u) {
  double v[RECON];
  if constexpr (RECON == 8) {
    v[0] = u.re[0][1]; v[1] = u.im[0][1];
    v[2] = u.re[0][2]; v[3] = u.im[0][2];
    v[4] = u.re[1][0]; v[5] = u.im[1][0];
    v[6] = atan2(u.im[0][0], u.re[0][0]);
    v[7] = atan2(u.im[2][0], u.re[2][0]);
  } else {
#pragma unroll
    for (int k = 0; k < RECON / 2; ++k) {
      v[2 * k] = u.re[k / 3][k % 3];
      v[2 * k + 1] = u.im[k / 3][k % 3];
    }
  }
  store_site<S, RECON, double>(base, vh, s, v);
}

// One thread per (site of one parity); loops over the 4 directions.
// form_long: pack the 3-hop product U_mu(x) U_mu(x+mu) U_mu(x+2mu).
template <typename S, int RECON>
__global__ void __launch_bounds__(128) gauge_import_kernel(Geom g, S *packed, const double *nat, int form_long) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= 2 * g.Vh) return;
  const int parity = idx >= g.Vh ? 1 : 0;
  const int s = idx - parity * g.Vh;
  const Site x = decode_site(g, s, parity);
  int X[4];
  site_global(g, x, X);
  for (int mu = 0; mu < 4; ++mu) {
    DLink u = nat_link(g, nat, X, mu);
    if (form_long) {
      int Y[4], Z[4];
      shift(g, X, mu, 1, Y);
      shift(g, X, mu, 2, Z);
      u = dmul(dmul(u, false, nat_link(g, nat, Y, mu), false), false, nat_link(g, nat, Z, mu), false);
    }
    pack_link<S, RECON>(packed + (int64_t)(2 * mu + parity) * g.Vh * RECON, g.Vh, s, u);
  }
}

template <int RECON>
static hipError_t gauge_io(const Geom &g, int prec, void *packed, const double *nat, int form_long, hipStream_t st) {
  const int bt = 128, nwg = (2 * g.Vh + bt - 1) / bt;
  switch (prec) {
#define CASE(P)                                                                                                   \
  case P:                                                                                                         \
    hipLaunchKernelGGL((gauge_import_kernel<Prec<P>::S, RECON>), dim3(nwg), dim3(bt), 0, st, g,                  \
                       (Prec<P>::S *)packed, nat, form_long);                                                     \
    return hipGetLastError();
    CASE(LQCD_F64)
    CASE(LQCD_F32)
    CASE(LQCD_F16)
    CASE(LQCD_BF16)
    CASE(LQCD_HALF)
#undef CASE
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gauge_import(const Geom &g, int prec, int recon, void *packed, const double *natural, int form_long,
                               hipStream_t st) {
  if (g.Vh == 0) return hipSuccess;
  switch (recon) {
    case 18: return gauge_io<18>(g, prec, packed, natural, form_long, st);
    case 12: return gauge_io<12>(g, prec, packed, natural, form_long, st);
    case 8: return gauge_io<8>(g, prec, packed, natural, form_long, st);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// clover term
//
// F_munu = (Q_munu - Q_munu^+)/8 from the four clover leaves (Q_numu is the
// adjoint of Q_munu). In the chiral basis sigma_munu is block diagonal:
// sigma_jk = -eps_jkl diag(s_l, s_l) for spatial j,k and
// sigma_k4 = diag(s_k, -s_k), so per chirality block
//   sum_{mu<nu} sigma F = s_1 (+-F_14 - F_23) + s_2 (F_13 +- F_24) + s_3 (+-F_34 - F_12)
// (upper signs for spins 0,1). Each block, 1 + i kappa c_sw (...), is a
// Hermitian 6x6 stored as 6 real diagonal entries plus the lower triangle.

// A parity block of the clover field: 72 reals per site, and for fixed-point
// storage the FP32 site norms after them (two code slots per norm).
template <typename S> __host__ __device__ constexpr int64_t clover_block_elems(int64_t vh) {
  return vh * 72 + (is_fixed<S>() ? 2 * vh : 0);
}

// One chirality block b of a site's clover field (reals 36 b .. 36 b + 35), in
// pieces of at most 4 reals (a 16-bit chunk of 8 may belong to both blocks).
// Fixed point: codes of v times the reciprocal of the site norm.
template <typename S>
__device__ __forceinline__ void store_clover_block(S *base, int64_t vh, int s, int b, const double (&v)[36],
                                                   float inv) {
  constexpr int CH = chunk_reals<S, 72>(), PW = CH < 4 ? CH : 4;
#pragma unroll
  for (int k = 0; k < 36; k += PW) {
    Chunk<S, PW> w;
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      if constexpr (is_fixed<S>())
        w.v[j] = Store<S>::from((float)v[k + j] * inv);
      else
        w.v[j] = Store<S>::from(v[k + j]);
    }
    const int r = 36 * b + k;
    *reinterpret_cast<Chunk<S, PW> *>(base + ((int64_t)(r / CH) * vh + s) * CH + r % CH) = w;
  }
}

typedef double d2v __attribute__((ext_vector_type(2)));

struct DRow {
  double re[3], im[3];
};

// acc += or -= row-streamed products of 3x3 complex matrices; r is one row of
// the streamed operand.
template <bool SUB> __device__ __forceinline__ void dmac(double &re, double &im, double ar, double ai, double br, double bi) {
  const double xr = SUB ? -ar : ar, xi = SUB ? -ai : ai;
  re = fma(xr, br, re);
  re = fma(-xi, bi, re);
  im = fma(xr, bi, im);
  im = fma(xi, br, im);
}

// The clover field, 64 sites and two waves per workgroup. The sites are taken in
// columns of (Lx, ey, ez) sites that run along t, so that a link's neighbours
// along t are read soon after it: an XCD has 8192 sites in flight, and in the
// natural order every link came from beyond its L2 several times (21.7 GB
// fetched at 32^3x64 for 1.2 GB of links; 3.0 ms, in columns 2.4 ms). Wave w forms F of the planes 3w .. 3w + 2, then the chirality
// block w of A and its inverse for the same sites. A wave stages one link of
// each of its sites at a time in its own part of LDS: the natural links are
// 144-byte pieces 576 bytes apart, which lanes read 16 bytes at a time in the
// order of the pieces (a load touches 7 links) and take back row by row; the
// next link's loads are in flight meanwhile. With
//   W = U_mu(x) [S - S'] + [T - T'] U_mu(x-mu),  (the second term first: only its 9 reals stay)
//   S  = U_nu(x+mu) (U_nu(x) U_mu(x+nu))^+,       S' = (U_mu(x-nu) U_nu(x+mu-nu))^+ U_nu(x-nu),
//   T  = U_nu(x) (U_nu(x-mu) U_mu(x-mu+nu))^+,    T' = (U_mu(x-mu-nu) U_nu(x-nu))^+ U_nu(x-mu-nu)
// W holds the leaves 1 and 2 and minus the adjoints of 4 and 3, so that
// F = (W - W^+) / 8 takes 10 products per plane instead of 12 (no unitarity
// used). Everything stays in registers: one thread per site with all six planes
// in local arrays moved 30-36 GB through scratch memory (4.4 ms at 32^3x64).
// What bounds it now is the L1: a 16-byte load of 144-byte pieces takes about 31
// tag lookups a wave instead of 16, 14 links per plane (about 1.3 ms).
constexpr int kCloverPlane = 9 * 64;                      // doubles: F of one plane (anti-Hermitian: 9 reals)
constexpr int kCloverWave = 2 * kCloverPlane + 64 * 18;   // two planes, then the staged links (later the third plane)

template <typename S>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2, 2)))
clover_build_kernel(Geom g, int ey, int ez, double kc, S *clov, S *clov_inv, const double *__restrict__ nat,
                    int *fail) {
  __shared__ __align__(16) double lds[2][kCloverWave];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int V = 2 * g.Vh;
  const int own = xcd_remap(blockIdx.x, gridDim.x) * 64 + lane;
  const bool valid = own < V;
  const int o = valid ? own : V - 1;
  int X[4];
  {
    const uint32_t lx = g.L[0], lt = g.L[3], nyc = g.L[1] / ey;
    uint32_t q = (uint32_t)o;
    X[0] = q % lx, q /= lx;
    X[1] = q % ey, q /= ey;
    X[2] = q % ez, q /= ez;
    X[3] = q % lt, q /= lt;
    X[1] += ey * (q % nyc);
    X[2] += ez * (q / nyc);
  }
  const int n = X[0] + g.L[0] * (X[1] + g.L[1] * (X[2] + g.L[2] * X[3]));
  // offsets of the neighbours in the natural order
  int fw[4], bw[4], stride = 1;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    fw[m] = X[m] + 1 == g.L[m] ? -(g.L[m] - 1) * stride : stride;
    bw[m] = X[m] == 0 ? (g.L[m] - 1) * stride : -stride;
    stride *= g.L[m];
  }
  double *F = lds[wave];
  d2v *stage = reinterpret_cast<d2v *>(F + 2 * kCloverPlane);
  d2v raw[9];
  auto load = [&](int site, int mu) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const int e = lane + 64 * k, j = e / 9;
      raw[k] = reinterpret_cast<const d2v *>(nat + 18 * (4 * (int64_t)__shfl(site, j, 64) + mu))[e - 9 * j];
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // publish the loaded link to its site's lane and start loading the next one
  auto put = [&](int next, int mu) __attribute__((always_inline)) {
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < 9; ++k) stage[lane + 64 * k] = raw[k];
    __builtin_amdgcn_wave_barrier();
    load(next, mu);
  };
  auto row = [&](int i) __attribute__((always_inline)) {
    DRow r;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const d2v z = stage[9 * lane + 3 * i + c];
      r.re[c] = z.x;
      r.im[c] = z.y;
    }
    return r;
  };
  // (the compiler may not move a product behind this point: left alone it puts
  // all of a plane's arithmetic behind all of its loads, and spills)
  auto pin = [&](DRow (&A)[3]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        __asm__ volatile("" : "+v"(A[i].re[c]));
        __asm__ volatile("" : "+v"(A[i].im[c]));
      }
  };
  auto whole = [&](DRow (&A)[3]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 3; ++i) A[i] = row(i);
    pin(A);
  };
  auto clear = [&](DRow (&A)[3]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) A[i].re[c] = A[i].im[c] = 0;
  };
  // C += A L, L the staged link
  auto mul_left = [&](DRow (&C)[3], const DRow (&A)[3]) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      __builtin_amdgcn_sched_barrier(0);
      const DRow r = row(k);
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) dmac<false>(C[i].re[j], C[i].im[j], A[i].re[k], A[i].im[k], r.re[j], r.im[j]);
    }
    pin(C);
  };
  // C = L A^+ (row i of L gives row i of C)
  auto mul_adj = [&](DRow (&C)[3], const DRow (&A)[3]) __attribute__((always_inline)) {
    clear(C);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      const DRow r = row(i);
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int k = 0; k < 3; ++k) dmac<false>(C[i].re[j], C[i].im[j], r.re[k], r.im[k], A[j].re[k], -A[j].im[k]);
    }
    pin(C);
  };
  // C -= A^+ L
  auto sub_adj_mul = [&](DRow (&C)[3], const DRow (&A)[3]) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      __builtin_amdgcn_sched_barrier(0);
      const DRow r = row(k);
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) dmac<true>(C[i].re[j], C[i].im[j], A[k].re[i], -A[k].im[i], r.re[j], r.im[j]);
    }
    pin(C);
  };
  // C = L A
  auto mul_right = [&](DRow (&C)[3], const DRow (&A)[3]) __attribute__((always_inline)) {
    clear(C);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      const DRow r = row(i);
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) dmac<false>(C[i].re[j], C[i].im[j], r.re[k], r.im[k], A[k].re[j], A[k].im[j]);
    }
    pin(C);
  };
  // planes 0..5: (x,y) (x,z) (x,t) (y,z) (y,t) (z,t)
  auto mu_of = [](int p) { return p < 3 ? 0 : (p < 5 ? 1 : 2); };
  auto nu_of = [](int p) { return p < 3 ? p + 1 : (p < 5 ? p - 1 : 3); };
  auto pick = [](const int (&d)[4], int m) { return m == 0 ? d[0] : m == 1 ? d[1] : m == 2 ? d[2] : d[3]; };
  load(n + pick(bw, mu_of(3 * wave)), nu_of(3 * wave));
#pragma unroll 1
  for (int pl = 0; pl < 3; ++pl) {
    const int p = 3 * wave + pl, pn = pl < 2 ? p + 1 : p;
    const int mu = mu_of(p), nu = nu_of(p);
    const int fm = pick(fw, mu), bm = pick(bw, mu), fn = pick(fw, nu), bn = pick(bw, nu);
    DRow P[3], Q[3], A[3];
    double f[9];
    // f += the 9 reals of (P - P^+) / 8: real parts of (0,1) (0,2) (1,2), imaginary parts of the lower triangle
    auto add_f = [&](bool first) __attribute__((always_inline)) {
      const double t[9] = {P[0].re[1] - P[1].re[0], P[0].re[2] - P[2].re[0], P[1].re[2] - P[2].re[1],
                           P[0].im[0] + P[0].im[0], P[1].im[0] + P[0].im[1], P[1].im[1] + P[1].im[1],
                           P[2].im[0] + P[0].im[2], P[2].im[1] + P[1].im[2], P[2].im[2] + P[2].im[2]};
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        f[k] = first ? 0.125 * t[k] : fma(0.125, t[k], f[k]);
        __asm__ volatile("" : "+v"(f[k]));
      }
    };
    put(n + bm + fn, mu);  // U_nu(x-mu)
    whole(P);
    put(n, nu);  // U_mu(x-mu+nu)
    clear(Q);
    mul_left(Q, P);
    put(n + bm + bn, mu);  // U_nu(x)
    mul_adj(A, Q);         // T
    put(n + bn, nu);       // U_mu(x-mu-nu)
    whole(P);
    put(n + bm + bn, nu);  // U_nu(x-nu)
    clear(Q);
    mul_left(Q, P);
    put(n + bm, mu);  // U_nu(x-mu-nu)
    sub_adj_mul(A, Q);  // T - T'
    put(n, nu);         // U_mu(x-mu)
    clear(P);
    mul_left(P, A);
    add_f(true);
    put(n + fn, mu);  // U_nu(x)
    whole(P);
    put(n + fm, nu);  // U_mu(x+nu)
    clear(Q);
    mul_left(Q, P);
    put(n + bn, mu);  // U_nu(x+mu)
    mul_adj(A, Q);    // S
    put(n + fm + bn, nu);  // U_mu(x-nu)
    whole(P);
    put(n + bn, nu);  // U_nu(x+mu-nu)
    clear(Q);
    mul_left(Q, P);
    put(n, mu);         // U_nu(x-nu)
    sub_adj_mul(A, Q);  // S - S'
    put(n + pick(bw, mu_of(pn)), nu_of(pn));  // U_mu(x); next: the first link of the next plane
    mul_right(P, A);
    add_f(false);
    __builtin_amdgcn_wave_barrier();
    // (the third plane takes the place of the staged links)
    double *o = F + pl * kCloverPlane + lane;
#pragma unroll
    for (int k = 0; k < 9; ++k) o[64 * k] = f[k];
  }
  __syncthreads();
  // block b of A = 1 + i kc [ s1 B1 + s2 B2 + s3 B3 ] on (spin-in-block, colour)
  const int b = wave;
  const double c = b == 0 ? 1.0 : -1.0;
  double B1[9], B2[9], B3[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    auto at = [&](int p) { return lds[p / 3][(p % 3) * kCloverPlane + k * 64 + lane]; };
    B1[k] = c * at(2) - at(3);
    B2[k] = at(1) + c * at(4);
    B3[k] = c * at(5) - at(0);
  }
  auto re = [](const double (&f)[9], int i, int j) {
    const double v = f[i + j - 1 < 0 ? 0 : i + j - 1];  // (0,1) 0, (0,2) 1, (1,2) 2
    return i == j ? 0.0 : (i < j ? v : -v);
  };
  auto im = [](const double (&f)[9], int i, int j) {
    return f[3 + (i > j ? i * (i + 1) / 2 + j : j * (j + 1) / 2 + i)];
  };
  // packed as stored: 6 diagonal entries, then the strictly lower triangle (re, im)
  double v[36];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    v[i] = 1.0 - kc * im(B3, i, i);
    v[3 + i] = 1.0 + kc * im(B3, i, i);
  }
  constexpr int kOff = 6;
  auto tri = [](int i, int j) { return kOff + i * (i - 1) + 2 * j; };
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      if (j < i) {  // (0,0): i kc B3; (1,1): -i kc B3
        v[tri(i, j)] = -kc * im(B3, i, j);
        v[tri(i, j) + 1] = kc * re(B3, i, j);
        v[tri(3 + i, 3 + j)] = kc * im(B3, i, j);
        v[tri(3 + i, 3 + j) + 1] = -kc * re(B3, i, j);
      }
      // (1,0): i kc (B1 + i B2)
      v[tri(3 + i, j)] = -kc * im(B1, i, j) - kc * re(B2, i, j);
      v[tri(3 + i, j) + 1] = kc * re(B1, i, j) - kc * im(B2, i, j);
    }
  const int t0 = (X[0] >> 1) / (g.B[0] >> 1), t1 = X[1] / g.B[1], t2 = X[2] / g.B[2], t3 = X[3] / g.B[3];
  const int tc[4] = {t0, t1, t2, t3};
  const int lc[4] = {X[0] - t0 * g.B[0], X[1] - t1 * g.B[1], X[2] - t2 * g.B[2], X[3] - t3 * g.B[3]};
  const int s = encode_site(g, tc, lc), parity = (X[0] + X[1] + X[2] + X[3]) & 1;
  double *xch = lds[0];  // site norms of the two blocks (fixed point)
  auto store = [&](S *field) __attribute__((always_inline)) {
    S *base = field + (int64_t)parity * clover_block_elems<S>(g.Vh);
    float inv = 1.f;
    if constexpr (is_fixed<S>()) {
      double m = 0;
#pragma unroll
      for (int k = 0; k < 36; ++k) m = fabs(v[k]) > m ? fabs(v[k]) : m;
      __syncthreads();  // F, or the norms of A, have been read
      xch[64 * b + lane] = m;
      __syncthreads();
      const double o = xch[64 * (1 - b) + lane];
      const float fm = (float)(o > m ? o : m);
      inv = fm > 0 ? 1.0f / fm : 0.0f;
      if (b == 0 && valid) site_norms<S, 72>(base, g.Vh)[s] = fm;
    }
    if (valid) store_clover_block<S>(base, g.Vh, s, b, v, inv);
  };
  store(clov);
  // Cholesky A = L L^+, in place (diagonal: 1 / L_jj)
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    double d = v[j];
#pragma unroll
    for (int k = 0; k < j; ++k) {
      d = fma(-v[tri(j, k)], v[tri(j, k)], d);
      d = fma(-v[tri(j, k) + 1], v[tri(j, k) + 1], d);
    }
    ok = ok && d > 0;
    v[j] = 1.0 / sqrt(d);
#pragma unroll
    for (int i = j + 1; i < 6; ++i) {
      double sr = v[tri(i, j)], si = v[tri(i, j) + 1];
#pragma unroll
      for (int k = 0; k < j; ++k)  // - L_ik conj(L_jk)
        dmac<true>(sr, si, v[tri(i, k)], v[tri(i, k) + 1], v[tri(j, k)], -v[tri(j, k) + 1]);
      v[tri(i, j)] = sr * v[j];
      v[tri(i, j) + 1] = si * v[j];
    }
  }
  if (!ok && valid) fail[0] = 1;
  // W = L^-1 in place, last row first: W_ij = -(1 / L_ii) sum_{j <= k < i} L_ik W_kj
#pragma unroll
  for (int i = 1; i < 6; ++i) {
    double wr[5], wi[5];
#pragma unroll
    for (int j = 0; j < i; ++j) {
      double sr = v[tri(i, j)] * v[j], si = v[tri(i, j) + 1] * v[j];
#pragma unroll
      for (int k = j + 1; k < i; ++k)
        dmac<false>(sr, si, v[tri(i, k)], v[tri(i, k) + 1], v[tri(k, j)], v[tri(k, j) + 1]);
      wr[j] = -sr * v[i];
      wi[j] = -si * v[i];
    }
#pragma unroll
    for (int j = 0; j < i; ++j) {
      v[tri(i, j)] = wr[j];
      v[tri(i, j) + 1] = wi[j];
    }
  }
  // A^-1 = W^+ W, in place: entry (i, j), i >= j, needs the rows k >= i, so
  // rows are finished from the top
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    double or_[6], oi[6];
#pragma unroll
    for (int j = 0; j <= i; ++j) {
      double sr = 0, si = 0;
#pragma unroll
      for (int k = i; k < 6; ++k) {  // conj(W_ki) W_kj
        const double ar = k == i ? v[i] : v[tri(k, i)], ai = k == i ? 0.0 : -v[tri(k, i) + 1];
        const double br = k == j ? v[j] : v[tri(k, j)], bi = k == j ? 0.0 : v[tri(k, j) + 1];
        dmac<false>(sr, si, ar, ai, br, bi);
      }
      or_[j] = sr;
      oi[j] = si;
    }
#pragma unroll
    for (int j = 0; j < i; ++j) {
      v[tri(i, j)] = or_[j];
      v[tri(i, j) + 1] = oi[j];
    }
    v[i] = or_[i];
  }
  store(clov_inv);
}

hipError_t launch_clover_build(const Geom &g, int prec, double kappa, double csw, void *clov, void *clov_inv,
                               const double *natural_gauge, int *d_fail, hipStream_t st) {
  if (g.Vh == 0) return hipSuccess;
  const int bt = 128, nwg = (2 * g.Vh + 63) / 64;  // 64 sites per workgroup of two waves
  const double kc = kappa * csw;
  // columns of 8 x 8 sites along y and z (of the largest even extent up to 8
  // that divides the lattice's)
  auto fit = [](int l) {
    int e = 8;
    while (l % e) e -= 2;
    return e;
  };
  const int ey = fit(g.L[1]), ez = fit(g.L[2]);
  switch (prec) {
#define CASE(P)                                                                                              \
  case P:                                                                                                    \
    hipLaunchKernelGGL((clover_build_kernel<Prec<P>::S>), dim3(nwg), dim3(bt), 0, st, g, ey, ez, kc,               \
                       (Prec<P>::S *)clov, (Prec<P>::S *)clov_inv, natural_gauge, d_fail);                  \
    return hipGetLastError();
    CASE(LQCD_F64)
    CASE(LQCD_F32)
    CASE(LQCD_F16)
    CASE(LQCD_BF16)
    CASE(LQCD_HALF)
#undef CASE
  }
  return hipErrorInvalidValue;
}

}  // namespace lqcd
