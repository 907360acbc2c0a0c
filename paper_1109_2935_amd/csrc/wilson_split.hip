// Wilson-clover kernels for launches with few sites: a site's eight hops run in
// eight waves.
//
// With one thread per site a launch of 2048 sites is 32 waves on 256 CUs and its
// time is one thread's chain of eight hops (load, project, multiply) and the
// clover product. Here a workgroup takes 64 points (site, source); wave w forms
// the half spinor of hop w for all of them (in order +x, -x, +y, ...) and leaves
// it in LDS, then six waves sum two spin-colour components each over the hops in
// that order and apply the epilogue, two rows of the clover product per wave.
// Every value is formed by the operations of the one-thread kernel in the same
// order, so that both give the same result bit for bit.
#include "lqcd_internal.h"
#include "wilson_device.h"

namespace lqcd {

constexpr int kSplitPoints = 64;
constexpr int kSplitThreads = 512;

// component (spin, colour) of hop MU's expansion: the row of the half spinor it
// takes and the factor, g the projection sign (expand_acc)
template <typename R>
__device__ __forceinline__ cpx<R> split_term(int mu, int sp, R g, const cpx<R> &u0, const cpx<R> &u1) {
  if (sp < 2) return sp == 0 ? u0 : u1;
  // rows 2, 3: x: (g i u1, g i u0), y: (g u1, -g u0), z: (g i u0, -g i u1), t: (g u0, g u1)
  const bool swap = mu < 2;
  const cpx<R> v = (sp == 2) == swap ? u1 : u0;
  const R f = (sp == 3 && (mu == 1 || mu == 2)) ? -g : g;
  return f * ((mu & 1) == 0 && mu < 3 ? times_i(v) : v);
}

template <int MU, int DIR, typename S, typename R, int RECON>
__device__ __forceinline__ void split_hop(const WArgs<S> &a, const Site &x, int s, int rhs, R sgn, bool valid, R *lds) {
  cpx<R> u[2][3];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int c = 0; c < 3; ++c) u[k][c] = mk<R>(0, 0);
  if (valid && hop_kept<MU>(a.g, x, DIR)) {
    HopIn<S, RECON> h;
    hop_fetch<MU, DIR, false, S, RECON>(a, x, s, rhs, h);
    hop_product<MU, DIR, S, R, RECON>(h, DIR > 0 ? -sgn : sgn, a.g.bc_t, u);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      lds[(6 * k + 2 * c) * kSplitPoints] = u[k][c].re;
      lds[(6 * k + 2 * c + 1) * kSplitPoints] = u[k][c].im;
    }
}

// One row of a chirality block: its diagonal entry and the other five entries in
// column order (those right of the diagonal as stored below it, to be conjugated)
template <typename R> struct CloverRow {
  R d;
  cpx<R> o[5];
};
template <typename S, typename R>
__device__ __forceinline__ void load_clover_row(const S *__restrict__ clov, int64_t vh, int s, int b, int i,
                                                CloverRow<R> &r) {
  constexpr int CH = chunk_reals<S, 72>();
  auto at = [&](int k) { return clov + ((int64_t)((36 * b + k) / CH) * vh + s) * CH + (36 * b + k) % CH; };
  r.d = to_real<R>(*at(i));
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const int j = m < i ? m : m + 1;            // column
    const int hi = j < i ? i : j, lo = j < i ? j : i;
    const Chunk<S, 2> v = *reinterpret_cast<const Chunk<S, 2> *>(at(6 + hi * (hi - 1) + 2 * lo));
    r.o[m] = mk<R>(to_real<R>(v.v[0]), to_real<R>(v.v[1]));
  }
}
template <typename R>
__device__ __forceinline__ cpx<R> clover_row_mul(const CloverRow<R> &r, int i, const cpx<R> (&x)[6]) {
  R xr = x[0].re, xi = x[0].im;
#pragma unroll
  for (int j = 1; j < 6; ++j) {
    xr = j == i ? x[j].re : xr;
    xi = j == i ? x[j].im : xi;
  }
  cpx<R> y = r.d * mk<R>(xr, xi);
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    // right of the diagonal: the conjugate of the stored entry
    const R ar = r.o[m].re, ai = m < i ? r.o[m].im : -r.o[m].im;
    const R br = m < i ? x[m].re : x[m + 1].re, bi = m < i ? x[m].im : x[m + 1].im;
    cmac(y, mk<R>(ar, ai), mk<R>(br, bi));
  }
  return y;
}

// Sum of the n partials of a device-driven CG step, the same in every thread.
__device__ __forceinline__ double cg_total(const double *part, int n) {
  double t = 0;
  for (int j = threadIdx.x & 63; j < n; j += 64) t += part[j];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
  return t;
}

// CG: 0 none; 1: q = the result; x += a p, r -= a q (p the input xin, q not
// stored); 2: p = the result + b p.
enum { kCgNone = 0, kCgUpdate = 1, kCgDirection = 2 };

template <typename S, typename R, int RECON, int MODE, int CG = kCgNone>
__global__ void __launch_bounds__(kSplitThreads) wilson_split_kernel(WArgs<S> a, CgStep cg) {
  constexpr bool CLOV = MODE == W_HOP_CLOV || MODE == W_XPAY_CLOV, XPAY = MODE == W_XPAY_CLOV || MODE == W_XPAY;
  __shared__ R half[8 * 12 * kSplitPoints];
  __shared__ R full[MODE == W_HOP_CLOV ? 24 * kSplitPoints : 1];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // points in the order of rhs_block: source group fastest
  const int ng = a.nrhs / a.rg, spb = kSplitPoints / a.rg;
  const int rhs = a.rg * ((int)blockIdx.x % ng) + (lane & (a.rg - 1));
  const int s = ((int)blockIdx.x / ng) * spb + lane / a.rg;
  const bool valid = s < a.g.Vh;
  const int64_t vh = a.g.Vh, vs = vh * a.nrhs, v = rhs_index(rhs, s, vh, a.rg);
  const R sgn = a.dagger ? R(-1) : R(1);
  // the epilogue's waves: components c0 = 2w and c0 + 1 (spin-colour 3 sp + c), rows i0 and i0 + 1 of block b
  const int c0 = 2 * w, b = c0 / 6, i0 = c0 - 6 * b;
  const bool epi = w < 6 && valid;
  CloverRow<R> row[2];
  cpx<R> xv[6];
  if (epi) {  // loaded ahead of the hops
    if constexpr (CLOV) {
      load_clover_row<S, R>(a.clov, vh, s, b, i0, row[0]);
      load_clover_row<S, R>(a.clov, vh, s, b, i0 + 1, row[1]);
    }
    if constexpr (XPAY) {
      // chunk k of the spinor: components 2k, 2k + 1; the block's three chunks (or this wave's)
#pragma unroll
      for (int k = 0; k < (CLOV ? 3 : 1); ++k) {
        const Chunk<S, 4> q = *reinterpret_cast<const Chunk<S, 4> *>(a.xin + ((int64_t)(CLOV ? 3 * b + k : w) * vs + v) * 4);
        xv[2 * k] = mk<R>(to_real<R>(q.v[0]), to_real<R>(q.v[1]));
        xv[2 * k + 1] = mk<R>(to_real<R>(q.v[2]), to_real<R>(q.v[3]));
      }
    }
  }
  {
    const Site x = decode_site(a.g, valid ? s : 0, a.parity);
    R *o = half + w * 12 * kSplitPoints + lane;
    switch (w) {
      case 0: split_hop<0, +1, S, R, RECON>(a, x, s, rhs, sgn, valid, o); break;
      case 1: split_hop<0, -1, S, R, RECON>(a, x, s, rhs, sgn, valid, o); break;
      case 2: split_hop<1, +1, S, R, RECON>(a, x, s, rhs, sgn, valid, o); break;
      case 3: split_hop<1, -1, S, R, RECON>(a, x, s, rhs, sgn, valid, o); break;
      case 4: split_hop<2, +1, S, R, RECON>(a, x, s, rhs, sgn, valid, o); break;
      case 5: split_hop<2, -1, S, R, RECON>(a, x, s, rhs, sgn, valid, o); break;
      case 6: split_hop<3, +1, S, R, RECON>(a, x, s, rhs, sgn, valid, o); break;
      default: split_hop<3, -1, S, R, RECON>(a, x, s, rhs, sgn, valid, o); break;
    }
  }
  __syncthreads();
  const R coef = (R)a.coef;
  cpx<R> acc[2], res[2];
  if (w < 6) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int sp = (c0 + e) / 3, c = (c0 + e) - 3 * sp;
      cpx<R> t = mk<R>(0, 0);
#pragma unroll
      for (int h = 0; h < 8; ++h) {
        const R *u = half + (h * 12 + 2 * c) * kSplitPoints + lane;
        const cpx<R> u0 = mk<R>(u[0], u[kSplitPoints]);
        const cpx<R> u1 = mk<R>(u[6 * kSplitPoints], u[7 * kSplitPoints]);
        t = t + split_term<R>(h >> 1, sp, (h & 1) ? sgn : -sgn, u0, u1);
      }
      acc[e] = t;
    }
  }
  if constexpr (MODE == W_HOP) {
    res[0] = coef * acc[0];
    res[1] = coef * acc[1];
  } else if constexpr (MODE == W_HOP_CLOV) {
    if (w < 6)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        acc[e] = coef * acc[e];
        full[(2 * (c0 + e)) * kSplitPoints + lane] = acc[e].re;
        full[(2 * (c0 + e) + 1) * kSplitPoints + lane] = acc[e].im;
      }
    __syncthreads();
    if (w < 6) {
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        const R *f = full + 2 * (6 * b + j) * kSplitPoints + lane;
        xv[j] = mk<R>(f[0], f[kSplitPoints]);
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) res[e] = clover_row_mul(row[e], i0 + e, xv);
    }
  } else {
    if (w < 6)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if constexpr (CLOV)
          res[e] = scale_add<true>(coef, acc[e], clover_row_mul(row[e], i0 + e, xv));
        else
          res[e] = scale_add<true>(coef, acc[e], xv[e]);
      }
  }
  if constexpr (CG != kCgNone) {
    // Every wave forms the totals of the earlier launches (fixed order); the
    // updates end, leaving x, r and p as they are, once |r|^2 <= stop or |p|^2
    // is not positive.
    const int n = gridDim.x, b0 = (cg.iter & 1) ^ 1, b1 = cg.iter & 1;
    const double rr = cg_total(cg.rr[b0], n), pp = cg_total(cg.pp[b0], n);
    double *now = CG == kCgUpdate ? cg.rr[b1] : cg.pp[b1];
    double own = 0;
    auto chunk = [&](double *f) { return reinterpret_cast<Chunk<double, 4> *>(f + ((int64_t)w * vs + v) * 4); };
    const double q[4] = {res[0].re, res[0].im, res[1].re, res[1].im};
    if constexpr (CG == kCgUpdate) {
      const bool go = rr > cg.stop && pp > 0;
      if (epi && go) {
        const double f = rr / pp;
        Chunk<double, 4> x = *chunk(cg.x), r = *chunk(cg.r);
        const Chunk<double, 4> p = *chunk(cg.p);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          x.v[k] += f * p.v[k];
          r.v[k] -= f * q[k];
          own += r.v[k] * r.v[k];
        }
        *chunk(cg.x) = x;
        *chunk(cg.r) = r;
      }
      if (!go && threadIdx.x == 0 && blockIdx.x == 0) own = rr;
    } else {
      const double next = cg_total(cg.rr[b1], n);
      const bool go = next > cg.stop && pp > 0;
      if (blockIdx.x == 0 && threadIdx.x == 0) {
        CgRing *e = cg.ring + cg.iter % kCgRing;
        e->rr = next;
        e->pp = pp;
        __hip_atomic_store(&e->iter, cg.iter, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
      }
      if (epi && go) {
        const double f = next / rr;
        Chunk<double, 4> p = *chunk(cg.p);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          p.v[k] = q[k] + f * p.v[k];
          own += p.v[k] * p.v[k];
        }
        *chunk(cg.p) = p;
      }
      if (!go && threadIdx.x == 0 && blockIdx.x == 0) own = pp;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) own += __shfl_xor(own, off, 64);
    __shared__ double waves[kSplitThreads / 64];
    if (lane == 0) waves[w] = own;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0;
      for (int j = 0; j < kSplitThreads / 64; ++j) t += waves[j];
      now[blockIdx.x] = t;
    }
    return;
  }
  if (!epi) return;
  Chunk<S, 4> o;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    o.v[2 * e] = Store<S>::from(res[e].re);
    o.v[2 * e + 1] = Store<S>::from(res[e].im);
  }
  *reinterpret_cast<Chunk<S, 4> *>(a.out + ((int64_t)w * vs + v) * 4) = o;
}

// Where the split form is taken: FP64 and FP32 storage, no partial inner
// products, every tile, and at most 16384 points. Measured (Schur operator, two
// launches, split against one thread per site): FP64 18 reals 2048 sites 13.6 /
// 19.4 us, 10368 sites 17.6 / 27.7, 16384 sites 19.3 / 26.4, 32768 sites 39.7 /
// 36.4; FP32 12 reals 2048 sites 11.7 / 12.4, 16384 sites 12.8 / 13.8, 32768
// sites 18.5 / 17.6. Beyond 16384 points the waves of the one-thread form fill
// the chip. Points are counted over the sources: with 2 to 24 sources on 128 to 8192
// sites, 8, 12 and 18 reals, hop and Schur operator, no launch below the line is
// slower (1.01 to 1.9 times as fast, the FP32 ones near the line the least), and cut
// ones gain as much. The 16-bit kernels gained 3-10% and keep the one-thread form: its
// epilogue rounds some results once where this one would round twice.
constexpr int64_t kSplitMost = 16384;
bool wilson_split_fits(const WilsonLaunch &w) {
  return (w.prec == LQCD_F64 || w.prec == LQCD_F32) && !w.partials && w.g.colour < 0 && !w.mfma && (int64_t)w.g.Vh * w.nrhs <= kSplitMost;
}

template <int P, int RECON> static hipError_t launch_split2(const WilsonLaunch &w, hipStream_t st) {
  using S = typename Prec<P>::S;
  using R = typename Prec<P>::R;
  WArgs<S> a;
  a.g = w.g;
  a.out = (S *)w.out;
  a.in = (const S *)w.in;
  a.gauge = (const S *)w.gauge;
  a.clov = (const S *)w.clov;
  a.xin = (const S *)w.xin;
  a.partials = nullptr;
  a.coef = w.coef;
  a.parity = w.parity;
  a.dagger = w.dagger;
  a.nrhs = w.nrhs;
  a.rg = rhs_group(w.nrhs);
  const dim3 grid(rhs_grid(w.g.Vh, w.nrhs, kSplitPoints)), block(kSplitThreads);
  switch (w.mode) {
#define CASE(M)                                                                                       \
  case M:                                                                                             \
    hipLaunchKernelGGL((wilson_split_kernel<S, R, RECON, M>), grid, block, 0, st, a, CgStep{});       \
    return hipGetLastError();
    CASE(W_HOP)
    CASE(W_HOP_CLOV)
    CASE(W_XPAY_CLOV)
    CASE(W_XPAY)
#undef CASE
  }
  return hipErrorInvalidValue;
}

template <int P> static hipError_t launch_split1(const WilsonLaunch &w, hipStream_t st) {
  switch (w.recon) {
    case 18: return launch_split2<P, 18>(w, st);
    case 12: return launch_split2<P, 12>(w, st);
    case 8: return launch_split2<P, 8>(w, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_wilson_split(const WilsonLaunch &w, hipStream_t st) {
  if (w.g.Vh == 0) return hipSuccess;
  switch (w.prec) {
    case LQCD_F64: return launch_split1<LQCD_F64>(w, st);
    case LQCD_F32: return launch_split1<LQCD_F32>(w, st);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// CGNE iterations without a host round trip: the recurrences of lqcd_cg_solve on
// Mhat in FP64, for lattices that take the split form. An iteration is the four
// launches of the two Schur applications; a lattice of 2048 sites took eight and
// two stream synchronisations (62 us an iteration, 30 us of them kernels).

bool cg_device_fits(const OpInfo &info) {
  return info.prec == LQCD_F64 && info.op->action == LQCD_WILSON_CLOVER && (int64_t)info.vh <= kSplitMost;
}
int cg_device_groups(const OpInfo &info) { return rhs_grid((int)info.vh, 1, kSplitPoints); }

__global__ void __launch_bounds__(256) cg_start_kernel(CgStep c, int n, double rr, double pp) {
  for (int j = threadIdx.x; j < n; j += 256) {
    c.rr[0][j] = j == 0 ? rr : 0;
    c.pp[0][j] = j == 0 ? pp : 0;
  }
}

hipError_t launch_cg_start(const OpInfo &info, const CgStep &c, double rr, double pp, hipStream_t st) {
  hipLaunchKernelGGL(cg_start_kernel, dim3(1), dim3(256), 0, st, c, cg_device_groups(info), rr, pp);
  return hipGetLastError();
}

template <int RECON> static hipError_t cg_iteration(const OpInfo &info, const CgStep &c, void *tmp, hipStream_t st) {
  const lqcd_operator *op = info.op;
  WArgs<double> a;
  a.g = info.g;
  a.gauge = (const double *)op->gauge;
  a.partials = nullptr;
  a.nrhs = a.rg = 1;
  const dim3 grid(cg_device_groups(info)), block(kSplitThreads);
  for (int dagger = 0; dagger < 2; ++dagger) {
    const double *in = dagger ? c.r : c.p;
    a.dagger = dagger;
    a.out = (double *)tmp;
    a.in = in;
    a.xin = nullptr;
    a.clov = (const double *)op->clover_inv + info.vh * 72;  // odd sites
    a.parity = 1;
    a.coef = 1.0;
    hipLaunchKernelGGL((wilson_split_kernel<double, double, RECON, W_HOP_CLOV>), grid, block, 0, st, a, CgStep{});
    a.out = nullptr;
    a.in = (const double *)tmp;
    a.xin = in;
    a.clov = (const double *)op->clover;  // even sites
    a.parity = 0;
    a.coef = -op->kappa * op->kappa;
    if (dagger)
      hipLaunchKernelGGL((wilson_split_kernel<double, double, RECON, W_XPAY_CLOV, kCgDirection>), grid, block, 0, st, a, c);
    else
      hipLaunchKernelGGL((wilson_split_kernel<double, double, RECON, W_XPAY_CLOV, kCgUpdate>), grid, block, 0, st, a, c);
  }
  return hipGetLastError();
}

hipError_t launch_cg_iteration(const OpInfo &info, const CgStep &c, void *tmp, hipStream_t st) {
  switch (info.recon) {
    case 18: return cg_iteration<18>(info, c, tmp, st);
    case 12: return cg_iteration<12>(info, c, tmp, st);
    case 8: return cg_iteration<8>(info, c, tmp, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lqcd
