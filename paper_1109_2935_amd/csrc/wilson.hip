// Wilson-clover operator kernels for gfx950 (eq. (2) of the paper, kappa
// normalisation M = A - kappa D).
//
// One thread per output site of one parity. For each of the 8 hops the
// neighbour spinor is spin-projected to a half spinor (2 colour vectors) with
// (1 -/+ gamma_mu) before the SU(3) multiply, and the product is expanded back
// to 4 spins; the boundary phase and the Dirichlet cut are applied in-kernel.
// Epilogues fuse the clover term (A or A^-1), an xpay and, for the Schwarz
// block solver, per-workgroup partial inner products.
#include <type_traits>

#include "lqcd_internal.h"
#include "wilson_device.h"

namespace lqcd {

// One direction of the hopping term, each hop checked against the cut.
template <int MU, typename S, typename R, int RECON>
__device__ __forceinline__ void wilson_dir(const WArgs<S> &a, const Site &x, int s, int rhs, R sgn,
                                           cpx<R> (&acc)[4][3]) {
  if constexpr (half_hop<S, RECON>()) {
    // raw loads and the packed-half hop, as in the pipelined form
    HopIn<S, RECON> h;
    if (hop_kept<MU>(a.g, x, +1)) {
      if (a.nrhs == 1)
        hop_fetch<MU, +1, true, S, RECON>(a, x, s, rhs, h);
      else
        hop_fetch<MU, +1, false, S, RECON>(a, x, s, rhs, h);
      hop_apply<MU, +1, S, R, RECON>(h, sgn, a.g.bc_t, acc);
    }
    if (hop_kept<MU>(a.g, x, -1)) {
      if (a.nrhs == 1)
        hop_fetch<MU, -1, true, S, RECON>(a, x, s, rhs, h);
      else
        hop_fetch<MU, -1, false, S, RECON>(a, x, s, rhs, h);
      hop_apply<MU, -1, S, R, RECON>(h, sgn, a.g.bc_t, acc);
    }
    return;
  }
  const int64_t vh = a.g.Vh, vs = vh * a.nrhs;
  // forward: (1 - sgn gamma_mu) U_mu(x) psi(x+mu)
  if (hop_kept<MU>(a.g, x, +1)) {
    int w;
    const int n = hop1<MU, +1>(a.g, x, &w);
    cpx<R> psi[4][3], h[2][3], u[2][3];
    load_spinor<S, R>(a.in, vs, rhs_index(rhs, n, vh, a.rg), psi);
    project<MU, R>(psi, -sgn, h);
    const Link<R> U = load_link<S, R, RECON>(a.gauge, vh, MU, x.p, s, a.nrhs == 1);
    su3_mv<fused_products<S>()>(U, h[0], u[0]);
    su3_mv<fused_products<S>()>(U, h[1], u[1]);
    if constexpr (MU == 3) {
      const R ph = ((w & 1) && a.g.bc_t < 0) ? R(-1) : R(1);
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) u[k][c] = ph * u[k][c];
    }
    expand_acc<MU, R>(acc, u, -sgn);
  }
  // backward: (1 + sgn gamma_mu) U_mu(x-mu)^+ psi(x-mu)
  if (hop_kept<MU>(a.g, x, -1)) {
    int w;
    const int n = hop1<MU, -1>(a.g, x, &w);
    cpx<R> psi[4][3], h[2][3], u[2][3];
    load_spinor<S, R>(a.in, vs, rhs_index(rhs, n, vh, a.rg), psi);
    project<MU, R>(psi, sgn, h);
    const Link<R> U = load_link<S, R, RECON>(a.gauge, vh, MU, 1 - x.p, n, a.nrhs == 1);
    su3_adj_mv<fused_products<S>()>(U, h[0], u[0]);
    su3_adj_mv<fused_products<S>()>(U, h[1], u[1]);
    if constexpr (MU == 3) {
      const R ph = ((w & 1) && a.g.bc_t < 0) ? R(-1) : R(1);
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) u[k][c] = ph * u[k][c];
    }
    expand_acc<MU, R>(acc, u, sgn);
  }
}

// Where the pipelined hops pay (measured at 32^3x64): FP32 storage with 18,
// 12 or 8 link reals (8: since the rebuild takes the hardware sine and cosine,
// 110.5 -> 105.8 us), 16-bit storage with 12 or 18, and the FP64 hopping term
// with 12 (257 -> 222 us). FP64 Schur kernels and the FP64 recon-18 hop spill
// with them, and the 16-bit xpay-only kernel (W_XPAY) spills.
template <typename S, int RECON, int MODE> constexpr bool pipelined_hops() {
  if constexpr (std::is_same<S, double>::value) return MODE == W_HOP && RECON == 12;
  if constexpr (is_fixed<S>()) return false;  // the neighbour's norm is read with its codes
  if constexpr (sizeof(S) == 4) return true;
  return RECON != 8 && MODE != W_XPAY;
}

// Apply the hop held in HA, then refill HA with the hop two ahead; the other
// buffer's loads stay in flight meanwhile.
#define HOP_STEP(MUa, DIRa, HA, MUn, DIRn)                      \
  __builtin_amdgcn_sched_barrier(0);                           \
  hop_apply<MUa, DIRa, S, R, RECON>(HA, sgn, a.g.bc_t, acc);   \
  __builtin_amdgcn_sched_barrier(0);                           \
  hop_fetch<MUn, DIRn, STREAM, S, RECON>(a, x, s, rhs, HA);

template <bool STREAM, typename S, typename R, int RECON>
__device__ __forceinline__ void wilson_hops_pipelined(const WArgs<S> &a, const Site &x, int s, int rhs, R sgn,
                                                      cpx<R> (&acc)[4][3]) {
  HopIn<S, RECON> A, B;
  hop_fetch<0, +1, STREAM, S, RECON>(a, x, s, rhs, A);
  hop_fetch<0, -1, STREAM, S, RECON>(a, x, s, rhs, B);
  HOP_STEP(0, +1, A, 1, +1)
  HOP_STEP(0, -1, B, 1, -1)
  HOP_STEP(1, +1, A, 2, +1)
  HOP_STEP(1, -1, B, 2, -1)
  HOP_STEP(2, +1, A, 3, +1)
  HOP_STEP(2, -1, B, 3, -1)
  __builtin_amdgcn_sched_barrier(0);
  hop_apply<3, +1, S, R, RECON>(A, sgn, a.g.bc_t, acc);
  __builtin_amdgcn_sched_barrier(0);
  hop_apply<3, -1, S, R, RECON>(B, sgn, a.g.bc_t, acc);
  __builtin_amdgcn_sched_barrier(0);
}
#undef HOP_STEP

// ---------------------------------------------------------------------------
// Link products of several right-hand sides on the matrix cores (16-bit
// storage). With N sources per site the products of one hop are
// U [3 x 2N] (3 colours x (2 half-spinor rows x N sources)), in real form
// [[Ur, -Ui], [Ui, Ur]] (6 x 6) times (h_re; h_im) (6 x 2N). They run on
// v_mfma_f32_4x4x4_16b_{f16,bf16}: 16 independent 4x4x4 products per
// instruction, FP32 accumulation. A block is one site and 4 of its sources
// (lanes 4b .. 4b+3): lane j supplies row j of the link (A operand) and the
// half spinor of its own source (B column j), and receives U h for its own
// source (D column j). Rows and K both run (c0 re, c0 im, c1 re, c1 im | c2 re,
// c2 im, 0, 0): 2 M blocks x 2 K steps x 2 half-spinor rows = 8 instructions
// per hop. Link and half-spinor entries are rounded to the storage format
// (a reconstructed third row and the projection sums are the only new
// roundings), products are exact and sums are FP32.

template <typename S>
__device__ __forceinline__ void mf_mul(const typename Mf4<S>::T (&a)[2][2], const cpx<float> (&h)[2][3],
                                       cpx<float> (&u)[2][3]) {
  using M = Mf4<S>;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const typename M::T b0 = M::pack(h[k][0].re, h[k][0].im, h[k][1].re, h[k][1].im);
    const typename M::T b1 = M::pack(h[k][2].re, h[k][2].im, 0.f, 0.f);
    mf_f4 d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};
    d0 = M::mma(a[0][0], b0, d0);
    d0 = M::mma(a[0][1], b1, d0);
    d1 = M::mma(a[1][0], b0, d1);
    d1 = M::mma(a[1][1], b1, d1);
    u[k][0] = mk<float>(d0[0], d0[1]);
    u[k][1] = mk<float>(d0[2], d0[3]);
    u[k][2] = mk<float>(d1[0], d1[1]);
  }
}

// Both hops of direction MU for (site s, source rhs) with the link products on
// the matrix cores. Every lane takes part in the products (a lane without a
// contribution supplies zeros), so there is no divergence around them.
template <int MU, typename S, int RECON>
__device__ __forceinline__ void wilson_dir_mf(const WArgs<S> &a, const Site &x, int s, int rhs, bool valid, float sgn,
                                              cpx<float> (&acc)[4][3]) {
  const int64_t vh = a.g.Vh, vs = vh * a.nrhs;
  const int j = threadIdx.x & 3;
#pragma unroll
  for (int dir = 0; dir < 2; ++dir) {
    const int step = dir == 0 ? 1 : -1;
    const float g = dir == 0 ? -sgn : sgn;
    const bool kept = valid && hop_kept<MU>(a.g, x, step);
    int w = 0;
    cpx<float> h[2][3];
    Link<float> U;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) U.m[r][c] = mk<float>(0, 0);
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) h[k][c] = mk<float>(0, 0);
    if (kept) {
      const int n = hop<MU>(a.g, x, step, &w);
      cpx<float> psi[4][3];
      load_spinor<S, float>(a.in, vs, rhs_index(rhs, n, vh, a.rg), psi);
      project<MU, float>(psi, g, h);
      U = dir == 0 ? load_link<S, float, RECON>(a.gauge, vh, MU, x.p, s, false)
                   : load_link<S, float, RECON>(a.gauge, vh, MU, 1 - x.p, n, false);
    }
    typename Mf4<S>::T A[2][2];
    if (dir == 0)
      mf_link_rows<S, false>(U, j, A);
    else
      mf_link_rows<S, true>(U, j, A);
    cpx<float> u[2][3];
    mf_mul<S>(A, h, u);
    if (MU == 3 && (w & 1) && a.g.bc_t < 0) {
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) u[k][c] = -1.f * u[k][c];
    }
    if (dir == 0)
      expand_acc<MU, float>(acc, u, -sgn);
    else
      expand_acc<MU, float>(acc, u, sgn);
  }
}

// Per-segment sums of 3 values for the Schwarz block solver. A segment is
// seg = min(sites per tile and parity, 64) consecutive sites (a power of two:
// the tile's site count divides 64 or is a multiple of it), so a segment never
// spans two waves and the layout of the partials does not depend on the
// workgroup size. Segment j covers sites [j*seg, (j+1)*seg); its sums go to
// dst[3*j .. 3*j+2].
__device__ __forceinline__ void segment_reduce_store(double (&v)[3], int seg, int site, int vh, double *dst) {
#pragma unroll
  for (int k = 0; k < 3; ++k)
    for (int off = seg >> 1; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
  if ((site & (seg - 1)) == 0 && site < vh)
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[3 * (site / seg) + k] = v[k];
}

// How a launch takes its hops: checked one by one at run time (any cut), or
// pipelined (no cut). A pipelined form for cuts at the tile faces (the dropped
// hop loaded like any other and zeroed by a select) measured 2.5% slower in
// the Schwarz preconditioner than the checked form, which skips the dropped
// hops' loads, and is not kept.
enum HopForm { kHopsChecked = 0, kHopsPipe = 1 };

// One output (site s, right-hand side rhs) of the hopping term and its epilogue.
// MF: link products on the matrix cores (16-bit storage, sources in groups of
// 4 lanes); then every lane of the wave calls this, `valid` marks real work.
template <typename S, typename R, int RECON, int MODE, bool REDUCE, bool MF = false, int HOPS = kHopsChecked>
__device__ __forceinline__ void wilson_point(const WArgs<S> &a, int s, int rhs, double (&red)[3], bool valid = true) {
  const Site x = decode_site(a.g, s, a.parity);
  const R sgn = a.dagger ? R(-1) : R(1);
  cpx<R> acc[4][3];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[i][c] = mk<R>(0, 0);
  if constexpr (MF) {
    wilson_dir_mf<0, S, RECON>(a, x, s, rhs, valid, sgn, acc);
    wilson_dir_mf<1, S, RECON>(a, x, s, rhs, valid, sgn, acc);
    wilson_dir_mf<2, S, RECON>(a, x, s, rhs, valid, sgn, acc);
    wilson_dir_mf<3, S, RECON>(a, x, s, rhs, valid, sgn, acc);
    if (!valid) return;
  } else {
    if constexpr (HOPS != kHopsChecked) {
      // The same arithmetic for every source count, so a site's rounding does not
      // depend on nrhs. The branch between two calls of it is deliberate: as one
      // basic block with the epilogue, the clover kernels spill (measured:
      // 700-900 bytes per lane); split like this they need 137-158 VGPRs and no
      // scratch. Where a site block has several source groups, the hopping term
      // of FP32 and FP64 fields loads links through the caches, since the next
      // workgroup reads them again (24^3 x 48, 12 sources: FP32 326 us with
      // streamed loads, 310 so; FP64 670, 623). One group reads a link once
      // (4 FP32 sources: 106 streamed, 116 cached); links of 16-bit fields are
      // half the bytes and take more room than they save (12 FP16 sources: 208,
      // 230), and beside clover terms, which are cached then, streamed links are
      // the faster (12 FP16 sources, Schur matvec: 499, 551).
      constexpr bool kStream = MODE != W_HOP || sizeof(S) == 2;
      // (One source has a call of its own, whose addresses the compiler simplifies:
      // without it launches of 10-30 us took 2% longer.)
      if (a.nrhs == 1)
        wilson_hops_pipelined<true, S, R, RECON>(a, x, s, rhs, sgn, acc);
      else if (kStream || a.nrhs == a.rg)
        wilson_hops_pipelined<true, S, R, RECON>(a, x, s, rhs, sgn, acc);
      else
        wilson_hops_pipelined<false, S, R, RECON>(a, x, s, rhs, sgn, acc);
    } else {
      wilson_dir<0, S, R, RECON>(a, x, s, rhs, sgn, acc);
      wilson_dir<1, S, R, RECON>(a, x, s, rhs, sgn, acc);
      wilson_dir<2, S, R, RECON>(a, x, s, rhs, sgn, acc);
      wilson_dir<3, S, R, RECON>(a, x, s, rhs, sgn, acc);
    }
  }
  // the epilogue's loads (xin, clover) are not hoisted into the hop pipeline,
  // where they would hold registers through all eight hops
  if constexpr (HOPS != kHopsChecked) __builtin_amdgcn_sched_barrier(0);
  const R coef = (R)a.coef;
  const int64_t vh = a.g.Vh, vs = vh * a.nrhs, v = rhs_index(rhs, s, vh, a.rg);
  cpx<R> res[4][3];
  if constexpr (MODE == W_HOP) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) res[i][c] = coef * acc[i][c];
  } else if constexpr (MODE == W_HOP_CLOV) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[i][c] = coef * acc[i][c];
    clover_mul<S, R>(a.clov, vh, s, acc, res, a.nrhs == 1);
  } else {
    cpx<R> xv[4][3];
    load_spinor<S, R>(a.xin, vs, v, xv);
    if constexpr (is_float16<S>()) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          __asm__ volatile("" : "+v"(xv[i][c].re));
          __asm__ volatile("" : "+v"(xv[i][c].im));
        }
    }
    if constexpr (MODE == W_XPAY_CLOV) {
      clover_mul<S, R>(a.clov, vh, s, xv, res, a.nrhs == 1);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) res[i][c] = scale_add<fused_products<S>()>(coef, acc[i][c], res[i][c]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) res[i][c] = scale_add<fused_products<S>()>(coef, acc[i][c], xv[i][c]);
    }
    if constexpr (REDUCE) {
      // inner products of the values as stored
      R fx[24];
      if constexpr (is_fixed<S>()) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            fx[6 * i + 2 * c] = res[i][c].re;
            fx[6 * i + 2 * c + 1] = res[i][c].im;
          }
        fixed_round<24, R>(fx);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          double qr, qi;
          if constexpr (is_fixed<S>()) {
            qr = fx[6 * i + 2 * c];
            qi = fx[6 * i + 2 * c + 1];
          } else {
            qr = quantize<S, R>(res[i][c].re);
            qi = quantize<S, R>(res[i][c].im);
          }
          const double rr = xv[i][c].re, ri = xv[i][c].im;
          red[0] += qr * rr + qi * ri;
          red[1] += qr * ri - qi * rr;
          red[2] += qr * qr + qi * qi;
        }
    }
  }
  store_spinor<S, R, true>(a.out, vs, v, res);
}

// One thread per (site, rhs): the lanes of a site block's source group are
// adjacent in the workgroup and the workgroups of its groups are adjacent in
// the launch (rhs_block), so link and clover loads are shared.
template <typename S, typename R, int RECON, int MODE, bool REDUCE, int HOPS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) wilson_kernel(WArgs<S> a) {
  const RhsBlock rb = rhs_block(a.nrhs, a.rg);
  double red[3] = {0, 0, 0};
  int s = rb.s;
  if constexpr (MODE == W_HOP_CLOV || MODE == W_XPAY_CLOV) {
    // one colour of tiles (single right-hand side; the host checks)
    if (a.g.colour >= 0) s = rb.s < (a.g.Vh >> 1) ? colour_site(a.g, rb.s) : a.g.Vh;
  }
  if (s < a.g.Vh) wilson_point<S, R, RECON, MODE, REDUCE, false, HOPS>(a, s, rb.rhs, red);
  if constexpr (REDUCE) {  // single right-hand side only
    segment_reduce_store(red, a.g.Vt2 < 64 ? a.g.Vt2 : 64, s, a.g.Vh, a.partials);
  }
}

// Matrix-core variant for 16-bit storage and a multiple of 4 right-hand sides:
// lanes 4b .. 4b+3 (one 4x4x4 block) are one site and its 4 sources of one
// group (the lane mapping of wilson_kernel with 4 sources per group). All
// lanes stay active through the products.
template <typename S, int RECON, int MODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) wilson_mf_kernel(WArgs<S> a) {
  const RhsBlock rb = rhs_block(a.nrhs, 4);  // rg == 4 here
  const bool valid = rb.s < a.g.Vh;
  double red[3];
  wilson_point<S, float, RECON, MODE, false, true>(a, valid ? rb.s : 0, rb.rhs, red, valid);
}

// Persistent launch over several operators (uneven lattices, several
// right-hand sides each): a fixed grid of workgroups takes work items from a
// global counter until every item of every job is done. An item is one
// workgroup's worth of (site, rhs) pairs, numbered job after job and, within a
// job, in the order of the non-persistent launch (source fastest).
constexpr int kMaxBatchJobs = 8;
constexpr int kBatchQueues = 8;  // one work queue per XCD
template <typename S> struct BatchArgs {
  WArgs<S> job[kMaxBatchJobs];
  int begin[kMaxBatchJobs + 1];  // first work item of each job (prefix sums)
  int njobs;
  int chunk;
  int mfma;           // 16-bit jobs with a multiple of 4 sources: link products on the matrix cores
  unsigned *counter;  // kBatchQueues counters, zero at launch
};

// Items are split into kBatchQueues contiguous ranges; workgroup b serves queue
// b % kBatchQueues, i.e. the XCD it runs on, so the items of one site block
// (its source groups, adjacent in the numbering) share that XCD's L2. The grid
// is a multiple of kBatchQueues, so every queue is drained.
template <typename S, typename R, int RECON>
__device__ __forceinline__ void batch_item(const BatchArgs<S> &b, int it) {
  int j = 0;
  while (j + 1 < b.njobs && it >= b.begin[j + 1]) ++j;
  const WArgs<S> &a = b.job[j];
  const RhsBlock rb = rhs_block_at(it - b.begin[j], a.nrhs, a.rg);
  const bool valid = rb.s < a.g.Vh;
  double red[3];
  if constexpr (is_float16<S>()) {
    if (b.mfma && a.nrhs % 4 == 0) {  // uniform over the workgroup
      wilson_point<S, R, RECON, W_HOP, false, true>(a, valid ? rb.s : 0, rb.rhs, red, valid);
      return;
    }
  }
  // jobs carry no cut: the same hop code as the per-operator launch
  if (valid)
    wilson_point<S, R, RECON, W_HOP, false, false, pipelined_hops<S, RECON, W_HOP>() ? kHopsPipe : kHopsChecked>(
        a, rb.s, rb.rhs, red);
}

// Single launch with one workgroup per item (items remapped per XCD like the
// single-operator launch): the alternative the autotuner weighs against the
// persistent queue.
template <typename S, typename R, int RECON>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) wilson_batch_flat_kernel(BatchArgs<S> b) {
  batch_item<S, R, RECON>(b, xcd_remap(blockIdx.x, gridDim.x));
}

template <typename S, typename R, int RECON>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) wilson_batch_kernel(BatchArgs<S> b) {
  __shared__ int next;
  const int total = b.begin[b.njobs];
  const int q = blockIdx.x % kBatchQueues;
  const int lo = (int)((int64_t)q * total / kBatchQueues), hi = (int)((int64_t)(q + 1) * total / kBatchQueues);
  // the index of the following item is fetched while the current one runs
  if (threadIdx.x == 0) next = lo + (int)atomicAdd(b.counter + q, 1u);
  __syncthreads();
  int it = next;
  while (it < hi) {
    __syncthreads();  // every thread has read `next`
    if (threadIdx.x == 0) next = lo + (int)atomicAdd(b.counter + q, 1u);
    batch_item<S, R, RECON>(b, it);
    __syncthreads();  // `next` is written
    it = next;
  }
}

__global__ void zero_counter_kernel(unsigned *c) { c[threadIdx.x] = 0u; }  // one workgroup, one thread per counter

template <typename S, typename R>
__global__ void __launch_bounds__(256) clover_apply_kernel(Geom g, S *out, const S *in, const S *clov, int nrhs) {
  const RhsBlock rb = rhs_block(nrhs, rhs_group(nrhs));
  const int s = rb.s;
  if (s >= g.Vh) return;
  const int64_t pidx = rhs_index(rb.rhs, s, g.Vh, rhs_group(nrhs));
  const int64_t vs = (int64_t)g.Vh * nrhs;
  cpx<R> x[4][3], y[4][3];
  load_spinor<S, R>(in, vs, pidx, x);
  clover_mul<S, R>(clov, g.Vh, s, x, y, nrhs == 1);
  store_spinor<S, R, true>(out, vs, pidx, y);
}

// Schwarz MR step on every block at once, after q = Mhat_B r and the
// per-segment partials of <q,r> and <q,q>: alpha_B = <q,r>_B / <q,q>_B,
// x += alpha_B r (x = alpha_B r on the first step), r -= alpha_B q.
template <typename S, typename R>
__global__ void __launch_bounds__(256) mr_update_kernel(Geom g, S *x, S *r, const S *q, const double *part, int nps,
                                                        int first, double omega) {
  int s = xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
  if (s >= launch_sites(g)) return;
  if (g.colour >= 0) s = colour_site(g, s);
  const int b = (int)fdiv((uint32_t)s, g.dVt2);
  double qr = 0, qi = 0, qq = 0;
  for (int j = 0; j < nps; ++j) {
    const double *p = part + 3 * (b * nps + j);
    qr += p[0];
    qi += p[1];
    qq += p[2];
  }
  const R ar = qq > 0 ? (R)(omega * qr / qq) : R(0), ai = qq > 0 ? (R)(omega * qi / qq) : R(0);
  R rv[24], qv[24], xv[24];
  load_spinor_reals<S, 24, R>(r, g.Vh, s, rv);
  load_spinor_reals<S, 24, R>(q, g.Vh, s, qv);
  if (first) {
#pragma unroll
    for (int k = 0; k < 24; ++k) xv[k] = R(0);
  } else {
    load_spinor_reals<S, 24, R>(x, g.Vh, s, xv);
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const R re = rv[2 * k], im = rv[2 * k + 1];
    xv[2 * k] += ar * re - ai * im;
    xv[2 * k + 1] += ar * im + ai * re;
    rv[2 * k] = re - (ar * qv[2 * k] - ai * qv[2 * k + 1]);
    rv[2 * k + 1] = im - (ar * qv[2 * k + 1] + ai * qv[2 * k]);
  }
  store_spinor_reals<S, 24, R>(x, g.Vh, s, xv);
  store_spinor_reals<S, 24, R>(r, g.Vh, s, rv);
}

hipError_t launch_mr_update(const Geom &g, int prec, void *x, void *r, const void *q, const double *partials, int nps,
                            bool first, double omega, hipStream_t st) {
  const int bt = 256, nwg = (launch_sites(g) + bt - 1) / bt;
  if (g.Vh == 0) return hipSuccess;
  switch (prec) {
#define CASE(P)                                                                                              \
  case P:                                                                                                    \
    hipLaunchKernelGGL((mr_update_kernel<Prec<P>::S, Prec<P>::R>), dim3(nwg), dim3(bt), 0, st, g,            \
                       (Prec<P>::S *)x, (Prec<P>::S *)r, (const Prec<P>::S *)q, partials, nps, (int)first, omega);  \
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


template <int P, int RECON, int MODE, bool RED>
static hipError_t launch_w3(const WilsonLaunch &w, hipStream_t st) {
  using S = typename Prec<P>::S;
  using R = typename Prec<P>::R;
  WArgs<S> a;
  a.g = w.g;
  a.out = (S *)w.out;
  a.in = (const S *)w.in;
  a.gauge = (const S *)w.gauge;
  a.clov = (const S *)w.clov;
  a.xin = (const S *)w.xin;
  a.partials = w.partials;
  a.coef = w.coef;
  a.parity = w.parity;
  a.dagger = w.dagger;
  a.nrhs = w.nrhs;
  a.rg = rhs_group(w.nrhs);
  // colour-restricted launches: the cut Schur pieces, one source, tiles
  // alternating in colour along x, and a cut (blocks of one colour are
  // independent only through it)
  if (w.g.colour >= 0 && ((MODE != W_HOP_CLOV && MODE != W_XPAY_CLOV) || w.nrhs != 1 || w.mfma || (w.g.NT[0] & 1) ||
                          !w.g.has_cut))
    return hipErrorInvalidValue;
  const int nwg = rhs_grid(launch_sites(w.g), w.nrhs, w.block_threads);
  if constexpr ((P == LQCD_F16 || P == LQCD_BF16) && !RED) {
    if (w.mfma) {
      if (w.nrhs % 4 || w.block_threads % 64) return hipErrorInvalidValue;
      hipLaunchKernelGGL((wilson_mf_kernel<S, RECON, MODE>), dim3(nwg), dim3(w.block_threads), 0, st, a);
      return hipGetLastError();
    }
  }
  if (w.mfma) return hipErrorInvalidValue;
  // launches without a cut take the pipelined hops where they pay (measured);
  // the others keep the runtime-checked hops
  if constexpr (pipelined_hops<S, RECON, MODE>()) {
    if (!w.g.has_cut) {
      hipLaunchKernelGGL((wilson_kernel<S, R, RECON, MODE, RED, kHopsPipe>), dim3(nwg), dim3(w.block_threads), 0, st,
                         a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((wilson_kernel<S, R, RECON, MODE, RED, kHopsChecked>), dim3(nwg), dim3(w.block_threads), 0, st,
                     a);
  return hipGetLastError();
}

template <int P, int RECON>
static hipError_t launch_w2(const WilsonLaunch &w, hipStream_t st) {
  switch (w.mode) {
    case W_HOP: return launch_w3<P, RECON, W_HOP, false>(w, st);
    case W_HOP_CLOV: return launch_w3<P, RECON, W_HOP_CLOV, false>(w, st);
    case W_XPAY_CLOV:
      return w.partials ? launch_w3<P, RECON, W_XPAY_CLOV, true>(w, st) : launch_w3<P, RECON, W_XPAY_CLOV, false>(w, st);
    case W_XPAY:
      return w.partials ? launch_w3<P, RECON, W_XPAY, true>(w, st) : launch_w3<P, RECON, W_XPAY, false>(w, st);
  }
  return hipErrorInvalidValue;
}

template <int P>
static hipError_t launch_w1(const WilsonLaunch &w, hipStream_t st) {
  switch (w.recon) {
    case 18: return launch_w2<P, 18>(w, st);
    case 12: return launch_w2<P, 12>(w, st);
    case 8:
      if constexpr (P == LQCD_F64 || P == LQCD_F32) return launch_w2<P, 8>(w, st);
      break;
  }
  return hipErrorInvalidValue;
}

hipError_t launch_wilson(const WilsonLaunch &w, hipStream_t st) {
  if (w.g.Vh == 0) return hipSuccess;
  switch (w.prec) {
    case LQCD_F64: return launch_w1<LQCD_F64>(w, st);
    case LQCD_F32: return launch_w1<LQCD_F32>(w, st);
    case LQCD_F16: return launch_w1<LQCD_F16>(w, st);
    case LQCD_BF16: return launch_w1<LQCD_BF16>(w, st);
    case LQCD_HALF: return launch_w1<LQCD_HALF>(w, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_clover_apply(const Geom &g, int prec, void *out, const void *in, const void *clov, int nrhs,
                               hipStream_t st) {
  const int bt = 256, nwg = rhs_grid(g.Vh, nrhs, bt);
  if (g.Vh == 0) return hipSuccess;
  switch (prec) {
#define CASE(P)                                                                                           \
  case P:                                                                                                 \
    hipLaunchKernelGGL((clover_apply_kernel<Prec<P>::S, Prec<P>::R>), dim3(nwg), dim3(bt), 0, st, g,      \
                       (Prec<P>::S *)out, (const Prec<P>::S *)in, (const Prec<P>::S *)clov, nrhs);        \
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

template <int P, int RECON>
static hipError_t launch_b2(const BatchJob *jobs, int njobs, int dagger, const BatchTune &t, int mfma,
                            unsigned *counter, hipStream_t st) {
  using S = typename Prec<P>::S;
  using R = typename Prec<P>::R;
  BatchArgs<S> b;
  b.njobs = njobs;
  b.chunk = t.chunk;
  b.mfma = mfma;
  if (t.chunk != t.block_threads || t.block_threads % 64) return hipErrorInvalidValue;
  b.counter = counter;
  b.begin[0] = 0;
  for (int j = 0; j < njobs; ++j) {
    WArgs<S> &a = b.job[j];
    a.g = jobs[j].g;
    a.out = (S *)jobs[j].out;
    a.in = (const S *)jobs[j].in;
    a.gauge = (const S *)jobs[j].gauge;
    a.clov = nullptr;
    a.xin = nullptr;
    a.partials = nullptr;
    a.coef = 1.0;
    a.parity = jobs[j].parity;
    a.dagger = dagger;
    a.nrhs = jobs[j].nrhs;
    a.rg = rhs_group(jobs[j].nrhs);
    // items of this job: one per workgroup of the non-persistent launch
    b.begin[j + 1] = b.begin[j] + rhs_grid(jobs[j].g.Vh, jobs[j].nrhs, t.block_threads);
  }
  if (t.grid == 0) {  // one workgroup per item
    hipLaunchKernelGGL((wilson_batch_flat_kernel<S, R, RECON>), dim3(b.begin[njobs]), dim3(t.block_threads), 0, st, b);
    return hipGetLastError();
  }
  if (t.grid % kBatchQueues) return hipErrorInvalidValue;
  hipLaunchKernelGGL(zero_counter_kernel, dim3(1), dim3(kBatchQueues), 0, st, counter);
  hipLaunchKernelGGL((wilson_batch_kernel<S, R, RECON>), dim3(t.grid), dim3(t.block_threads), 0, st, b);
  return hipGetLastError();
}

template <int P>
static hipError_t launch_b1(int recon, const BatchJob *jobs, int njobs, int dagger, const BatchTune &t, int mf,
                            unsigned *c, hipStream_t st) {
  switch (recon) {
    case 18: return launch_b2<P, 18>(jobs, njobs, dagger, t, mf, c, st);
    case 12: return launch_b2<P, 12>(jobs, njobs, dagger, t, mf, c, st);
    case 8:
      if constexpr (P == LQCD_F64 || P == LQCD_F32) return launch_b2<P, 8>(jobs, njobs, dagger, t, mf, c, st);
      break;
  }
  return hipErrorInvalidValue;
}

hipError_t launch_wilson_batch(int prec, int recon, const BatchJob *jobs, int njobs, int dagger, const BatchTune &t,
                               int mfma, unsigned *counter, hipStream_t st) {
  if (njobs < 1 || njobs > kMaxBatchJobs) return hipErrorInvalidValue;
  if (mfma && prec != LQCD_F16 && prec != LQCD_BF16) return hipErrorInvalidValue;
  switch (prec) {
    case LQCD_F64: return launch_b1<LQCD_F64>(recon, jobs, njobs, dagger, t, mfma, counter, st);
    case LQCD_F32: return launch_b1<LQCD_F32>(recon, jobs, njobs, dagger, t, mfma, counter, st);
    case LQCD_F16: return launch_b1<LQCD_F16>(recon, jobs, njobs, dagger, t, mfma, counter, st);
    case LQCD_BF16: return launch_b1<LQCD_BF16>(recon, jobs, njobs, dagger, t, mfma, counter, st);
    case LQCD_HALF: return launch_b1<LQCD_HALF>(recon, jobs, njobs, dagger, t, mfma, counter, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lqcd
