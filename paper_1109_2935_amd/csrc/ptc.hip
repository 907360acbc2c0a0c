// Gauge-equivariant parallel-transport convolution (PTC) network kernels.
//
// One layer maps Cin channels of colour-spinor fields to Cout channels:
//   psi'_o(x) = sum_i sum_p W[o,i,p] (T_p psi_i)(x),
// p = 0 identity, 1+2mu forward hop (U_mu(x) psi(x+mu)), 2+2mu backward hop
// (U_mu(x-mu)^+ psi(x-mu)), W[o,i,p] a complex 4x4 spin matrix. The paper has
// no such network; it is used as a learned preconditioner of flexible GCR
// (Section III-B: the outer solver must be flexible).
//
// Activations between layers are BF16, one record of 24 reals (48 bytes, in the
// order spin, colour, re/im) per packed index site * C + channel of a parity
// block; the network output is an FP32 packed spinor. The channel mixing is a complex GEMM
//   O[(o,s)][(c,x)] = sum_{(i,p,s')} W[(o,s)][(i,p,s')] Y[(i,p,s')][(c,x)],
// Y = T_p psi_i, run on the BF16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32
// accumulation) in real form with interleaved real/imaginary rows:
//   A[2m+r][2k+r'] = [[Wr, -Wi],[Wi, Wr]][r][r'],  B[2k+r'][n] = (Yr, Yi)[r'].
// General form: a workgroup owns 64 or 32 sites of one parity; it builds Y for a
// chunk of input channels in LDS (parallel transport, converted to BF16), then
// each of its 4 waves runs the MFMA tiles it owns. Layers from 16 channels keep Y
// in registers (ptc_forward16_kernel). Weights come pre-packed in the per-lane
// A-operand order, so each A fragment is one coalesced 16-byte load.
#include <algorithm>
#include <type_traits>

#include "lqcd_internal.h"
#include "lqcd_ptc.h"

namespace lqcd {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// (x, y) rounded to nearest-even BF16, x in the low half
__device__ __forceinline__ bf16x2_t pack_bf16x2(float x, float y) {
  return __builtin_convertvector(f32x2_t{x, y}, bf16x2_t);
}

constexpr int kTile = 16;      // sites per workgroup tile
constexpr int kPtcThreads = 256;
constexpr int kLdsPad = 8;     // bf16 padding per LDS row (bank spread)

// activation access: the 24 reals (48 bytes) of packed index idx in a parity block
__device__ __forceinline__ void act_load(const bf16 *__restrict__ blk, int64_t idx, float *r) {
  load_chunks<bf16, 24, 8, float>(blk + idx * 24, 1, 0, r);
}

// An FP32 link from 12 or 18 stored reals.
template <int RC> __device__ __forceinline__ Link<float> ptc_link(const float *v) {
  Link<float> u = unpack_link<RC == 12 ? 12 : 18, float>(v);
  if constexpr (RC == 12) {
    // conj(row 0 x row 1), its sums in the order that the activations' roundings have had
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int k = (j + 1) % 3, l = (j + 2) % 3;
      const cpx<float> a = u.m[0][k], b = u.m[1][l], c = u.m[0][l], d = u.m[1][k];
      u.m[2][j] = mk<float>((a.re * b.re - a.im * b.im) - (c.re * d.re - c.im * d.im),
                            -((a.re * b.im + a.im * b.re) - (c.re * d.im + c.im * d.re)));
    }
  }
  return u;
}

__device__ __forceinline__ f32x4_t mfma_bf16(const bf16x8_t &a, const bf16x8_t &b, const f32x4_t &c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Neighbour table of the transport paths: entry [par][p-1][s] (p = 1..8) is
// the index of the site reached by path p from site s of parity par, with
// bit 31 set where the hop crosses the antiperiodic time boundary.
__global__ void ptc_nbr_kernel(Geom g, int *tab) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  const int par = blockIdx.y;
  if (s >= g.Vh) return;
  const Site x = decode_site(g, s, par);
  int *t = tab + (int64_t)par * 8 * g.Vh + s;
  int w, n;
#define PTC_NBR(MU)                                                              \
  n = hop<MU>(g, x, 1, &w);                                                      \
  t[(2 * MU) * (int64_t)g.Vh] = n | ((MU == 3 && (w & 1) && g.bc_t < 0) << 31);  \
  n = hop<MU>(g, x, -1, &w);                                                     \
  t[(2 * MU + 1) * (int64_t)g.Vh] = n | ((MU == 3 && (w & 1) && g.bc_t < 0) << 31);
  PTC_NBR(0)
  PTC_NBR(1)
  PTC_NBR(2)
  PTC_NBR(3)
#undef PTC_NBR
}

// Transport of NCH channels i0, i0 + kstep, ... of one path p at site s of
// parity par, written to LDS as BF16 (row stride `cstride` between colours, 8
// K values per channel: spin-major, re/im interleaved; channel i0 + k kstep at
// column 8 k kstep). The link and the neighbour are read once; the NCH
// channel loads are issued together.
template <int RECON, int NCH>
__device__ __forceinline__ void transportn_lds(const PtcGeo &q, const int *__restrict__ nbr, const bf16 *__restrict__ act,
                                               int C, int i0, int kstep, int p, int par, int s, __bf16 *dst,
                                               int cstride) {
  const int64_t vh = q.g.Vh, vs = vh * C;
  int n = s;
  float ph = 1.f;
  if (p != 0) {
    const int e = nbr[((int64_t)par * 8 + p - 1) * vh + s];
    n = e & 0x7fffffff;
    ph = e < 0 ? -1.f : 1.f;
  }
  const bf16 *blk = act + (int64_t)(p == 0 ? par : 1 - par) * vs * 24;
  float r[NCH][24];
#pragma unroll
  for (int k = 0; k < NCH; ++k) act_load(blk, (int64_t)n * C + i0 + k * kstep, r[k]);
  if (p != 0) {
    const int mu = (p - 1) >> 1;
    const bool fwd = ((p - 1) & 1) == 0;
    float lv[RECON];
    // forward: U_mu(x) at x; backward: U_mu(x - mu)^+ at the neighbour
    load_site<float, RECON, float>(q.gauge + (int64_t)(2 * mu + (fwd ? par : 1 - par)) * vh * RECON, vh, fwd ? s : n,
                                   lv);
    const Link<float> U0 = ptc_link<RECON>(lv);
    // the matrix applied: U, or U^+ for a backward hop (selected once), times the boundary sign
    Link<float> U;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const cpx<float> e = fwd ? U0.m[a][b] : conj(U0.m[b][a]);
        U.m[a][b] = ph * e;
      }
#pragma unroll
    for (int k = 0; k < NCH; ++k)
#pragma unroll
      for (int sp = 0; sp < 4; ++sp) {
        cpx<float> v[3], u[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = mk<float>(r[k][6 * sp + 2 * c], r[k][6 * sp + 2 * c + 1]);
        su3_mv(U, v, u);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          r[k][6 * sp + 2 * c] = u[c].re;
          r[k][6 * sp + 2 * c + 1] = u[c].im;
        }
      }
  }
#pragma unroll
  for (int k = 0; k < NCH; ++k)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      bf16x8_t v;
#pragma unroll
      for (int sp = 0; sp < 4; ++sp) {
        v[2 * sp] = (__bf16)r[k][6 * sp + 2 * c];
        v[2 * sp + 1] = (__bf16)r[k][6 * sp + 2 * c + 1];
      }
      *reinterpret_cast<bf16x8_t *>(dst + c * cstride + 8 * k * kstep) = v;
    }
}

__device__ __forceinline__ bf16x8_t lds_frag(const __bf16 *row) {
  return *reinterpret_cast<const bf16x8_t *>(row);
}

// ---------------------------------------------------------------------------
// forward: out (Cout channels, parity par) = sum W (T psi_in)
//
// A workgroup owns NS sites, i.e. N = 3 * NS GEMM columns
// (n = colour * NS + site). Per K chunk its 256 threads transport
// kFwSites x fw_ipc items into LDS (BF16, row n holds the chunk's K values),
// then each wave multiplies its block of 16x16 output tiles: m-tiles
// {mbase + 4j} by n-tiles [nbase, nbase + nn), so each B fragment read from
// LDS feeds up to two MFMAs and each A fragment (pre-packed, one 16-byte load
// per lane) up to 3 NS / 16. NS = 64 halves the weight traffic per site of
// NS = 32 but needs twice the accumulators; the launch picks one by timing
// (both give identical results: the K order of every output is the same).

constexpr int kFwRow = 16 * 8 + kLdsPad;  // bf16 per LDS row: 16 items x 8 K values + padding

template <int NS>
__global__ void __launch_bounds__(kPtcThreads) __attribute__((amdgpu_waves_per_eu(2)))
ptc_forward_kernel(PtcGeo q, PtcLayerDev L, const int *nbr, const bf16 *in, void *out, int out_f32, int par_arg,
                   int zero_par) {
  constexpr int kFwSites = NS, NT = 3 * NS / 16;
  constexpr int NWC = kPtcThreads / 64;       // waves
  constexpr int JM = (8 + NWC - 1) / NWC;     // m-tiles per wave at most (8 m-tiles for 16 output channels)
  __shared__ __align__(16) __bf16 Bt[3 * NS * kFwRow];
  // each XCD takes a contiguous range of site tiles, so that the neighbours'
  // activations are read from its own L2; with par_arg < 0 both output
  // parities are computed, workgroups 2t and 2t + 1 taking tile t of the even
  // and the odd sites, so that an input site's reads as a hop input (by one
  // parity) and as its own identity input (by the other) come close in time
  int wl = xcd_remap(blockIdx.x, gridDim.x);
  const int par = par_arg < 0 ? (wl & 1) : par_arg;
  if (par_arg < 0) wl >>= 1;
  const int s0 = wl * kFwSites;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // this wave's output tiles
  int mbase, nm, nbase = 0, nn;
  if (L.mtiles >= NWC) {
    mbase = wave;
    nm = (L.mtiles - wave + NWC - 1) / NWC;
    nn = NT;
  } else {
    const int split = NWC / L.mtiles;  // waves per m-tile
    mbase = wave % L.mtiles;
    nm = 1;
    nn = (NT + split - 1) / split;
    nbase = (wave / L.mtiles) * nn;
    nn = max(0, min(nn, NT - nbase));
  }
  f32x4_t acc[JM][NT];
#pragma unroll
  for (int j = 0; j < JM; ++j)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[j][t] = f32x4_t{0, 0, 0, 0};
  const bf16x8_t *A = (const bf16x8_t *)L.A;
  // one K chunk (items q0 .. q0+ipc-1) from LDS into the accumulators
  auto mma_chunk = [&](auto &ac, const __bf16 *Bb, int q0, int ipc) {
    for (int kl = 0; kl < ipc / 4; ++kl) {
      const int ks = q0 / 4 + kl;
      bf16x8_t a[JM];
#pragma unroll
      for (int j = 0; j < JM; ++j)
        if (j < nm) a[j] = A[((size_t)(mbase + NWC * j) * L.fw_ks + ks) * 64 + lane];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t < nn) {
          const bf16x8_t b = lds_frag(Bb + ((nbase + t) * 16 + (lane & 15)) * kFwRow + kl * 32 + 8 * (lane >> 4));
#pragma unroll
          for (int j = 0; j < JM; ++j)
            if (j < nm) ac[j][t] = mfma_bf16(a[j], b, ac[j][t]);
        }
      }
    }
  };
  // Output. Row m = 16 mt + 4 g + jj (g = lane / 16) of a tile is channel
  // o = 2 mt + g / 2, spin 2 (g % 2) + jj / 2, real/imaginary part jj % 2;
  // column n = 16 nt + lane % 16. The tile is staged in LDS as
  // [site][channel][24 reals] (rows padded against bank conflicts) by stage(),
  // then stored in whole 16-byte chunks by store_out() (after a barrier).
  const int g = lane >> 4;
  const int64_t vs = (int64_t)q.g.Vh * L.cout;
  const int srow = L.cout * 24 + (out_f32 ? 4 : 8);  // staging row, in elements of the output type
  auto stage = [&](const f32x4_t (&ac)[JM][NT]) {
#pragma unroll
    for (int j = 0; j < JM; ++j) {
      if (j >= nm) continue;
      const int o = 2 * (mbase + NWC * j) + (g >> 1);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t >= nn) continue;
        const int n = (nbase + t) * 16 + (lane & 15);
        const int c = n / kFwSites, sl = n % kFwSites;
        if (o < L.cout) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int r = (2 * (g & 1) + h) * 6 + 2 * c;
            if (!out_f32) {
              Bt[sl * srow + o * 24 + r] = (__bf16)ac[j][t][2 * h];
              Bt[sl * srow + o * 24 + r + 1] = (__bf16)ac[j][t][2 * h + 1];
            } else {
              *reinterpret_cast<float2 *>(reinterpret_cast<float *>(Bt) + sl * srow + o * 24 + r) =
                  make_float2(ac[j][t][2 * h], ac[j][t][2 * h + 1]);
            }
          }
        }
      }
    }
  };
  auto store_out = [&]() {
    if (!out_f32) {
      // the workgroup's records are one range of memory, stored in 16-byte pieces in its order (first layer, 1 -> 16
      // channels, of an application at 16^4: both launches 24 us; piece after piece of a record, 34 us)
      const int per = 3 * L.cout;
      uint4 *blk = reinterpret_cast<uint4 *>((bf16 *)out + ((int64_t)par * vs + (int64_t)s0 * L.cout) * 24);
      for (int w = threadIdx.x; w < per * min(kFwSites, q.g.Vh - s0); w += kPtcThreads) {
        const int sl = w / per;
        blk[w] = *reinterpret_cast<const uint4 *>(Bt + sl * srow + 8 * (w - sl * per));
      }
    } else {
      const int per_chunk = kFwSites * L.cout;
      // FP32 packed spinor (chunks of 4 reals); the network's last layer (one channel)
      const float *Sf = reinterpret_cast<const float *>(Bt);
      float *blk = (float *)out + (int64_t)par * vs * 24;
      for (int w = threadIdx.x; w < 6 * per_chunk; w += kPtcThreads) {
        const int k = w / per_chunk, rem = w - k * per_chunk;
        const int sl = rem / L.cout, o = rem - sl * L.cout;
        const int s = s0 + sl;
        if (s < q.g.Vh)
          *reinterpret_cast<float4 *>(blk + ((int64_t)k * vs + (int64_t)s * L.cout + o) * 4) =
              *reinterpret_cast<const float4 *>(Sf + sl * srow + o * 24 + 4 * k);
      }
    }
  };
  // input known to vanish on parity zero_par (the network input lives on even
  // sites): the items reading that parity are zero, and when every hop is
  // zero only the identity items' K steps are multiplied
  const int hop_par = 1 - par;
  const int q_end = zero_par == hop_par ? 4 * ((L.cin + 3) / 4) : 4 * L.fw_ks;
  for (int q0 = 0; q0 < q_end; q0 += L.fw_ipc) {
    const int ipc = min(L.fw_ipc, q_end - q0);
    __syncthreads();
    if (L.cin % 4 == 0) {
      // kNch items (one site and path) per thread: channels un and un + gn of
      // the chunk when it is one path (lanes of a site then read whole cache
      // lines), else kNch consecutive channels
      constexpr int kNch = 2;
      const int gn = ipc / kNch;
      const bool one_path = ipc == L.cin;
#pragma unroll 1
      for (int w = threadIdx.x; w < kFwSites * gn; w += kPtcThreads) {
        const int un = w % gn, sl = w / gn;
        const int u0 = one_path ? un : kNch * un, kstep = one_path ? gn : 1;
        const int qi = q0 + u0, s = s0 + sl;
        __bf16 *dst = Bt + sl * kFwRow + 8 * u0;
        const int pq = qi / L.cin;
        if (s < q.g.Vh && qi < L.fw_items && (pq == 0 ? par : hop_par) != zero_par) {
          const int p = pq, i0 = qi - p * L.cin;
          if (q.recon == 12)
            transportn_lds<12, kNch>(q, nbr, in, L.cin, i0, kstep, p, par, s, dst, kFwSites * kFwRow);
          else
            transportn_lds<18, kNch>(q, nbr, in, L.cin, i0, kstep, p, par, s, dst, kFwSites * kFwRow);
        } else {
          const bf16x8_t zero = {};
#pragma unroll
          for (int k = 0; k < kNch; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c)
              *reinterpret_cast<bf16x8_t *>(dst + c * kFwSites * kFwRow + 8 * k * kstep) = zero;
        }
      }
    } else {
      // one item per thread, sites fastest (narrow activations)
#pragma unroll 1
      for (int w = threadIdx.x; w < kFwSites * ipc; w += kPtcThreads) {
        const int sl = w % kFwSites, u = w / kFwSites;
        const int qi = q0 + u, s = s0 + sl;
        __bf16 *dst = Bt + sl * kFwRow + 8 * u;
        const int pq = qi / L.cin;
        if (s < q.g.Vh && qi < L.fw_items && (pq == 0 ? par : hop_par) != zero_par) {
          const int p = pq, i = qi - p * L.cin;
          if (q.recon == 12)
            transportn_lds<12, 1>(q, nbr, in, L.cin, i, 1, p, par, s, dst, kFwSites * kFwRow);
          else
            transportn_lds<18, 1>(q, nbr, in, L.cin, i, 1, p, par, s, dst, kFwSites * kFwRow);
        } else {
          const bf16x8_t zero = {};
#pragma unroll
          for (int c = 0; c < 3; ++c) *reinterpret_cast<bf16x8_t *>(dst + c * kFwSites * kFwRow) = zero;
        }
      }
    }
    __syncthreads();
    mma_chunk(acc, Bt, q0, ipc);
  }
  __syncthreads();
  stage(acc);
  __syncthreads();
  store_out();
}

// ---------------------------------------------------------------------------
// forward from 16 channels
//
// The colour products U v run on v_mfma_f32_4x4x4_16b_bf16 with the vectors as
// the A operand and the link as the B operand: block (site, channel), row = spin
// (its colour vector as stored), column j = row j of U in real form, once for
// the real and once for the imaginary parts. Lane 16 kg + 4 s + j then holds the
// four spins of (site s, channel kg, colour j), which, rounded to BF16, is its B
// operand of the 16x16x32 channel product with column 4 s + j and K group kg:
// the transported inputs never leave the registers. (Column 4 s + 3 is unused: a
// quarter of the channel product is spent on it.) The links are read as BF16 rows
// from a table made once per application, the activations as 12-byte rows of the
// 48-byte records: four channels of a site are 192 bytes in a row.
// A wave owns 8 sites and all output channels; the weights of a path (32 KB)
// are staged in LDS for the workgroup's 64 sites, and the activations, links and
// weights of path p + 1 are loaded while path p is multiplied, an eighth of them
// at a time: issued together they hold up every wave of the SIMD until the last
// is accepted (3.45 instead of 2.95 ms). Loads are unconditional and tile counts
// compile-time, as in ptc_bwd_data_kernel. 16 sites per wave or loads two paths
// ahead need more registers than two waves per SIMD have (4.1 and 3.9 ms).
// Bound by the matrix cores and the loads together: at 32^3 x 64, 16 -> 16, 2.95 ms
// for both parities, of which the products take 1.6 ms at the cores' peak and
// a wave's 1 KB loads 34 cycles each; 16 -> 1, one parity: 0.80 ms. The form that
// transported through LDS (producer and consumer waves) took 3.23 and 1.00 ms.
// U is rounded to BF16, colour and channel sums are in FP32, and the transported
// inputs are rounded to BF16, each sum in the order of that form.

// Link table of the hop paths, and the neighbour table (as ptc_nbr_kernel) in the
// same launch: entry [par][p - 1][s] of the links, for par < npar, holds the applied
// matrix (U, or U^+ for a backward hop, times the boundary sign), 9 words (Re, -Im)
// in BF16.
__global__ void __launch_bounds__(256) ptc_link_kernel(PtcGeo q, int npar, int *__restrict__ nbr,
                                                       uint32_t *__restrict__ tab) {
  const int64_t vh = q.g.Vh;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int par = blockIdx.y >> 3, p = blockIdx.y & 7, mu = p >> 1;
  const bool fwd = (p & 1) == 0;
  if (s >= vh) return;
  const Site x = decode_site(q.g, (int)s, par);
  int w, n;
  switch (mu) {
    case 0: n = hop<0>(q.g, x, fwd ? 1 : -1, &w); break;
    case 1: n = hop<1>(q.g, x, fwd ? 1 : -1, &w); break;
    case 2: n = hop<2>(q.g, x, fwd ? 1 : -1, &w); break;
    default: n = hop<3>(q.g, x, fwd ? 1 : -1, &w); break;
  }
  const int e = n | ((mu == 3 && (w & 1) && q.g.bc_t < 0) << 31);
  nbr[((int64_t)par * 8 + p) * vh + s] = e;
  if (par >= npar) return;
  const int64_t ls = fwd ? s : n;
  const float *base = q.gauge + (int64_t)(2 * mu + (fwd ? par : 1 - par)) * vh * q.recon;
  Link<float> U0;
  if (q.recon == 12) {
    float lv[12];
    load_site<float, 12, float>(base, vh, ls, lv);
    U0 = ptc_link<12>(lv);
  } else {
    float lv[18];
    load_site<float, 18, float>(base, vh, ls, lv);
    U0 = ptc_link<18>(lv);
  }
  const float ph = e < 0 ? -1.f : 1.f;
  uint32_t *o = tab + (((int64_t)par * 8 + p) * vh + s) * 9;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const cpx<float> m = fwd ? U0.m[a][b] : conj(U0.m[b][a]);
      o[3 * a + b] = __builtin_bit_cast(uint32_t, pack_bf16x2(ph * m.re, -(ph * m.im)));
    }
}

constexpr int kF16Sites = 64;
constexpr int kF16Threads = 512;
constexpr int kF16Waves = kF16Threads / 64;
constexpr int kF16Own = kF16Sites / kF16Waves;  // sites of a wave
constexpr int kF16N = kF16Own / 4;              // its column tiles

struct Word3 {
  uint32_t x, y, z;
};

// LDS written by some lanes of a wave is read by others after this point.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int MT>
__global__ void __launch_bounds__(kF16Threads) __attribute__((amdgpu_waves_per_eu(MT == 8 ? 2 : MT == 4 ? 3 : 4)))
ptc_forward16_kernel(PtcGeo q, PtcLayerDev L, const int *__restrict__ nbr, const uint32_t *__restrict__ links,
                     const bf16 *__restrict__ in, void *__restrict__ out, int out_f32, int par_arg) {
  constexpr int NFRAG = MT * 4 * 64, PER = (NFRAG + kF16Threads - 1) / kF16Threads, NT = kF16N;
  constexpr int kRow = 196;                      // words per site of the output staging (768 bytes and a pad)
  constexpr int kStage = kF16Sites * (MT == 1 ? 28 : kRow) * 4;  // bytes of it
  constexpr int kLds = 2 * NFRAG * 16 > kStage ? 2 * NFRAG * 16 : kStage;
  __shared__ __align__(16) unsigned char smem[kLds];
  __shared__ int nbL[kF16Waves][8][kF16Own];
  bf16x8_t *As = reinterpret_cast<bf16x8_t *>(smem);
  int wl = xcd_remap(blockIdx.x, gridDim.x);
  const int par = par_arg < 0 ? (wl & 1) : par_arg;
  if (par_arg < 0) wl >>= 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 3, sl = (lane >> 2) & 3, kg = lane >> 4;
  const int64_t vh = q.g.Vh, vs = vh * 16;
  const int s0 = wl * kF16Sites + kF16Own * wave;  // sites beyond the last repeat it; they are not stored
  const bf16x8_t *A = (const bf16x8_t *)L.A;
  static_assert(kF16Own * 8 == 64, "one neighbour entry per lane");
  nbL[wave][lane >> 3][lane & 7] =
      nbr[((int64_t)par * 8 + (lane >> 3)) * vh + min(s0 + (lane & 7), (int)vh - 1)] & 0x7fffffff;
  f32x4_t acc[MT][NT];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[t][n] = f32x4_t{0, 0, 0, 0};

  bf16x8_t ap[PER];
  auto load_a1 = [&](int p, int k) __attribute__((always_inline)) {
    const int e = (threadIdx.x + k * kF16Threads) % NFRAG, t = min(e >> 8, L.mtiles - 1);
    ap[k] = A[((size_t)t * L.fw_ks + 4 * p + ((e >> 6) & 3)) * 64 + (e & 63)];
  };
  auto store_a = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < PER; ++k) As[buf * NFRAG + (threadIdx.x + k * kF16Threads) % NFRAG] = ap[k];
  };
  const uint32_t *same = reinterpret_cast<const uint32_t *>(in) + (int64_t)par * vs * 12;
  const uint32_t *other = reinterpret_cast<const uint32_t *>(in) + (int64_t)(1 - par) * vs * 12;
  Word3 raw[NT][4], lw[NT];
  // The loads of path p in 8 parts, issued between the products of path p - 1:
  // all at once they hold up every wave's products until the last is accepted.
  auto issue = [&](int p, int part) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      if (part / 2 != n) continue;  // parts 0 .. 2 NT - 1: half of tile n's channels
      const int64_t nb = nbL[wave][p - 1][4 * n + sl], s = min(s0 + 4 * n + sl, (int)vh - 1);
      if (part % 2 == 0)
        lw[n] = *reinterpret_cast<const Word3 *>(links + (((int64_t)par * 8 + p - 1) * vh + s) * 9 + 3 * min(j, 2));
      const uint32_t *r = other + nb * 192 + kg * 12 + 3 * j;
#pragma unroll
      for (int ks = 2 * (part % 2); ks < 2 * (part % 2) + 2; ++ks) raw[n][ks] = *reinterpret_cast<const Word3 *>(r + 48 * ks);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (part == 2 * NT + k * 3 / PER) load_a1(p, k);  // parts 2 NT ..: the weights
  };
  uint4 b[NT][4];
  // Products of the path in buffer buf, 8 parts of 4 MT / 8 (K step, m-tile) steps
  // (one part for few m-tiles); a part's weights are read from LDS one part ahead.
  constexpr int STEPS = 4 * MT, PARTS = STEPS >= 8 ? 8 : 1, SP = STEPS / PARTS;
  auto products = [&](int buf, int next) __attribute__((always_inline)) {
    const bf16x8_t *a0 = As + buf * NFRAG + lane;
    auto frag = [&](int i) { return a0[((i % MT) * 4 + i / MT) * 64]; };  // step i: m-tile i % MT, K step i / MT
    bf16x8_t a[2][SP];
#pragma unroll
    for (int m = 0; m < SP; ++m) a[0][m] = frag(m);
#pragma unroll
    for (int c = 0; c < PARTS; ++c) {
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (PARTS == 8)
        issue(next, c);
      else
#pragma unroll
        for (int k = 0; k < 8; ++k) issue(next, k);
      if (c + 1 < PARTS)
#pragma unroll
        for (int m = 0; m < SP; ++m) a[(c + 1) & 1][m] = frag((c + 1) * SP + m);
#pragma unroll
      for (int m = 0; m < SP; ++m) {
        const int i = c * SP + m;
#pragma unroll
        for (int n = 0; n < NT; ++n)
          acc[i % MT][n] = mfma_bf16(a[c & 1][m], __builtin_bit_cast(bf16x8_t, b[n][i / MT]), acc[i % MT][n]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // identity path: the words of colour j
#pragma unroll
  for (int k = 0; k < PER; ++k) load_a1(0, k);
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const uint32_t *r = same + (int64_t)min(s0 + 4 * n + sl, (int)vh - 1) * 192 + kg * 12 + min(j, 2);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) b[n][ks] = make_uint4(r[48 * ks], r[48 * ks + 3], r[48 * ks + 6], r[48 * ks + 9]);
  }
  store_a(0);
  __syncthreads();
  products(0, 1);
  store_a(1);
#pragma unroll 1
  for (int p = 1; p < 9; ++p) {
    // transport of path p
    const mf_f4 zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      // real parts: (Re, -Im); imaginary parts: (Im, Re)
      const uint32_t x[3] = {lw[n].x, lw[n].y, lw[n].z};
      uint32_t y[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) y[c] = ((x[c] >> 16) | (x[c] << 16)) ^ 0x00008000u;
      const mf_s4 x0 = __builtin_bit_cast(mf_s4, u32x2_t{x[0], x[1]}), x1 = __builtin_bit_cast(mf_s4, u32x2_t{x[2], 0u});
      const mf_s4 y0 = __builtin_bit_cast(mf_s4, u32x2_t{y[0], y[1]}), y1 = __builtin_bit_cast(mf_s4, u32x2_t{y[2], 0u});
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const mf_s4 v0 = __builtin_bit_cast(mf_s4, u32x2_t{raw[n][ks].x, raw[n][ks].y});
        const mf_s4 v1 = __builtin_bit_cast(mf_s4, u32x2_t{raw[n][ks].z, 0u});
        mf_f4 re = Mf4<bf16>::mma(v0, x0, zero4), im = Mf4<bf16>::mma(v0, y0, zero4);
        re = Mf4<bf16>::mma(v1, x1, re);
        im = Mf4<bf16>::mma(v1, y1, im);
        b[n][ks] = make_uint4(__builtin_bit_cast(uint32_t, pack_bf16x2(re[0], im[0])),
                              __builtin_bit_cast(uint32_t, pack_bf16x2(re[1], im[1])),
                              __builtin_bit_cast(uint32_t, pack_bf16x2(re[2], im[2])),
                              __builtin_bit_cast(uint32_t, pack_bf16x2(re[3], im[3])));
      }
    }
    __syncthreads();  // the weights of path p are in LDS, those of p - 1 have been used
    products(p & 1, min(p + 1, 8));
    store_a((p + 1) & 1);
  }
  __syncthreads();
  // Row 16 t + 4 kg + jj is channel 2 t + kg / 2, spin 2 (kg % 2) + jj / 2, part
  // jj % 2; column 16 n + 4 sl + j is site 4 n + sl, colour j. Staged per wave in
  // the order of the output, then stored in 16-byte pieces.
  uint32_t *st = reinterpret_cast<uint32_t *>(smem) + wave * kF16Own * (MT == 1 ? 28 : kRow);
  if (out_f32) {  // one channel, FP32 packed spinor: [site][24 reals]
    if (j < 3 && kg < 2)
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          *reinterpret_cast<float2 *>(st + (4 * n + sl) * 28 + (2 * kg + h) * 6 + 2 * j) =
              make_float2(acc[0][n][2 * h], acc[0][n][2 * h + 1]);
    wave_lds_fence();
    float *blk = (float *)out + (int64_t)par * vh * 24;
    if (const int k = lane >> 3, site = lane & 7; k < 6) {
      if (s0 + site < vh)
        *reinterpret_cast<float4 *>(blk + ((int64_t)k * vh + s0 + site) * 4) =
            *reinterpret_cast<const float4 *>(st + site * 28 + 4 * k);
    }
    return;
  }
  if (j < 3)
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int o = 2 * t + (kg >> 1);
      if (o >= L.cout) continue;
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          st[(4 * n + sl) * (MT == 1 ? 28 : kRow) + o * 12 + (2 * (kg & 1) + h) * 3 + j] =
              __builtin_bit_cast(uint32_t, pack_bf16x2(acc[t][n][2 * h], acc[t][n][2 * h + 1]));
    }
  wave_lds_fence();
  const int per = L.cout * 3;  // pieces per site
  uint4 *blk = reinterpret_cast<uint4 *>((bf16 *)out) + ((int64_t)par * vh + s0) * per;
  for (int e = lane; e < kF16Own * per; e += 64) {
    const int site = e / per;
    if (s0 + site < vh) blk[e] = *reinterpret_cast<const uint4 *>(st + site * (MT == 1 ? 28 : kRow) + 4 * (e - site * per));
  }
}

// ---------------------------------------------------------------------------
// backward pass. The cotangents delta between layers are held as the BF16
// operands both GEMMs take them as (each reader of an FP32 field would round
// it first), per site [colour][channel][spin][re/im]: a 16-byte piece is the 8
// K values of one channel and colour in the B operand of a 16x16x32 product.

// (colour c of channel o is ch pieces after colour c - 1)
__device__ __forceinline__ const uint4 *delta_at(const bf16 *delta, int64_t vh, int ch, int par, int s, int o) {
  return reinterpret_cast<const uint4 *>(delta) + ((int64_t)par * vh + s) * 3 * ch + o;
}

// The output cotangent (FP32 packed even spinor, one channel) in that layout.
__global__ void __launch_bounds__(256) ptc_delta_kernel(int64_t vh, const float *in_even, bf16 *delta) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= vh) return;
  float r[24];
  load_spinor_reals<float, 24, float>(in_even, vh, s, r);
  uint4 *d = reinterpret_cast<uint4 *>(delta) + 3 * s;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    bf16x8_t v;
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) {
      v[2 * sp] = (__bf16)r[6 * sp + 2 * c];
      v[2 * sp + 1] = (__bf16)r[6 * sp + 2 * c + 1];
    }
    d[c] = __builtin_bit_cast(uint4, v);
  }
}

// Data: gpsi_i(x) = sum_p T_p^+ (sum_o W[o,i,p]^+ delta_o)(x), T_{+mu}^+ = T_{-mu}.
// The adjoint product is taken at the site T_p^+ reads from and transported in
// registers: in the 16x16 result tiles a lane holds the same site and rows for
// each of the three colours (one tile per colour), so the SU(3) product of a
// (channel, spin) vector mixes registers of one lane, in FP32, and the 9 paths
// are summed in FP32 accumulators. Nothing but delta is read and gpsi written:
// the form with the 9 Cin intermediate fields in memory (13.8 KB per site at 16
// channels, written and read in FP32) was bound by them.
// A wave owns 16 sites; the weights of a path (32 KB at 16 -> 16) are staged in
// LDS for the workgroup's 64 sites, and the cotangents, link and weights of hop
// p + 1 are loaded before hop p is multiplied: one wave per SIMD with the
// registers of both (two waves of half the rows each spill). The loads of the
// hop loop are unconditional (the last one repeats hop 8) and the tile counts
// compile-time: a branch around a prefetch makes the compiler wait for all
// outstanding loads where the paths join.
// MT m-tiles (16 rows, 2 input channels each) and KS K steps (4 output
// channels each), both rounded up from the layer's.
// zero_par: parity on which delta vanishes (the output cotangent lives on even
// sites), -1: none.
constexpr int kBwSites = 64;
constexpr int kBwThreads = 256;

template <int RC, int KS> struct BwPath {
  bf16x8_t b[KS][3];
  float lv[RC];
  float ph;
};

template <int RC, int MT, int KS>
__global__ void __launch_bounds__(kBwThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
ptc_bwd_data_kernel(PtcGeo q, PtcLayerDev L, const int *__restrict__ nbr, const bf16 *__restrict__ delta,
                    bf16 *__restrict__ gpsi, int zero_par) {
  constexpr int NFRAG = MT * KS * 64, PER = (NFRAG + kBwThreads - 1) / kBwThreads;
  __shared__ bf16x8_t As[2][NFRAG];
  const int wl0 = xcd_remap(blockIdx.x, gridDim.x);
  const int par = wl0 & 1, s0 = (wl0 >> 1) * kBwSites;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4;
  const int64_t vh = q.g.Vh;
  const int s_own = s0 + 16 * wave + (lane & 15);
  const bool valid = s_own < vh;
  const int s = valid ? s_own : 0;
  const int nks = L.kadj / 32, rows = 8 * L.cin;
  const bf16x8_t *A = (const bf16x8_t *)L.Aadj;

  f32x4_t acc[MT][3];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[t][c] = f32x4_t{0, 0, 0, 0};

  // channels beyond Cout meet zero weights: those lanes load channel 0
  auto fetch_delta = [&](bf16x8_t (&b)[KS][3], int np, int n) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int o = 4 * ks + g;
      const uint4 *d = delta_at(delta, vh, L.cout, np, n, o < L.cout ? o : 0);
#pragma unroll
      for (int c = 0; c < 3; ++c) b[ks][c] = __builtin_bit_cast(bf16x8_t, d[c * L.cout]);
    }
  };
  // T_p^+ reads the site that path p' reaches, p' the opposite hop (entry of path p)
  auto entry = [&](int p) { return nbr[((int64_t)par * 8 + ((p - 1) ^ 1)) * vh + s]; };
  auto fetch = [&](BwPath<RC, KS> &f, int p, int e) __attribute__((always_inline)) {
    const int n = e & 0x7fffffff, mu = (p - 1) >> 1;
    const bool at_n = ((p - 1) & 1) == 0;  // U_mu(x - mu)^+ from x - mu, else U_mu(x) from x + mu
    f.ph = e < 0 ? -1.f : 1.f;
    load_site<float, RC, float>(q.gauge + (int64_t)(2 * mu + (at_n ? 1 - par : par)) * vh * RC, vh, at_n ? n : s,
                                f.lv);
    fetch_delta(f.b, 1 - par, n);
  };
  // fragments of path p: rows p rows .. + 16 MT (a tile may run into the next
  // path's rows, whose results are unused; beyond the last row it is clamped)
  bf16x8_t ap[PER];
  auto load_a = [&](int p) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = threadIdx.x + k * kBwThreads;
      const int ln = e & 63, t = (e >> 6) / KS, ks = (e >> 6) % KS;
      const int r = p * rows + 16 * t + (ln & 15), rt = min(r >> 4, L.madj_tiles - 1);
      ap[k] = A[((size_t)rt * nks + min(ks, nks - 1)) * 64 + ((ln & 48) | (r & 15))];
    }
  };
  auto store_a = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = threadIdx.x + k * kBwThreads;
      // K steps beyond the layer's are zero (masked without a branch)
      uint4 w = __builtin_bit_cast(uint4, ap[k]);
      const uint32_t keep = (e >> 6) % KS < nks ? ~0u : 0u;
      w = make_uint4(w.x & keep, w.y & keep, w.z & keep, w.w & keep);
      if (NFRAG % kBwThreads == 0 || e < NFRAG) As[buf][e] = __builtin_bit_cast(bf16x8_t, w);
    }
  };
  // one path's product W_p^+ delta for m-tile t
  auto product = [&](const bf16x8_t (&b)[KS][3], int buf, int t, f32x4_t (&C)[3]) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 3; ++c) C[c] = f32x4_t{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8_t a = As[buf][(t * KS + ks) * 64 + lane];
#pragma unroll
      for (int c = 0; c < 3; ++c) C[c] = mfma_bf16(a, b[ks][c], C[c]);
    }
  };
  if (zero_par != par) {  // identity path
    bf16x8_t b[KS][3];
    load_a(0);
    fetch_delta(b, par, s);
    store_a(0);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < MT; ++t) product(b, 0, t, acc[t]);
  }
  if (zero_par != 1 - par) {  // hops: weights of hop p in buffer p % 2
    BwPath<RC, KS> fa, fb;
    int e1 = entry(1);
    load_a(1);
    fetch(fa, 1, e1);
    e1 = entry(2);
    store_a(1);
    auto step = [&](auto at_n, const BwPath<RC, KS> &f, BwPath<RC, KS> &next, int p) __attribute__((always_inline)) {
      __syncthreads();  // hop p is in LDS, hop p - 1 has been multiplied
      const int pn = min(p + 1, 8), e = e1;
      load_a(pn);
      fetch(next, pn, e);
      e1 = entry(min(p + 2, 8));
      __builtin_amdgcn_sched_barrier(0);
      const Link<float> U = ptc_link<RC>(f.lv);
      // the matrix products of tile t + 1 run beside the transport of tile t;
      // the barriers keep the compiler from opening more tiles (it spills)
      f32x4_t C[2][3];
      product(f.b, p & 1, 0, C[0]);
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < MT) product(f.b, p & 1, t + 1, C[(t + 1) & 1]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          cpx<float> v[3], u[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) v[c] = mk<float>(C[t & 1][c][2 * h], C[t & 1][c][2 * h + 1]);
          if constexpr (at_n.value)
            su3_adj_mv(U, v, u);
          else
            su3_mv(U, v, u);
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            acc[t][c][2 * h] += f.ph * u[c].re;
            acc[t][c][2 * h + 1] += f.ph * u[c].im;
          }
        }
        // (the sums are formed here: left alone they are sunk to the end of the
        // hop loop, with the products of all tiles held in registers until then)
#pragma unroll
        for (int c = 0; c < 3; ++c) __asm__ volatile("" : "+v"(acc[t][c]));
      }
      __builtin_amdgcn_sched_barrier(0);
      store_a((p + 1) & 1);
    };
#pragma unroll 1
    for (int p = 1; p < 9; p += 2) {
      step(std::true_type(), fa, fb, p);
      step(std::false_type(), fb, fa, p + 1);
    }
  }
  if (!valid) return;
  // row 16 t + 4 g + jj: channel 2 t + g / 2, spin 2 (g % 2) + jj / 2, part jj % 2
  uint2 *out = reinterpret_cast<uint2 *>(gpsi) + ((int64_t)par * vh + s) * 6 * L.cin;
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int i = 2 * t + (g >> 1);
    if (i >= L.cin) continue;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      out[2 * (c * L.cin + i) + (g & 1)] =
          make_uint2(__builtin_bit_cast(uint32_t, pack_bf16x2(acc[t][c][0], acc[t][c][1])),
                     __builtin_bit_cast(uint32_t, pack_bf16x2(acc[t][c][2], acc[t][c][3])));
  }
}

// Weights: partial sums over site tiles of
//   G[(m', r)][k'] = sum_{(n, r')} D[(m', r)][(n, r')] Y'[(n, r')][k'],
//   D = [[dr, di],[di, -dr]],  Y' = (Yr, Yi),
// i.e. G = (Re, Im) of sum_x delta (T psi)^+. A workgroup owns a chunk of 16
// items (q = p Cin + i: with 16 channels one path) and a contiguous range of
// tiles of 16 sites; thread (site, item) transports one channel in FP32 and writes it
// as BF16 to LDS, row (item, spin), K = (colour, site, re/im); delta is staged
// the same way (row (channel, spin); the rows r = 1 are formed from the words
// on reading). The next tile's loads are issued before the products. The
// PATH: 16 input channels, chunk = path (uniform over the workgroup); JW: m-tiles
// per wave (the layer's halved and rounded up; rows beyond Cout are unused). The
// transports bound it (about 350 vector instructions per wave and tile against
// 24 matrix instructions): 172 us for a 16 -> 16 layer at 16^4 with the sum over
// groups; 942 us when a workgroup took 4 channels with all 9 paths, one parity,
// and wrote its operands to LDS in 2-byte pieces.
constexpr int kWgThreads = 256;
constexpr int kWgRow = 2 * 3 * kTile + kLdsPad;  // bf16 per LDS row

template <int RC, bool PATH, int JW>
__global__ void __launch_bounds__(kWgThreads)
ptc_bwd_weight_kernel(PtcGeo q, PtcLayerDev L, const int *__restrict__ nbr, const bf16 *__restrict__ in,
                      const bf16 *__restrict__ delta, float *__restrict__ partial, int groups, int zero_par) {
  __shared__ __align__(16) __bf16 At[2][64 * kWgRow];
  __shared__ __align__(16) __bf16 Bt[2][64 * kWgRow];
  // the chunks of one group of tiles run side by side on one XCD (the
  // dispatcher deals workgroups round-robin over 8), so that they share its L2
  const int nck = gridDim.y, b8 = blockIdx.x + gridDim.x * blockIdx.y, loc = b8 / 8;
  const int grp = (b8 % 8) * (groups / 8) + loc / nck, ck = loc % nck;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sl = threadIdx.x & 15, it = threadIdx.x >> 4;
  const int64_t vh = q.g.Vh, vs = vh * L.cin;
  // items beyond the last and channels beyond Cout (rows and columns of the
  // result that are not used) repeat the first
  const int qi = 16 * ck + it < L.fw_items ? 16 * ck + it : 0;
  const int p = PATH ? ck : qi / L.cin, i = PATH ? it : qi - p * L.cin, o = it < L.cout ? it : 0;
  const int ph_ = p == 0 ? 1 : p, mu = (ph_ - 1) >> 1;
  const bool fwd = ((ph_ - 1) & 1) == 0;
  const int ntile = (int)((vh + kTile - 1) / kTile);
  // tiles of both parities in turn, or those of the parity where delta lives
  const int npar = zero_par < 0 ? 2 : 1, total = npar * ntile;
  const int first = (int)((int64_t)grp * total / groups), last = (int)((int64_t)(grp + 1) * total / groups) - 1;
  const int nmt = L.mw_tiles, wm = wave & 1, wn = wave >> 1;

  f32x4_t acc[JW][2];
#pragma unroll
  for (int j = 0; j < JW; ++j)
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[j][t] = f32x4_t{0, 0, 0, 0};

  auto run = [&](auto ident) __attribute__((always_inline)) {
    constexpr bool IDENT = decltype(ident)::value;  // every item of the chunk is on the identity path
    uint4 dr[3], yr[3];
    float lv[RC];
    float ph = 1.f;
    // (tiles and sites beyond the last are clamped; such sites' delta is zeroed)
    auto site_of = [&](int tile) { return (npar == 2 ? tile >> 1 : tile) * kTile + sl; };
    auto clamped = [&](int tile) { return min(site_of(tile), (int)vh - 1); };
    auto par_of = [&](int tile) { return npar == 2 ? (tile & 1) : 1 - zero_par; };
    // the site that path p reaches (loaded a tile ahead of the operands)
    auto entry = [&](int tile) {
      const int s = clamped(tile);
      if constexpr (IDENT) return s;
      const int e = nbr[((int64_t)par_of(tile) * 8 + ph_ - 1) * vh + s];
      return PATH || p != 0 ? e : s;
    };
    auto fetch = [&](int tile, int e) __attribute__((always_inline)) {
      const int par = par_of(tile), s = clamped(tile), n = e & 0x7fffffff;
      const uint4 *d = delta_at(delta, vh, L.cout, par, s, o);
#pragma unroll
      for (int c = 0; c < 3; ++c) dr[c] = d[c * L.cout];
      if constexpr (!IDENT) {
        ph = e < 0 ? -1.f : 1.f;
        load_site<float, RC, float>(q.gauge + (int64_t)(2 * mu + (fwd ? par : 1 - par)) * vh * RC, vh, fwd ? s : n,
                                    lv);
      }
      const uint4 *y = reinterpret_cast<const uint4 *>(in) + ((p == 0 ? par : 1 - par) * vs + (int64_t)n * L.cin + i) * 3;
#pragma unroll
      for (int c = 0; c < 3; ++c) yr[c] = y[c];
    };
    if (last < first) return;
    int buf = 0, e1 = entry(first);
    fetch(first, e1);
    e1 = entry(min(first + 1, last));
#pragma unroll 1
    for (int tile = first; tile <= last; ++tile, buf ^= 1) {
      // words: delta [colour][spin], Y [spin][colour]
      uint32_t dw[12], yw[12];
      const bool valid = site_of(tile) < vh;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        dw[4 * c] = dr[c].x, dw[4 * c + 1] = dr[c].y, dw[4 * c + 2] = dr[c].z, dw[4 * c + 3] = dr[c].w;
        yw[4 * c] = yr[c].x, yw[4 * c + 1] = yr[c].y, yw[4 * c + 2] = yr[c].z, yw[4 * c + 3] = yr[c].w;
      }
      __bf16 *Ab = At[buf] + 4 * it * kWgRow + 2 * sl, *Bb = Bt[buf] + 4 * it * kWgRow + 2 * sl;
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int c = 0; c < 3; ++c)
          *reinterpret_cast<uint32_t *>(Ab + sp * kWgRow + 2 * c * kTile) = valid ? dw[4 * c + sp] : 0u;
      if constexpr (IDENT) {
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
          for (int c = 0; c < 3; ++c) *reinterpret_cast<uint32_t *>(Bb + sp * kWgRow + 2 * c * kTile) = yw[3 * sp + c];
      } else {
        const Link<float> U0 = ptc_link<RC>(lv);
        // U, or U^+ for a backward hop, times the boundary sign, on one spin at a time
        auto apply = [&](auto adj) __attribute__((always_inline)) {
#pragma unroll
          for (int sp = 0; sp < 4; ++sp) {
            cpx<float> v[3], u[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const uint32_t w = yw[3 * sp + c];
              v[c] = mk<float>(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
            }
            if constexpr (decltype(adj)::value)
              su3_adj_mv(U0, v, u);
            else
              su3_mv(U0, v, u);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const uint32_t w = __builtin_bit_cast(uint32_t, pack_bf16x2(ph * u[c].re, ph * u[c].im));
              *reinterpret_cast<uint32_t *>(Bb + sp * kWgRow + 2 * c * kTile) = PATH || p != 0 ? w : yw[3 * sp + c];
            }
          }
        };
        if (fwd)
          apply(std::false_type());
        else
          apply(std::true_type());
      }
      fetch(min(tile + 1, last), e1);
      e1 = entry(min(tile + 2, last));
      __syncthreads();  // this tile is in LDS (and the last but one has been multiplied)
#pragma unroll
      for (int ks = 0; ks < 3; ++ks) {
        bf16x8_t b[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
          b[t] = lds_frag(Bt[buf] + ((2 * wn + t) * 16 + (lane & 15)) * kWgRow + ks * 32 + 8 * (lane >> 4));
#pragma unroll
        for (int j = 0; j < JW; ++j) {
          const int mt = wm + 2 * j;
          // row 16 mt + lane % 16 = 2 (channel, spin) + r
          uint4 w = *reinterpret_cast<const uint4 *>(At[buf] + (8 * mt + ((lane & 15) >> 1)) * kWgRow + ks * 32 +
                                                     8 * (lane >> 4));
          if (lane & 1) {  // (dr, di) -> (di, -dr)
            w.x = ((w.x >> 16) | (w.x << 16)) ^ 0x80000000u;
            w.y = ((w.y >> 16) | (w.y << 16)) ^ 0x80000000u;
            w.z = ((w.z >> 16) | (w.z << 16)) ^ 0x80000000u;
            w.w = ((w.w >> 16) | (w.w << 16)) ^ 0x80000000u;
          }
          const bf16x8_t a = __builtin_bit_cast(bf16x8_t, w);
#pragma unroll
          for (int t = 0; t < 2; ++t) acc[j][t] = mfma_bf16(a, b[t], acc[j][t]);
        }
      }
    }
  };
  if (PATH && ck == 0)
    run(std::true_type());
  else
    run(std::false_type());
  // partial[ck][grp][16 mw_tiles rows][64 columns (item, spin)]
  float *dst = partial + ((size_t)ck * groups + grp) * (size_t)nmt * 16 * 64;
#pragma unroll
  for (int j = 0; j < JW; ++j) {
    const int mt = wm + 2 * j;
    if (mt >= nmt) continue;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        dst[(16 * mt + 4 * (lane >> 4) + jj) * 64 + (2 * wn + t) * 16 + (lane & 15)] = acc[j][t][jj];
  }
}

// gW[o][i][p][s][s'] (complex, FP32) = sum over groups of the partials, in a
// fixed order: a quarter of the groups per thread, then the four sums. 64
// threads run along a row of the partials (one chunk's columns).
__global__ void __launch_bounds__(256) ptc_weight_reduce_kernel(PtcLayerDev L, const float *partial, int groups,
                                                                float *gw) {
  __shared__ double sum[4][64][2];
  const int col = threadIdx.x & 63, part = threadIdx.x >> 6;
  const int m = blockIdx.x, ck = blockIdx.y;  // m = 4 o + s
  const size_t ld = (size_t)L.mw_tiles * 16 * 64;
  const float *base = partial + (size_t)ck * groups * ld + (size_t)2 * m * 64 + col;
  const int g0 = part * groups / 4, g1 = (part + 1) * groups / 4;
  double re = 0, im = 0;
#pragma unroll 4
  for (int g = g0; g < g1; ++g) {
    re += base[g * ld];
    im += base[g * ld + 64];
  }
  sum[part][col][0] = re;
  sum[part][col][1] = im;
  __syncthreads();
  const int qi = 16 * ck + (col >> 2);
  if (part != 0 || qi >= L.fw_items) return;
  const int p = qi / L.cin, i = qi - p * L.cin, o = m >> 2, s = m & 3;
  const size_t idx = ((((size_t)o * L.cin + i) * 9 + p) * 4 + s) * 4 + (col & 3);
  gw[2 * idx] = (float)(((sum[0][col][0] + sum[1][col][0]) + sum[2][col][0]) + sum[3][col][0]);
  gw[2 * idx + 1] = (float)(((sum[0][col][1] + sum[1][col][1]) + sum[2][col][1]) + sum[3][col][1]);
}

// ---------------------------------------------------------------------------
// weight packing: master FP32 complex W[o][i][p][s][s'] -> MFMA A fragments.

__device__ __forceinline__ float wval(const float *W, int cin, int o, int i, int p, int s, int s2, int im) {
  return W[2 * ((((o * cin + i) * 9 + p) * 4 + s) * 4 + s2) + im];
}

// forward A: row m = 2*(o*4+s) + r, col k = 2*(q*4+s') + r' with q = p*Cin + i.
__global__ void ptc_pack_forward_kernel(PtcLayerDev L, const float *W, bf16x8_t *A) {
  const int total = L.mtiles * L.fw_ks * 64;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int lane = idx % 64, ks = (idx / 64) % L.fw_ks, mt = idx / (64 * L.fw_ks);
  const int m = mt * 16 + (lane & 15);
  const int mp = m >> 1, r = m & 1, o = mp >> 2, s = mp & 3;
  bf16x8_t v;
  for (int j = 0; j < 8; ++j) {
    const int k = ks * 32 + 8 * (lane >> 4) + j;
    const int kp = k >> 1, r2 = k & 1;
    const int qi = kp >> 2, s2 = kp & 3;
    const int p = qi / L.cin, i = qi % L.cin;
    float val = 0.f;
    if (o < L.cout && qi < L.fw_items) {
      const float wr = wval(W, L.cin, o, i, p, s, s2, 0), wi = wval(W, L.cin, o, i, p, s, s2, 1);
      val = (r == 0) ? (r2 == 0 ? wr : -wi) : (r2 == 0 ? wi : wr);
    }
    v[j] = (__bf16)val;
  }
  A[idx] = v;
}

// adjoint A: row m = 2*((p*Cin+i)*4+s') + r, col k = 2*(o*4+s) + r'; conj(W)^T embedded.
__global__ void ptc_pack_adjoint_kernel(PtcLayerDev L, const float *W, bf16x8_t *A) {
  const int ks_n = L.kadj / 32;
  const int total = L.madj_tiles * ks_n * 64;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int lane = idx % 64, ks = (idx / 64) % ks_n, mt = idx / (64 * ks_n);
  const int m = mt * 16 + (lane & 15);
  const int kp = m >> 1, r = m & 1;
  const int qi = kp >> 2, p = qi / L.cin, i = qi - p * L.cin, s2 = kp & 3;
  bf16x8_t v;
  for (int j = 0; j < 8; ++j) {
    const int k = ks * 32 + 8 * (lane >> 4) + j;
    const int mp = k >> 1, r2 = k & 1, o = mp >> 2, s = mp & 3;
    float val = 0.f;
    if (p < 9 && o < L.cout) {
      const float wr = wval(W, L.cin, o, i, p, s, s2, 0), wi = wval(W, L.cin, o, i, p, s, s2, 1);
      // conj(W)^T: [[Wr, Wi], [-Wi, Wr]]
      val = (r == 0) ? (r2 == 0 ? wr : wi) : (r2 == 0 ? -wi : wr);
    }
    v[j] = (__bf16)val;
  }
  A[idx] = v;
}

// ---------------------------------------------------------------------------
// host launchers

hipError_t launch_ptc_nbr(const Geom &g, int *tab, hipStream_t st) {
  if (g.Vh == 0) return hipSuccess;
  hipLaunchKernelGGL(ptc_nbr_kernel, dim3((g.Vh + 255) / 256, 2), dim3(256), 0, st, g, tab);
  return hipGetLastError();
}

hipError_t launch_ptc_links(const PtcGeo &q, int npar, int *nbr, void *tab, hipStream_t st) {
  hipLaunchKernelGGL(ptc_link_kernel, dim3((q.g.Vh + 255) / 256, 16), dim3(256), 0, st, q, npar, nbr, (uint32_t *)tab);
  return hipGetLastError();
}

hipError_t launch_ptc_forward(const PtcGeo &q, const PtcLayerDev &L, const int *nbr, const void *links, const void *in,
                              void *out, int out_f32, int par, int variant, int zero_par, hipStream_t st) {
  // LDS staging of the output tile: BF16 up to 16 channels; FP32 one channel
  if (out_f32 && L.cout != 1) return hipErrorInvalidValue;
  if (par < -1 || par > 1) return hipErrorInvalidValue;
  const int npar = par < 0 ? 2 : 1;  // par -1: both parities in one launch
  switch (variant) {
#define PTC_FWD(NS)                                                                                        \
  hipLaunchKernelGGL((ptc_forward_kernel<NS>), dim3(npar * ((q.g.Vh + NS - 1) / NS)), dim3(kPtcThreads), 0, \
                     st, q, L, nbr, (const bf16 *)in, out, out_f32, par, zero_par);                         \
  break;
    case 642: PTC_FWD(64)
    case 322: PTC_FWD(32)
#undef PTC_FWD
    case kPtcForward16: {
      // it reads every path, so no input parity may be known zero
      if (L.cin != 16 || zero_par >= 0 || !links) return hipErrorInvalidValue;
      const dim3 grid(npar * ((q.g.Vh + kF16Sites - 1) / kF16Sites)), block(kF16Threads);
#define PTC_F16(MT)                                                                                        \
  hipLaunchKernelGGL((ptc_forward16_kernel<MT>), grid, block, 0, st, q, L, nbr, (const uint32_t *)links,    \
                     (const bf16 *)in, out, out_f32, par)
      if (L.mtiles == 1)
        PTC_F16(1);
      else if (L.mtiles == 2)
        PTC_F16(2);
      else if (L.mtiles <= 4)
        PTC_F16(4);
      else
        PTC_F16(8);
#undef PTC_F16
      break;
    }
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Layer-0 input: the even field (FP32 packed spinor) as BF16 activations
// with one channel, zero on odd sites.
__global__ void ptc_input_kernel(int64_t vh, const float *in_even, bf16 *act) {
  // one 16-byte piece of a record per thread
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, s = e / 3;
  if (s >= vh) return;
  float r[8];
  load_chunks<float, 8, 4, float>(in_even + 8 * (e - 3 * s) * vh, vh, s, r);
  store_chunks<bf16, 8, 8, float>(act + 8 * e, 1, 0, r);
  float z[8] = {};
  store_chunks<bf16, 8, 8, float>(act + vh * 24 + 8 * e, 1, 0, z);
}

hipError_t launch_ptc_input(int64_t vh, const void *in_even, void *act, hipStream_t st) {
  if (vh == 0) return hipSuccess;
  hipLaunchKernelGGL(ptc_input_kernel, dim3((unsigned)((3 * vh + 255) / 256)), dim3(256), 0, st, vh,
                     (const float *)in_even, (bf16 *)act);
  return hipGetLastError();
}

hipError_t launch_ptc_delta(int64_t vh, const float *in_even, void *delta, hipStream_t st) {
  hipLaunchKernelGGL(ptc_delta_kernel, dim3((unsigned)((vh + 255) / 256)), dim3(256), 0, st, vh, in_even, (bf16 *)delta);
  return hipGetLastError();
}

hipError_t launch_ptc_bwd_data(const PtcGeo &q, const PtcLayerDev &L, const int *nbr, const void *delta, void *gpsi,
                               int zero_par, hipStream_t st) {
  const dim3 grid(2 * ((q.g.Vh + kBwSites - 1) / kBwSites));
  const int nmt = (8 * L.cin + 15) / 16, nks = L.kadj / 32;
#define PTC_DY(RC, MT, KS)                                                                                \
  hipLaunchKernelGGL((ptc_bwd_data_kernel<RC, MT, KS>), grid, dim3(kBwThreads), 0, st, q, L, nbr,          \
                     (const bf16 *)delta, (bf16 *)gpsi, zero_par)
#define PTC_DY_KS(RC, MT)   \
  if (nks == 1)             \
    PTC_DY(RC, MT, 1);      \
  else if (nks == 2)        \
    PTC_DY(RC, MT, 2);      \
  else                      \
    PTC_DY(RC, MT, 4)
#define PTC_DY_MT(RC)       \
  if (nmt <= 2) {           \
    PTC_DY_KS(RC, 2);       \
  } else if (nmt <= 4) {    \
    PTC_DY_KS(RC, 4);       \
  } else {                  \
    PTC_DY_KS(RC, 8);       \
  }
  if (q.recon == 12) {
    PTC_DY_MT(12)
  } else {
    PTC_DY_MT(18)
  }
#undef PTC_DY_MT
#undef PTC_DY_KS
#undef PTC_DY
  return hipGetLastError();
}

int ptc_weight_chunks(const PtcLayerDev &L) { return (L.fw_items + 15) / 16; }

// Three workgroups per CU fit (LDS, registers): their number over all chunks
// stays at or below 768, so that no second wave of a few workgroups follows
// (792 took twice the time of 720). A multiple of 8, one share per XCD, and no
// more than there are tiles (rounded up: a group may be empty).
int ptc_weight_groups(const PtcLayerDev &L, size_t vh, int zero_par) {
  const size_t tiles = (zero_par < 0 ? 2 : 1) * ((vh + kTile - 1) / kTile);
  const size_t most = 768 / ptc_weight_chunks(L) / 8 * 8;
  return (int)std::min(most, (tiles + 7) / 8 * 8);
}
size_t ptc_weight_partial_bytes(const PtcLayerDev &L, size_t vh, int zero_par) {
  return (size_t)ptc_weight_chunks(L) * ptc_weight_groups(L, vh, zero_par) * L.mw_tiles * 16 * 64 * sizeof(float);
}

hipError_t launch_ptc_bwd_weight(const PtcGeo &q, const PtcLayerDev &L, const int *nbr, const void *in,
                                 const void *delta, float *partial, float *gw, int zero_par, hipStream_t st) {
  const int groups = ptc_weight_groups(L, q.g.Vh, zero_par), nck = ptc_weight_chunks(L);
#define PTC_DW(RC, PATH, JW)                                                                                      \
  hipLaunchKernelGGL((ptc_bwd_weight_kernel<RC, PATH, JW>), dim3(groups, nck), dim3(kWgThreads), 0, st, q, L, nbr, \
                     (const bf16 *)in, (const bf16 *)delta, partial, groups, zero_par)
#define PTC_DW_JW(RC, PATH) \
  if (L.mw_tiles <= 2)      \
    PTC_DW(RC, PATH, 1);    \
  else if (L.mw_tiles <= 4) \
    PTC_DW(RC, PATH, 2);    \
  else                      \
    PTC_DW(RC, PATH, 4)
  if (q.recon == 12) {
    if (L.cin == 16) {
      PTC_DW_JW(12, true);
    } else {
      PTC_DW_JW(12, false);
    }
  } else {
    if (L.cin == 16) {
      PTC_DW_JW(18, true);
    } else {
      PTC_DW_JW(18, false);
    }
  }
#undef PTC_DW_JW
#undef PTC_DW
  hipLaunchKernelGGL(ptc_weight_reduce_kernel, dim3(4 * L.cout, nck), dim3(256), 0, st, L, (const float *)partial,
                     groups, gw);
  return hipGetLastError();
}

hipError_t launch_ptc_pack(const PtcLayerDev &L, const float *W, hipStream_t st) {
  const int bt = 256;
  const int nf = L.mtiles * L.fw_ks * 64;
  hipLaunchKernelGGL(ptc_pack_forward_kernel, dim3((nf + bt - 1) / bt), dim3(bt), 0, st, L, W, (bf16x8_t *)L.A);
  const int na = L.madj_tiles * (L.kadj / 32) * 64;
  hipLaunchKernelGGL(ptc_pack_adjoint_kernel, dim3((na + bt - 1) / bt), dim3(bt), 0, st, L, W, (bf16x8_t *)L.Aadj);
  return hipGetLastError();
}

__global__ void adam_kernel(float *w, float *m, float *v, const float *g, size_t n, float lr, float b1, float b2,
                            float eps, float bc1, float bc2, float gscale) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = gscale * g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

hipError_t launch_adam(float *w, float *m, float *v, const float *g, size_t n, float lr, float b1, float b2, float eps,
                       float bc1, float bc2, float gscale, hipStream_t st) {
  const int bt = 256;
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + bt - 1) / bt)), dim3(bt), 0, st, w, m, v, g, n, lr, b1, b2, eps,
                     bc1, bc2, gscale);
  return hipGetLastError();
}

}  // namespace lqcd
