// Kernels of the gauge-covariant linear network used as the flexible-CG preconditioner.
//
// A layer maps C_in colour-vector channels to C_out on the full lattice:
//   y_c(n) = sum_c' [ W_0[c][c'] psi_c'(n) + sum_{d=1..8} W_d[c][c'] (T_d psi_c')(n) ]
// with T_{+mu} psi(n) = F~_mu(n) psi(n+mu) and T_{-mu} psi(n) = F~_mu(n-mu)^dag psi(n-mu)
// (d = 1..4: +x,+y,+z,+t; d = 5..8: -x,-y,-z,-t).  The transports reuse the packed FP32
// one-hop matrices of the Dslash: for output parity p, k = 4 mu is F~_mu(n) and
// k = 4 mu + 1 is -F~_mu(n-mu)^dag, so T_{-mu} = -L_{4mu+1}.
//
// Activations are complex64, stored per parity.  With C >= 2 channels they are interleaved in
// channel pairs, [parity][C/2][3 colours][V/2][2 channels], so that reading all channels of a
// neighbour takes 3C/2 16-byte loads, each 1 KiB contiguous over a wave (with the colours of a site next
// to each other it spread over 3 KiB, and the load units set the pace of the layers); a single channel is
// [parity][3][V/2].  A null input pointer stands for a field that is zero on that parity.
#include "device.h"
#include "net.h"
#include "launch.h"

namespace stag {

__device__ __forceinline__ void cmac_f(Cx<float>& acc, const float2 w, const Cx<float>& v) {
  acc.re = fmaf(w.x, v.re, acc.re);
  acc.re = fmaf(-w.y, v.im, acc.re);
  acc.im = fmaf(w.x, v.im, acc.im);
  acc.im = fmaf(w.y, v.re, acc.im);
}

// Channels c0 .. c0 + G - 1 of a C-channel activation at site cb (c0 even when G >= 2).
template <int C, int G>
__device__ __forceinline__ void load_channels(const float2* base, long half, long cb, int c0, Cx<float> t[G][3]) {
  if constexpr (C == 1) {
    gptr<f2v> p = as_global<f2v>(base) + cb;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const f2v w = p[i * half];
      t[0][i] = Cx<float>{w.x, w.y};
    }
  } else {
    static_assert(G % 2 == 0, "channel pairs are loaded whole");
#pragma unroll
    for (int q = 0; q < G / 2; ++q) {
      gptr<f4v> p = as_global<f4v>(base) + (long)(c0 / 2 + q) * 3 * half + cb;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const f4v w = p[i * half];
        t[2 * q][i] = Cx<float>{w.x, w.y};
        t[2 * q + 1][i] = Cx<float>{w.z, w.w};
      }
    }
  }
}

template <int C>
__device__ __forceinline__ void store_channels(float2* base, long half, long cb, const Cx<float> v[C][3]) {
  if constexpr (C == 1) {
    gptr_w<f2v> p = as_global_w<f2v>(base) + cb;
#pragma unroll
    for (int i = 0; i < 3; ++i) p[i * half] = f2v{v[0][i].re, v[0][i].im};
  } else {
#pragma unroll
    for (int q = 0; q < C / 2; ++q) {
      gptr_w<f4v> p = as_global_w<f4v>(base) + (long)q * 3 * half + cb;
#pragma unroll
      for (int i = 0; i < 3; ++i)
        p[i * half] = f4v{v[2 * q][i].re, v[2 * q][i].im, v[2 * q + 1][i].re, v[2 * q + 1][i].im};
    }
  }
}

// One side of a launch as a workgroup sees it.  The geometry stays a reference to the kernel argument: its
// arrays are indexed by a run-time direction, which a copy would turn into scratch memory.
struct NetView {
  const Geo& g;
  const char* links;
  int out_par;
  const float2* in_same;
  const float2* in_other;
  float2* out;
  const float2* w;
  const float2* gy;
};
__device__ __forceinline__ NetView net_view(const NetLaunch& l, bool second) {
  return NetView{l.a[0].g,
                 second ? l.a[1].links : l.a[0].links,
                 second ? l.a[1].out_par : l.a[0].out_par,
                 second ? l.a[1].in_same : l.a[0].in_same,
                 second ? l.a[1].in_other : l.a[0].in_other,
                 second ? l.a[1].out : l.a[0].out,
                 l.a[0].w,
                 second ? l.gy[1] : l.gy[0]};
}
constexpr int kNetVecWG = kWave;  // k_net_layer

// A layer launch: workgroups in XCD-sweep order (xcd_sweep_site), the two parities of a tile next to each
// other, so that the activations which both sides and the neighbouring sites read are shared in an XCD's L2.
__device__ __forceinline__ NetView net_side(const NetLaunch& l, int& cb) {
  const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  const Geo& g = l.a[0].g;
  cb = xcd_sweep_site(xcd, (l.n == 2 ? j >> 1 : j) * blockDim.x + threadIdx.x, g.stride[3], g.L[3]);
  return net_view(l, l.n == 2 && (j & 1));
}

// The same with one contiguous range of whole 64-site link blocks per XCD, net_range_len sites, and one side after
// the other: the first layer's even side reads its own sites only, and in between the odd side's workgroups it was
// in their way.  A call of two layers with 2 channels at 24^3x48 takes 103 us, 114 interleaved (111 as two
// launches), with 8 channels 148 and 164.
__host__ __device__ inline int net_range_len(int half) { return ceil_div(half, 8 * kWave) * kWave; }
__device__ __forceinline__ NetView net_range_side(const NetLaunch& l, int& cb) {
  const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int half = l.a[0].g.half, n = net_range_len(half), per = n / kNetVecWG;
  const bool second = l.n == 2 && j < per;
  const int i = (l.n == 2 && !second ? j - per : j) * kNetVecWG + threadIdx.x;
  cb = xcd * n + i < half ? xcd * n + i : -1;
  return net_view(l, second);
}

// Transported colour vectors of all input channels along direction d (1..8) for the site s.
template <int CIN>
__device__ __forceinline__ void transported(const NetView& a, const Site& s, long blk, int lane, int d,
                                            Cx<float> t[CIN][3]) {
  const int mu = (d - 1) & 3;
  const bool fwd = d <= 4;
  const int nb = neighbour(s, a.g, mu, a.g.h1[mu], fwd);
  Cx<float> u[9];
  if (a.g.long12)
    load_link<P32, true>(a.links, blk, 4 * mu + (fwd ? 0 : 1), lane, 1.f, u);
  else
    load_link<P32, false>(a.links, blk, 4 * mu + (fwd ? 0 : 1), lane, 1.f, u);
  if (!fwd)
#pragma unroll
    for (int e = 0; e < 9; ++e) u[e] = Cx<float>{-u[e].re, -u[e].im};
  Cx<float> v[CIN][3];
  load_channels<CIN, CIN>(a.in_other, a.g.half, nb, 0, v);
#pragma unroll
  for (int c = 0; c < CIN; ++c) {
#pragma unroll
    for (int i = 0; i < 3; ++i) t[c][i] = Cx<float>{0.f, 0.f};
    matvec_acc(u, v[c], t[c]);
  }
}

// Layers with one channel on a side.  Large lattices are bound by reads (24^3x48: 1 -> 8 335 MB, 191 of it links,
// in 58 us; 8 -> 1 327 MB in 80 us, its neighbours read eight times through L2), small ones by the chain of load latencies: the next direction's link and
// channels are in flight while a direction is transported and mixed, in single-wave workgroups, so that a small
// lattice spreads over more CUs.  Without that 8 -> 1 took 96 us, and a whole network call with 1, 8, 8 and 1
// channels at 8^4 45 us instead of 39, with 1, 4 and 1 at 10x8x8x14 28 instead of 19.  XCD ranges of whole link
// blocks: a wave whose sites straddle two blocks reads twice the cache lines of a link (26x26x20x30, 1, 4 and 1
// channels: 92 us in the sweep, 87 in ranges).
template <int CIN, int COUT>
__global__ __launch_bounds__(kNetVecWG) void k_net_layer(NetLaunch l) {
  int cb;
  const NetView a = net_range_side(l, cb);
  if (cb < 0) return;
  const Site s = site_of(cb, a.out_par, a.g);
  const long blk = cb >> 6;
  const int lane = cb & 63;
  Cx<float> acc[COUT][3];
#pragma unroll
  for (int c = 0; c < COUT; ++c)
#pragma unroll
    for (int i = 0; i < 3; ++i) acc[c][i] = Cx<float>{0.f, 0.f};
  if (a.in_same) {
    Cx<float> v[CIN][3];
    load_channels<CIN, CIN>(a.in_same, a.g.half, cb, 0, v);
#pragma unroll
    for (int ci = 0; ci < CIN; ++ci) {
#pragma unroll
      for (int c = 0; c < COUT; ++c) {
        const float2 w = a.w[c * CIN + ci];
#pragma unroll
        for (int i = 0; i < 3; ++i) cmac_f(acc[c][i], w, v[ci][i]);
      }
    }
  }
  if (a.in_other) {
    Cx<float> u[2][9], v[2][CIN][3];
    auto fetch = [&](int d) {
      const int mu = (d - 1) & 3;
      const bool fwd = d <= 4;
      if (a.g.long12)
        load_link<P32, true>(a.links, blk, 4 * mu + (fwd ? 0 : 1), lane, 1.f, u[d & 1]);
      else
        load_link<P32, false>(a.links, blk, 4 * mu + (fwd ? 0 : 1), lane, 1.f, u[d & 1]);
      load_channels<CIN, CIN>(a.in_other, a.g.half, neighbour(s, a.g, mu, a.g.h1[mu], fwd), 0, v[d & 1]);
      asm volatile("" ::: "memory");  // these loads stay ahead of the products, and the products of the next fetch
    };
    fetch(1);
#pragma unroll
    for (int d = 1; d <= 8; ++d) {
      if (d < 8) fetch(d + 1);
      Cx<float> w9[9];
#pragma unroll
      for (int e = 0; e < 9; ++e) {
        const Cx<float> w = u[d & 1][e];
        w9[e] = d <= 4 ? w : Cx<float>{-w.re, -w.im};
      }
      const float2* wd = a.w + d * COUT * CIN;
#pragma unroll
      for (int ci = 0; ci < CIN; ++ci) {
        Cx<float> t[3] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
        matvec_acc(w9, v[d & 1][ci], t);
#pragma unroll
        for (int c = 0; c < COUT; ++c) {
          const float2 w = wd[c * CIN + ci];
#pragma unroll
          for (int i = 0; i < 3; ++i) cmac_f(acc[c][i], w, t[i]);
        }
      }
      asm volatile("" ::: "memory");
    }
  }
  store_channels<COUT>(a.out, a.g.half, cb, acc);
}

// Channel mixing on the matrix cores.  For the 64 sites of one wave and one term d (identity or a
// transport), the mixing is the complex product Y[c][n] += sum_c' W_d[c][c'] X_d[c'][n] over the
// 192 columns n = (site, colour).  It runs as a real GEMM with the 2x2 real form of each complex
// weight: rows i = 2c + {re, im}, inner index k = 2c' + {re, im},
//   A[2c][2c'] = Re W, A[2c][2c'+1] = -Im W, A[2c+1][2c'] = Im W, A[2c+1][2c'+1] = Re W,
// on v_mfma_f32_16x16x4_f32 (A 16x4, B 4x16, C 16x16 in FP32): twelve 16-column tiles (colour i, lanes
// 16 q .. 16 q + 15), and ceil(CIN/2) steps of 4 inner indices per term.
//   MFMA lane layout (16x16x4): lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and
//   C[4 (l / 16) + r][l % 16], r = 0..3.
// The transports stay on the vector units, one lane per site.  FP32 products on the matrix cores do not
// overlap other vector instructions, so the two add up (about 24 thousand cycles per wave at 8 channels) and
// bound the kernel; the rest has to stay out of their way.  One stage is one channel pair of one term: its
// four components go to the operand layout through LDS (12 four-byte writes, 3 sixteen-byte reads, free of
// bank conflicts) while the products of the stage before run, and the pair's registers take the loads of
// the next term at once.  Both parities of an 8-channel layer at 24^3x48 take 180 to 194 us (145 us with every
// load left out, 82 us without the products too); two launches in launch order of the sites, whose operand reads
// waited out an LDS latency for each pair of products, took 272 us.
template <int CIN, int COUT>
__global__ __launch_bounds__(256, 2) void k_net_layer_mfma(NetLaunch l) {
  static_assert(CIN >= 2 && CIN <= 8 && CIN % 2 == 0, "the matrix-core layer takes channel pairs, at most 4");
  static_assert(COUT >= 2 && COUT <= 8 && COUT % 2 == 0, "matrix-core layers write whole channel pairs");
  constexpr int KS = CIN / 2;  // inner steps of 4 reals (2 input channels) per term
  __shared__ __align__(16) float xs[256 / kWave][2][kWave * 12];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  int own;
  const NetView a = net_side(l, own);
  if (__ballot(own >= 0) == 0) return;  // the whole wave is past the lattice
  const int cb = own >= 0 ? own : 0;  // dead lanes compute a valid site; their columns are not stored
  const Site s = site_of(cb, a.out_par, a.g);
  const long half = a.g.half;
  const int row = lane & 15, kq = lane >> 4;
  f4v acc[3][4];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[i][q] = f4v{0.f, 0.f, 0.f, 0.f};
  // A operand of this lane: row `row` (channel c, part ri), inner index 4 ks + kq (channel 2 ks + kq / 2, part ki)
  const int c = row >> 1, ri = row & 1, ki = kq & 1;
  const float* wl = reinterpret_cast<const float*>(a.w) + 2 * ((c < COUT ? c : 0) * CIN + (kq >> 1)) + (ri ^ ki);
  auto load_weights = [&](int d, float w[KS]) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) w[ks] = c < COUT ? wl[2 * (d * COUT * CIN + 2 * ks)] : 0.f;
  };
  auto load_u = [&](int d, Cx<float> u[9]) {
    const int k = 4 * ((d - 1) & 3) + (d <= 4 ? 0 : 1);
    if (a.g.long12)
      load_link<P32, true>(a.links, cb >> 6, k, cb & 63, 1.f, u);
    else
      load_link<P32, false>(a.links, cb >> 6, k, cb & 63, 1.f, u);
  };
  auto source = [&](int d) {  // the site whose channels term d reads
    return d == 0 ? cb : neighbour(s, a.g, (d - 1) & 3, a.g.h1[(d - 1) & 3], d <= 4);
  };
  Cx<float> v[KS][2][3], u[2][9];
  float w[3][KS];
  load_weights(0, w[0]);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) load_channels<CIN, 2>(a.in_same, half, cb, 2 * ks, v[ks]);
  float* xw = xs[wave][0];
  const int wr = 12 * row + kq;            // this lane as the site 16 kq + row: [part of k][row][colour][q]
  const int rd = (kq * 16 + row) * 12;     // ... and as an operand lane
  f4v bv[3];
#pragma unroll
  for (int d = 0; d < 9; ++d) {
    int nb = 0;
    if (d < 8) {
      nb = source(d + 1);
      load_weights(d + 1, w[(d + 1) % 3]);
      load_u(d + 1, u[(d + 1) & 1]);
    }
    if (d > 4)
#pragma unroll
      for (int e = 0; e < 9; ++e) u[d & 1][e] = Cx<float>{-u[d & 1][e].re, -u[d & 1][e].im};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      Cx<float> t[2][3];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (d == 0) {
#pragma unroll
          for (int i = 0; i < 3; ++i) t[h][i] = v[ks][h][i];
        } else {
#pragma unroll
          for (int i = 0; i < 3; ++i) t[h][i] = Cx<float>{0.f, 0.f};
          matvec_acc(u[d & 1], v[ks][h], t[h]);
        }
      }
      if (d < 8) load_channels<CIN, 2>(a.in_other, half, nb, 2 * ks, v[ks]);
      const int stage = d * KS + ks;
      float* x = xw + (stage & 1) * (kWave * 12);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        x[wr + 4 * i] = t[0][i].re;
        x[wr + 4 * i + 192] = t[0][i].im;
        x[wr + 4 * i + 384] = t[1][i].re;
        x[wr + 4 * i + 576] = t[1][i].im;
      }
      __builtin_amdgcn_wave_barrier();
      if (stage > 0) {
        const int pd = ks ? d : d - 1, pk = ks ? ks - 1 : KS - 1;  // the stage before
        const float av = ri == 0 && ki == 1 ? -w[pd % 3][pk] : w[pd % 3][pk];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[i][q], acc[i][q], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 3; ++i) bv[i] = *reinterpret_cast<const f4v*>(x + rd + 4 * i);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  {
    const float av = ri == 0 && ki == 1 ? -w[8 % 3][KS - 1] : w[8 % 3][KS - 1];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[i][q], acc[i][q], 0, 0, 0);
  }
  // C rows 4 kq .. 4 kq + 3 are channels 2 kq and 2 kq + 1, (re, im) each: one pair of the interleaved layout
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int site = __shfl(own, 16 * q + row, kWave);
    if (site < 0 || 2 * kq >= COUT) continue;
    gptr_w<f4v> o = as_global_w<f4v>(a.out) + (long)kq * 3 * half + site;
#pragma unroll
    for (int i = 0; i < 3; ++i) o[(long)i * half] = acc[i][q];
  }
}

// A workgroup of a weight-gradient launch: block b of nblk adds the sites b, b + nblk, ... (in units of a
// workgroup or wave), for one of nd directions (or pairs) and one side.  Eight consecutive workgroups go to
// the eight XCDs; on each, the directions and sides of one block follow each other and run together, reading
// the same output gradients and neighbourhood through one L2, and consecutive blocks stay on one XCD.
// nblk is a multiple of 8.
struct WgradBlock {
  int b, d, side;
};
__device__ __forceinline__ WgradBlock wgrad_block(int nblk, int nd, int nside) {
  const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3, per = nd * nside, k = j % per;
  return WgradBlock{xcd * (nblk >> 3) + j / per, k % nd, k / nd};
}

// Weight gradient, one direction d per workgroup (wgrad_block), all output channels:
//   partial[p][d][c][c'] = sum_n sum_a G_c(n)_a conj((T_d psi_c')(n)_a)
// over the output sites of parity a.out_par; each block walks sites with a grid stride and
// writes one partial (complex, FP64) per (d, c, c') for a fixed-order second stage.
template <int CIN, int COUT>
__global__ __launch_bounds__(256) void k_net_wgrad(NetLaunch l, double* partial, int nblk) {
  const WgradBlock wb = wgrad_block(nblk, 9, l.n);
  const NetView a = net_view(l, wb.side != 0);
  const float2* gy = a.gy;
  const int b = wb.b, d = wb.d;
  Cx<float> acc[COUT][CIN];
#pragma unroll
  for (int c = 0; c < COUT; ++c)
#pragma unroll
    for (int ci = 0; ci < CIN; ++ci) acc[c][ci] = Cx<float>{0.f, 0.f};
  const bool have = d == 0 ? a.in_same != nullptr : a.in_other != nullptr;
  if (have && gy) {
    for (int cb = b * blockDim.x + threadIdx.x; cb < a.g.half; cb += nblk * blockDim.x) {
      const Site s = site_of(cb, a.out_par, a.g);
      Cx<float> t[CIN][3];
      if (d == 0) {
        load_channels<CIN, CIN>(a.in_same, a.g.half, cb, 0, t);
      } else {
        transported<CIN>(a, s, cb >> 6, cb & 63, d, t);
      }
      Cx<float> gvs[COUT][3];
      load_channels<COUT, COUT>(gy, a.g.half, cb, 0, gvs);
#pragma unroll
      for (int c = 0; c < COUT; ++c) {
        const Cx<float>* gv = gvs[c];
#pragma unroll
        for (int ci = 0; ci < CIN; ++ci)
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            // g * conj(t)
            acc[c][ci].re = fmaf(gv[i].re, t[ci][i].re, acc[c][ci].re);
            acc[c][ci].re = fmaf(gv[i].im, t[ci][i].im, acc[c][ci].re);
            acc[c][ci].im = fmaf(gv[i].im, t[ci][i].re, acc[c][ci].im);
            acc[c][ci].im = fmaf(-gv[i].re, t[ci][i].im, acc[c][ci].im);
          }
      }
    }
  }
  // block reduction, one (c, c') pair at a time, in FP64
  __shared__ double lds[2 * 4];
#pragma unroll
  for (int c = 0; c < COUT; ++c)
#pragma unroll
    for (int ci = 0; ci < CIN; ++ci) {
      double v[2] = {(double)acc[c][ci].re, (double)acc[c][ci].im};
      block_sum<2>(v, lds);
      if (threadIdx.x == 0) {
        const long idx = ((((long)a.out_par * 9 + d) * COUT + c) * CIN + ci) * nblk + b;
        partial[2 * idx] = v[0];
        partial[2 * idx + 1] = v[1];
      }
      __syncthreads();
    }
}

// Weight gradient on the matrix cores, two directions d per workgroup (wgrad_block):
//   P[c][c'] = sum_n sum_a G_c(n)_a conj(X_d,c'(n)_a),  X_d = T_d psi (or psi for d = 0),
// as a real GEMM over the inner index k = 2 n + part (n = 3 site + colour) with rows i = 2c + {re, im}:
//   A[2c][(n,0)] = Re G, A[2c][(n,1)] = Im G, A[2c+1][(n,0)] = Im G, A[2c+1][(n,1)] = -Re G,
//   B[(n,0)][c'] = Re X, B[(n,1)][c'] = Im X,  columns 0-7 for the first direction and 8-15 for the second
// (unused columns are zero).  Each wave walks 64-site chunks with a grid stride and accumulates one 16x16
// FP32 tile; the waves of a block are summed in FP64 in a fixed order and written as one partial per block
// in the layout of k_net_wgrad.
// Half a wave works on each direction, 32 sites at a time, and on half of the output channels.  G and X reach
// the operand layout through LDS (18.8 KB per wave at 8 channels, eight waves per CU), stored as
// [channel][k of the step][step], so that a lane reads the operands of four consecutive steps with one
// 16-byte load.  Row strides of 196 floats spread the 16 rows over the banks; the rows were 384 floats apart
// before, all on one bank, and those conflicts were 60% of the launch.  The loads of the next 32 sites are in
// flight during the products.  Both parities of an 8-channel layer at 24^3x48 take 283 to 293 us; with one direction
// per workgroup, half the columns empty, 655 us.
constexpr int kWgradMfmaWG = 128;

template <int CIN, int COUT>
__global__ __launch_bounds__(kWgradMfmaWG, 2) void k_net_wgrad_mfma(NetLaunch l, double* partial, int nblk) {
  static_assert(CIN >= 2 && CIN <= 8 && COUT >= 2 && COUT <= 8, "the matrix-core gradient needs 2..8 channels");
  constexpr int NW = kWgradMfmaWG / kWave;
  constexpr int HS = kWave / 2;        // sites staged at a time
  constexpr int NS = 3 * HS / 2;       // inner steps of 4 (two n, both parts) they make
  constexpr int RS = 4 * NS + 4;       // row stride of a staged channel
  __shared__ __align__(16) float xs[NW][2][CIN][RS];
  __shared__ __align__(16) float gs[NW][COUT][RS];
  double(*red)[kWave][4] = reinterpret_cast<double(*)[kWave][4]>(&xs[0][0][0][0]);  // after the last chunk
  static_assert(sizeof(xs) >= sizeof(double) * NW * kWave * 4, "the reduction reuses the staging buffer");
  const WgradBlock wb = wgrad_block(nblk, 5, l.n);
  const NetView a = net_view(l, wb.side != 0);
  const float2* gy = a.gy;
  const int b = wb.b, d0 = 2 * wb.d;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int row = lane & 15, kq = lane >> 4;
  f4v acc = f4v{0.f, 0.f, 0.f, 0.f};
  if (gy) {
    const int nhalf = ceil_div(a.g.half, kWave) * 2;  // 32-site halves of the chunks
    // operands of this lane: row c, part ri of G; column row & 7 of direction row >> 3 of X
    const int c = row >> 1, ri = row & 1;
    const bool bcol = (row & 7) < CIN;
    const float* xl = &xs[wave][row >> 3][bcol ? row & 7 : 0][kq * NS];
    const float* gl = &gs[wave][c < COUT ? c : 0][(kq ^ ri) * NS];
    const float gsign = c < COUT ? (ri == 1 && (kq & 1) == 1 ? -1.f : 1.f) : 0.f;
    // what this lane loads: direction d0 + q, and GC channels of G from gc0 on (with two channels both halves
    // load the pair and each stages one)
    constexpr int GC = COUT >= 4 ? COUT / 2 : 2;
    const int q = lane >> 5, ls = lane & (HS - 1), d = d0 + q, gc0 = COUT >= 4 ? q * GC : 0;
    const int mu0 = (d0 - 1) & 3, mu1 = d0 & 3;
    const int k = q ? 4 * mu1 + (d0 + 1 <= 4 ? 0 : 1) : 4 * mu0 + (d0 <= 4 ? 0 : 1);
    Cx<float> u[9], v[CIN][3], gvs[GC][3];
    auto load_half = [&](int hc) {  // sites 32 hc ..
      const int cb = min(hc * HS + ls, a.g.half - 1);
      const Site s = site_of(cb, a.out_par, a.g);
      if (d == 0) {
        load_channels<CIN, CIN>(a.in_same, a.g.half, cb, 0, v);
      } else if (d < 9) {
        const int n0 = d0 == 0 ? 0 : neighbour(s, a.g, mu0, a.g.h1[mu0], d0 <= 4);
        const int n1 = d0 == 8 ? 0 : neighbour(s, a.g, mu1, a.g.h1[mu1], d0 + 1 <= 4);
        if (a.g.long12)
          load_link<P32, true>(a.links, cb >> 6, k, cb & 63, 1.f, u);
        else
          load_link<P32, false>(a.links, cb >> 6, k, cb & 63, 1.f, u);
        load_channels<CIN, CIN>(a.in_other, a.g.half, q ? n1 : n0, 0, v);
      }
      load_channels<COUT, GC>(gy, a.g.half, cb, gc0, gvs);
    };
    const int wv = b * NW + wave, step = 2 * nblk * NW;
    int hc = 2 * wv;
    if (hc < nhalf) load_half(hc);
    while (hc < nhalf) {  // uniform per wave
      Cx<float> t[CIN][3];
      const bool live = hc * HS + ls < a.g.half;
      const float sg = d > 4 ? -1.f : 1.f;
#pragma unroll
      for (int e = 0; e < 9; ++e) u[e] = Cx<float>{sg * u[e].re, sg * u[e].im};
#pragma unroll
      for (int ci = 0; ci < CIN; ++ci) {
#pragma unroll
        for (int i = 0; i < 3; ++i) t[ci][i] = Cx<float>{0.f, 0.f};
        matvec_acc(u, v[ci], t[ci]);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          if (d == 0) t[ci][i] = v[ci][i];
          if (!live || d > 8) t[ci][i] = Cx<float>{0.f, 0.f};
        }
      }
      // entry n = 3 ls + i: step n / 2, k = 2 (n & 1) + part
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const int n = 3 * ls + i, at = 2 * (n & 1) * NS + (n >> 1);
#pragma unroll
        for (int ci = 0; ci < CIN; ++ci) {
          xs[wave][q][ci][at] = t[ci][i].re;
          xs[wave][q][ci][at + NS] = t[ci][i].im;
        }
#pragma unroll
        for (int j = 0; j < (COUT >= 4 ? GC : 1); ++j) {
          const Cx<float> gv = COUT >= 4 ? gvs[j][i] : (q ? gvs[1][i] : gvs[0][i]);
          float* o = &gs[wave][COUT >= 4 ? gc0 + j : q][at];
          o[0] = live ? gv.re : 0.f;
          o[NS] = live ? gv.im : 0.f;
        }
      }
      __builtin_amdgcn_wave_barrier();
      hc = hc & 1 ? hc - 1 + step : hc + 1;
      if (hc < nhalf) load_half(hc);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NS / 4; ++j) {
        const f4v av = reinterpret_cast<const f4v*>(gl)[j], bv = reinterpret_cast<const f4v*>(xl)[j];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(gsign == 0.f ? 0.f : gsign * av[e], bcol ? bv[e] : 0.f, acc, 0, 0,
                                                     0);
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][lane][r] = (double)acc[r];
  __syncthreads();
  if (wave != 0) return;
  double v[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    v[r] = red[0][lane][r];
    for (int w = 1; w < NW; ++w) v[r] += red[w][lane][r];
  }
  // C rows 4 kq + r: channel 2 kq + (r >> 1), part r & 1; column row: c' = row & 7 of direction d0 + (row >> 3)
  const int cp = row & 7, d = d0 + (row >> 3);
  if (cp >= CIN || d >= 9) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int co = 2 * kq + h;
    if (co >= COUT) continue;
    const long idx = ((((long)a.out_par * 9 + d) * COUT + co) * CIN + cp) * nblk + b;
    partial[2 * idx] = v[2 * h];
    partial[2 * idx + 1] = v[2 * h + 1];
  }
}

// out[d][c][c'] += sum over parities and blocks of the partials, in a fixed order.  One wave per (d, c, c'):
// the partials of one parity and output are contiguous and go through LDS, so that the serial sum waits on
// LDS and not on memory (one lane walking them in memory took 60 us of dependent loads, this 5).
constexpr int kWgradReduceMax = 512;
__global__ __launch_bounds__(64) void k_net_wgrad_reduce(const double* partial, int n, int nblk, int npar,
                                                         double* out) {
  __shared__ double2 s[kWgradReduceMax];
  const int j = blockIdx.x;  // (d, c, c') flat, of n
  const double2* src = reinterpret_cast<const double2*>(partial);
  for (int i = threadIdx.x; i < npar * nblk; i += kWave) {
    const int p = i / nblk;
    s[i] = src[((long)p * n + j) * nblk + (i - p * nblk)];
  }
  __syncthreads();
  if (threadIdx.x > 1) return;
  const double* v = reinterpret_cast<const double*>(s) + threadIdx.x;  // lane 0 real, lane 1 imaginary parts
  double sum = 0.0;
#pragma unroll 16
  for (int i = 0; i < npar * nblk; ++i) sum += v[2 * i];
  out[2 * j + threadIdx.x] += sum;
}

// Place in a single-channel activation [3][V/2] of entry i of an even-site vector [V/2][3], n = 3 V/2.
__device__ __forceinline__ long plane_of(long i, long n) { return (i % 3) * (n / 3) + i / 3; }

// even-site complex128 vector -> channel 0 of a complex64 activation (parity 0)
__global__ __launch_bounds__(256) void k_net_embed(const double2* in, float2* out, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 v = in[i];
  out[plane_of(i, n)] = make_float2((float)v.x, (float)v.y);
}

// channel 0 of a complex64 activation (parity 0) -> even-site complex128 vector
__global__ __launch_bounds__(256) void k_net_extract(const float2* in, double2* out, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float2 v = in[plane_of(i, n)];
  out[i] = make_double2((double)v.x, (double)v.y);
}

// Loss gradient at the output: g = scale (N(b) - x) on even sites; partial |N(b) - x|^2 per block.
__global__ __launch_bounds__(256) void k_net_loss(const float2* out, const double2* x, double scale, float2* g,
                                                  double* partial, long n) {
  __shared__ double lds[4];
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  double s[1] = {0.0};
  if (i < n) {
    const long j = plane_of(i, n);
    const float2 o = out[j];
    const double2 xv = x[i];
    const double dr = (double)o.x - xv.x, di = (double)o.y - xv.y;
    s[0] = dr * dr + di * di;
    g[j] = make_float2((float)(scale * dr), (float)(scale * di));
  }
  block_sum<1>(s, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = s[0];
}

__global__ __launch_bounds__(256) void k_sum_partials(const double* partial, int n, double* out) {
  __shared__ double lds[4];
  double s[1] = {0.0};
  for (int i = threadIdx.x; i < n; i += blockDim.x) s[0] += partial[i];
  block_sum<1>(s, lds);
  if (threadIdx.x == 0) *out = s[0];
}

// ---- launchers ---------------------------------------------------------------------
hipError_t launch_net_layer(const NetLaunch& l, int cin, int cout, hipStream_t st) {
  if (l.n == 0) return hipSuccess;
  const Geo& g = l.a[0].g;
  const long len = xcd_sweep_len(g.stride[3], g.L[3]);
  // The matrix-core layer too takes single-wave workgroups below two waves per SIMD (a network of 1, 8, 8 and 1
  // channels at 12^3x16: 47 us against 54); at 16^3x32, just there, four waves are faster: 84 us against 93.
  const int wg = 8 * l.n * len < 2048L * kWave ? kWave : 256;
  const int nv = 8 * l.n * (net_range_len(g.half) / kNetVecWG), nb = 8 * l.n * (int)((len + wg - 1) / wg);
  // layers with at least two channels on both sides mix on the matrix cores; 1 -> C and C -> 1
  // would fill at most a quarter of an MFMA tile and stay on the vector units
#define STAG_NET_LAYER(I, O) \
  if (cin == I && cout == O) { k_net_layer<I, O><<<nv, kNetVecWG, 0, st>>>(l); return hipGetLastError(); }
#define STAG_NET_LAYER_MFMA(I, O) \
  if (cin == I && cout == O) { \
    for (int i = 0; i < l.n; ++i) \
      if (!l.a[i].in_same || !l.a[i].in_other) return hipErrorInvalidValue;  /* inner layers: both parities set */ \
    k_net_layer_mfma<I, O><<<nb, wg, 0, st>>>(l); return hipGetLastError(); }
  STAG_NET_LAYER(1, 1) STAG_NET_LAYER(1, 2) STAG_NET_LAYER(2, 1) STAG_NET_LAYER_MFMA(2, 2)
  STAG_NET_LAYER(1, 4) STAG_NET_LAYER(4, 1) STAG_NET_LAYER_MFMA(4, 4)
  STAG_NET_LAYER(1, 8) STAG_NET_LAYER(8, 1) STAG_NET_LAYER_MFMA(8, 8)
#undef STAG_NET_LAYER
#undef STAG_NET_LAYER_MFMA
  return hipErrorInvalidValue;
}

hipError_t launch_net_wgrad(const NetLaunch& l, double* partial, int cin, int cout, int nblk, hipStream_t st) {
  if (nblk % 8) return hipErrorInvalidValue;
#define STAG_NET_WG(I, O)                                                          \
  if (cin == I && cout == O) {                                                     \
    k_net_wgrad<I, O><<<nblk * 9 * l.n, 256, 0, st>>>(l, partial, nblk);           \
    return hipGetLastError();                                                      \
  }
#define STAG_NET_WG_MFMA(I, O)                                                     \
  if (cin == I && cout == O) {                                                     \
    for (int i = 0; i < l.n; ++i) /* inner layers: both parities set */            \
      if (!l.a[i].in_same || !l.a[i].in_other) return hipErrorInvalidValue;        \
    k_net_wgrad_mfma<I, O><<<nblk * 5 * l.n, kWgradMfmaWG, 0, st>>>(l, partial, nblk); \
    return hipGetLastError();                                                      \
  }
  STAG_NET_WG(1, 1) STAG_NET_WG(1, 2) STAG_NET_WG(2, 1) STAG_NET_WG_MFMA(2, 2)
  STAG_NET_WG(1, 4) STAG_NET_WG(4, 1) STAG_NET_WG_MFMA(4, 4)
  STAG_NET_WG(1, 8) STAG_NET_WG(8, 1) STAG_NET_WG_MFMA(8, 8)
#undef STAG_NET_WG
#undef STAG_NET_WG_MFMA
  return hipErrorInvalidValue;
}

hipError_t launch_net_wgrad_reduce(const double* partial, int cin, int cout, int nblk, int npar, double* out,
                                   hipStream_t st) {
  if (npar * nblk > kWgradReduceMax) return hipErrorInvalidValue;
  const int n = 9 * cout * cin;
  k_net_wgrad_reduce<<<n, kWave, 0, st>>>(partial, n, nblk, npar, out);
  return hipGetLastError();
}

hipError_t launch_net_embed(const void* in, float2* out, long nsites, hipStream_t st) {
  const long n = nsites * 3;
  if (n == 0) return hipSuccess;
  k_net_embed<<<(n + 255) / 256, 256, 0, st>>>(reinterpret_cast<const double2*>(in), out, n);
  return hipGetLastError();
}

hipError_t launch_net_extract(const float2* in, void* out, long nsites, hipStream_t st) {
  const long n = nsites * 3;
  if (n == 0) return hipSuccess;
  k_net_extract<<<(n + 255) / 256, 256, 0, st>>>(in, reinterpret_cast<double2*>(out), n);
  return hipGetLastError();
}

hipError_t launch_net_loss(const float2* out, const void* x, double scale, float2* g, double* partial, double* sum,
                           long nsites, hipStream_t st) {
  const long n = nsites * 3;
  const int nb = (int)((n + 255) / 256);
  k_net_loss<<<nb, 256, 0, st>>>(out, reinterpret_cast<const double2*>(x), scale, g, partial, n);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_sum_partials<<<1, 256, 0, st>>>(partial, nb, sum);
  return hipGetLastError();
}

}  // namespace stag

namespace stag {

__global__ __launch_bounds__(256) void k_norm2_c128(const double2* x, double* partial, long n) {
  __shared__ double lds[4];
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  double s[1] = {0.0};
  if (i < n) {
    const double2 v = x[i];
    s[0] = v.x * v.x + v.y * v.y;
  }
  block_sum<1>(s, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = s[0];
}

hipError_t launch_norm2_c128(const void* x, double* partial, double* sum, long nsites, hipStream_t st) {
  const long n = nsites * 3;
  const int nb = (int)((n + 255) / 256);
  k_norm2_c128<<<nb, 256, 0, st>>>(reinterpret_cast<const double2*>(x), partial, n);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_sum_partials<<<1, 256, 0, st>>>(partial, nb, sum);
  return hipGetLastError();
}

}  // namespace stag

namespace stag {

// out = a - b (complex128), partial |out|^2 per block
__global__ __launch_bounds__(256) void k_sub_norm(const double2* a, const double2* b, double2* out, double* partial,
                                                  long n) {
  __shared__ double lds[4];
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  double s[1] = {0.0};
  if (i < n) {
    const double2 u = a[i], v = b[i];
    const double2 w = make_double2(u.x - v.x, u.y - v.y);
    out[i] = w;
    s[0] = w.x * w.x + w.y * w.y;
  }
  block_sum<1>(s, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = s[0];
}

// even-site complex128 vector times a real scale -> single-channel complex64 activation
__global__ __launch_bounds__(256) void k_scale_to_f32(const double2* in, double scale, float2* out, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 v = in[i];
  out[plane_of(i, n)] = make_float2((float)(scale * v.x), (float)(scale * v.y));
}

hipError_t launch_sub_norm(const void* a, const void* b, void* out, double* partial, double* sum, long nsites,
                           hipStream_t st) {
  const long n = nsites * 3;
  const int nb = (int)((n + 255) / 256);
  k_sub_norm<<<nb, 256, 0, st>>>(reinterpret_cast<const double2*>(a), reinterpret_cast<const double2*>(b),
                                 reinterpret_cast<double2*>(out), partial, n);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_sum_partials<<<1, 256, 0, st>>>(partial, nb, sum);
  return hipGetLastError();
}

hipError_t launch_scale_to_f32(const void* in, double scale, float2* out, long nsites, hipStream_t st) {
  const long n = nsites * 3;
  k_scale_to_f32<<<(n + 255) / 256, 256, 0, st>>>(reinterpret_cast<const double2*>(in), scale, out, n);
  return hipGetLastError();
}

}  // namespace stag
